"""HSIC tests past 2048 pairs in the FP64 form, and of more permutations than one pass over the
1 GiB of tables and partial sums takes."""
import numpy as np
import pytest

import oracle
from paper_2406_06488_amd import api
from tests.gpu_helpers import TOL, say
from tests.test_gpu_hsic import _dev, _pair, _term_scale, compare_hsic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,B", [(2049, 5), (3000, 33), (4096, 6)])
def test_largest_row_stage_f64(n, B):
    X, Y = _pair(n, 6, 5, n, 0.2, "f64")
    g = api.hsic(_dev(X, "f64"), _dev(Y, "f64"), B, 7, 0.1, 0.15, "f64")
    compare_hsic(g, oracle.hsic_test(X, Y, B, 7, 0.1, 0.15), "f64", X, Y, 0.1, 0.15)


@pytest.mark.parametrize("prec,rows", [("f64", 4), ("f32", 8)])
def test_second_pass(prec, rows):
    """The permutations around the end of the first pass, and the last, against the oracle's
    HSIC of each; the first ones bit for bit those of a test of one pass."""
    n, seed, gx, gy = 4096, 9, 0.1, 0.15
    first = 2 ** 30 // (4 * n + 8 * (n // 256) * (n // rows))  # tables, partial sums
    B = first + 300
    X, Y = _pair(n, 6, 5, 11, 0.1, prec)
    Xd, Yd = _dev(X, prec), _dev(Y, prec)
    say("hsic passes", prec, first, B)
    g = api.hsic(Xd, Yd, B, seed, gx, gy, prec)
    ps = g["perm_stats"].cpu().numpy()
    few = api.hsic(Xd, Yd, 300, seed, gx, gy, prec)
    assert few["statistic"] == g["statistic"]
    assert np.array_equal(few["perm_stats"].cpu().numpy(), ps[:300])
    assert g["count_ge"] == int(np.sum(ps >= g["threshold"]))
    from scipy.spatial.distance import cdist
    X, Y = X.astype(np.float64), Y.astype(np.float64)
    K, L = np.exp(-gx * cdist(X, X, "sqeuclidean")), np.exp(-gy * cdist(Y, Y, "sqeuclidean"))
    picks = [first - 2, first - 1, first, first + 1, first + 150, B - 1]
    want = np.array([oracle.hsic(K, L, oracle.permutation(n, seed, b)) for b in picks])
    floor = np.mean(np.abs(ps))
    extra = 1e-14 * _term_scale(X, Y, gx, gy) if prec == "f64" else 0.0
    err = np.abs(ps[picks] - want)
    assert np.all(err <= TOL[prec] * np.maximum(np.abs(want), floor) + extra), (err, want)
    assert abs(g["statistic"] - oracle.hsic(K, L)) <= TOL[prec] * abs(g["statistic"]) + extra
