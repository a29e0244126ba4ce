"""HSIC term pass at the edges of its 256-column slices, 128-row tiles, row groups and batches
of four permutations, and with kernel entries that vanish or are far below 1."""
import numpy as np
import pytest

import oracle
from paper_2406_06488_amd import api
from tests.test_gpu_hsic import _dev, _pair, compare_hsic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n,B", [(5, 1), (127, 3), (128, 4), (129, 5), (255, 31), (256, 32),
                                 (257, 33), (384, 40), (513, 66), (1025, 9)])
def test_slice_edges(n, B, prec):
    X, Y = _pair(n, 6, 5, n + B, 0.7, prec)
    g = api.hsic(_dev(X, prec), _dev(Y, prec), B, 7, 0.1, 0.15, prec)
    compare_hsic(g, oracle.hsic_test(X, Y, B, 7, 0.1, 0.15), prec, X, Y, 0.1, 0.15)


def test_small_entries():
    """Entries of L around 1e-9: the row sums keep their relative accuracy beside the unit
    diagonal (FP64 form; an entry's own error grows with its exponent in the FP32 form)."""
    X, Y = _pair(150, 6, 5, 3, 0.7, "f64")
    g = api.hsic(_dev(X, "f64"), _dev(Y, "f64"), 40, 7, 0.1, 2.0, "f64")
    compare_hsic(g, oracle.hsic_test(X, Y, 40, 7, 0.1, 2.0), "f64", X, Y, 0.1, 2.0)


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_vanishing_entries_tie(prec):
    """Every entry of L underflows to 0: all permutations tie at 0 and all count."""
    X, Y = _pair(300, 6, 5, 3, 0.7, prec)
    g = api.hsic(_dev(X, prec), _dev(Y, prec), 50, 7, 0.1, 1e6, prec)
    assert g["statistic"] == 0.0 and g["count_ge"] == 50 and g["p_value"] == 1.0
    assert not np.any(g["perm_stats"].cpu().numpy())
