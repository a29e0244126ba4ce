"""Work lists that one dispatch does not hold go in several: the second and later ones against
values of other paths (sizes just past each limit)."""
import numpy as np
import pytest

from paper_2406_06488_amd import _lib, api, inputs
from tests.gpu_helpers import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _cross_means(X, Y):
    """U, sigma and the mean distance of the cross test in FP64, by blocks of rows."""
    X, Y = X.double(), Y.double()
    hx, hy = X.shape[0] // 2, Y.shape[0] // 2

    def means(A, C):
        out = []
        for a in torch.split(A, 1024):
            d2 = torch.zeros((a.shape[0], C.shape[0]), dtype=torch.float64, device="cuda")
            for k in range(A.shape[1]):
                d2 += (a[:, k, None] - C[None, :, k]) ** 2
            out.append(d2.sqrt_().mean(1))
        return torch.cat(out)

    vx = means(X[:hx], Y[hy:]) - (m := means(X[:hx], X[hx:]))
    vy = means(Y[:hy], Y[hy:]) - means(Y[:hy], X[hx:])
    u = float(vx.mean() - vy.mean())
    sigma = float((vx.var(unbiased=False) / hx + vy.var(unbiased=False) / hy).sqrt())
    return u, sigma, float(m.mean())


@pytest.mark.parametrize("prec,n,tol", [
    ("f64", 93000, 1e-12),    # 727^2 tiles: past 2^22 parts of a tile
    ("f32", 262150, 1e-5),    # 2049^2 tiles: past 2^22 tiles
])
def test_cross_tiles(prec, n, tol):
    say("cross dispatches", prec, n)
    X, Y = inputs.device_pair(n, n, 2, 3, mean_shift=0.05)
    if prec == "f64":
        X, Y = X.double(), Y.double()
    g = api.cross(X, Y, "ed", prec)
    u, sigma, scale = _cross_means(X, Y)
    assert abs(g["statistic"] - u) <= tol * scale and abs(g["sigma"] - sigma) <= tol * scale, (g, u, sigma)


def test_standard_pass_f64():
    """A pass of 162 splits of 4278 tiles each, eight parts a tile: past 2^22.  The
    pre-computation test gives the same statistics; either's error is a few roundings of the
    mean distance (about 3)."""
    X, Y = inputs.device_pair(6000, 5700, 4, 5, mean_shift=0.05)
    X, Y, B = X.double(), Y.double(), 165
    say("standard dispatches")
    a = api.standard(X, Y, B, 3, "ed", "f64")["perm_stats"]
    b = api.precomputed(X, Y, B, 3, "ed", "f64")["perm_stats"]
    assert float((a - b).abs().max()) <= 1e-13 * 3


def test_precomputed_strips():
    """60 strips x 139 900 groups of 64 splits: past 2^23 workgroups.  The first splits bit for
    bit those of a short test; all of them by the efficient test's statistics (1e-5 each)."""
    X, Y = inputs.device_pair(400, 100, 5, 6, mean_shift=0.05)
    B = 64 * 139900 - 1
    say("precomputed dispatches", B)
    a = api.precomputed(X, Y, B, 3, "ed", "f32")
    few = api.precomputed(X, Y, 1000, 3, "ed", "f32")["perm_stats"]
    assert torch.equal(a["perm_stats"][:1000], few)
    b = api.run(X, Y, B, 3, "ed", "f32")["perm_stats"]
    floor = float(b.abs().mean())
    err = (a["perm_stats"] - b).abs() / torch.clamp(b.abs(), min=floor)
    assert float(err.max()) <= 2e-5
    assert a["count_ge"] == int((a["perm_stats"] >= a["threshold"]).sum())


def test_resampling_units_f64():
    """Units of one tile and one chunk: 60 x 17 500 of them, past 2^20, a dispatch per quarter.
    The first and the last splits bit for bit those of short tests."""
    X, Y = inputs.device_pair(400, 100, 5, 7, mean_shift=0.05)
    X, Y, few = X.double(), Y.double(), 1000
    B = 256 * 17500 - 1
    say("resampling dispatches", B)
    _lib.check(_lib.load().etest_tune_set(_lib.PREC_F64, 500, 501, 1, 1))
    try:
        a = api.run(X, Y, B, 3, "ed", "f64")
        head = api.run(X, Y, few, 3, "ed", "f64")
        words = api.membership(400, 100, 3, B - few, few)
        tail = api.perm_stats_from_membership(X, Y, words, "ed", "f64")
    finally:
        _lib.check(_lib.load().etest_tune_clear())
    assert a["threshold"] == head["threshold"] == tail["threshold"]
    assert torch.equal(a["perm_stats"][:few], head["perm_stats"])
    assert torch.equal(a["perm_stats"][B - few:], tail["perm_stats"])
