"""Strip sums of the pre-computation test."""
import numpy as np
import pytest

import oracle
from paper_2406_06488_amd import api
from tests.test_gpu_hsic import _dev

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


def test_small_entries_beside_a_large_one():
    """One item at distance 1 from all others, whose own distances d are just below 2^-53, half
    an ulp of 1: a row's sum over the x* columns starts with the 1 and loses every d that is added
    to it one by one.  Chains of 32 columns lose at most 31 of the 126; what a row's x* sum lacks
    goes to its y* sum (row total less x* sum), hence into S_XY, of which the statistic takes 2 /
    (nx ny); beside that two roundings of each row's sums."""
    nx, ny = 128, 2
    d = 0.98 * U
    W = np.zeros((nx + ny, nx + ny))
    W[1:, 0] = 1.0
    W[1:, 1:] += np.eye(nx + ny - 1) * (d / np.sqrt(2.0))
    X, Y = W[:nx].copy(), W[nx:].copy()
    XX, YY, XY = (b.cpu().numpy() for b in api.blocks(_dev(X, "f64"), _dev(Y, "f64"), "ed", "f64"))
    assert np.all(XX[0, 1:] == 1.0) and abs(XX[1, 2] / U - 0.98) < 1e-9
    g = api.precomputed(_dev(X, "f64"), _dev(Y, "f64"), 0, 1, "ed", "f64")
    err = abs(g["statistic"] - oracle.threshold(XX, YY, XY))
    allowed = nx * (31 * d + 2 * U) * (2.0 / (nx * ny) + 1.0 / (nx * nx))
    assert err <= allowed, (err / U, allowed / U)
