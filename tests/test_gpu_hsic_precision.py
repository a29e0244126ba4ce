"""What T1 = sum over i, j of K[i][j] L[pi_i][pi_j] of the HSIC test is held to, on data whose
kernel entries are known exactly: every coordinate, mean, norm and squared distance is exact in
each form's arithmetic, so the entries are those that api.blocks() gives for the same rows."""
import numpy as np
import pytest

from paper_2406_06488_amd import api
from tests.test_gpu_hsic import _dev

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


def _kernel(X, gamma, prec):
    """The kernel matrix of the rows of X as the library forms it, zero diagonal."""
    h = X.shape[0] // 2
    Xd = _dev(X, prec)
    kxx, kyy, kxy = (b.cpu().numpy() for b in api.blocks(Xd[:h], Xd[h:], "mmd", prec, gamma))
    K = np.block([[kxx, kxy], [kxy.T, kyy]])
    np.fill_diagonal(K, 0.0)
    return K


def test_products_far_below_one():
    """FP32 entries of 2^-124: their products (2^-248) keep every bit.  Rows +-e_m: squared
    distance 4 within a pair (the entry vanishes), 2 otherwise.  Bound: T1's lane chains and
    tree, and the row sums behind T2 and T3, take fewer than 40 and 80 roundings."""
    n, gamma, B, seed = 256, 43.0, 20, 5
    X = np.zeros((n, n // 2), dtype=np.float32)
    X[0::2] = np.eye(n // 2)
    X[1::2] = -np.eye(n // 2)
    K = _kernel(X, gamma, "f32")
    assert set(np.unique(K)) == {np.float32(0.0), K[0, 2]} and 2.0 ** -126 < K[0, 2] < 2.0 ** -120
    g = api.hsic(_dev(X, "f32"), _dev(X, "f32"), B, seed, gamma, gamma, "f32")
    got = np.append(g["perm_stats"].cpu().numpy(), g["statistic"])
    P = np.vstack([api.permutations(n, seed, 0, B).cpu().numpy(), np.arange(n)])
    Kl = K.astype(np.longdouble)  # exponents as far as 2^-16382
    r = Kl.sum(1)
    t2 = r.sum() ** 2 / ((n - 1) * (n - 2))
    for b in range(B + 1):
        t1 = (Kl * Kl[np.ix_(P[b], P[b])]).sum()
        t3 = 2 * (r @ r[P[b]]) / (n - 2)
        scale = float((t1 + t2 + t3) / (n * (n - 3)))
        err = abs(got[b] - float((t1 + t2 - t3) / (n * (n - 3)))) / scale
        assert err <= 200 * U, (b, err / U)
