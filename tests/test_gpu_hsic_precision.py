"""What T1 = sum over i, j of K[i][j] L[pi_i][pi_j] of the HSIC test is held to, on data whose
kernel entries are known exactly: every coordinate, mean, norm and squared distance is exact in
each form's arithmetic, so the entries are those that api.blocks() gives for the same rows."""
from fractions import Fraction

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


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n,chain", [(256, 1), (512, 2), (1024, 4), (2048, 4)])
def test_small_products_beside_a_large_one(n, chain, prec):
    """One pair of equal rows (K = 1) and k^2 just below half an ulp of 1 for every other
    product: added one by one to the large product, they would all vanish.  A lane adds `chain`
    products before a compensated step, so at most chain - 1 of them do, of 2 k^2 < 2^-52 each;
    beside them the partial sum's rounding (2^-52 at its size of 2) and those of the final
    formula (2^-52 + 2^-53 + 2^-52, and T2's and T3's of 2^-55)."""
    j = n - 56
    X = np.zeros((n, n - 1), dtype=np.float64 if prec == "f64" else np.float32)
    X[:j] = np.eye(n - 1)[:j]
    X[j] = X[0]
    X[j + 1:] = np.eye(n - 1)[j:]
    gamma = -0.25 * np.log(0.98 * U)
    K = _kernel(X, gamma, prec)
    k = Fraction(float(K[0, 1]))
    assert K[0, j] == 1.0 and len(np.unique(K)) == 3 and 0.97 < float(k * k) / U < 0.99
    g = api.hsic(_dev(X, prec), _dev(X, prec), 0, 1, gamma, gamma, prec)
    t1 = 2 + (n * (n - 1) - 2) * k * k
    r0, r = 1 + (n - 2) * k, (n - 1) * k  # row sums of the pair, of the others
    t2 = (2 * r0 + (n - 2) * r) ** 2 / ((n - 1) * (n - 2))
    t3 = 2 * (2 * r0 * r0 + (n - 2) * r * r) / (n - 2)
    err = abs(Fraction(g["statistic"]) * n * (n - 3) - (t1 + t2 - t3))
    allowed = 2 * U * (chain - 1) + 2 * U + 2 * U + U + 2 * U + U
    assert float(err) <= allowed, (float(err) / U, allowed / U)
