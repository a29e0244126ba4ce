"""FP64 block stage at the edges of its 32 x 64 parts and 32-coordinate rounds: blocks, their
row / column sums (through the observed and the cross statistic) against long-double values."""
import numpy as np
import pytest

from paper_2406_06488_amd import api

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -53


def _dist(A, C):
    d = A.astype(np.longdouble)[:, None, :] - C.astype(np.longdouble)[None, :, :]
    return np.sqrt((d * d).sum(-1))


@pytest.mark.parametrize("nx,ny", [(1, 1), (31, 33), (64, 65), (97, 127), (129, 160), (200, 257)])
@pytest.mark.parametrize("p", [1, 15, 16, 17, 32, 33, 63, 100])
def test_blocks_and_sums(nx, ny, p):
    import torch
    g = np.random.Generator(np.random.PCG64(nx * 1000 + ny * 10 + p))
    X, Y = g.standard_normal((nx, p)), g.standard_normal((ny, p)) + 0.1
    tx, ty = torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda()
    want = _dist(X, X), _dist(Y, Y), _dist(X, Y)
    # d^2: a difference and an addition per coordinate, each half an ulp of a partial sum no
    # larger than the result; the square root halves the relative error and adds half an ulp
    tol = (2 * p + 4) * EPS
    for got, w in zip(api.blocks(tx, ty, "ed", "f64"), want):
        assert np.all(np.abs(got.cpu().numpy() - w) <= tol * w)
    # the statistic from FP64 sums of those blocks: entry errors, and one rounding for each of
    # the log-depth steps of the sums (under 64 on these sizes)
    sxx, syy, sxy = (float(w.mean()) for w in want)
    st = api.run(tx, ty, 0, 1, "ed", "f64", with_perm_stats=False)["statistic"]
    assert abs(st - float(2 * want[2].mean() - want[0].mean() - want[1].mean())) <= \
        (tol + 64 * EPS) * (2 * sxy + sxx + syy)
    if nx >= 2 and ny >= 2:
        hx, hy = nx // 2, ny // 2
        u = (want[2][:hx, hy:].mean() - want[0][:hx, hx:].mean()) - \
            (want[1][:hy, hy:].mean() - want[2][hx:, :hy].mean())
        c = api.cross(tx, ty, "ed", "f64")
        assert abs(c["statistic"] - float(u)) <= (tol + 64 * EPS) * (2 * sxy + sxx + syy + 4)


@pytest.mark.parametrize("nx,ny", [(1, 1), (15, 17), (33, 95), (128, 129), (260, 381)])
@pytest.mark.parametrize("B", [1, 255, 256, 700])
@pytest.mark.parametrize("kind", ["ed", "mmd"])
def test_resampling_edges(nx, ny, B, kind):
    """Centring and resampling at the edges of their 16-row blocks, 32-row strips and 256-split
    chunks, by the oracle's rules for the FP64 form."""
    import torch

    import oracle
    from tests.gpu_helpers import compare_run
    g = np.random.Generator(np.random.PCG64(nx + 7 * ny + B))
    X, Y = g.standard_normal((nx, 5)), g.standard_normal((ny, 5)) + 0.3
    got = api.run(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda(), B, 3, kind, "f64", 0.2)
    want = oracle.run_test(X, Y, B, 3, api.KINDS[kind], 0.2)
    compare_run(got, want, "f64")


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("nx,ny,B", [(1, 1, 1), (31, 33, 63), (129, 100, 64), (200, 260, 257)])
def test_precomputed_edges(nx, ny, B, dense, prec):
    """Per-split entry sums at the edges of 32-row strips and groups of 64 splits."""
    import torch

    import oracle
    from tests.gpu_helpers import compare_run
    g = np.random.Generator(np.random.PCG64(nx + 3 * ny + B))
    dt = np.float64 if prec == "f64" else np.float32
    X = g.standard_normal((nx, 5)).astype(dt)
    Y = (g.standard_normal((ny, 5)) + 0.3).astype(dt)
    got = api.precomputed(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda(), B, 3, "ed", prec,
                          dense=dense)
    compare_run(got, oracle.run_test(X.astype(np.float64), Y.astype(np.float64), B, 3), prec)
