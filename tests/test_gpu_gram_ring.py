"""Gram kernels of small grids (half tiles up to 128 stored tiles, whole tiles up to 256) against
the one of large grids: each test alone, and in a batch whose grid is past both, must agree bit
for bit, at the edges of tiles, half tiles and operand stages."""
import numpy as np
import pytest

from paper_2406_06488_amd import api, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "bf16r"])
@pytest.mark.parametrize("kind", ["ed", "mmd"])
@pytest.mark.parametrize("p", [1, 32, 63, 64, 65, 129, 200, 448])
def test_alone_equals_large_grid(p, kind, prec):
    import torch
    sizes = [(1, 1), (64, 63), (65, 129), (300, 170), (1100, 900), (1500, 1400)]
    B = 40
    data, reqs, outs = [], [], []
    for t, (nx, ny) in enumerate(sizes):
        X, Y = inputs.gaussian_pair(nx, ny, p, seed=t + p, mean_shift=0.1)
        X[nx // 2], Y[0] = X[0], X[0]  # near pairs, within and across the samples
        data.append((torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda()))
        outs.append(torch.zeros(B, dtype=torch.float64, device="cuda"))
        reqs.append(api.make_request(*data[-1], B, t, kind, prec, 1.0 / p, outs[-1]))
    tiles = [(-(-nx // 128) + -(-ny // 128)) for nx, ny in sizes]
    assert sum(t * (t + 1) // 2 for t in tiles) > 256
    batch = api.batch(reqs)
    for t, (X, Y) in enumerate(data):
        alone = api.run(X, Y, B, t, kind, prec, 1.0 / p)
        for k in ("statistic", "threshold", "p_value", "count_ge", "n_refined"):
            assert alone[k] == batch[t][k], (sizes[t], k)
        assert np.array_equal(alone["perm_stats"].cpu().numpy(), outs[t].cpu().numpy()), sizes[t]


@pytest.mark.parametrize("prec", ["f32", "bf16r"])
@pytest.mark.parametrize("p", [64, 129])
def test_shared_blocks_equal_own_blocks_in_every_shape(p, prec):
    """An MMD test fed by the energy-distance test of the same samples, on grids of 6, 153, 276
    and 741 stored tiles (one per kernel shape), and all of them in one launch of more than 640:
    bit for bit the test that forms its own blocks."""
    import torch
    B = 30
    data, reqs, outs, own = [], [], [], []
    for t, (nx, ny) in enumerate([(65, 129), (1100, 900), (1500, 1400), (2500, 2300)]):
        X, Y = inputs.gaussian_pair(nx, ny, p, seed=t + p, mean_shift=0.1)
        X[nx // 2], Y[0] = X[0], X[0]
        X, Y = torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda()
        data.append((X, Y))  # the requests hold addresses only
        pair, po = [], []
        for kind in ("ed", "mmd"):
            own.append(api.run(X, Y, B, t, kind, prec, 1.0 / p))
            po.append(torch.zeros(B, dtype=torch.float64, device="cuda"))
            pair.append(api.make_request(X, Y, B, t, kind, prec, 1.0 / p, po[-1]))
        for r, o, w in zip(api.batch(pair), po, own[-2:]):
            assert r["statistic"] == w["statistic"] and r["n_refined"] == w["n_refined"], (nx, ny)
            assert np.array_equal(o.cpu().numpy(), w["perm_stats"].cpu().numpy()), (nx, ny)
            o.zero_()
        reqs += pair
        outs += po
    for r, o, w in zip(api.batch(reqs), outs, own):
        assert r["statistic"] == w["statistic"] and r["n_refined"] == w["n_refined"]
        assert np.array_equal(o.cpu().numpy(), w["perm_stats"].cpu().numpy())
