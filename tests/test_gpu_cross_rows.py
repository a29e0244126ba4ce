"""The cross statistic's split of the x-side tiles over workgroups (16 workgroups, eight threads
per row, four column tiles each at a time; rows past 4096 are read again from memory): sizes past
each of those, against the FP64 oracle, with the cross tests' tolerances."""
import numpy as np
import pytest

import oracle
from paper_2406_06488_amd import api, inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("nx,ny", [(2100, 2030),   # 17 x-side tiles
                                   (300, 8900)])   # 36 tiles of 4600 rows on either side
def test_cross_rows_past_the_split(nx, ny, prec):
    dt = np.float64 if prec == "f64" else np.float32
    X, Y = inputs.gaussian_pair(nx, ny, 3, 7, mean_shift=0.1, dtype=dt)
    g = api.cross(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda(), "ed", prec)
    X, Y = X.astype(np.float64), Y.astype(np.float64)
    o = oracle.cross(X, Y, oracle.ED, 0.0)
    h = nx // 2
    tol = {"f64": 1e-12, "f32": 1e-5}[prec] * np.abs(oracle.block(X[:h], X[h:], oracle.ED, 0.0)).mean()
    assert abs(g["statistic"] - o["statistic"]) <= tol, (g, o)
    assert abs(g["sigma"] - o["sigma"]) <= tol, (g, o)
    dz = (tol + abs(o["z"]) * tol) / o["sigma"]
    assert abs(g["z"] - o["z"]) <= dz * 1.01 + 1e-12, (g, o)
