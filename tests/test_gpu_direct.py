"""The exact product at the edges of its kernel's tiles (16 or 32 targets per workgroup, source tiles of 1024 rows in
runs of 32) against fp64 sums formed with numpy."""
import numpy as np
import pytest
import torch

from paper_2202_01085_amd import f3m, inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("nx,ny,D", [(1, 1, 3), (15, 33, 1), (16, 1023, 2), (17, 1024, 3), (33, 1025, 4), (64, 5000, 5),
                                     (1000, 31, 6), (4097, 2049, 7), (65536, 1500, 3), (65537, 777, 2), (70001, 1056, 5)])
def test_direct_at_tile_edges(nx, ny, D):
    gamma = 0.4
    print("direct_kmvm_xy nx=%d ny=%d D=%d" % (nx, ny, D), flush=True)
    X = inputs.points_uniform(nx, D, 11, device=DEV)
    Y = inputs.points_normal(ny, D, 12, device=DEV)
    b = inputs.rhs_normal(ny, 13, device=DEV)
    y = f3m.direct_kmvm_xy(X, Y, b, gamma).cpu().numpy().astype(np.float64)
    rows = np.unique(np.concatenate([np.arange(min(nx, 40)), np.arange(max(0, nx - 40), nx),
                                     np.linspace(0, nx - 1, 60).astype(np.int64)]))
    Xr, Yh = X.cpu().numpy().astype(np.float64)[rows], Y.cpu().numpy().astype(np.float64)
    bh = b.cpu().numpy().astype(np.float64)
    g = float(np.float32(gamma))
    e = -((Xr[:, None, :] - Yh[None, :, :]) ** 2).sum(-1) / (2.0 * g * g)
    k = np.exp(e)
    want = k @ bh
    # fp32 rounding of the exponent: D + 3 operations, each 2^-24 of it; of the exponential (1 ulp) and the product;
    # of a running sum of 32 terms
    bound = 2.0 ** -24 * (((D + 3) * k * np.abs(e) + 35.0 * k) @ np.abs(bh)) + 1e-30
    assert np.all(np.abs(y[rows] - want) <= bound)
