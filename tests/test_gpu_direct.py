"""The exact products.  direct_kmvm at the edges of its kernels (64 targets a wavefront, or 16 or 32 targets a workgroup and
source tiles of 1024 rows; both in runs of 32) against fp64 sums formed with numpy;
direct_kmvm_xy_rows_f64 where its tiles (64, 128 or 256 rows, 256 sources), slices and exponentials end."""
import numpy as np
import pytest
import torch

from paper_2202_01085_amd import f3m, inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("nx,ny,D", [(1, 1, 3), (15, 33, 1), (16, 1023, 2), (17, 1024, 3), (33, 1025, 4), (64, 5000, 5),
                                     (1000, 31, 6), (4097, 2049, 7), (65536, 1500, 3), (65537, 777, 2), (70001, 1056, 5),
                                     # both sides of the rule for few sources: a lane per target, or tiles of sources
                                     (1, 129, 3), (17, 160, 7), (63, 128, 1), (65, 129, 2), (2_097_151, 400, 3),
                                     (2_097_151, 401, 1), (2_097_151, 700, 5), (2_097_151, 701, 7), (2_097_153, 1100, 2),
                                     (2_097_153, 1101, 3), (160_000, 200, 6), (159_999, 200, 4), (2_097_152, 3001, 4)])
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


def test_direct_with_few_sources_is_bound_by_its_targets():
    # 1e7 targets, ten sources: 160 MB in and out; a workgroup's share of a tile of sources for every few targets
    # (600 us) would be several times what the traffic takes (40 us; 250 us are 0.64 TB/s)
    X, Y = inputs.points_uniform(10_000_000, 3, 14, device=DEV), inputs.points_uniform(10, 3, 15, device=DEV)
    b, y = inputs.rhs_normal(10, 16, device=DEV), torch.empty(10_000_000, device=DEV)
    times = []
    for _ in range(8):
        t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0.record()
        f3m.direct_kmvm_xy(X, Y, b, 0.5, y=y)
        t1.record()
        t1.synchronize()
        times.append(t0.elapsed_time(t1))
    assert min(times) <= 0.25


@pytest.mark.parametrize("m,ny,D,gamma", [(1, 1, 3, 0.5), (63, 255, 1, 0.3), (65, 257, 2, 0.02), (256, 4095, 3, 0.4),
                                          (257, 8193, 4, 0.6), (2048, 3000, 7, 1.0), (2049, 12289, 3, 0.3)])
def test_fp64_rows_at_tile_edges(m, ny, D, gamma):
    print("direct_kmvm_xy_rows_f64 m=%d ny=%d D=%d gamma=%g" % (m, ny, D, gamma), flush=True)
    X = inputs.points_uniform(3000, D, 21, device=DEV)
    Y = inputs.points_normal(ny, D, 22, device=DEV)
    b = inputs.rhs_normal(ny, 23, device=DEV)
    rows = inputs.sample_rows(3000, m, 24).to(DEV)
    y = f3m.direct_kmvm_xy_rows_f64(X, Y, b, gamma, rows).cpu().numpy()
    at = np.unique(np.concatenate([np.arange(min(m, 30)), np.arange(max(0, m - 30), m)]))
    Xr = X[rows].cpu().numpy().astype(np.float64)[at]
    Yh, bh = Y.cpu().numpy().astype(np.float64), b.cpu().numpy().astype(np.float64)
    g = float(np.float32(gamma))
    e = -((Xr[:, None, :] - Yh[None, :, :]) ** 2).sum(-1) / (2.0 * g * g)
    k = np.exp(e)
    # fp64 rounding of the exponent on both sides, of the exponential and of the sum (ny / slices terms in a row, at
    # most 4096 + 64); denormal kernel values are exact to 2^-1074 each
    bound = 2.0 ** -53 * ((2 * (D + 3) * k * np.abs(e) + 4200.0 * k) @ np.abs(bh)) + 2.0 ** -1073 * ny * np.abs(bh).max()
    assert np.all(np.abs(y[at] - k @ bh) <= bound)


def test_fp64_rows_of_far_points_are_exactly_zero():
    # exponents far below the smallest fp64 number, and beyond what a 32-bit power of two can hold
    X = torch.tensor([[0.0, 0.0, 0.0], [1e18, 0.0, 0.0]], device=DEV)
    Y = torch.tensor([[50.0, 0.0, 0.0], [1e15, 1e15, 0.0]], device=DEV)
    y = f3m.direct_kmvm_xy_rows_f64(X, Y, torch.ones(2, device=DEV), 1e-3, torch.arange(2)).cpu().numpy()
    assert np.all(y == 0.0)


def test_fp64_rows_of_points_that_are_not_numbers():
    """A squared distance that is NaN makes the sum NaN, an infinite one contributes nothing, in every row kernel
    (64, 128 and 256 rows per workgroup) and through every entry point."""
    inf, nan = float("inf"), float("nan")
    bad_src = [[nan, 0.2, 0.3], [0.1, inf, 0.3], [0.1, 0.2, -inf]]
    bad_row = [[0.5, nan, 0.5], [0.5, inf, 0.5], [0.5, 0.5, -inf], [0.5, -inf, 0.5], [inf, inf, 0.5], [0.5, 0.5, inf]]
    bh = inputs.rhs_normal(5000, 33)
    for m in (40, 300, 3000):
        for last in range(len(bad_src) + 1):
            Yh = inputs.points_uniform(5000, 3, 31)
            for k in range(last):                     # in the first and the last tile and in the middle
                Yh[(0, 4999, 2500)[k]] = torch.tensor(bad_src[::-1][k])
            Xh = inputs.points_uniform(m, 3, 32)
            at = np.arange(len(bad_row)) * 6 + 1
            Xh[at] = torch.tensor(bad_row)
            rows = torch.arange(m, device=DEV)
            y = f3m.direct_kmvm_xy_rows_f64(Xh.to(DEV), Yh.to(DEV), bh.to(DEV), 0.3, rows)[:400].cpu().numpy()
            with np.errstate(invalid="ignore"):
                diff = Xh[:400].numpy().astype(np.float64)[:, None, :] - Yh.numpy().astype(np.float64)[None, :, :]
                g = float(np.float32(0.3))
                k = np.exp(-(diff ** 2).sum(-1) / (2.0 * g * g))
            want = np.where(np.isnan(k).any(1), np.nan, np.nan_to_num(k) @ bh.numpy().astype(np.float64))
            assert np.isnan(want[1]) and (last == 3) == bool(np.isnan(want[0])) and np.isnan(want[13]) == (last >= 1)
            assert np.array_equal(np.isnan(y), np.isnan(want))
            ok = ~np.isnan(want)
            assert np.allclose(y[ok], want[ok], rtol=1e-11, atol=1e-11)
    # one point set, and the entry point that allocates nothing
    X = inputs.points_uniform(5000, 3, 34)
    X[77, 2] = nan
    X, b, rows = X.to(DEV), bh.to(DEV), torch.arange(60, 90, device=DEV)
    y64 = torch.empty(30, dtype=torch.float64, device=DEV)
    f3m.direct_kmvm_rows_f64_static(X, b, 0.3, rows, y64)
    assert bool(torch.isnan(f3m.direct_kmvm_rows_f64(X, b, 0.3, rows)).all()) and bool(torch.isnan(y64).all())
    X[77, 2] = inf                                    # the row itself only
    f3m.direct_kmvm_rows_f64_static(X, b, 0.3, rows, y64)
    for v in (f3m.direct_kmvm_rows_f64(X, b, 0.3, rows), y64):
        assert torch.isnan(v).nonzero().flatten().tolist() == [17]
