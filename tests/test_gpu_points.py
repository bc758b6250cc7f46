"""The far field that goes from point to point (more than three dimensions, few points per box) against the CPU F3M."""
import numpy as np
import pytest
import torch

import oracle
from paper_2202_01085_amd import f3m, inputs
from parity_util import TOL_F3M, assert_close, say

pytestmark = pytest.mark.gpu


# n, D, dist, p, theta, zeta, eta_smooth, adaptive, rows compared: runs of targets above and below 16, a row of 359 near
# boxes (7-D, above the 256 taken at once), one source per box, a depth whose pairs are all interpolated, smaller ratios
@pytest.mark.parametrize("n,D,dist,p,theta,zeta,eta_smooth,adaptive,rows", [
    (2_001, 4, "uniform", 3, 2.0, 4, 0.0, False, 60),
    (3_000, 4, "normal", 2, 2.0, 2, 0.0, False, 100),
    (1_003, 5, "mixture", 3, 2.0, 8, 0.0, False, 40),
    (2_000, 5, "uniform", 2, 1.5, 4, 0.0, False, 100),
    (400, 6, "normal", 3, 2.0, 6, 0.0, False, 6),
    (2_001, 6, "uniform", 2, 1.0, 6, 0.0, False, 100),
    (40_000, 7, "uniform", 2, 2.0, 4, 0.0, False, 6),
    (150, 7, "mixture", 3, 2.0, 4, 0.0, False, 5),
    (17, 7, "uniform", 2, 2.0, 1, 0.0, False, 17),
    (1_500, 4, "uniform", 3, 2.0, 4, 0.15, False, 60),
    (1_000, 5, "uniform", 3, 2.0, 4, 0.1, True, 20),
])
def test_far_field_between_points(n, D, dist, p, theta, zeta, eta_smooth, adaptive, rows):
    say("points n=%d D=%d %s p=%d theta=%g zeta=%d eta_smooth=%g" % (n, D, dist, p, theta, zeta, eta_smooth))
    gamma = 0.9
    gen = {"uniform": inputs.points_uniform, "normal": inputs.points_normal, "mixture": inputs.points_mixture}[dist]
    X, b = gen(n, D, 60 + D), inputs.rhs_normal(n, 61)
    g = float(np.float32(gamma))
    T = oracle.Tree(X.numpy(), theta=theta, zeta=zeta, gamma=g, eta_smooth=float(np.float32(eta_smooth)))
    plan = f3m.Plan(X.to("cuda:0"), gamma, p, theta, leaf_max=zeta, eta_smooth=eta_smooth, adaptive_far=adaptive)
    assert plan.info().depth == T.L
    # the depths that go from point to point: point pairs of the near boxes one depth up against nodes and far pairs
    used, info = plan.product_info(), plan.info()
    for l in range(1, T.L + 1):
        size = np.diff(T.boxes(l - 1)[1].astype(np.int64))
        ptr, cols = T.interactions(l - 1, 0)
        near = np.add.reduceat(size[cols], ptr[:-1]) if cols.size else np.zeros(size.size, np.int64)
        pairs, far, r = int((near * size).sum()), T.interactions(l, 1)[1].size, int(info.level_nodes[l]) ** D
        pays = far > 0 and info.level_nodes[l] in (2, 3) and (1.0 if r > 512 else 0.5) * pairs <= far * r
        assert bool(used.far_points[l]) == pays, l
    assert any(used.far_points) and used.near_depth == 0
    y = plan.kmvm(b.to("cuda:0"))
    torch.cuda.synchronize()
    idx = np.arange(rows) * (n // rows)
    want = T.apply_rows(b.numpy(), g, p, idx, adaptive=adaptive)
    assert_close(y.cpu().numpy()[idx], want, TOL_F3M, "vs CPU F3M")
    for l in range(1, T.L + 1):
        if used.far_points[l]:
            p2m, m2l, l2p = plan.level_times(l)
            assert p2m == 0.0 and l2p == 0.0 and m2l > 0.0
    # the far rows are not kept at such a depth: they come out of the plan on request
    for l in range(1, T.L + 1):
        ptr, cols = plan.interactions(l, 1)
        optr, ocols = T.interactions(l, 1)
        assert np.array_equal(ptr.astype(np.int64), optr) and np.array_equal(cols.astype(np.int64), ocols)
    plan.close()
