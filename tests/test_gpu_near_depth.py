"""Products whose near pairs are interpolated to within fp32 rounding (3-D, 4 nodes per dimension, wide kernels)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2202_01085_amd import f3m, inputs
from parity_util import TOL_F3M, assert_close, say

pytestmark = pytest.mark.gpu


# the bound 0.2395 (l^2 / (2 gamma^2))^2 <= 2^-24 holds from l <= 0.0316 gamma on: n, dist, gamma, zeta put that depth at
# the last depth, above it, at depth 2, and (the narrow kernels: 0) nowhere
@pytest.mark.parametrize("n,dist,gamma,zeta,depth", [
    (30_001, "uniform", 2.0, 12, 4),     # l = 1/16 at depth 4 of 5
    (20_000, "uniform", 4.0, 128, 3),    # l = 1/8 at depth 3 of 3
    (20_000, "uniform", 8.0, 64, 2),
    (20_000, "uniform", 7.5, 64, 3),
    (30_001, "uniform", 1.7, 12, 5),     # l = 1/32 at depth 5 of 5
    (20_000, "uniform", 3.5, 128, 0),    # it would be depth 4 of 3
    (40_000, "normal", 60.0, 64, 3),
    (20_000, "uniform", 1.0, 128, 0),
])
def test_interpolated_near_field(n, dist, gamma, zeta, depth):
    say("near depth n=%d %s gamma=%g zeta=%d" % (n, dist, gamma, zeta))
    X = (inputs.points_uniform if dist == "uniform" else inputs.points_normal)(n, 3, 71)
    B = inputs.rhs_normal(3 * n, 72).view(3, n)
    g = float(np.float32(gamma))
    T = oracle.Tree(X.numpy(), theta=2.0, zeta=zeta)
    plan = f3m.Plan(X.to("cuda:0"), gamma, 4, 2.0, leaf_max=zeta)
    assert plan.info().depth == T.L
    assert plan.product_info().near_depth == depth and not any(plan.product_info().far_points)
    want = np.stack([T.apply(B[j].numpy(), g, 4) for j in range(3)])
    Bd = B.to("cuda:0")
    y = plan.kmvm(Bd[0])
    t = plan.stage_times()
    assert (t["p2p"] == 0.0) == (depth > 0)
    worked = [l for l in range(1, T.L + 1) if plan.level_times(l)[1] > 0.0]
    assert max(worked) == (depth or T.L)
    Y = plan.kmvm_multi(Bd)
    torch.cuda.synchronize()
    assert_close(y.cpu().numpy(), want[0], TOL_F3M, "vs CPU F3M")
    for j in range(3):
        assert_close(Y[j].cpu().numpy(), want[j], TOL_F3M, "column %d" % j)
    lists = [plan.interactions(T.L, kind)[1].size for kind in (0, 1)]
    assert lists == [T.interactions(T.L, kind)[1].size for kind in (0, 1)]
    # the solver keeps its vectors in box order
    lam = 0.1 * n
    x, it, _ = plan.cg_solve(Bd[0], lam, tol=1e-6, max_iter=20)
    res = plan.kmvm(x) + lam * x - Bd[0]
    assert float(res.norm() / Bd[0].norm()) <= 1e-5
    plan.close()


def test_interpolated_near_field_of_one_large_box():
    """Node weights of a box with more than 2 x 512 chunks of 256 points are summed in two stages; a cluster of 600 000
    points lies in one box of depth 2, and two points far from it set the cube."""
    n = 600_001
    X = inputs.points_normal(n, 3, 73) * 0.02 + 0.375
    X[0], X[n // 2] = 0.0, 1.0
    b = inputs.rhs_normal(n, 74).abs()
    Xd, bd = X.to("cuda:0"), b.to("cuda:0")
    plan = f3m.Plan(Xd, 8.0, 4, 2.0)
    inf = plan.info()
    assert plan.product_info().near_depth == 2 and inf.max_box[2] > 2 * 512 * 256
    y = plan.kmvm(bd)
    rows = torch.cat([torch.tensor([0, n // 2, n - 1]), inputs.sample_rows(n, 200, 75)]).to("cuda:0")
    want = f3m.direct_kmvm_rows_f64(Xd, bd, 8.0, rows).cpu().numpy()
    # all weights positive and every kernel value above 0.95: the truncation is at most 2^-24 of the sum
    assert_close(y[rows].cpu().numpy(), want, TOL_F3M, "vs exact rows")
    plan.close()
