"""Products whose near pairs are interpolated between weighted points (3-D, 4 nodes per dimension)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2202_01085_amd import f3m, inputs
from parity_util import TOL_F3M, assert_close, say

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def points(dist, n):
    if dist == "shell":       # boxes missing on one side of a parent, parents with one child
        X = inputs.points_uniform(n, 3, 321) - 0.5
        return (X / X.norm(dim=1, keepdim=True)).contiguous()
    return (inputs.points_uniform if dist == "uniform" else inputs.points_normal)(n, 3, 321)


# few leaf boxes: the last depth; from 8192 on: the first depth with l <= 0.166 gamma (box edge l), whose boxes then hold
# less than one, and more than one run of 256 points; narrow kernels: not at all (0)
@pytest.mark.parametrize("n,dist,gamma,zeta,depth", [
    (20_000, "uniform", 1.0, 128, 3),     # 64 parents, 39 points a box, one chunk each
    (3_001, "uniform", 2.0, 128, 2),      # 8 parents
    (40_001, "uniform", 0.4, 8, 4),       # depth 4 of 6
    (90_000, "normal", 3.5, 90, 4),       # depth 4 of 6, boxes of 1 to 890 points: up to four chunks
    (60_001, "shell", 0.9, 24, 4),        # depth 4 of 6
    (20_000, "uniform", 0.7, 128, 0),
])
def test_weighted_near_field(n, dist, gamma, zeta, depth):
    say("weighted near n=%d %s gamma=%g zeta=%d" % (n, dist, gamma, zeta))
    X = points(dist, n)
    B = inputs.rhs_normal(3 * n, 322).view(3, n)
    g = float(np.float32(gamma))
    T = oracle.Tree(X.numpy(), theta=2.0, zeta=zeta)
    want = T.apply(B[0].numpy(), g, 4)
    Bd = B.to(DEV)
    for overlap in (False, True):
        plan = f3m.Plan(X.to(DEV), gamma, 4, 2.0, leaf_max=zeta, overlap=overlap)
        assert plan.info().depth == T.L and plan.near_weighted() == depth and plan.product_info().near_depth == 0
        y = plan.kmvm(Bd[0])
        t = plan.stage_times()
        assert t["p2p"] > 0.0
        if depth:
            assert max(l for l in range(1, T.L + 1) if plan.level_times(l)[1] > 0.0) == depth
        Y = plan.kmvm_multi(Bd)
        torch.cuda.synchronize()
        assert_close(y.cpu().numpy(), want, TOL_F3M, "vs CPU F3M")
        assert_close(Y[0].cpu().numpy(), want, TOL_F3M, "column 0")
        for j in (1, 2):
            assert_close(Y[j].cpu().numpy(), plan.kmvm(Bd[j]).cpu().numpy(), 2e-6, "column %d" % j)
        # the solver keeps its vectors in box order
        lam = 0.1 * n
        x, it, _ = plan.cg_solve(Bd[0], lam, tol=1e-6, max_iter=20)
        res = plan.kmvm(x) + lam * x - Bd[0]
        assert float(res.norm() / Bd[0].norm()) <= 1e-5
        plan.close()


def test_weighted_near_field_of_one_large_box():
    """Node weights of a box with more than 2 x 512 chunks of 256 points are summed in two stages; two thirds
    of a cluster of 600 000 points lie in one box of depth 4, and two points far from it set the cube."""
    n = 600_001
    X = inputs.points_normal(n, 3, 323) * 0.02 + 0.40625
    X[0], X[n // 2] = 0.0, 1.0
    b = inputs.rhs_normal(n, 324).abs()
    Xd, bd = X.to(DEV), b.to(DEV)
    plan = f3m.Plan(Xd, 1.6, 4, 2.0, max_depth=4)
    inf = plan.info()
    assert plan.near_weighted() == 4 and inf.max_box[4] > 2 * 512 * 256
    y = plan.kmvm(bd)
    rows = torch.cat([torch.tensor([0, n // 2, n - 1]), inputs.sample_rows(n, 200, 325)]).to(DEV)
    want = f3m.direct_kmvm_rows_f64(Xd, bd, 1.6, rows).cpu().numpy()
    # all weights positive and every kernel value above 0.5: the error is that of the far pairs, boxes of edge 1/4 and less
    assert_close(y[rows].cpu().numpy(), want, TOL_F3M, "vs exact rows")
    plan.close()


@pytest.mark.parametrize("two", [False, True])
def test_no_bias_against_exact_near_sums(two):
    """Positive weights, so that rounding in one direction shows: the mean difference from the same products with exact near
    sums (which the small field of one point a pair, i.e. of none, asks for).  The fp32 basis is 3e-8 too large in each of the six
    applications, 1.8e-7, of which the near pairs, a quarter of the sum here, would pass on 4e-8; what remains are the roundings of the
    table's factors, some 2e-8 in any direction for one lengthscale, and less over five."""
    n = 3_000
    X, b = inputs.points_uniform(n, 3, 31, device=DEV), inputs.rhs_normal(n, 32, device=DEV).abs()
    more = dict(Y=inputs.points_uniform(n, 3, 33, device=DEV)) if two else {}
    mean = []
    for gamma in (2.0, 2.15, 2.3, 3.0, 4.0):
        plan, exact = f3m.Plan(X, gamma, 4, 2.0, **more), f3m.Plan(X, gamma, 4, 2.0, small_field=1, **more)
        assert plan.near_weighted() == plan.info().depth == exact.info().depth == 2 and exact.near_weighted() == 0
        y, y_exact = plan.kmvm(b).double(), exact.kmvm(b).double()
        mean.append(float(((y - y_exact) / y_exact).mean()))
        plan.close()
        exact.close()
    say("  mean differences " + " ".join("%.1e" % m for m in mean))
    assert abs(sum(mean) / len(mean)) <= 2e-8
