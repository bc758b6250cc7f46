"""P2M and L2P by long runs (boxes of thousands of points, 3-D, 4 nodes per dimension) against the CPU F3M on sampled rows."""
import numpy as np
import pytest
import torch

import oracle
from paper_2202_01085_amd import f3m, inputs
from parity_util import TOL_F3M, assert_close, say

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


# 64 boxes of depth 2 with 2050 to 2300 points (runs of 2048 and a few more), with normal points of 1 to 20 000; every pair
# interpolated plainly, between weighted points, at a smooth depth 1 and 2, and not at all near (exact near field)
@pytest.mark.parametrize("n,dist,gamma,depth,more", [
    (140_001, "uniform", 8.0, 2, {}),
    (140_001, "uniform", 1.6, 2, {}),
    (140_001, "normal", 60.0, 2, {}),
    (131_072, "uniform", 0.7, 2, {}),
    (140_001, "uniform", 1.0, 1, dict(eta_smooth=0.5)),
    (140_001, "uniform", 0.7, 2, dict(eta_smooth=0.1)),
])
def test_long_runs(n, dist, gamma, depth, more):
    say("long runs n=%d %s gamma=%g %r" % (n, dist, gamma, more))
    X = (inputs.points_uniform if dist == "uniform" else inputs.points_normal)(n, 3, 331)
    b = inputs.rhs_normal(n, 332)
    g = float(np.float32(gamma))
    T = oracle.Tree(X.numpy(), theta=2.0, zeta=128, max_depth=2, gamma=g, **{k: float(np.float32(v)) for k, v in more.items()})
    plan = f3m.Plan(X.to(DEV), gamma, 4, 2.0, max_depth=2, **more)
    assert plan.info().depth == T.L == depth
    y = plan.kmvm(b.to(DEV))
    torch.cuda.synchronize()
    rows = inputs.sample_rows(n, 300, 333).numpy()
    assert_close(y.cpu().numpy()[rows], T.apply_rows(b.numpy(), g, 4, rows), TOL_F3M, "vs CPU F3M")
    plan.close()


def test_long_runs_summed_in_two_stages():
    """2.5 million points in one box of depth 2: more than 1024 runs.  Positive weights, wide kernel: the exact rows."""
    n = 2_500_001
    X = inputs.points_uniform(n, 3, 334, device=DEV) * 0.2
    X[0], X[n - 1] = 0.0, 1.0
    b = inputs.rhs_normal(n, 335, device=DEV).abs()
    plan = f3m.Plan(X, 1.6, 4, 2.0, max_depth=2)
    assert plan.info().max_box[2] > 1024 * 2048
    y = plan.kmvm(b)
    rows = torch.cat([torch.tensor([0, n - 1]), inputs.sample_rows(n, 100, 336)]).to(DEV)
    want = f3m.direct_kmvm_rows_f64(X, b, 1.6, rows)
    # only the two corner points are far pairs (2 of 2.5e6 terms); near pairs are exact to 2^-24
    assert_close(y[rows][2:].cpu().numpy(), want[2:].cpu().numpy(), 2e-6, "vs exact rows")
    plan.close()


def test_long_runs_add_no_more_rounding_than_short_ones():
    """Every point twice, with weights of opposite sign: the product is zero, and what comes out is the rounding of the sums of
    the node weights (the terms of a pair round alike).  Relative to the norm of the weights, rms over 48 right-hand sides of one
    smooth depth: 1.5e-9 with runs of 256 points, 4.8e-9 with 32 points to a lane and the lanes added in fp32, 1.2e-9 with 16 points
    to a lane and the rest in fp64.  48 random numbers of one spread give it to
    within a tenth."""
    h = 1 << 17
    X = inputs.points_uniform(h, 3, 337, device=DEV)
    X = torch.cat([X, X])
    B = inputs.rhs_normal(48 * h, 338, device=DEV).view(48, h)
    B = torch.cat([B, -B], dim=1).contiguous()
    plan = f3m.Plan(X, 1.0, 4, 2.0, eta_smooth=0.5)
    inf = plan.info()
    assert inf.depth == 1 and inf.near_pairs[1] == 0 and 2 * h // inf.nboxes[1] >= 2048      # long runs, every pair interpolated
    Y = plan.kmvm_multi(B)
    e = float((Y.double().pow(2).mean() / B.double().pow(2).sum(dim=1).mean()).sqrt())
    say("  rounding of node weights %.2e" % e)
    assert e <= 2.2e-9
    plan.close()
