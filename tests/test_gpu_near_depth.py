"""Products whose near pairs are interpolated to within fp32 rounding (3-D, 4 nodes per dimension, wide kernels)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2202_01085_amd import f3m, inputs
from parity_util import TOL_F3M, assert_close, say

pytestmark = pytest.mark.gpu


# the bound 0.2395 (l^2 / (2 gamma^2))^2 <= 2^-24 holds from l <= 0.0316 gamma on: n, dist, gamma, zeta put that depth at
# the last depth, above it, at depth 2, and (the narrow kernels) nowhere
@pytest.mark.parametrize("n,dist,gamma,zeta", [
    (30_001, "uniform", 2.0, 12),    # l = 1/16 at depth 4 of 5
    (20_000, "uniform", 4.0, 128),   # l = 1/8 at depth 3 of 3
    (20_000, "uniform", 8.0, 64),    # depth 2
    (20_000, "uniform", 7.5, 64),    # depth 3
    (30_001, "uniform", 1.7, 12),    # l = 1/32 at depth 5 of 5
    (20_000, "uniform", 3.5, 128),   # nowhere: it would be depth 4 of 3
    (40_000, "normal", 60.0, 64),
    (20_000, "uniform", 1.0, 128),   # nowhere: exact near field
])
def test_interpolated_near_field(n, dist, gamma, zeta):
    say("near depth n=%d %s gamma=%g zeta=%d" % (n, dist, gamma, zeta))
    X = (inputs.points_uniform if dist == "uniform" else inputs.points_normal)(n, 3, 71)
    B = inputs.rhs_normal(3 * n, 72).view(3, n)
    g = float(np.float32(gamma))
    T = oracle.Tree(X.numpy(), theta=2.0, zeta=zeta)
    plan = f3m.Plan(X.to("cuda:0"), gamma, 4, 2.0, leaf_max=zeta)
    assert plan.info().depth == T.L
    want = np.stack([T.apply(B[j].numpy(), g, 4) for j in range(3)])
    Bd = B.to("cuda:0")
    y, Y = plan.kmvm(Bd[0]), plan.kmvm_multi(Bd)
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
