"""Plans whose products end at a depth of at most 512 boxes group the points by those boxes in one pass; the option
route_min_points brings small inputs onto that path."""
import numpy as np
import pytest
import torch

import oracle
from paper_2202_01085_amd import f3m, inputs
from parity_util import TOL_F3M, assert_close, say

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def points(dist, n):
    return (inputs.points_uniform if dist == "uniform" else inputs.points_normal)(n, 3, 341)


# tiles of 32768: one that is nearly empty, full ones, a last one of one point; 64 and 512 boxes, unoccupied ones among
# them (normal points), 8 boxes of a smooth depth; the weighted depth although the plain one exists (gamma 3: depth 4)
@pytest.mark.parametrize("n,dist,gamma,zeta,more", [
    (3_000, "uniform", 1.0, 8, {}), (32_768, "uniform", 1.0, 64, {}), (65_537, "uniform", 1.6, 64, {}),
    (140_001, "normal", 8.0, 64, {}), (100_000, "uniform", 3.0, 16, {}), (50_000, "uniform", 1.0, 64, dict(eta_smooth=0.5)),
    (50_000, "normal", 6.0, 64, dict(eta_smooth=0.3, adaptive_far=True)),
])
def test_grouped_points(n, dist, gamma, zeta, more):
    say("grouped n=%d %s gamma=%g zeta=%d %r" % (n, dist, gamma, zeta, more))
    X = points(dist, n)
    b = inputs.rhs_normal(2 * n, 342).view(2, n)
    Xd, bd = X.to(DEV), b.to(DEV)
    ref = f3m.Plan(Xd, gamma, 4, 2.0, leaf_max=zeta, **more)
    plan = f3m.Plan(Xd, gamma, 4, 2.0, leaf_max=zeta, route_min_points=1, **more)
    # the tree that is reported does not change
    assert np.array_equal(plan.perm(), ref.perm()) and np.array_equal(plan.point_keys(), ref.point_keys())
    L = ref.info().depth
    assert plan.info().depth == L
    for l in range(L + 1):
        assert all(np.array_equal(p, q) for p, q in zip(plan.boxes(l), ref.boxes(l)))
        assert all(np.array_equal(p, q) for p, q in zip(plan.interactions(l, 0), ref.interactions(l, 0)))
    if not more:
        k = plan.near_weighted()
        assert k in (2, 3) and int(plan.info().nboxes[k]) <= 512
    y, y_ref = plan.kmvm(bd[0]), ref.kmvm(bd[0])
    torch.cuda.synchronize()
    # two plans that stop at different depths and add in another order: both within rounding of the CPU F3M's method
    assert_close(y.cpu().numpy(), y_ref.cpu().numpy(), 4e-6, "against the plan in box order")
    again = f3m.Plan(Xd, gamma, 4, 2.0, leaf_max=zeta, route_min_points=1, **more)
    assert torch.equal(again.kmvm(bd[0]), y)   # the order depends on the points only
    again.close()
    Y = plan.kmvm_multi(bd)
    assert torch.equal(Y[0], y) and torch.equal(Y[1], plan.kmvm(bd[1]))
    lam = 0.1 * n
    x, it, _ = plan.cg_solve(bd[0], lam, tol=1e-6, max_iter=20)
    res = plan.kmvm(x) + lam * x - bd[0]
    assert float(res.norm() / bd[0].norm()) <= 1e-5
    if n <= 32_768:
        T = oracle.Tree(X.numpy(), theta=2.0, zeta=zeta)
        assert_close(y.cpu().numpy(), T.apply(b[0].numpy(), float(np.float32(gamma)), 4), TOL_F3M, "vs CPU F3M")
    got = torch.empty_like(y)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        plan.kmvm(bd[0], y=got)
    for _ in range(3):
        got.zero_()
        graph.replay()
        plan.kmvm(bd[1])
        torch.cuda.synchronize()
        assert torch.equal(got, y)
    plan.close()
    ref.close()


def test_solve_to_a_tolerance_on_grouped_points():
    """The tree goes deeper than the depth the points are grouped by; the solver's vectors are in the grouped order."""
    n, gamma, lam = 40_000, 1.0, 4_000.0
    X, b = points("uniform", n).to(DEV), inputs.rhs_normal(n, 345, device=DEV)
    plan = f3m.Plan(X, gamma, 4, 2.0, leaf_max=16, route_min_points=1)
    ref = f3m.Plan(X, gamma, 4, 2.0, leaf_max=16, route_min_points=n + 1)
    assert 0 < plan.near_weighted() <= 3 < plan.info().depth
    (x, it, h), (x_ref, it_ref, h_ref) = (p.cg_solve(b, lam, tol=1e-4, max_iter=200) for p in (plan, ref))
    say("  %d and %d iterations" % (it, it_ref))
    assert it < 200 and abs(it - it_ref) <= 1 and h[-1] <= 1e-4 and (h[:-1] > 1e-4).all() and len(h) == it + 1
    # both solve their system to 1e-4 of |b|, and the smallest eigenvalue is lam
    assert float((x - x_ref).norm()) <= 2e-4 * float(b.norm()) / lam
    res = plan.kmvm(x) + lam * x - b
    assert float(res.norm() / b.norm()) <= 1.1e-4
    plan.close()
    ref.close()


def thin_points(name, n):
    """Point sets with few occupied boxes at deep depths: the keys there go beyond the 512 cells of depth 3."""
    rng = np.random.default_rng(343)
    X = rng.random((n, 3))
    if name == "line":
        X[:, 1] = X[:, 2] = X[:, 0]
    elif name == "plane":
        X[:, 2] = 0.25
    elif name == "outliers":        # one cluster and two points far away: no far pairs at the depths down to the cluster
        X = 0.45 + 0.08 * X
        X[0], X[1] = 0.0, 1.0
    else:                           # tight clusters in corners
        X = 0.02 * X + np.array([[0.0, 0.0, 0.0], [0.9, 0.9, 0.9], [0.0, 0.0, 0.9]])[rng.integers(0, 3, n)]
    return torch.from_numpy(X.astype(np.float32))


@pytest.mark.parametrize("name", ["line", "plane", "outliers", "corners"])
@pytest.mark.parametrize("gamma", [0.5, 0.8, 1.0, 2.0, 3.0, 8.0])
def test_few_boxes_of_a_deep_depth(name, gamma):
    n = 9_000
    say("thin points %s gamma=%g" % (name, gamma))
    X, b = thin_points(name, n), inputs.rhs_normal(n, 344)
    ref = f3m.Plan(X.to(DEV), gamma, 4, 2.0, leaf_max=8, route_min_points=n + 1)
    plan = f3m.Plan(X.to(DEV), gamma, 4, 2.0, leaf_max=8, route_min_points=1)
    say("  depth %d, products end at: plain %d, weighted %d" % (plan.info().depth, plan.product_info().near_depth, plan.near_weighted()))
    T = oracle.Tree(X.numpy(), theta=2.0, zeta=8)
    want = T.apply(b.numpy(), float(np.float32(gamma)), 4)
    y = plan.kmvm(b.to(DEV))
    torch.cuda.synchronize()
    assert_close(y.cpu().numpy(), want, TOL_F3M, "vs CPU F3M")
    assert_close(ref.kmvm(b.to(DEV)).cpu().numpy(), want, TOL_F3M, "the ungrouped plan")
    assert np.array_equal(plan.perm(), ref.perm())
    plan.close()
    ref.close()
