"""The two-pass permutation (the default from 2^21 to 512 x 28 x 1024 points) moves data and nothing else: the bits of the plan that
gathers and scatters directly (the option route_min_points above the size) and of the one that takes three passes (below it)."""
import pytest
import torch

from paper_2202_01085_amd import f3m, inputs
from parity_util import say

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


DIRECT = 2 ** 31 - 1      # as route_min_points: no passes at any size


# 8192 values to a tile: the smallest, a last tile of one, full; 20480; 28672 and the largest.  The kernel couples neighbours, so
# a value, a point or a result in another's place changes the sums.
@pytest.mark.parametrize("n", [1 << 21, (1 << 21) + 1, 512 * 8192, 512 * 8192 + 1, 10_000_000, 512 * 20480 + 1, 512 * 28672])
def test_two_passes_equal_the_direct_way_at_every_tile(n):
    say("two passes n=%d" % n)
    X = inputs.points_uniform(n, 3, 371, device=DEV)
    b = inputs.rhs_normal(n, 372, device=DEV)
    y = {}
    for min_points in (0, DIRECT):
        plan = f3m.Plan(X, 0.02, 4, 2.0, route_min_points=min_points)
        y[min_points] = plan.kmvm(b)
        tables = plan.info().device_bytes
        plan.close()
        if min_points:
            assert with_passes - tables >= 12 * n       # the other plan has the tables and work vectors of two passes
        with_passes = tables
    assert torch.equal(y[0], y[DIRECT])
    rows = inputs.sample_rows(n, 200, 373).to(DEV)
    want = f3m.direct_kmvm_rows_f64(X, b, 0.02, rows)
    assert float((y[0][rows] - want).norm() / want.norm()) <= 1e-2       # the error of 4 nodes; a wrong place gives 1


def test_two_passes_equal_three():
    """Targets, sources, one set, several right-hand sides and the solver."""
    n, m = 2_200_001, 50_000
    X = inputs.points_uniform(n, 3, 373, device=DEV)
    Y = X[:: n // m][:m].contiguous()
    b = inputs.rhs_normal(m, 374, device=DEV)
    a = f3m.Plan(X, 0.03, 4, 2.0, Y=Y)                             # targets in two passes
    c = f3m.Plan(X, 0.03, 4, 2.0, Y=Y, route_min_points=2_000_000)  # ... in three
    assert torch.equal(a.kmvm(b), c.kmvm(b))
    w = inputs.rhs_normal(n, 375, device=DEV)
    a2 = f3m.Plan(Y, 0.03, 4, 2.0, Y=X)                            # sources in two passes
    c2 = f3m.Plan(Y, 0.03, 4, 2.0, Y=X, route_min_points=2_000_000)
    assert torch.equal(a2.kmvm(w), c2.kmvm(w))
    p, q = f3m.Plan(X, 0.03, 4, 2.0), f3m.Plan(X, 0.03, 4, 2.0, route_min_points=2_000_000)
    assert torch.equal(p.kmvm(w), q.kmvm(w))
    B = torch.stack([w, -w, 2 * w])
    assert torch.equal(p.kmvm_multi(B), q.kmvm_multi(B))
    x1, x2 = (k.cg_solve(w, 100.0, tol=0.0, max_iter=3)[0] for k in (p, q))
    assert torch.equal(x1, x2)
