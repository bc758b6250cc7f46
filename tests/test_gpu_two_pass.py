"""The two-pass permutation (2^21 points and more) moves data and nothing else: the bits of the plan that gathers and scatters
directly (the option route_min_points above the size, which leaves sizes below 2^21 and above 28 * 2^19 to the direct way)."""
import pytest
import torch

from paper_2202_01085_amd import f3m, inputs
from parity_util import say

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


# 8192 to a tile: the smallest, a last tile of one, full; 20480; 28672 and the largest.  Every point its own weight, and a
# kernel so narrow that a product is the right-hand side itself up to near neighbours: a misplaced value shows.
@pytest.mark.parametrize("n", [1 << 21, (1 << 21) + 1, 512 * 8192, 512 * 8192 + 1, 10_000_000, 512 * 20480 + 1, 512 * 28672])
def test_two_passes_put_every_value_in_its_place(n):
    say("two passes n=%d" % n)
    X = inputs.points_uniform(n, 3, 371, device=DEV)
    b = inputs.rhs_normal(n, 372, device=DEV)
    plan = f3m.Plan(X, 1e-6, 4, 2.0)
    y = plan.kmvm(b)
    # neighbours closer than a few 1e-6 are rare: all but a few rows are the right-hand side bit for bit
    same = (y == b).sum().item()
    assert same >= n - 2_000
    y2 = plan.kmvm(-b)
    assert torch.equal(y2, -y)
    plan.close()


def test_two_passes_equal_the_direct_way():
    """The same points with the two passes and as the targets of a plan whose sources go the direct way."""
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
