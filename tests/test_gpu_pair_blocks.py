"""The paired near field (two sibling boxes per wavefront, their targets packed into as few column blocks as hold them)
against the kernel that takes the boxes one at a time, which the products with several right-hand sides use."""
import pytest
import torch

from paper_2202_01085_amd import f3m, inputs
from parity_util import say

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


# mean points per leaf box of 32^3: one block for two boxes, two for three, three for four, every tile full, more than
# one tile per box; normal points mix all of them.  Two fp32 sums of some 1000 terms in another order: 2e-6.
@pytest.mark.parametrize("n,dist", [(400_000, "uniform"), (655_361, "uniform"), (1_000_003, "uniform"),
                                    (1_250_000, "uniform"), (1_600_001, "uniform"), (2_097_152, "uniform"),
                                    (2_000_000, "normal")])
def test_packed_pairs_equal_single_tiles(n, dist):
    say("pair blocks n=%d %s" % (n, dist))
    X = (inputs.points_uniform if dist == "uniform" else inputs.points_normal)(n, 3, 51, device=DEV)
    B = inputs.rhs_normal(2 * n, 52, device=DEV).view(2, n)
    plan = f3m.Plan(X, 0.05 if dist == "uniform" else 0.3, 4, 2.0, leaf_max=128)
    assert int(plan.info().nboxes[plan.info().depth]) >= 8192
    Y = plan.kmvm_multi(B)
    for j in range(2):
        y = plan.kmvm(B[j])
        diff = (y - Y[j]).double()
        assert float(diff.norm() / Y[j].double().norm()) <= 2e-6
        assert float(diff.abs().max() / Y[j].abs().max()) <= 8e-6
    plan.close()
