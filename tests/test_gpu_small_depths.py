"""Several small depths of the tensor in one M2L launch, and right-hand sides read and results written through the permutation."""
import pytest
import torch

import oracle
from paper_2202_01085_amd import f3m, inputs
from parity_util import TOL_F3M, assert_close, say

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


# one depth; two; all of them small; a last depth of 4096 boxes with small ones above (fewer than 1024 parents) and one of
# 32768 boxes, whose parents are too many to share a launch; chunks and pairs of chunks; exact and weighted near pairs
@pytest.mark.parametrize("n,D,gamma,zeta", [
    (257, 3, 1.0, 64), (2_051, 3, 1.0, 32), (9_001, 3, 3.0, 64), (60_001, 3, 0.3, 32), (120_007, 3, 0.6, 8), (120_007, 3, 0.1, 8),
    (70_003, 3, 0.05, 300)])
def test_depths_together(n, D, gamma, zeta):
    say("depths together n=%d gamma=%g zeta=%d" % (n, gamma, zeta))
    X = inputs.points_uniform(n, D, 401)
    b = inputs.rhs_normal(n, 402)
    T = oracle.Tree(X.numpy(), theta=2.0, zeta=zeta)
    want = T.apply(b.numpy(), gamma, 4)
    bd = b.to(DEV)
    got = []
    for overlap in (False, True):
        plan = f3m.Plan(X.to(DEV), gamma, 4, 2.0, leaf_max=zeta, overlap=overlap)
        y = plan.kmvm(bd)
        torch.cuda.synchronize()
        assert_close(y.cpu().numpy(), want, TOL_F3M, "vs CPU F3M")
        assert torch.equal(plan.kmvm(-bd), -y)   # nothing is left over from the product before
        got.append(y)
        plan.close()
    assert torch.equal(got[0], got[1])
