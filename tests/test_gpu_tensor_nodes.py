"""P2M and L2P of every number of dimensions and nodes per dimension (not 3-D with 4 nodes) against the two-set CPU F3M:
one division, most points of either set in one box, the sets two cubes apart, so that every pair is interpolated."""
import numpy as np
import pytest
import torch

import oracle
from paper_2202_01085_amd import f3m, inputs
from parity_util import assert_close, say

pytestmark = pytest.mark.gpu

SHAPES = [(D, p) for D in range(1, 8) for p in range(2, 9) if p ** D <= 4096 and (D, p) != (3, 4)]


def cluster(n, D, seed):
    """n points, all but one in the lowest box of depth 1; the last one at the far corner of the cube"""
    X = inputs.points_uniform(n, D, seed) * 0.45
    X[0], X[n - 1] = 0.0, 1.0
    return X


# points: one chunk of 256 that ends inside a step of 32 or 64, and two chunks; a lane, a group and a wavefront to spare
@pytest.mark.parametrize("nx,ny", [(70, 259), (257, 45)])
@pytest.mark.parametrize("D,p", SHAPES)
def test_node_weights_and_potentials(D, p, nx, ny):
    say("nodes D=%d p=%d nx=%d ny=%d" % (D, p, nx, ny))
    X, Y = cluster(nx, D, 311), cluster(ny, D, 312)
    Y[:, 0] += 2.5
    Y = Y.contiguous()
    # positive weights: with both signs the sum over this one cluster cancels to a few percent of its terms and less, and the
    # error is that of the terms over what is left (1.0e-5 at D = 4, p = 8).  Without cancellation: the rounding of
    # D basis values of either side, 2 D p 2^-24 (8e-6 at the most, as if all had one sign), a quarter of that.
    b = inputs.rhs_normal(ny, 313).abs()
    T = oracle.Tree2(X.numpy(), Y.numpy(), theta=2.0, zeta=16, max_depth=1)
    plan = f3m.Plan(X.to("cuda:0"), 1.5, p, 2.0, leaf_max=16, max_depth=1, Y=Y.to("cuda:0"))
    inf = plan.info()
    assert inf.depth == T.L == 1 and inf.near_pairs[1] == 0 and inf.far_pairs[1] == 4
    y = plan.kmvm(b.to("cuda:0"))
    torch.cuda.synchronize()
    assert_close(y.cpu().numpy(), T.apply(b.numpy(), float(np.float32(1.5)), p), 2e-6, "D=%d p=%d" % (D, p))
    plan.close()
