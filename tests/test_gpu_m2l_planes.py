"""The candidate-grid M2L (3-D, 4 nodes per dimension) where planes and lines of its 6 x 6 x 6 grid are empty, and where
none is: the far field of every depth against the CPU F3M."""
import numpy as np
import pytest
import torch

import oracle
from paper_2202_01085_amd import f3m, inputs
from parity_util import TOL_F3M, assert_close, say

pytestmark = pytest.mark.gpu


def points(kind, n):
    X = inputs.points_uniform(n, 3, 301)
    if kind == "plane":       # one plane of boxes in z
        X[:, 2] *= 1e-4
    elif kind == "line":      # boxes along x only
        X[:, 1:] *= 1e-4
    elif kind == "diagonal":  # along the diagonal: at most two candidates of a line are there
        X = X[:, :1] + 0.01 * (X - 0.5)
    elif kind == "shell":     # a sphere's surface: candidates missing on one side of a parent
        X = X - 0.5
        X = X / X.norm(dim=1, keepdim=True)
    return X.contiguous()


# depths with fewer than 1024 parents take the kernel with one parent to a workgroup, the others the one with four, whose last
# workgroup is full only where their number is a multiple of four; the kinds leave planes, lines or single places empty
@pytest.mark.parametrize("kind,n,zeta,gamma", [
    ("uniform", 12_000, 20, 0.2), ("uniform", 24_001, 12, 0.1), ("plane", 40_000, 8, 0.05), ("line", 4_000, 2, 0.005),
    ("diagonal", 16_000, 8, 0.15), ("shell", 30_000, 16, 0.3), ("shell", 30_001, 4, 0.2),
])
def test_far_field_on_partly_empty_grids(kind, n, zeta, gamma):
    say("m2l planes %s n=%d" % (kind, n))
    X = points(kind, n)
    b = inputs.rhs_normal(n, 302)
    T = oracle.Tree(X.numpy(), theta=2.0, zeta=zeta)
    plan = f3m.Plan(X.to("cuda:0"), gamma, 4, 2.0, leaf_max=zeta)
    inf = plan.info()
    assert inf.depth == T.L >= 3
    parents = [int(v) for v in inf.nboxes[1:inf.depth]]   # of depths 2 .. L
    assert min(parents) < 1024 and (max(parents) >= 1024) == (kind != "line" and n != 12_000)
    say("  parents", parents)
    y = plan.kmvm(b.to("cuda:0"))
    torch.cuda.synchronize()
    assert_close(y.cpu().numpy(), T.apply(b.numpy(), float(np.float32(gamma)), 4), TOL_F3M, kind)
    plan.close()
