"""P2M of 3-D boxes with 4 nodes per dimension: every remainder of the runs of 8, 16, 32 and 64 points, an odd number of boxes."""
import numpy as np
import pytest
import torch

import oracle
from paper_2202_01085_amd import f3m, inputs
from parity_util import assert_close, say

pytestmark = pytest.mark.gpu


# points of the boxes of depth 1: one run a box (two boxes to a wavefront; an odd number of them; a half without points), and
# boxes of several runs of 256
@pytest.mark.parametrize("counts", [
    [1, 2, 7, 8, 9, 15, 16, 17], [31, 32, 33, 1, 63, 64, 65, 24], [255, 1, 256, 40, 39, 41, 127], [129, 3, 96],
    [257, 1, 64, 65, 256, 300], [511, 512, 513, 16, 17, 1_100, 2, 5]])
def test_node_weights_of_boxes(counts):
    say("node weights %s" % counts)
    parts = []
    for i, c in enumerate(counts):
        corner = torch.tensor([i & 1, (i >> 1) & 1, i >> 2], dtype=torch.float32) * 0.5
        parts.append(inputs.points_uniform(c, 3, 411 + i) * 0.4 + corner)
    Y = torch.cat(parts)
    Y[0] = 0.0
    Y[:, 0] += 2.5
    Y = Y.contiguous()
    X = inputs.points_uniform(90, 3, 410)
    X[0], X[-1] = 0.0, 1.0
    # positive weights: the rounding of the 12 basis values and 3 products of either side, without cancellation (2e-6, as if
    # all 36 roundings of 2^-24 had one sign)
    b = inputs.rhs_normal(len(Y), 412).abs()
    T = oracle.Tree2(X.numpy(), Y.numpy(), theta=2.0, zeta=1, max_depth=1)
    plan = f3m.Plan(X.to("cuda:0"), 1.5, 4, 2.0, leaf_max=1, max_depth=1, Y=Y.to("cuda:0"))
    inf = plan.info()
    assert inf.depth == T.L == 1 and inf.near_pairs[1] == 0
    y = plan.kmvm(b.to("cuda:0"))
    torch.cuda.synchronize()
    assert_close(y.cpu().numpy(), T.apply(b.numpy(), float(np.float32(1.5)), 4), 2e-6, "counts %s" % counts)
    plan.close()
