"""Box tables of all depths from one pass over the sorted keys: equal to the oracle's, bit for bit, at the edges of its blocks
(2048 points) and with runs of equal keys."""
import numpy as np
import pytest
import torch

import oracle
from paper_2202_01085_amd import f3m, inputs
from parity_util import say
from test_gpu_parity import check_plan_bit_exact

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def points(kind, n, D):
    X = inputs.points_uniform(n, D, 351)
    if kind == "equal":       # runs of hundreds of equal points: the tree goes down to the depth of the keys
        X = X[torch.arange(n) // 300 * 300].clone()
    elif kind == "two":       # two places only
        X = (torch.arange(n)[:, None] % 2).float().expand(n, D).clone()
    elif kind == "line":
        X[:, 1:] *= 1e-6
    return X.contiguous()


@pytest.mark.parametrize("kind,n,D,zeta,depth", [
    ("uniform", 129, 3, 128, 0), ("uniform", 128, 3, 128, 0), ("uniform", 2_048, 3, 8, 0), ("uniform", 2_049, 3, 9, 0),
    ("uniform", 4_097, 1, 1, 0), ("uniform", 6_143, 2, 7, 0), ("uniform", 10_000, 7, 16, 0), ("equal", 5_001, 3, 64, 0),
    ("equal", 3_001, 1, 16, 0), ("two", 2_500, 3, 128, 0), ("two", 2_500, 2, 2_000, 3), ("line", 9_000, 3, 1, 0),
    ("uniform", 9_000, 4, 3, 2),
])
def test_box_tables(kind, n, D, zeta, depth):
    say("bulk tables %s n=%d D=%d zeta=%d depth=%d" % (kind, n, D, zeta, depth))
    X = points(kind, n, D)
    T = oracle.Tree(X.numpy(), theta=2.0, zeta=zeta, max_depth=depth)
    plan = f3m.Plan(X.to(DEV), 1.0, 3 if D <= 4 else 2, 2.0, leaf_max=zeta, max_depth=depth)
    check_plan_bit_exact(plan, T)
    inf = plan.info()
    assert [int(inf.max_box[l]) for l in range(T.L + 1)] == [int(np.diff(T.boxes(l)[1].astype(np.int64)).max()) for l in range(T.L + 1)]
    plan.close()


def test_the_largest_set_that_takes_one_pass_and_the_next():
    """2^24 and 2^24 + 1 points: the tables of the pass over all depths against those made depth by depth."""
    n = (1 << 24) + 1
    X = inputs.points_normal(n, 3, 352, device=DEV)
    plans = [f3m.Plan(X[:m].contiguous(), 0.1, 4, 2.0) for m in (n - 1, n)]
    infos = [p.info() for p in plans]
    assert infos[0].depth == infos[1].depth
    for l in range(infos[0].depth + 1):
        (k0, s0), (k1, s1) = (p.boxes(l) for p in plans)
        # one point more: one box holds one more, or there is one box more
        assert abs(int(infos[1].nboxes[l]) - int(infos[0].nboxes[l])) <= 1
        if len(k0) == len(k1):
            d = np.diff(s1.astype(np.int64)) - np.diff(s0.astype(np.int64))
            assert np.array_equal(k0, k1) and d.sum() == 1 and (d >= 0).all()
    for p in plans:
        p.close()
