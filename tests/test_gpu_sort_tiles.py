"""The order of the points is that of their keys, equal keys in the caller's order, with tiles of either size (8 x 256 keys below
2^20, 32 x 256 from there on) and at their edges."""
import numpy as np
import pytest

from paper_2202_01085_amd import f3m, inputs
from parity_util import say

pytestmark = pytest.mark.gpu


# one key and a tile more or less one; a whole round of tiles over the dies and one more; the last small tiles, the first large
@pytest.mark.parametrize("n", [2, 2_047, 2_048, 2_049, 8 * 2_048, 8 * 2_048 + 1, 100_003, (1 << 20) - 1, 1 << 20, (1 << 20) + 1])
@pytest.mark.parametrize("D", [2, 3])
def test_points_in_the_order_of_their_keys(n, D):
    say("sort n=%d D=%d" % (n, D))
    X = inputs.points_uniform(n, D, 421)
    X[: n // 2] = X[n - n // 2:].clone()      # pairs of equal points half the set apart, in tiles of their own
    X[n // 4: n // 4 + n // 8] = X[0]         # and a run of one key through many tiles
    plan = f3m.Plan(X.to("cuda:0"), 1.0, 4, 2.0)
    perm, keys = plan.perm().astype(np.int64), plan.point_keys().astype(np.int64)
    assert np.array_equal(np.sort(perm), np.arange(n))
    assert (np.diff(keys) >= 0).all() and (np.diff(perm)[np.diff(keys) == 0] > 0).all()
    plan.close()
