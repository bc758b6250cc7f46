"""The rule for the depth that products end at and for the one-pass grouping of the points (host code of the library; no GPU
needed): the tables of the grouping have a place for every cell of the depth, so the keys of the points must stay below that."""
import ctypes
import os

import numpy as np
import pytest

import oracle
from paper_2202_01085_amd import build, f3m

PLACES = 512      # of the grouping's tables


@pytest.fixture(scope="module")
def rule():
    if not os.path.exists(f3m.LIB_PATH):
        build.build_lib()
    lib = f3m.lib()
    depths = lib._ZN3f3m14product_depthsEilbbbbiPiS0_Pb
    depths.restype = None
    depths.argtypes = [ctypes.c_int, ctypes.c_int64] + [ctypes.c_bool] * 4 + [ctypes.c_int] + [ctypes.POINTER(ctypes.c_int)] * 2 \
        + [ctypes.POINTER(ctypes.c_bool)]
    plain, weighted = lib._ZN3f3m17near_interp_errorEdid, lib._ZN3f3m19near_weighted_errorEdidd
    plain.restype = weighted.restype = ctypes.c_double
    plain.argtypes = [ctypes.c_double, ctypes.c_int, ctypes.c_double]
    weighted.argtypes = plain.argtypes + [ctypes.c_double]

    def run(L, nboxes, far, near_left, E, gamma):
        """As a plan of one set does it: nboxes and far by depth; returns near_depth, near_weighted, grouped."""
        ok = [weighted(E, l, gamma, 1.0) <= 2.0 ** -24 for l in range(L + 1)]
        may_group = any(weighted(E, l, gamma, 1.0) <= 2.0 ** -24 for l in (2, 3))
        nd, first = ctypes.c_int(0), 0
        for l in range(2, L + 1):
            if far[l] and nd.value == 0:
                if plain(E, l, gamma) <= 2.0 ** -24:
                    nd.value = l
                elif first == 0 and ok[l]:
                    first = l
        nw, grouped = ctypes.c_int(0), ctypes.c_bool(False)
        depths(L, nboxes[L], far[L], near_left, False, may_group, first, ctypes.byref(nd), ctypes.byref(nw), ctypes.byref(grouped))
        return nd.value, nw.value, grouped.value

    return run


def clusters(rng, n, centres, width):
    return np.asarray(centres)[rng.integers(0, len(centres), n)] + rng.uniform(0.0, width, (n, 3))


def point_sets():
    rng = np.random.default_rng(11)
    n = 6000
    line = np.repeat(rng.random((n, 1)), 3, axis=1)
    plane = rng.random((n, 3))
    plane[:, 2] = 0.25
    one = rng.uniform(0.45, 0.53, (n, 3))
    one[:2] = [[0.0] * 3, [1.0] * 3]      # a cluster and two outliers
    return {"uniform": rng.random((n, 3)), "line": line, "plane": plane, "outliers": one,
            "clusters": clusters(rng, n, [[0.0] * 3, [0.95] * 3], 0.05),
            "corner": clusters(rng, n, [[0.0] * 3, [0.9] * 3, [0.0, 0.0, 0.9]], 0.02)}


@pytest.mark.parametrize("name", ["uniform", "line", "plane", "outliers", "clusters", "corner"])
def test_keys_of_grouped_points_fit_the_tables(rule, name):
    X = point_sets()[name].astype(np.float32)
    T = oracle.Tree(X, theta=2.0, zeta=4)
    E, L = T.E, T.L
    nboxes = [T.nboxes(l) for l in range(L + 1)]
    keys = T.point_keys()
    far = [l > 0 and T.interactions(l, 1)[1].size > 0 for l in range(L + 1)]
    near_left = T.interactions(L, 0)[1].size > 0
    seen = set()
    for ratio in (0.5, 0.7, 0.76, 0.8, 1.0, 1.2, 1.5, 2.0, 2.5, 3.0, 5.0, 8.0, 20.0):
        nd, nw, grouped = rule(L, nboxes, far, near_left, E, ratio * E)
        last = nd or nw or L
        assert not (nd and nw)
        if grouped:
            cells = keys >> np.uint32(3 * (T.Lq - last))
            assert int(cells.max()) < PLACES, (name, ratio, last, nboxes[last])
        seen.add((last, grouped))
    if name in ("line", "plane", "clusters"):
        assert any(g for _, g in seen)                                     # grouped at a coarse depth
    if name in ("outliers", "clusters", "corner"):
        assert any(not g and l > 3 and nboxes[l] <= PLACES for l, g in seen)   # few boxes of a deep depth: not grouped
