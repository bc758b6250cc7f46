"""The bound that decides where the near pairs are interpolated between weighted points, against the interpolation error itself
(host code of the library; no GPU needed)."""
import ctypes
import os

import numpy as np
import pytest

from paper_2202_01085_amd import build, f3m
from test_near_bound import NODES, basis


@pytest.fixture(scope="module")
def bound():
    if not os.path.exists(f3m.LIB_PATH):
        build.build_lib()
    f = f3m.lib()._ZN3f3m19near_weighted_errorEdidd   # double f3m::near_weighted_error(E, int depth, gamma, reach)
    f.restype, f.argtypes = ctypes.c_double, [ctypes.c_double, ctypes.c_int, ctypes.c_double, ctypes.c_double]
    return f


# reach: the largest offset of two near boxes in one dimension, in box edges: 1 for one set, the far ratio for two
@pytest.mark.parametrize("depth,ratio,reach", [(2, 0.166, 1.0), (3, 0.3, 1.0), (5, 0.1, 1.0), (4, 0.5, 1.0), (3, 0.128, 2.0), (4, 0.3, 2.0)])
def test_bound_covers_the_interpolation_error(bound, depth, ratio, reach):
    E = 1.7
    l = E / 2.0 ** depth
    gamma = l / ratio
    c = (0.5 * l / gamma) ** 2
    t = np.linspace(-1.0, 1.0, 201)
    L = basis(t)
    terms = sum((5.0 / 3.0) ** k for k in range(6))
    b = bound(E, depth, gamma, reach)
    e = np.exp(-0.5 * c * t * t)

    def smooth(x, y, o):                               # F of two boxes o cells apart, local coordinates, one dimension
        return np.exp(c * (x[:, None] * y[None, :] + 2.0 * o * (x[:, None] - y[None, :] - o)))

    exact = {o: e[:, None] * smooth(t, t, o) * e[None, :] for o in (0, reach)}
    d = t[:, None] - t[None, :] - 2.0 * reach
    assert np.allclose(exact[reach], np.exp(-0.5 * c * d * d), rtol=1e-13)
    inter = {o: e[:, None] * (L @ smooth(NODES, NODES, o) @ L.T) * e[None, :] for o in (0, reach)}
    # one of the six interpolations: the bound's share covers it, and is no more than a third too large
    e1 = max(np.abs(e[:, None] * (L @ smooth(NODES, t, o) - smooth(t, t, o)) * e[None, :]).max() for o in (0, reach))
    assert e1 <= b / terms <= 1.35 * e1 * np.exp((1.0 + reach) * ratio * ratio)
    rng = np.random.default_rng(5)
    i, j = rng.integers(0, t.size, (2, 3, 200_000))
    for o in ((0, 0, 0), (reach, 0, 0), (reach, reach, 0), (reach, reach, reach)):
        k, ki = (np.prod([m[o[d]][i[d], j[d]] for d in range(3)], axis=0) for m in (exact, inter))
        assert np.abs(ki - k).max() <= b


def test_where_the_bound_reaches_fp32_rounding(bound):
    assert bound(1.0, 3, 0.125 / 0.165, 1.0) <= 2.0 ** -24 < bound(1.0, 3, 0.125 / 0.167, 1.0)
    assert bound(1.0, 3, 0.125 / 0.128, 2.0) <= 2.0 ** -24 < bound(1.0, 3, 0.125 / 0.1295, 2.0)


def test_error_at_the_limit_is_far_below_rounding():
    """Where the bound has just reached 2^-24 the error itself (fp64): single pairs, and the sum over the 27 near boxes of
    evenly spread points with weights of one sign, where errors of one sign would add up."""
    c = (0.5 * 0.166) ** 2
    t = np.linspace(-1.0, 1.0, 81)
    L, e = basis(t), np.exp(-0.5 * c * t * t)
    exact, inter = {}, {}
    for o in (-1, 0, 1):
        f = np.exp(c * (NODES[:, None] * NODES[None, :] + 2.0 * o * (NODES[:, None] - NODES[None, :] - o)))
        exact[o] = np.exp(-0.5 * c * (t[:, None] - t[None, :] - 2.0 * o) ** 2)
        inter[o] = e[:, None] * (L @ f @ L.T) * e[None, :]
    rng = np.random.default_rng(6)
    i, j = rng.integers(0, t.size, (2, 3, 100_000))
    err = np.array([np.prod([inter[o[d]][i[d], j[d]] for d in range(3)], axis=0)
                    - np.prod([exact[o[d]][i[d], j[d]] for d in range(3)], axis=0) for o in np.ndindex(3, 3, 3) for o in [np.array(o) - 1]])
    assert np.abs(err).max() <= 2.0 ** -24 / 8 and np.sqrt((err ** 2).mean()) <= 2.0 ** -24 / 50
    s, a = (sum(m[o].mean(axis=1) for o in m) for m in (exact, inter))
    rel = np.einsum("i,j,k->ijk", a, a, a) / np.einsum("i,j,k->ijk", s, s, s) - 1.0
    assert np.abs(rel).max() <= 2.0 ** -24 / 30
