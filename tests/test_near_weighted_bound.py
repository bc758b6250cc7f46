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
    f = f3m.lib()._ZN3f3m19near_weighted_errorEdid   # double f3m::near_weighted_error(double E, int depth, double gamma)
    f.restype, f.argtypes = ctypes.c_double, [ctypes.c_double, ctypes.c_int, ctypes.c_double]
    return f


@pytest.mark.parametrize("depth,ratio", [(2, 0.166), (3, 0.3), (5, 0.1), (4, 0.5)])
def test_bound_covers_the_interpolation_error(bound, depth, ratio):
    E = 1.7
    l = E / 2.0 ** depth
    gamma = l / ratio
    c = (0.5 * l / gamma) ** 2
    t = np.linspace(-1.0, 1.0, 201)
    L = basis(t)
    terms = sum((5.0 / 3.0) ** k for k in range(6))
    b = bound(E, depth, gamma)
    e = np.exp(-0.5 * c * t * t)

    def smooth(x, y, o):                               # F of two boxes o cells apart, local coordinates, one dimension
        return np.exp(c * (x[:, None] * y[None, :] + 2.0 * o * (x[:, None] - y[None, :] - o)))

    exact = {o: e[:, None] * smooth(t, t, o) * e[None, :] for o in (0, 1)}
    d = t[:, None] - t[None, :] - 2.0 * 1
    assert np.allclose(exact[1], np.exp(-0.5 * c * d * d), rtol=1e-13)
    inter = {o: e[:, None] * (L @ smooth(NODES, NODES, o) @ L.T) * e[None, :] for o in (0, 1)}
    # one of the six interpolations: the bound's share covers it, and is no more than a third too large
    e1 = max(np.abs(e[:, None] * (L @ smooth(NODES, t, o) - smooth(t, t, o)) * e[None, :]).max() for o in (0, 1))
    assert e1 <= b / terms <= 1.35 * e1 * np.exp(2.0 * ratio * ratio)
    rng = np.random.default_rng(5)
    i, j = rng.integers(0, t.size, (2, 3, 200_000))
    for o in ((0, 0, 0), (1, 0, 0), (1, 1, 0), (1, 1, 1)):
        k, ki = (np.prod([m[o[d]][i[d], j[d]] for d in range(3)], axis=0) for m in (exact, inter))
        assert np.abs(ki - k).max() <= b


def test_where_the_bound_reaches_fp32_rounding(bound):
    assert bound(1.0, 3, 0.125 / 0.165) <= 2.0 ** -24 < bound(1.0, 3, 0.125 / 0.167)
