"""The bound that decides at which depth the near pairs are interpolated, against the interpolation error itself (host code
of the library; no GPU needed)."""
import ctypes
import os

import numpy as np
import pytest

from paper_2202_01085_amd import build, f3m

NODES = np.array([1.0, 0.5, -0.5, -1.0])


@pytest.fixture(scope="module")
def bound():
    if not os.path.exists(f3m.LIB_PATH):
        build.build_lib()
    f = f3m.lib()._ZN3f3m17near_interp_errorEdid      # double f3m::near_interp_error(double E, int depth, double gamma)
    f.restype, f.argtypes = ctypes.c_double, [ctypes.c_double, ctypes.c_int, ctypes.c_double]
    return f


def basis(t):
    """Lagrange basis of the nodes at t: [points, 4]"""
    return np.stack([np.prod([(t - NODES[j]) / (NODES[i] - NODES[j]) for j in range(4) if j != i], axis=0)
                     for i in range(4)], axis=1)


@pytest.mark.parametrize("depth,q", [(2, 1e-3), (3, 1e-2), (5, 5e-4), (4, 5e-2)])
def test_bound_covers_the_interpolation_error(bound, depth, q):
    E = 1.7
    l = E / 2.0 ** depth
    gamma = l / np.sqrt(2.0 * q)                       # q = l^2 / (2 gamma^2)
    t = np.linspace(-1.0, 1.0, 201)
    L = basis(t)
    lebesgue = np.abs(L).sum(1).max()
    assert abs(lebesgue - 5.0 / 3.0) < 1e-3
    terms = sum((5.0 / 3.0) ** k for k in range(6))
    b = bound(E, depth, gamma)

    def kernel(x, y, o):                               # local coordinates in boxes o cells apart, one dimension
        return np.exp(-((x[:, None] - y[None, :]) * 0.5 * l - o * l) ** 2 / (2.0 * gamma * gamma))

    exact = {o: kernel(t, t, o) for o in (0, 1)}
    inter = {o: L @ kernel(NODES, NODES, o) @ L.T for o in (0, 1)}
    # one of the six interpolations: the bound's share covers it, and is no more than a tenth too large
    e1 = max(np.abs(L @ kernel(NODES, t, o) - exact[o]).max() for o in (0, 1))
    assert e1 <= b / terms <= 1.1 * e1 * (1.0 + 10.0 * q)
    # all six: random points of pairs of boxes up to one cell apart in every dimension
    rng = np.random.default_rng(5)
    i, j = rng.integers(0, t.size, (2, 3, 200_000))
    for o in ((0, 0, 0), (1, 0, 0), (1, 1, 0), (1, 1, 1)):
        k, ki = (np.prod([m[o[d]][i[d], j[d]] for d in range(3)], axis=0) for m in (exact, inter))
        assert np.abs(ki - k).max() <= b
