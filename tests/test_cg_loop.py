"""The host's side of the conjugate-gradient loop, compiled by itself and run on made-up residuals: how many products a solve
launches, and how far it runs ahead of what it knows.  No GPU needed."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "cg_loop.h"
// residuals: of iteration k = 0, 1, ...; out: launched, looked at, most iterations under way, waits with nothing queued behind
extern "C" void run(const double *residuals, int max_iter, double limit, int *out) {
    int launched = 0, seen = 0, ahead = 0, idle = 0;
    f3m::cg_iterate(max_iter, 1.0, limit,
                    [&](int k) {
                        if (k != launched) ahead = 99;
                        ++launched;
                        if (launched - seen > ahead) ahead = launched - seen;
                    },
                    [&](int k, double *residual) {
                        if (k != seen || k >= launched) ahead = 99;
                        ++seen;
                        if (seen == launched) ++idle;
                        *residual = residuals[k];
                        return residuals[k] <= limit;
                    });
    out[0] = launched; out[1] = seen; out[2] = ahead; out[3] = idle;
}
"""


@pytest.fixture(scope="module")
def loop(tmp_path_factory):
    d = tmp_path_factory.mktemp("cg_loop")
    src, lib = d / "run.cpp", d / "run.so"
    src.write_text(SOURCE)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-I",
                           os.path.join(ROOT, "paper_2202_01085_amd", "csrc"), str(src), "-o", str(lib)])
    f = ctypes.CDLL(str(lib)).run
    f.restype = None
    f.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_double, ctypes.c_void_p]

    def run(residuals, max_iter, limit):
        r = np.ascontiguousarray(residuals, dtype=np.float64)
        assert r.size >= max_iter
        out = np.zeros(4, dtype=np.int32)
        f(r.ctypes.data, max_iter, limit, out.ctypes.data)
        return [int(v) for v in out]

    return run


def needed(r, max_iter, limit):
    hit = np.nonzero(np.asarray(r)[:max_iter] <= limit)[0]
    return int(hit[0]) + 1 if hit.size else max_iter


# steady decrease, slow to very fast; one that speeds up (as the spectrum is worked off), one that stalls, one that goes up and down
@pytest.mark.parametrize("name,r", [
    *[("rate %g" % q, q ** np.arange(1, 401)) for q in (0.97, 0.8, 0.5, 0.1, 0.01, 1e-7)],
    ("faster and faster", np.exp(-0.02 * np.arange(1, 401) ** 1.5)),
    ("stall", np.maximum(0.5 ** np.arange(1, 401), 3e-5)),
    ("up and down", 0.8 ** np.arange(1, 401) * (1.0 + 0.6 * np.cos(2.0 * np.arange(1, 401)))),
])
@pytest.mark.parametrize("tol", [0.5, 1e-2, 1e-4, 1e-6])
def test_no_product_for_nothing(loop, name, r, tol):
    for max_iter in (1, 2, 3, 17, 400):
        launched, seen, ahead, _ = loop(r, max_iter, tol)
        assert seen == launched == needed(r, max_iter, tol), (name, tol, max_iter)
        assert ahead <= 2


def test_a_fixed_number_of_iterations_never_waits(loop):
    for k in (1, 2, 5, 40):
        assert loop(0.5 ** np.arange(1, 41), k, 0.0) == [k, k, min(k, 2), 1]     # the only wait is for the last one
    assert loop([1.0], 0, 0.0) == [0, 0, 0, 0]


def test_far_from_the_tolerance_the_next_iteration_is_queued(loop):
    launched, seen, ahead, idle = loop(0.8 ** np.arange(1, 201), 200, 1e-6)
    assert launched == seen == 62 and ahead == 2
    assert idle <= 13     # the first, and the last factor of ten (ten iterations) and a little more


def test_a_jump_below_the_tolerance_costs_one_product(loop):
    r = np.concatenate([0.9 ** np.arange(1, 20), np.full(20, 1e-9)])     # eight digits at once: nothing foretells it
    launched, seen, _, _ = loop(r, 39, 1e-6)
    assert seen == 20 and launched == 21
