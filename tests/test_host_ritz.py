"""Lowest eigenvalue of the Lanczos tridiagonal matrix (host code, no GPU).

The stop rule follows it through the growing matrix (LowestRitz), the result
comes from a bisection of the last one (tridiag_lowest); both against LAPACK
and each other: random matrices, converging runs, and matrices whose bisection
meets a pivot of exactly zero (a constant diagonal).  Both stop at a bracket of
two rounding units; a pivot recurrence of m <= 60 rows is good to a few of |T|,
hence 1e-14 |T|.
"""
import ctypes
import os

import numpy as np
import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2105_06806_amd", "libedx.so")
pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libedx.so not built")
_D = ctypes.POINTER(ctypes.c_double)


@pytest.fixture(scope="module")
def solvers():
    lib = ctypes.CDLL(LIB)
    bisect = lib._ZN3edx14tridiag_lowestEPKdS1_ii
    bisect.restype, bisect.argtypes = ctypes.c_double, [_D, _D, ctypes.c_int, ctypes.c_int]
    follow = lib._ZN3edx10LowestRitz4nextEPKdS2_i
    follow.restype, follow.argtypes = ctypes.c_double, [ctypes.c_void_p, _D, _D, ctypes.c_int]
    return bisect, follow


def _matrices():
    rng = np.random.default_rng(5)
    for m in (2, 3, 5, 17, 60):
        for kind in range(5):
            a, b = rng.normal(size=m), np.abs(rng.normal(size=m)) + 0.1
            if kind == 1:
                a[:] = 0.0
            elif kind == 2:
                a[:], b[:] = -3.25, 0.5
            elif kind == 3:
                b *= 10.0 ** (-0.2 * np.arange(m))       # a converging run
            elif kind == 4:
                a[1::2] = a[0]
            yield a, b


def test_lowest_ritz_value(solvers):
    bisect, follow = solvers
    for a, b in _matrices():
        pa, pb = a.ctypes.data_as(_D), b.ctypes.data_as(_D)
        state = (ctypes.c_double * 16)()                   # a fresh LowestRitz
        for m in range(1, a.size + 1):
            t = np.diag(a[:m]) + np.diag(b[: m - 1], 1) + np.diag(b[: m - 1], -1)
            ev = np.linalg.eigvalsh(t)
            tol = 1e-14 * max(np.abs(ev).max(), 1e-300)
            assert abs(follow(state, pa, pb, m) - ev[0]) <= tol
            for k in range(m):
                assert abs(bisect(pa, pb, m, k) - ev[k]) <= tol, (m, k)


def test_followed_value_is_the_bisected_one(solvers):
    """To the last bit, after every row, so that a run which has converged sees
    the same value again (a stop rule with tol = 0 waits for that)."""
    bisect, follow = solvers
    rng = np.random.default_rng(8)
    settled = 0
    for trial in range(60):
        m = int(rng.integers(2, 120))
        a, b = rng.normal(size=m), np.abs(rng.normal(size=m)) + 0.2
        a[0] -= rng.choice([0.0, 4.0])        # a level that converges within a few rows
        a *= 10.0 ** rng.integers(-3, 4)
        b *= 10.0 ** rng.integers(-3, 1)
        pa, pb = a.ctypes.data_as(_D), b.ctypes.data_as(_D)
        state = (ctypes.c_double * 16)()
        last = None
        for k in range(1, m + 1):
            e = follow(state, pa, pb, k)
            assert e == bisect(pa, pb, k, 0)
            settled += e == last
            last = e
    assert settled > 1000
