"""The plan of the sign kernels that stop early (sdp_sign_plan, host only):
independently of the library's grid, every eigenvalue's scalar iterates meet the
bound it states, on a grid ten times finer, for the worst case and for every
entry of the stop table; and the iterates stay in the fast step's basin.

An eigenvalue delta starts at x_0 = c delta with c >= 1.25, so it is off by
delta |1 - s| / 2 <= x_0 |1 - s| / 2, and at most n - 1 eigenvalues sit at the worst
point.  2% for what lies between the points of the library's grid; 1.5e-16 is what
double-precision iterates resolve."""
import math

import numpy as np
import pytest

import paper_1707_05058_amd as sdp
from test_sign_schedule_cpu import fast

X_MAX, THETA = 1.25, 0.9
GRID = np.concatenate([np.logspace(-18, 0, 18 * 2560 + 1), np.linspace(0, X_MAX, 10241)[1:]])
CASES = [(t, n) for t in (0.5, 0.1, 1e-2, 1e-4, 4e-5, 1e-6, 1e-7, 1e-10, 1e-14, 1e-16)
         for n in (1, 2, 16, 32, 48, 64, 80, 96, 112, 128)]


def finish(x, j, n):
    c = 0.5 if n <= 32 else 0.9375
    b0, b1, b2 = ((1.002014, 0.523437, 0.325222) if j == 0
                  else (1.0, 0.5 + (c * 0.00338 ** 2 if j == 1 else 0.0), 0.375))
    r = 1.0 - x * x
    return x * (b0 + r * (b1 + r * b2))


def error(x, steps, n):
    for j in range(steps):
        x = finish(x, j, n)
    return GRID * np.abs(1.0 - x) / 2.0


@pytest.mark.parametrize("tol,n", CASES)
def test_worst_case_and_every_stop(tol, n):
    k1, k2, stop = sdp.sign_plan(tol, n)
    target = tol / (2.0 * math.sqrt(max(n - 1, 1)))
    assert k2 >= 1 and stop[0] == 0
    x = GRID.copy()
    for k in range(k1):
        near = np.abs(1.0 - x * x) <= THETA
        x = fast(x)
        assert x.max() <= X_MAX
        if k < len(stop) and stop[k] > 0:
            e = error(x, stop[k], n)[near].max()
            assert e <= 1.02 * max(target / 3, min(target, 1.5e-16)), (k, stop[k], e / target)
    assert error(x, k2, n).max() <= max(1.02 * target, 1.2e-16), (k1, k2)
    assert all(s == 0 for s in stop[k1:])


def test_defaults_have_a_stop_after_every_step():
    for tol, n in ((1e-6, 16), (1e-6, 128), (1e-14, 16), (1e-14, 128)):
        k1, _, stop = sdp.sign_plan(tol, n)
        assert all(1 <= s <= 3 for s in stop[1:k1])


def test_arguments():
    assert sdp.sign_plan(0.0, 16) == sdp.sign_plan(1e-16, 16)
    with pytest.raises(sdp.SdpError):
        sdp.sign_plan(1e-6, 0)
