"""The decoupling past its first attempt (iteration 64; before it the sign
function projects every FP32 clique of 49 and more vertices): it carries most
projections once the iterates have settled, and where its certificate keeps
failing the sign function takes over again after the attempts of iterations 64
and 128.

Certified projections: those that neither took the sign function (counted) nor
swept (a sweep each at least), so projections - sign_fallbacks - jacobi_sweeps
of a window is a lower bound.  Parity with the FP64 oracle: each FP32 projection
is accurate to ~1e-6 ||W||_F and the iteration is nonexpansive, 2e-4 relative to
the largest entry for up to 200 iterations."""
import pytest

import sdpgen
from test_gpu_decouple import rel_err
from test_gpu_hsde import compare_fixed_n_hsde

pytestmark = pytest.mark.gpu

TOL = 2e-4


def blocks_of_64():
    return sdpgen.block_arrow_instance(3, 58, 6, 40, seed=5, density=1.0)


def blocks_of_112():
    return sdpgen.block_arrow_instance(20, 106, 6, 400, seed=8, density=0.02)


def blocks_of_128():
    return sdpgen.block_arrow_instance(24, 122, 6, 600, seed=9, density=0.01)


def window(S, n):
    a = S.stats()
    S.step(n)
    b = S.stats()
    return {k: b[k] - a[k] for k in a}


def matches(S, oracle_mod, inst, n):
    sol = S.solution(0)
    P = oracle_mod.Problem(inst)
    P.run(n, tol=0.0)
    return rel_err(sol["u"], P.u()) <= TOL and rel_err(sol["y_dual"], P.y_dual()) <= TOL


@pytest.mark.timeout(600)
@pytest.mark.parametrize("make,before,n", [(blocks_of_64, 150, 50), (blocks_of_112, 100, 15),
                                           (blocks_of_128, 100, 15)])
def test_most_projections_are_certified(sdp, gpu, oracle_mod, make, before, n):
    inst = make()
    with sdp.Solver([inst], tol=0.0, max_iter=10 ** 6, precision="fp32") as S:
        first = window(S, 64)
        assert first["sign_fallbacks"] == first["projections"]
        S.step(before - 64)
        w = window(S, n)
        assert w["projections"] - w["sign_fallbacks"] - w["jacobi_sweeps"] > 0.5 * w["projections"], w
        assert matches(S, oracle_mod, inst, before + n)


@pytest.mark.timeout(600)
def test_failing_certificates(sdp, gpu, oracle_mod):
    """The attempts of iterations 64 and 128 sweep, and the sign function takes
    most of the others."""
    inst = sdpgen.block_arrow_instance(12, 74, 6, 150, seed=4, density=0.05)
    with sdp.Solver([inst], tol=0.0, max_iter=10 ** 6, precision="fp32") as S:
        S.step(64)
        for n in (40, 56):
            w = window(S, n)
            assert w["jacobi_sweeps"] > 0 and w["sign_fallbacks"] > 0.5 * w["projections"], w
        assert matches(S, oracle_mod, inst, 160)


@pytest.mark.timeout(600)
def test_homogeneous(sdp, gpu, oracle_mod):
    compare_fixed_n_hsde(sdp, oracle_mod, [blocks_of_64()], 120, precision="fp32", tol_rel=TOL)
