"""The split iteration of a few large FP64 cliques finishes with as many
Newton-Schulz steps as sdp_sign_schedule gives: blocks whose small eigenvalues
all sit at the point that is worst for one step fewer.

Bound: the schedule keeps the exact iteration's Frobenius error within tol/2
||W||_F, which one step fewer exceeds by 44 and 48% at the first two; FP64 adds
no rounding at these tolerances."""
import numpy as np
import pytest

import sdpgen
from test_sign_schedule_cpu import worst_error

pytestmark = pytest.mark.gpu


def worst_block(rng, n, tol, schedule):
    k1, k2 = schedule(tol, n)
    _, d = worst_error(k1, k2 - 1)
    q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    small = d * rng.choice([-1.0, 1.0], n - 1)
    w = (q * np.concatenate([[np.sqrt(1.0 - np.sum(small ** 2))], small])) @ q.T
    return 0.5 * (w + w.T)


def positive_part(w):
    t, v = np.linalg.eigh(w)
    return (v * np.maximum(t, 0.0)) @ v.T


@pytest.mark.parametrize("n,tol", [(96, 4e-5), (96, 1e-2), (128, 0.1)])
def test_split_iteration(sdp, gpu, n, tol):
    """Algorithm 2's first z-update from v = z = 0 is P+(-lambda / rho)."""
    inst = sdpgen.block_arrow_instance(1, n - 8, 8, 5, seed=1)
    w = worst_block(np.random.default_rng(n), n, tol, sdp.sign_schedule)
    with sdp.Solver([inst], algorithm="dual", precision="fp64", tol=0.0, max_iter=10,
                    jacobi_tol=tol) as S:
        S.set_state(0, np.zeros(S.npk[0]), -sdp.pack_blocks([w]), 1.0)
        S.step(1)
        x = S.blocks(0)[0][0]
    err = np.linalg.norm(x - positive_part(w))
    assert err <= tol / 2 * (1 + 1e-9) * np.linalg.norm(w), err / tol
