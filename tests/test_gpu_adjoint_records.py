"""The reverse sweep with every iteration's eigenvectors kept (up to 4 GiB) and
with segments recomputed from checkpoints (beyond): one instance alone, whose
records fit, against 64 copies of it in one handle, whose records do not.

Bar: both compute the same iterates from the same data in FP64, apart from
the order of sums; the 1e-8 that 20 iterations are held to against the oracle,
times T / 20.
"""
import numpy as np
import pytest

import sdpgen
from test_gpu_adjoint import gpu_vjp, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(600)
def test_kept_and_recomputed_eigenvectors_agree(sdp, gpu):
    inst = sdpgen.block_arrow_instance(4, 88, 8, 12, seed=2, density=0.1)
    T, copies = 240, 64
    assert 8 * 4 * 96 ** 2 * T * copies > 4 << 30 > 8 * 4 * 96 ** 2 * T
    ubar = np.random.default_rng(5).standard_normal(inst.nnz)
    u1, c1, b1 = gpu_vjp(sdp, [inst], T, 20, 1.0, ubar)
    u2, c2, b2 = gpu_vjp(sdp, [inst] * copies, T, 20, 1.0, np.tile(ubar, copies))
    for x, y in ((u1, u2), (c1, c2), (b1, b2)):
        y = y.reshape(copies, -1)
        for k in (0, 1, copies - 1):
            assert rel_err(y[k], x) <= 1e-8 * T / 20, k
