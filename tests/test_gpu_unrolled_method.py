"""The unrolled iterations run the eigensolver that projection_method names: u_T
is, bit for bit, what T cold-started iterations of the same plan give (no warm
start, no decoupling, the same kernels and data)."""
import numpy as np
import pytest

import sdpgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("s", [60, 76])
def test_two_level(sdp, gpu, precision, s):
    import torch
    inst = sdpgen.block_arrow_instance(3, s - 4, 4, 20, seed=s)
    T = 40
    with sdp.Solver([inst], rho=0.9, tol=0.0, max_iter=1000, precision=precision, autotune=0,
                    warm_start=0, decouple=0, projection_method="two_level") as S:
        assert all(sdp.projection_variant_two_level(int(precision == "fp32"), v)
                   for v in S.projection_plan_variants())
        S.step(T)
        want = S.solution(0)["u"]
        assert np.abs(S.solution(0)["X_packed"]).max() > 0
        u = torch.zeros(S.total_nnz, dtype=torch.float64, device="cuda")
        S.unrolled_forward(T, 8, u)
        assert np.array_equal(u.cpu().numpy(), want)
