"""FP32-eig iterations of cliques of up to 32 vertices on both forms of the
one-wave sign kernels, that for up to 4096 cliques of 16 and that for more and
for blocks of 32, at the edges of the padded sizes and of the count, against the
FP64 oracle.  Bar: each FP32 projection is accurate to ~1e-6 ||W||_F and the
iteration is nonexpansive, so N iterations differ by about N * 1e-6 of the
largest entry: 2e-4 for 40."""
import pytest

import sdpgen
from test_gpu_admm_sign import arrow_with_blocks
from test_gpu_decouple import parity
from test_gpu_dual import compare_fixed_n_dual
from test_gpu_hsde import compare_fixed_n_hsde

pytestmark = pytest.mark.gpu


def mixed():
    return arrow_with_blocks([s - 1 for s in (2, 3, 15, 16, 17, 31, 32)], 1, 30, seed=12)


@pytest.mark.timeout(300)
@pytest.mark.parametrize("l,d", [(4096, 2), (4097, 2), (64, 15), (64, 16)])
def test_counts(sdp, gpu, oracle_mod, l, d):
    inst = sdpgen.block_arrow_instance(l, d, 1, 8, seed=d, density=0.01)
    parity(sdp, oracle_mod, [inst], 40, "fp32", 2e-4)


def test_sizes(sdp, gpu, oracle_mod):
    parity(sdp, oracle_mod, [mixed()], 40, "fp32", 2e-4)


def test_dual_and_homogeneous(sdp, gpu, oracle_mod):
    compare_fixed_n_dual(sdp, oracle_mod, [mixed()], 40, precision="fp32", tol_rel=2e-4)
    compare_fixed_n_hsde(sdp, oracle_mod, [mixed()], 40, precision="fp32", tol_rel=2e-4)
