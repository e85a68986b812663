"""FP32-eig iterations whose cliques of 33-128 vertices take the matrix sign
function (up to 48, and above wherever the decoupling does not carry them):
clique sizes at the edges of the padded sizes, odd ones between, long enough
for the first decoupling probe (iteration 64) and some iterations after it,
against the FP64 oracle.  Bar: each FP32 projection is accurate to ~1e-6
||W||_F and the iteration is nonexpansive, so N iterations differ by about
N * 1e-6 of the largest entry: 2e-4 for 70."""
import pytest

from test_gpu_admm_sign import arrow_with_blocks
from test_gpu_decouple import parity
from test_gpu_dual import compare_fixed_n_dual

pytestmark = pytest.mark.gpu

SIZES = {"to_48": [33, 40, 47, 48], "to_80": [49, 63, 64, 65, 79, 80],
         "to_128": [81, 96, 97, 112, 113, 127, 128]}


def instance(name):
    return arrow_with_blocks([s - 4 for s in SIZES[name]], 4, 60, seed=11)


@pytest.mark.parametrize("name", SIZES)
def test_primal(sdp, gpu, oracle_mod, name):
    parity(sdp, oracle_mod, [instance(name)], 70, "fp32", 2e-4)


@pytest.mark.parametrize("name", SIZES)
def test_dual(sdp, gpu, oracle_mod, name):
    compare_fixed_n_dual(sdp, oracle_mod, [instance(name)], 70, precision="fp32", tol_rel=2e-4)
