"""Algorithm 3's scalars formed by every wave (instances of up to 256 partial
sums of 64 coordinates or rows) and by a workgroup per instance (above): fixed-N
parity with the FP64 oracle at the edge, alone and beside smaller instances (the
bar of the other tests of the iteration)."""
import pytest

import sdpgen
from test_gpu_hsde import compare_fixed_n_hsde

pytestmark = pytest.mark.gpu


def partials(inst):
    return (inst.nnz + 63) // 64 + (inst.m + 63) // 64


def band(n):
    return sdpgen.sparse_rows_instance(n, sdpgen.banded_cliques(n, 7), 40, 20, seed=n)


@pytest.mark.parametrize("n,parts", [(2042, 256), (2044, 257), (6000, 751)])
def test_edge(sdp, gpu, oracle_mod, n, parts):
    inst = band(n)
    assert partials(inst) == parts
    compare_fixed_n_hsde(sdp, oracle_mod, [inst], 12)


def test_batch(sdp, gpu, oracle_mod):
    compare_fixed_n_hsde(sdp, oracle_mod,
                         [band(60), band(3000), sdpgen.block_arrow_instance(4, 5, 3, 15, seed=1)],
                         12)
