"""Sparse row products with several rows per wave (handles of 16384 and more
short rows): rows of 1 to 300 entries side by side, a row count that is no
multiple of the group, and a small instance behind a large one in the same
handle, against the oracle's conjugate-gradient iteration (the bar of the
other tests of that iteration)."""
import numpy as np
import pytest

import sdpgen
from test_gpu_cg import compare_cg

pytestmark = pytest.mark.gpu


def mixed_rows_instance(n, w, m, lengths, seed):
    rng = np.random.default_rng(seed)
    cliques = sdpgen.banded_cliques(n, w)
    pr, pc = sdpgen.pattern_from_cliques(n, cliques)
    ks = np.minimum(rng.choice(lengths, m), pr.shape[0])
    cols = [np.sort(rng.choice(pr.shape[0], k, replace=False)).astype(np.int32) for k in ks]
    ptr = np.concatenate([[0], np.cumsum(ks)]).astype(np.int64)
    return sdpgen._finish(n, m, pr, pc, list(cliques), sdpgen.A_CSR, rng.standard_normal(ptr[-1]),
                          ptr, np.concatenate(cols), rng.standard_normal(m),
                          f"mixed_rows_n{n}_m{m}", dict(seed=seed))


@pytest.mark.timeout(600)
@pytest.mark.parametrize("m", [16382, 16385, 16387])   # (one row a wave; four, with tails)
def test_mixed_row_lengths(sdp, gpu, oracle_mod, m):
    insts = [mixed_rows_instance(6000, 5, m, [1, 3, 62, 63, 64, 65, 127, 129, 300], seed=m),
             mixed_rows_instance(9, 2, 1, [7], seed=1)]
    compare_cg(sdp, oracle_mod, insts, 5, K=2, factor=False)
