"""Sparse row products with several rows per wave, taken for rows of up to 64
entries on average: rows of 1 to 129 entries side by side, a row count that is no
multiple of the group, and a small instance behind a large one in the same
handle, at both sides of the average, against the oracle's conjugate-gradient
iteration (the bar of the other tests of that iteration)."""
import pytest

from test_gpu_cg import rel_err
from test_gpu_row_groups import mixed_rows_instance

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(600)
@pytest.mark.parametrize("m", [16384, 16385, 16387])
@pytest.mark.parametrize("lengths,short", [([1, 2, 3, 5, 62, 63, 64, 65, 127, 129], True),
                                           ([64, 65, 66], False)])
def test_mixed_row_lengths(sdp, gpu, oracle_mod, m, lengths, short):
    insts = [mixed_rows_instance(6000, 5, m, lengths, seed=m),
             mixed_rows_instance(9, 2, 1, [7], seed=1)]
    rows, nnz = m + 1, sum(int(i.a_rowptr[-1]) for i in insts)
    assert (nnz <= 64 * rows) == short
    n, K = 5, 2
    with sdp.Solver(insts, tol=0.0, max_iter=1000, cg_max_iter=K, cg_tol=0.0) as S:
        S.step(n)
        sols = [S.solution(i) for i in range(len(insts))]
    for inst, sol in zip(insts, sols):
        P = oracle_mod.Problem(inst, factor=False)
        P.set_affine_cg(K, 0.0)
        P.run(n, tol=0.0)
        assert rel_err(sol["u"], P.u()) <= 1e-8, inst.name
        assert rel_err(sol["y_dual"], P.y_dual()) <= 1e-8, inst.name
