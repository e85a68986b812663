"""Sparse row products with several rows per wave (handles of 16384 and more
short rows): rows of 1 to 300 entries side by side, a row count that is no
multiple of the group, and a small instance behind a large one in the same
handle, against the oracle's conjugate-gradient iteration (the bar of the
other tests of that iteration)."""
import numpy as np
import pytest

import sdpgen
from test_gpu_cg import rel_err

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
    n, K = 5, 2
    with sdp.Solver(insts, tol=0.0, max_iter=1000, cg_max_iter=K, cg_tol=0.0) as S:
        S.step(n)
        sols = [S.solution(i) for i in range(len(insts))]
        hists = [S.history(i) for i in range(len(insts))]
        steps = S.cg_steps()
    for inst, sol, (hc, hl, _) in zip(insts, sols, hists):
        P = oracle_mod.Problem(inst, factor=False)
        P.set_affine_cg(K, 0.0)
        r = P.run(n, tol=0.0)
        Xo, Lo = P.blocks()
        errs = dict(u=rel_err(sol["u"], P.u()), y=rel_err(sol["y_dual"], P.y_dual()),
                    X=rel_err(sol["X_packed"], sdp.pack_blocks(Xo)),
                    L=rel_err(sol["L_packed"], sdp.pack_blocks(Lo)),
                    eps_c=rel_err(hc, r.hist_eps_c), eps_l=rel_err(hl, r.hist_eps_l))
        for k, v in errs.items():
            assert v <= 1e-8, (inst.name, k, v)
    # the instance of one row is solved by its first step, and takes the second
    # only where the residual does not round to zero
    assert n * K <= steps <= 2 * n * K
