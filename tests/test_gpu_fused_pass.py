"""Both products with B = L^-1 A in one pass (dense instances of 20 MB and
more in a handle): fixed-N parity of Algorithms 1-3 with the FP64 oracle at
the edges of the plan (1e-8 relative to the largest entry, the bar of the two
separate passes: the sums are the same up to their order), and results that do
not depend on how the members of a cluster are scheduled.

Sizes: a member holds up to 4096 columns, so 3903, 4335 and 9480 coordinates
make clusters of one (ending in a partial member), two and three; the row
counts are odd, so the last group of eight rows is partial.
"""
import numpy as np
import pytest

import sdpgen
from test_gpu_admm import compare_fixed_n, rel_err
from test_gpu_dual import compare_fixed_n_dual
from test_gpu_hsde import compare_fixed_n_hsde

pytestmark = pytest.mark.gpu

FUSED_MIN_BYTES = 20 << 20


def members1():
    return sdpgen.block_arrow_instance(18, 16, 5, 801, seed=3)


def members2():
    return sdpgen.block_arrow_instance(20, 16, 5, 701, seed=4)


def members3():
    return sdpgen.banded_instance(600, 15, 301, seed=5)


@pytest.mark.parametrize("make,columns", [(members1, 3903), (members2, 4335), (members3, 9480)])
@pytest.mark.parametrize("chunk", [0, 5])
def test_primal_matches_oracle(sdp, gpu, oracle_mod, make, columns, chunk):
    inst = make()
    assert inst.nnz == columns and 8 * inst.m * inst.nnz >= FUSED_MIN_BYTES
    compare_fixed_n(sdp, oracle_mod, inst, 12, graph_chunk=chunk, rho=0.8)


def test_dual_and_homogeneous_match_oracle(sdp, gpu, oracle_mod):
    insts = [members2(), members3()]
    compare_fixed_n_dual(sdp, oracle_mod, insts, 12)
    compare_fixed_n_hsde(sdp, oracle_mod, insts, 12)


def test_uneven_batch_with_sparse_and_tiny_instances(sdp, gpu, oracle_mod):
    """Sparse instances beside the dense ones and dense ones of fewer rows
    than a group of eight: every one as the oracle has it."""
    insts = [sdpgen.block_arrow_instance(3, 5, 2, 1, seed=1),
             sdpgen.block_arrow_instance(6, 9, 4, 40, seed=2, density=0.2), members3(),
             sdpgen.block_arrow_instance(18, 16, 5, 7, seed=6)]
    n = 12
    with sdp.Solver(insts, tol=0.0, max_iter=1000) as S:
        S.step(n)
        sols = [S.solution(i) for i in range(len(insts))]
    for inst, sol in zip(insts, sols):
        P = oracle_mod.Problem(inst)
        P.run(n, tol=0.0)
        assert rel_err(sol["u"], P.u()) <= 1e-8, inst.name
        assert rel_err(sol["y_dual"], P.y_dual()) <= 1e-8, inst.name


def run(sdp, insts, n, stream=None):
    kw = {} if stream is None else dict(stream=stream.cuda_stream)
    with sdp.Solver(insts, tol=0.0, max_iter=10 ** 6, **kw) as S:
        S.step(n)
        return [S.solution(i)["u"] for i in range(len(insts))]


@pytest.mark.parametrize("copies", [4, 85, 128, 129])
def test_many_instances(sdp, gpu, oracle_mod, copies):
    """Copies of one instance of two members each: 4 and 85 (whose clusters
    leave units idle) and 128 (a workgroup per unit) take the fused pass, 129
    (more clusters than units, which would wait for members that have not
    started) the two separate passes.  Every copy comes out the same, and as the
    oracle has it."""
    inst = sdpgen.block_arrow_instance(20, 16, 5, 41, seed=7)
    assert 4096 < inst.nnz <= 8192
    if copies == 4:
        inst = members2()
    us = run(sdp, [inst] * copies, 10)
    for u in us[1:]:
        assert rel_err(u, us[0]) <= 1e-12
    P = oracle_mod.Problem(inst)
    P.run(10, tol=0.0)
    assert rel_err(us[0], P.u()) <= 1e-8


def test_two_streams_at_once_bitwise(sdp, gpu):
    """Two handles iterating at the same time compete for the units, so
    members wait for absent ones or compute their parts: the results are those
    of each handle alone, bit for bit."""
    import threading
    import torch
    sets = [[members2(), members3()], [members3(), members1()]]
    alone = [run(sdp, s, 300) for s in sets]
    out = [None, None]

    def work(i):
        out[i] = run(sdp, sets[i], 300, torch.cuda.Stream())

    ts = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for a, b in zip(alone, out):
        for x, y in zip(a, b):
            assert np.array_equal(x, y)
