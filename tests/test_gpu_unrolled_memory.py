"""What the unrolled forward keeps for the reverse sweep
(sdp_set_unrolled_records): every iteration's eigenvectors, or checkpoints from
which segments are recomputed, also where the device has no room for the
records.  Both against the oracle (FP64, 1e-8 relative to the largest entry)
and against each other (the recomputed iterates and records are the same
numbers, so every bit agrees)."""
import numpy as np
import pytest

import sdpgen
from test_gpu_adjoint import oracle_vjp, rel_err
from test_gpu_setup_memory import fill_device

pytestmark = pytest.mark.gpu


def run(sdp, insts, T, ckpt, ubar, precision, records=None):
    import torch
    with sdp.Solver(insts, rho=0.9, tol=0.0, max_iter=10 ** 6, precision=precision) as S:
        if records is not None:
            S.set_unrolled_records(records)
        u = torch.zeros(S.total_nnz, dtype=torch.float64, device="cuda")
        cb, bb = torch.zeros_like(u), torch.zeros(S.total_m, dtype=torch.float64, device="cuda")
        free = torch.cuda.mem_get_info()[0]
        S.unrolled_forward(T, ckpt, u)
        S.vjp(torch.from_numpy(ubar).cuda(), cb, bb)
        held = free - torch.cuda.mem_get_info()[0]
        return [x.cpu().numpy() for x in (u, cb, bb)], held


@pytest.mark.parametrize("T,ckpt", [(1, 1), (13, 5), (20, 20), (7, 9)])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_kept_and_recomputed(sdp, gpu, oracle_mod, T, ckpt, precision):
    insts = [sdpgen.block_arrow_instance(4, 5, 3, 15, seed=1),
             sdpgen.block_arrow_instance(2, 30, 4, 12, seed=2)]
    ubar = np.random.default_rng(1000 + T).standard_normal(sum(i.nnz for i in insts))
    kept, _ = run(sdp, insts, T, ckpt, ubar, precision)
    recomputed, _ = run(sdp, insts, T, ckpt, ubar, precision, records=0)
    for x, y in zip(kept, recomputed):
        assert np.array_equal(x, y)
    if precision == "fp64":
        for x, y in zip(kept, oracle_vjp(oracle_mod, insts, T, 0.9, ubar)):
            assert rel_err(x, y) <= 1e-8


def test_checkpoints_bound_the_memory(sdp, gpu):
    """Without records the reverse sweep holds those of ckpt_every iterations and
    the checkpoints, besides a dozen vectors (2 MB each with the device's
    granularity)."""
    inst = sdpgen.block_arrow_instance(30, 90, 6, 20, seed=3, density=0.05)
    T, ckpt, record = 100, 5, 8 * 30 * (96 * 96 + 96)
    ubar = np.random.default_rng(5).standard_normal(inst.nnz)
    kept, held = run(sdp, [inst], T, ckpt, ubar, "fp64")
    recomputed, held0 = run(sdp, [inst], T, ckpt, ubar, "fp64", records=0)
    assert held >= T * record
    assert held0 <= ckpt * record + T // ckpt * 16 * 30 * 96 * 97 // 2 + (12 << 21)
    for x, y in zip(kept, recomputed):
        assert np.array_equal(x, y)


@pytest.mark.timeout(300)
def test_no_room_for_the_records(sdp, gpu):
    inst = sdpgen.block_arrow_instance(30, 90, 6, 20, seed=3, density=0.05)
    T, ckpt, record = 250, 10, 8 * 30 * (96 * 96 + 96)
    ubar = np.random.default_rng(6).standard_normal(inst.nnz)
    kept, held = run(sdp, [inst], T, ckpt, ubar, "fp64")
    assert held >= T * record
    with fill_device(T * record // 2):
        recomputed, held0 = run(sdp, [inst], T, ckpt, ubar, "fp64")
    for x, y in zip(kept, recomputed):
        assert np.array_equal(x, y)
