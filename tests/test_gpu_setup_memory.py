"""Set-up where the device has room for A but not for B = L^-1 A beside it:
Algorithm 3 then iterates with A and both triangular passes, as it does for
small matrices.  The rest of the device is held by a tensor meanwhile, so an
allocation fails as it would beside another program.  Bar: 1e-8 relative to
the largest entry, as against the oracle, between the two forms."""
import contextlib
import gc

import numpy as np
import pytest

import sdpgen
from test_gpu_admm import rel_err

pytestmark = pytest.mark.gpu

STEPS = 30


@contextlib.contextmanager
def fill_device(room):
    """Everything on the device held by tensors but about `room` bytes."""
    import torch
    chunk = 64 << 20
    torch.cuda.empty_cache()
    hogs = [torch.empty(torch.cuda.mem_get_info()[0] - (4 << 30), dtype=torch.uint8, device="cuda")]
    try:
        for _ in range(512):                       # (the device holds more than it reports free)
            try:
                hogs.append(torch.empty(chunk, dtype=torch.uint8, device="cuda"))
            except torch.cuda.OutOfMemoryError:
                break
        del hogs[1:1 + (room + chunk - 1) // chunk]
        torch.cuda.empty_cache()
        yield
    finally:
        del hogs
        gc.collect()
        torch.cuda.empty_cache()


def solve(sdp, inst):
    with sdp.Solver([inst], algorithm="hsde", tol=0.0, max_iter=1000) as S:
        S.step(STEPS)
        return S.solution(0)


@pytest.mark.timeout(300)
def test_hsde_without_room_for_b(sdp, gpu):
    import torch
    inst = sdpgen.banded_instance(2000, 15, 1000, seed=0)
    b_bytes = 8 * inst.m * inst.nnz
    ref = solve(sdp, inst)   # (the first handle also loads the kernels and their scratch)
    torch.cuda.empty_cache()
    free0 = torch.cuda.mem_get_info()[0]
    with sdp.Solver([inst], algorithm="hsde", tol=0.0, max_iter=1000) as S:
        used = free0 - torch.cuda.mem_get_info()[0]
    assert 2 * b_bytes < used < 3 * b_bytes        # A and B are held
    print(f"held {used / 1e6:.0f} MB, A {b_bytes / 1e6:.0f} MB", flush=True)
    with fill_device(used - b_bytes // 2):
        got = solve(sdp, inst)
    for k in ("u", "y_dual", "X_packed", "L_packed"):
        assert rel_err(got[k], ref[k]) <= 1e-8, k
    assert not np.array_equal(got["u"], ref["u"])  # (the other form: other roundings)
