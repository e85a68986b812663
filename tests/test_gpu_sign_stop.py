"""The sign iteration's early stop: blocks whose smallest eigenvalues sit at
every stage of the iteration, from well separated to exactly zero, come out
within the projection tolerance (numpy.linalg.eigh in FP64 as reference).

Bound: the schedule and the stop table keep the Frobenius error of the exact
iteration within tol/2 ||W||_F; rounding of the products adds a multiple of
n eps ||W||_F (at most ~60 products of depth n, each with a relative error of
sqrt(n) eps, of which a fixed point forgets all but the last few)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SMALL = (0.3, 1e-2, 1e-4, 1e-6, 1e-7, 1e-9, 1e-12, 1e-15, 0.0)


def block(rng, s, small):
    """Random eigenvectors; eigenvalues of both signs in [0.3, 1] but the last,
    +-small (relative to the largest)."""
    q, _ = np.linalg.qr(rng.standard_normal((s, s)))
    t = rng.uniform(0.3, 1.0, s) * rng.choice([-1.0, 1.0], s)
    t[-1] = small * rng.choice([-1.0, 1.0])
    w = (q * t) @ q.T
    return 0.5 * (w + w.T)


def project(blocks, dtype):
    import torch
    import paper_1707_05058_amd as sdp
    sizes = np.array([b.shape[0] for b in blocks])
    offs = np.concatenate([[0], np.cumsum(sizes ** 2)])
    x = torch.from_numpy(np.concatenate([b.ravel() for b in blocks])).to("cuda", dtype)
    out = torch.zeros_like(x)
    sdp.psd_project_batched(torch.from_numpy(sizes.astype(np.int32)).cuda(),
                            torch.from_numpy(offs[:-1].astype(np.int64)).cuda(), x, out,
                            int(sizes.max()))
    y, back = out.double().cpu().numpy(), x.double().cpu().numpy()
    return [(back[o:o + s * s].reshape(s, s), y[o:o + s * s].reshape(s, s))
            for o, s in zip(offs, sizes)]


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("s", [1, 2, 15, 16, 17, 31, 32, 33, 48, 64, 65, 96, 112, 113, 128])
def test_every_stage_of_the_stop(s, prec):
    import torch
    dtype = torch.float32 if prec == "fp32" else torch.float64
    tol, eps = (1e-6, 2.0 ** -24) if prec == "fp32" else (1e-14, 2.0 ** -53)
    rng = np.random.default_rng(s)
    blocks = [block(rng, s, v) * scale for v in SMALL for scale in (1.0, 1e5)]
    blocks += [np.zeros((s, s)), np.eye(s), -np.eye(s)]
    for w, y in project(blocks, dtype):
        t, v = np.linalg.eigh(w)
        ref = (v * np.maximum(t, 0.0)) @ v.T
        err = np.linalg.norm(y - ref)
        assert err <= (tol + 16.0 * max(s, 16) * eps) * np.linalg.norm(w), (s, prec, err)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("s", [16, 24, 40])
def test_a_bad_block_stays_alone(s, prec):
    import torch
    dtype = torch.float32 if prec == "fp32" else torch.float64
    rng = np.random.default_rng(s)
    good = block(rng, s, 1e-3)
    bad = good.copy()
    bad[0, s - 1] = bad[s - 1, 0] = np.nan
    got = project([good, bad, good], dtype)
    assert np.isnan(got[1][1]).all()
    assert np.array_equal(got[0][1], got[2][1]) and np.isfinite(got[0][1]).all()
