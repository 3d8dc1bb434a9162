"""What otfs_lmmse_cg_noalloc leaves behind.  A refused call leaves the plan's layout and its
binding as they were; a plan that fits the static scratch without the register-resident tiles'
tables is solved there on the streaming kinds, and a later binding takes its own kinds again."""
import ctypes

import numpy as np
import pytest

import oracle as O
import paper_2604_02266_amd as otfs
import workloads as W
from helpers import say, split, to_dev

SCRATCH = 64 << 20
TILE_LDS = 159 * 1024
ITERS = 6


def _frames(M, N, n, seed):
    rng = np.random.default_rng(seed)
    return [W.small_frame(rng, M, N, 6, (0, 20), (-6, 6), qam=16, snr_db=25.0, max_iters=ITERS,
                          tol=0.0) for _ in range(n)]


def _plan(frames, **kw):
    return otfs.Plan([f.spec for f in frames], max_iters=ITERS, rel_tol=0.0, tune=False, **kw)


def test_refused_call_keeps_the_layout():
    # (refused before any device work: the addresses are not touched)
    plan = _plan(_frames(512, 512, 8, 91), bind=False)
    before = plan.workspace_bytes()
    assert before[0] > SCRATCH
    v = ctypes.c_void_p
    st = otfs.lib().otfs_lmmse_cg_noalloc(plan._h, v(256), v(512), None, None, None)
    assert st == otfs.E_NOMEM
    assert plan.workspace_bytes() == before


def _y(frames):
    return np.concatenate([O.received_frame(f)[2] for f in frames]).astype(np.complex64)


@pytest.mark.gpu
def test_refused_call_keeps_the_binding():
    import torch
    frames = _frames(512, 512, 8, 92)
    frames[0:0] = _frames(128, 64, 1, 93)          # one that is register-resident
    y = to_dev(_y(frames))
    say("refused noalloc on a bound plan")
    plan = _plan(frames)
    assert plan.workspace_bytes()[0] > SCRATCH and plan.info().lds_bytes == TILE_LDS
    ref = plan.lmmse_cg(y).cpu().numpy()
    h = plan.apply_H(y).cpu().numpy()
    with pytest.raises(otfs.OtfsError) as ei:
        plan.lmmse_cg_noalloc(y)
    assert ei.value.status == otfs.E_NOMEM
    assert plan.info().lds_bytes == TILE_LDS
    x = plan.lmmse_cg(y).cpu().numpy()
    assert np.array_equal(x.view(np.uint32), ref.view(np.uint32))
    assert np.array_equal(plan.apply_H(y).cpu().numpy(), h)
    torch.cuda.synchronize()


@pytest.mark.gpu
def test_plan_that_fits_only_without_tiles():
    import torch
    frames = _frames(256, 800, 8, 94)
    y = to_dev(_y(frames))
    say("noalloc on the streaming kinds")
    plan = _plan(frames)
    tile_ws, te = plan.workspace_bytes()[0], plan.info().tile_elems
    assert plan.info().lds_bytes == TILE_LDS
    stream = _plan(frames, tile_elems=te)
    assert stream.workspace_bytes()[0] <= SCRATCH < tile_ws
    ref, sref = plan.lmmse_cg(y).cpu().numpy(), stream.lmmse_cg(y).cpu().numpy()
    h, sh = plan.apply_H(y).cpu().numpy(), stream.apply_H(y).cpu().numpy()
    for _ in range(2):
        x = plan.lmmse_cg_noalloc(y).cpu().numpy()
        assert np.array_equal(x.view(np.uint32), sref.view(np.uint32))
        # bound to the scratch, on the streaming kinds throughout
        assert plan.info().lds_bytes != TILE_LDS
        assert np.array_equal(plan.apply_H(y).cpu().numpy(), sh)
        # its own workspace again: its own layout and kinds
        assert plan.workspace_bytes()[0] == tile_ws
        plan.bind()
        assert plan.info().lds_bytes == TILE_LDS
        x = plan.lmmse_cg(y).cpu().numpy()
        assert np.array_equal(x.view(np.uint32), ref.view(np.uint32))
        assert np.array_equal(plan.apply_H(y).cpu().numpy(), h)
    torch.cuda.synchronize()
    op = O.TwistedConvChannel(256, 800, frames[1].spec.h, frames[1].spec.tau, frames[1].spec.nu)
    xr, _, _ = O.cg_lmmse(split(y.cpu().numpy(), frames)[1].astype(np.complex128), op,
                          frames[1].spec.lam, ITERS, 0.0)
    for v in (ref, sref):
        assert O.nmse(split(v, frames)[1], xr) <= 1e-9
