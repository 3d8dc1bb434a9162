"""The direct kinds at device-wide fences (kernels of their own): the same bits as the XCD-local
kinds on the same tiling, and frames of more tiles than one XCD holds, which take them without
being asked, against the FP64 oracle -- with the direction in the gathers (up to 8 paths) and in
a pass of its own, with and without the refresh."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from helpers import say, split, to_dev

pytestmark = pytest.mark.gpu

ITERS = 10
NMSE_TOL = 1e-9   # unit roundoff times the conditioning of these frames (25 dB), as for the tiles


@pytest.fixture(scope="module")
def otfs():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_02266_amd as m
    m.lib()
    return m


def _batch(seed, P, shapes):
    rng = np.random.default_rng(seed)
    frames = [W.small_frame(rng, M, N, P, (0, 9), (-4, 4), qam=16, snr_db=25.0, max_iters=ITERS,
                            tol=0.0) for M, N in shapes]
    ops = [O.received_frame(f) for f in frames]
    return frames, [r[0] for r in ops], np.concatenate([r[2] for r in ops]).astype(np.complex64)


@pytest.mark.parametrize("refresh", [0, 4])
@pytest.mark.parametrize("P", [5, 11])
@pytest.mark.parametrize("tile_elems", [1500, 600])
def test_agent_equals_xcd_local(otfs, tile_elems, P, refresh):
    frames, _, y = _batch(71 + P, P, [(128, 64), (100, 30), (64, 16), (256, 20)])
    say("agent and xcd-local", tile_elems, P, refresh)
    got = []
    for flags in (otfs.NO_LDS_RESIDENT, otfs.NO_LDS_RESIDENT | otfs.AGENT_BARRIER):
        plan = otfs.Plan([f.spec for f in frames], max_iters=ITERS, rel_tol=0.0, refresh_every=refresh,
                         tile_elems=tile_elems, flags=flags)
        assert plan.info().xcd_local == (0 if flags & otfs.AGENT_BARRIER else 1)
        got.append(plan.lmmse_cg(to_dev(y)).cpu().numpy().view(np.uint32))
    assert np.array_equal(*got)


@pytest.mark.parametrize("P", [5, 11])
def test_more_tiles_than_an_xcd_holds(otfs, P):
    frames, ops, y = _batch(81 + P, P, [(64, 220), (64, 150)])
    say("more tiles than an XCD holds", P)
    plan = otfs.Plan([f.spec for f in frames], max_iters=ITERS, rel_tol=0.0, tile_elems=64)
    assert plan.info().xcd_local == 0
    x = plan.lmmse_cg(to_dev(y)).cpu().numpy()
    for f, op, a, b in zip(frames, ops, split(x, frames), split(y, frames)):
        xr, _, _ = O.cg_lmmse(b.astype(np.complex128), op, f.spec.lam, ITERS, 0.0)
        assert O.nmse(a, xr) <= NMSE_TOL
