"""Which batches keep the streaming kinds although their frames have register-resident cuts
(narrow frames of few paths in small batches, batches whose windows are mostly halo) and which,
just past each line, take the tiles: told by the bits of a plan with an explicit tiling, with both
forms' estimates against the FP64 oracle's on a few frames."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from helpers import say, split, to_dev

pytestmark = pytest.mark.gpu

ITERS = 12
# as for the tiles' own tests: unit roundoff times the conditioning of these frames (25 dB)
NMSE_TOL = 1e-9
TILE_LDS = 159 * 1024

CASES = [
    # M, N, P, delays, Dopplers, frames, the tiles are taken
    (64, 128, 2, (0, 4), (-8, 8), 6, False),       # one tile of 16 elements per thread each
    (32, 256, 4, (0, 2), (-8, 8), 3, False),
    (64, 128, 2, (0, 4), (-8, 8), 65, True),       # more streaming bands than CUs
    (64, 112, 5, (0, 4), (-8, 8), 6, True),        # five paths
    (64, 64, 2, (0, 4), (-4, 4), 6, True),         # 8 elements per thread
    (96, 80, 2, (0, 4), (-8, 8), 6, False),        # less than a full tile, rows leave lanes idle
    (128, 64, 2, (0, 4), (-8, 8), 6, True),        # wider
    (201, 116, 4, (0, 100), (-58, 58), 48, False),  # halos of more than 6.5 times the tiles
    (201, 116, 4, (0, 20), (-10, 10), 48, True),
]


@pytest.fixture(scope="module")
def otfs():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_02266_amd as m
    m.lib()
    return m


@pytest.mark.parametrize("case", range(len(CASES)))
def test_solve_forms(otfs, case):
    M, N, P, tr, vr, n, tiles = CASES[case]
    rng = np.random.default_rng(9950 + case)
    # one set of shifts for the batch, with the whole range in it; gains of their own
    first = W.small_frame(rng, M, N, P, tr, vr, qam=16, snr_db=25.0, max_iters=ITERS, tol=0.0)
    first.spec.tau[:2], first.spec.nu[:2] = (tr[0], tr[1]), (vr[0], vr[1])
    frames = [first]
    for _ in range(n - 1):
        f = W.small_frame(rng, M, N, P, tr, vr, qam=16, snr_db=25.0, max_iters=ITERS, tol=0.0)
        f.spec.tau[:], f.spec.nu[:] = first.spec.tau, first.spec.nu
        frames.append(f)
    say("solve forms", CASES[case])
    y = np.concatenate([O.received_frame(f)[2] for f in frames]).astype(np.complex64)
    specs = [f.spec for f in frames]
    plan = otfs.Plan(specs, max_iters=ITERS, rel_tol=0.0, tune=False)
    stream = otfs.Plan(specs, max_iters=ITERS, rel_tol=0.0, tune=False, tile_elems=plan.info().tile_elems)
    assert (plan.info().lds_bytes == TILE_LDS) == tiles and plan.info().launches == 1
    x, xs = plan.lmmse_cg(to_dev(y)).cpu().numpy(), stream.lmmse_cg(to_dev(y)).cpu().numpy()
    assert np.array_equal(x.view(np.uint32), xs.view(np.uint32)) != tiles
    for i in (0, n - 1):
        op = O.TwistedConvChannel(M, N, specs[i].h, specs[i].tau, specs[i].nu)
        xr, _, _ = O.cg_lmmse(split(y, frames)[i].astype(np.complex128), op, specs[i].lam, ITERS, 0.0)
        assert O.nmse(split(x, frames)[i], xr) <= NMSE_TOL
        assert O.nmse(split(xs, frames)[i], xr) <= NMSE_TOL
