"""The FP64 refresh of register-resident frames on the applications' tiles: every third
iteration, at strips of one and two columns per lane, tiles with wrapped gathers on one side, on
both and on none, negative delays, odd M (windows through registers, frames at odd offsets),
bf16 input -- the solution against the FP64 oracle, and the residual that the frame reports one
iteration after its last refresh against the true residual of its estimate."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from helpers import bf16_round, say, split, to_dev

pytestmark = pytest.mark.gpu

ITERS, EVERY = 10, 3
# as for the solves without refresh: the unit roundoff grown by the conditioning of these
# frames is below 3e-5 in the 2-norm
NMSE_TOL = 1e-9
# The reported residual is the refreshed one (rounded once to FP32, 6e-8 of itself) after one
# FP32 update; the estimate's own rounding moves the true one by 6e-8 ||A|| ||x|| <= 1e-6 ||b||,
# against residuals above 1e-3 ||b|| after 10 iterations
REL_TOL = 2e-3

CASES = [
    # M, N, P, delays, Dopplers
    (128, 64, 8, (0, 16), (-8, 8)),
    (130, 70, 6, (-9, 9), (-7, 7)),
    (1024, 32, 5, (0, 64), (-4, 4)),
    (96, 90, 7, (-11, 20), (-10, 9)),
    (257, 35, 6, (0, 32), (-3, 3)),
    (513, 40, 4, (-40, 40), (-20, 20)),
    (128, 96, 9, (-50, 50), (-10, 10)),
    (300, 200, 64, (0, 20), (-12, 12)),
    (1024, 256, 4, (0, 64), (-16, 16)),
]


@pytest.fixture(scope="module")
def otfs():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_02266_amd as m
    m.lib()
    return m


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_refresh_on_tiles(otfs, case, bf16):
    import torch
    M, N, P, tr, vr = CASES[case]
    rng = np.random.default_rng(9900 + case)
    frames = [W.small_frame(rng, M, N, P, tr, vr, qam=16, snr_db=25.0, max_iters=ITERS, tol=0.0)
              for _ in range(2)]
    say("refresh on tiles", CASES[case], "bf16" if bf16 else "complex64")
    rec = [O.received_frame(f) for f in frames]
    y = np.concatenate([r[2] for r in rec]).astype(np.complex64)
    yd = to_dev(y)
    if bf16:
        bits, y = bf16_round(y)
        yd = torch.from_numpy(bits.view(np.int16)).to("cuda").view(torch.bfloat16)
    plan = otfs.Plan([f.spec for f in frames], max_iters=ITERS, rel_tol=0.0, refresh_every=EVERY,
                     flags=otfs.Y_BF16 if bf16 else 0, tune=False)
    stats = plan.new_stats()
    x = plan.lmmse_cg(yd, stats=stats)
    torch.cuda.synchronize()
    st, x = stats.cpu().numpy(), x.cpu().numpy()
    for i, (f, r, xg, yy) in enumerate(zip(frames, rec, split(x, frames), split(y, frames))):
        yy = yy.astype(np.complex128)
        xr, _, _ = O.cg_lmmse(yy, r[0], f.spec.lam, ITERS, 0.0)
        assert O.nmse(xg, xr) <= NMSE_TOL, i
        x64 = xg.astype(np.complex128)
        b = r[0].apply_adjoint(yy)
        true = np.linalg.norm(b - r[0].apply_adjoint(r[0].apply(x64)) - f.spec.lam * x64) / np.linalg.norm(b)
        rel = float(st[i, 1:2].view(np.float32)[0])
        assert true > 1e-4 and abs(rel - true) <= REL_TOL * true, (i, rel, true)
