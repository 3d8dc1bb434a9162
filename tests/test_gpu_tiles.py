"""Register-resident tiles (the built-in kind of frames beyond one workgroup's LDS): solves at
the edges of the cut -- strips of one and two columns per lane, partial strips and row bands,
odd M (windows copied through registers), windows wider than the frame, negative delays, the
largest path count, one tile and 32 tiles -- against the FP64 oracle, and the forms that share
a frame's state between launches (one iteration per launch, the refresh, bf16 input)."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from helpers import bf16_round, check_decisions, say, split, to_dev

pytestmark = pytest.mark.gpu

ITERS = 12
# FP32 CG against FP64 CG after 12 iterations: the unit roundoff 6e-8 grown by the worst
# conditioning of these frames (25 dB: kappa below 5 / 3e-3, error growth at most its square
# root times the iteration count, about 500) is 3e-5 in the 2-norm, 1e-9 as an NMSE
NMSE_TOL = 1e-9
TILE_LDS = 159 * 1024

CASES = [
    # M, N, P, delays, Dopplers
    (128, 64, 8, (0, 16), (-8, 8)),         # one strip of 128 columns, one full tile
    (130, 70, 6, (0, 9), (-7, 7)),          # two strips of 66 columns, ragged bands
    (1024, 16, 5, (0, 64), (-4, 4)),        # eight strips of one row group
    (96, 90, 7, (-11, 20), (-10, 9)),       # one column per lane, negative delays
    (257, 35, 6, (0, 32), (-3, 3)),         # odd M: windows through registers
    (513, 40, 4, (-40, 40), (-39, 39)),     # odd M, window rows beyond the frame
    (64, 64, 9, (-63, 63), (-63, 63)),      # every shift: window beyond the frame both ways
    (2048, 8, 3, (0, 5), (-7, 7)),          # 16 strips, 8 rows
    (300, 200, 64, (0, 37), (-25, 25)),     # the largest path count
    (1024, 256, 4, (0, 64), (-16, 16)),     # 32 full tiles: the largest frame
]


@pytest.fixture(scope="module")
def otfs():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_02266_amd as m
    m.lib()
    return m


def _frames(case, n):
    M, N, P, tr, vr = CASES[case]
    rng = np.random.default_rng(9500 + case)
    return [W.small_frame(rng, M, N, P, tr, vr, qam=16, snr_db=25.0, max_iters=ITERS, tol=0.0)
            for _ in range(n)]


def _received(frames):
    rec = [O.received_frame(f) for f in frames]
    return [r[0] for r in rec], np.concatenate([r[2] for r in rec]).astype(np.complex64)


def _solve(otfs, plan, y):
    import torch
    sym = torch.zeros(plan.total_elems, dtype=torch.uint8, device="cuda")
    st = plan.new_stats()
    x = plan.lmmse_cg(y, sym=sym, stats=st)
    torch.cuda.synchronize()
    return x.cpu().numpy(), sym.cpu().numpy(), otfs.stats_numpy(st)


@pytest.mark.parametrize("case", range(len(CASES)))
def test_tiles_match_oracle(otfs, case):
    frames = _frames(case, 1 if CASES[case][0] * CASES[case][1] > 50000 else 3)
    ops, y = _received(frames)
    say("tiles", CASES[case])
    plan = otfs.Plan([f.spec for f in frames], max_iters=ITERS, rel_tol=0.0, tune=False)
    assert plan.info().lds_bytes == TILE_LDS, "the register-resident kind"
    x, sym, st = _solve(otfs, plan, to_dev(y))
    assert np.all(st["iters"] == ITERS) and np.all(st["status"] == otfs.FRAME_CAPPED)
    for f, op, xg, sg, yy in zip(frames, ops, split(x, frames), split(sym, frames), split(y, frames)):
        xr, _, _ = O.cg_lmmse(yy.astype(np.complex128), op, f.spec.lam, ITERS, 0.0)
        nm = O.nmse(xg, xr)
        assert nm <= NMSE_TOL, (CASES[case], nm)
        check_decisions(sg, xg, xr, 16)


def test_tiles_alone_in_a_batch_and_beside_other_kinds(otfs):
    # frames of one tile, of several, of odd M, LDS-resident ones, one beyond 32 tiles and a
    # small ragged one (streaming kinds)
    rng = np.random.default_rng(77)
    frames = [W.small_frame(rng, M, N, 5, (0, 12), (-4, 4), qam=16, snr_db=25.0, max_iters=ITERS,
                            tol=0.0)
              for M, N in ((128, 64), (64, 16), (512, 96), (37, 11), (255, 33), (1024, 272), (100, 30))]
    ops, y = _received(frames)
    say("tiles beside other kinds")
    plan = otfs.Plan([f.spec for f in frames], max_iters=ITERS, rel_tol=0.0, tune=False)
    assert plan.info().launches >= 3 and plan.info().resident_frames == 2
    x, sym, st = _solve(otfs, plan, to_dev(y))
    assert np.all(st["iters"] == ITERS)
    for f, op, xg, yy in zip(frames, ops, split(x, frames), split(y, frames)):
        xr, _, _ = O.cg_lmmse(yy.astype(np.complex128), op, f.spec.lam, ITERS, 0.0)
        assert O.nmse(xg, xr) <= NMSE_TOL, (f.spec.M, f.spec.N)


@pytest.mark.parametrize("case", [0, 1, 4, 9])
def test_tiles_across_launches(otfs, case):
    # one iteration per launch (the trace) carries x, c and p through memory: the same bits;
    # the FP64 refresh every 5 and bf16 input against the oracle
    import torch
    frames = _frames(case, 2)
    ops, y = _received(frames)
    specs = [f.spec for f in frames]
    say("tiles across launches", CASES[case])
    plan = otfs.Plan(specs, max_iters=ITERS, rel_tol=0.0, tune=False)
    x, sym, _ = _solve(otfs, plan, to_dev(y))
    tx = torch.from_numpy(np.concatenate([f.sym for f in frames]).astype(np.uint8)).cuda()
    xt, st, errs = plan.lmmse_cg_trace(to_dev(y), tx)
    torch.cuda.synchronize()
    assert np.array_equal(xt.cpu().numpy().view(np.uint32), x.view(np.uint32))
    assert np.array_equal(st.cpu().numpy(), sym)
    n = [O.bit_errors(s, f.sym, 16) for s, f in zip(split(sym, frames), frames)]
    assert list(errs[-1].cpu().numpy()) == n
    plan = otfs.Plan(specs, max_iters=ITERS, rel_tol=0.0, refresh_every=5, tune=False)
    assert plan.info().lds_bytes == TILE_LDS
    xr5, _, s5 = _solve(otfs, plan, to_dev(y))
    assert np.all(s5["iters"] == ITERS)
    bits, yr = bf16_round(y)
    plan = otfs.Plan(specs, max_iters=ITERS, rel_tol=0.0, flags=otfs.Y_BF16, tune=False)
    yb = torch.from_numpy(bits.view(np.int16)).to("cuda").view(torch.bfloat16)
    xb, _, _ = _solve(otfs, plan, yb)
    for f, op, a, b, yy, yq in zip(frames, ops, split(xr5, frames), split(xb, frames),
                                   split(y, frames), split(yr, frames)):
        assert O.nmse(a, O.cg_lmmse(yy.astype(np.complex128), op, f.spec.lam, ITERS, 0.0)[0]) <= NMSE_TOL
        assert O.nmse(b, O.cg_lmmse(yq.astype(np.complex128), op, f.spec.lam, ITERS, 0.0)[0]) <= NMSE_TOL


@pytest.mark.parametrize("case", range(len(CASES)))
def test_tile_applies_match_oracle(otfs, case):
    # H and H^H by tiles, the case's frames at an even and at an odd element offset of the batch
    # (an odd one cannot take 16-byte copies), beside a frame that keeps the streaming items
    M, N, P, tr, vr = CASES[case]
    rng = np.random.default_rng(9700 + case)
    specs = [W.small_frame(rng, *s, qam=4).spec for s in
             ((M, N, P, tr, vr), (45, 33, 3, (0, 4), (-2, 2)), (M, N, P, tr, vr), (64, 16, 2, (0, 3), (-2, 2)))]
    say("tile applies", CASES[case])
    plan = otfs.Plan(specs, tune=False)
    E = plan.total_elems
    x = (rng.standard_normal(E) + 1j * rng.standard_normal(E)).astype(np.complex64)
    y = (rng.standard_normal(E) + 1j * rng.standard_normal(E)).astype(np.complex64)
    yh = plan.apply_H(to_dev(x)).cpu().numpy()
    xh = plan.apply_HH(to_dev(y)).cpu().numpy()
    for s, xs, ys, a, b in zip(specs, split(x, specs), split(y, specs), split(yh, specs), split(xh, specs)):
        op = O.TwistedConvChannel(s.M, s.N, s.h, s.tau, s.nu)
        scale = 1e-5 * np.abs(s.h).sum()   # FP32 products and sums of P terms, as for every form
        assert np.abs(a - op.apply(xs.astype(np.complex128))).max() <= scale * np.abs(xs).max(), (s.M, s.N)
        assert np.abs(b - op.apply_adjoint(ys.astype(np.complex128))).max() <= scale * np.abs(ys).max(), (s.M, s.N)
