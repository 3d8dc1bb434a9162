"""The standalone applications in batches whose estimate takes the apply cuts (strips of one and
two columns per lane, partial strips and row bands, odd M, negative delays, many paths) and in
batches whose estimate keeps the streaming items (shifts that make most of a window a halo, a few
frames, two paths): the form that the rule names, told by the bits of a plan with an explicit
tiling, and every frame against the FP64 sums."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from helpers import say, split, to_dev

pytestmark = pytest.mark.gpu

CASES = [
    # M, N, P, delays, Dopplers, frames, the cuts are taken
    (128, 64, 8, (0, 4), (-2, 2), 160, True),
    (512, 128, 8, (0, 32), (-8, 8), 40, True),       # two columns per lane
    (130, 70, 12, (-4, 5), (-2, 2), 120, True),      # two partial strips, ragged bands
    (96, 90, 16, (-5, 5), (-3, 3), 100, True),
    (257, 35, 8, (0, 9), (-1, 1), 160, True),        # odd M: windows through registers
    (300, 200, 32, (0, 20), (-6, 6), 24, True),
    (2048, 16, 6, (0, 20), (-1, 1), 60, True),
    (512, 128, 2, (0, 128), (-50, 50), 40, False),
    (64, 64, 9, (-63, 63), (-63, 63), 64, False),
    (255, 129, 5, (0, 30), (-10, 10), 8, False),
    (1024, 256, 2, (0, 127), (-42, 42), 15, False),
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
def test_application_forms(otfs, case):
    M, N, P, tr, vr, n, cuts = CASES[case]
    rng = np.random.default_rng(9800 + case)
    specs = []
    for _ in range(n):
        pick = rng.choice((tr[1] - tr[0] + 1) * (vr[1] - vr[0] + 1), size=P, replace=False)
        h = (rng.standard_normal(P) + 1j * rng.standard_normal(P)) / np.sqrt(2 * P)
        specs.append(W.FrameSpec(M=M, N=N, tau=(pick // (vr[1] - vr[0] + 1) + tr[0]).astype(np.int32),
                                 nu=(pick % (vr[1] - vr[0] + 1) + vr[0]).astype(np.int32), h=h, qam=4,
                                 snr_db=20.0, lam=0.01, max_iters=1, tol=0.0))
    say("application forms", CASES[case])
    plan = otfs.Plan(specs, tune=False)
    stream = otfs.Plan(specs, tune=False, tile_elems=plan.info().tile_elems)
    E = plan.total_elems
    x = (rng.standard_normal(E) + 1j * rng.standard_normal(E)).astype(np.complex64)
    for fn, ref in (("apply_H", "apply"), ("apply_HH", "apply_adjoint")):
        got = getattr(plan, fn)(to_dev(x)).cpu().numpy()
        other = getattr(stream, fn)(to_dev(x)).cpu().numpy()
        if fn == "apply_HH":   # (H's wrapped terms can round alike in both forms)
            assert np.array_equal(got, other) != cuts
        elif not cuts:
            assert np.array_equal(got, other)
        parts = list(zip(specs, split(x, specs), split(got, specs), split(other, specs)))
        for i, (s, v, a, b) in enumerate(parts):
            # FP32 products and sums of P terms, as for every form
            tol = 1e-5 * np.abs(s.h).sum() * np.abs(v).max()
            assert np.abs(a - b).max() <= tol, (fn, i)
            if i in (0, 1, n // 2, n - 1):
                op = O.TwistedConvChannel(M, N, s.h, s.tau, s.nu)
                assert np.abs(a - getattr(op, ref)(v.astype(np.complex128))).max() <= tol, (fn, i)


def test_tiled_frames_at_odd_offsets(otfs):
    # an odd number of elements before frames of even M: no 16-byte copies of their windows
    rng = np.random.default_rng(9890)
    specs = [W.small_frame(rng, 45, 33, 3, (0, 4), (-2, 2)).spec]
    specs += [W.small_frame(rng, 512, 128, 8, (0, 32), (-8, 8)).spec for _ in range(40)]
    say("tiled frames at odd offsets")
    plan = otfs.Plan(specs, tune=False)
    stream = otfs.Plan(specs, tune=False, tile_elems=plan.info().tile_elems)
    E = plan.total_elems
    x = (rng.standard_normal(E) + 1j * rng.standard_normal(E)).astype(np.complex64)
    for fn, ref in (("apply_H", "apply"), ("apply_HH", "apply_adjoint")):
        got = split(getattr(plan, fn)(to_dev(x)).cpu().numpy(), specs)
        other = split(getattr(stream, fn)(to_dev(x)).cpu().numpy(), specs)
        assert fn == "apply_H" or all(not np.array_equal(a, b) for a, b in zip(got[1:], other[1:]))
        for i, (s, v, a, b) in enumerate(zip(specs, split(x, specs), got, other)):
            tol = 1e-5 * np.abs(s.h).sum() * np.abs(v).max()
            assert np.abs(a - b).max() <= tol, (fn, i)
            if i in (0, 1, 40):
                op = O.TwistedConvChannel(s.M, s.N, s.h, s.tau, s.nu)
                assert np.abs(a - getattr(op, ref)(v.astype(np.complex128))).max() <= tol, (fn, i)
