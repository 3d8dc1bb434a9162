"""The H^H coefficients of the tiled applications, one by one.  With the only nonzero row of the
input at Doppler bin 0, whose wrap factors are 1, and paths of distinct Dopplers, each output row
is one path's coefficient S_p[k] = conj(h_p) e^{-j 2 pi nu_p k / (MN)}, wrapped columns included:
it has to be that number rounded to FP32 once, half a unit in the last place of each component,
plus what the FP64 phases leave of the gain: three angles of up to 2 pi (two factors of the
table, one of the reference) with two roundings each, 38 times 2^-53, taken as 64.  The batches take the
tiled form (not the bits of a plan with an explicit tiling, which multiplies two FP32 tables)."""
import numpy as np
import pytest

import oracle as O
from helpers import SpecLike, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def otfs():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_02266_amd as m
    m.lib()
    return m


@pytest.mark.parametrize("M,N,P,dtau,n", [(512, 128, 16, 60, 64), (130, 70, 12, 9, 128), (257, 96, 9, 9, 96)])
def test_adjoint_coefficients_are_rounded_once(otfs, M, N, P, dtau, n):
    rng = np.random.default_rng(9600 + M)
    specs = []
    for _ in range(n):
        h = (rng.standard_normal(P) + 1j * rng.standard_normal(P)).astype(np.complex64)
        nu = rng.permutation(P) - P // 2
        specs.append(SpecLike(M, N, rng.integers(-dtau, dtau + 1, P), nu, h))
    say("adjoint coefficients", M, N, P, dtau, n)
    plan = otfs.Plan(specs, tune=False)
    y = np.zeros((len(specs), N, M), np.complex64)
    y[:, 0] = 1.0
    x = plan.apply_HH(to_dev(y.reshape(-1))).cpu().numpy().reshape(len(specs), N, M)
    stream = otfs.Plan(specs, tune=False, tile_elems=plan.info().tile_elems)
    xs = stream.apply_HH(to_dev(y.reshape(-1))).cpu().numpy().reshape(len(specs), N, M)
    assert all(not np.array_equal(a, b) for a, b in zip(x, xs))
    k = np.arange(M)
    for f, s in enumerate(specs[:8]):
        for p in range(P):
            h = complex(s.h[p])
            want = np.conj(h) * np.exp(-2j * np.pi * ((int(s.nu[p]) * k) % (M * N)) / (M * N))
            got = x[f, -int(s.nu[p]) % N].astype(np.complex128)
            for a, b in ((got.real, want.real), (got.imag, want.imag)):
                over = np.abs(a - b) - (2.0 ** -24 * np.abs(b) + 64 * 2.0 ** -53 * abs(h))
                assert over.max() <= 0, (f, p, int(over.argmax()), int(s.tau[p]), int(s.nu[p]))
        # and against the oracle's operator
        op = O.TwistedConvChannel(M, N, s.h, s.tau, s.nu)
        ref = op.apply_adjoint(y[f].reshape(-1).astype(np.complex128)).reshape(N, M)
        assert np.abs(x[f] - ref).max() <= 1e-6 * np.abs(s.h).sum()
