"""The DZT by passes of short DFTs (65 to 2048 Doppler bins that split into two or three factors
of at most 16) against direct sums in 64 bits: every radix, two and three
passes, ragged and single-strip column counts, both directions.

Tolerance per column, in its 2-norm: a pass forms each bin as a sum of at most 16 products of
twiddled values, so its relative error is at most (16 + 4) u with u = 2^-24 (the sum, the two
twiddles' rounding and products); three passes and the scaling stay below 64 u.
"""
import numpy as np
import pytest

from helpers import say, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def otfs():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_02266_amd as m
    m.lib()
    return m


TWO = [66, 70, 72, 75, 77, 78, 80, 81, 84, 88, 90, 96, 98, 100, 104, 110, 112, 117, 120, 121, 126, 128,
       130, 132, 135, 140, 143, 144, 150, 154, 165, 168, 169, 180, 182, 195, 196, 208, 210, 225, 240, 256]
THREE = [125, 162, 250, 264, 507, 512, 1001, 1024, 1536, 2048]
GEMM = [64, 67, 97, 2049]   # the other side of the rule


@pytest.mark.parametrize("N", TWO + THREE + GEMM)
@pytest.mark.parametrize("M,nf", [(1, 1), (67, 3), (128, 2), (64, 40)])
def test_passes_match_the_direct_transform(otfs, N, M, nf):
    if N > 600 and nf > 3:
        nf = 5
    say("dzt", M, N, nf)
    rng = np.random.default_rng(N * 1000 + M)
    x = (rng.standard_normal((nf, N, M)) + 1j * rng.standard_normal((nf, N, M))).astype(np.complex64)
    xd = to_dev(x.reshape(-1))
    F = np.exp(-2j * np.pi * (np.outer(np.arange(N), np.arange(N)) % N) / N) / np.sqrt(N)
    bound = (64 if N != 2049 else 4 * np.sqrt(N)) * 2.0 ** -24
    for inverse in (False, True):
        got = otfs.dzt(xd, M, N, inverse=inverse).cpu().numpy().reshape(nf, N, M)
        ref = (F.conj() if inverse else F) @ x.astype(np.complex128)
        err = np.linalg.norm(got - ref, axis=1) / np.linalg.norm(ref, axis=1)
        assert err.max() <= bound, (inverse, err.max())
