"""The pilot's path set where runs of bins are passed over: thresholds at, just below and just
above the magnitude of bins (zero and underflowing ones too), frames that end inside a run and
inside a group, NaN and infinite bins -- the counts against the rule evaluated bin by bin.

The rule's own rounding is below 1e-6 of |h|^2, so only bins within 4e-6 of theta^2 may differ."""
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


class Spec:
    def __init__(self, M, N):
        self.M, self.N, self.lam, self.qam = M, N, 0.1, 4
        self.tau = self.nu = np.zeros(64, dtype=np.int32)
        self.h = np.full(64, 0.1 + 0j)


@pytest.mark.parametrize("theta", [0.0, 1e-20, 0.08, 0.5])
@pytest.mark.parametrize("M,N", [(8, 4), (64, 64), (64, 65), (100, 41), (513, 24), (512, 128)])
def test_counts_follow_the_rule(otfs, M, N, theta):
    import torch
    say("pilot groups", M, N, theta)
    rng = np.random.default_rng(M * N)
    E = M * N
    y = ((rng.standard_normal(E) + 1j * rng.standard_normal(E)) * 0.01).astype(np.complex64)
    at = rng.permutation(E)[:12]
    mag = max(theta, 1e-3)
    y[at] = mag * np.array([1 - 1e-3, 1 - 3e-5, 1 + 3e-5, 1 + 1e-3, 2, 3, 4, 5, 0.5, 1, 1, 9]) * np.exp(
        1j * rng.uniform(0, 6.28, 12))
    y[at[9]], y[at[10]] = complex(np.nan, 0), complex(np.inf, 1.0)
    if theta == 0.0:
        y[rng.permutation(E)[:E // 2]] = 0
    plan = otfs.Plan([Spec(M, N)], max_iters=2, rel_tol=0.0, tune=False)
    n = int(plan.paths_from_pilot(to_dev(y), theta).cpu().numpy()[0])
    th2 = np.float32(theta) * np.float32(theta)
    with np.errstate(all="ignore"):
        p = y.real.astype(np.float64) ** 2 + y.imag.astype(np.float64) ** 2
        # an infinite bin rotates to NaN or infinity: selected or not
        lo = int(np.sum((p > th2 * (1 + 4e-6)) & np.isfinite(p) & (p > 1e-37)))
        hi = int(np.sum(((p >= th2 * (1 - 4e-6)) & (p > 0)) & np.isfinite(p))) + 1
    assert lo <= n <= hi, (lo, n, hi)
