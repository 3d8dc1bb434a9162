"""The per-iteration trace with the FP64 refresh on batches whose every frame is
register-resident: the refresh has to leave the partial norms that the next one-iteration
launch sums, so the trace ends on the solve's estimate, decisions and statistics bit for bit.
The frames' streaming tiling has fewer tiles than their register-resident cut, more, and as many."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from helpers import say, split, to_dev

pytestmark = pytest.mark.gpu

ITERS, EVERY = 12, 5
TILE_LDS = 159 * 1024


@pytest.fixture(scope="module")
def otfs():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_02266_amd as m
    m.lib()
    return m


@pytest.mark.parametrize("M,N,n", [(128, 64, 2), (130, 70, 2), (257, 35, 3), (512, 128, 1),
                                   (128, 32, 24), (1024, 256, 1), (512, 64, 16)])
def test_trace_with_refresh_equals_the_solve(otfs, M, N, n):
    import torch
    rng = np.random.default_rng(9300 + M + n)
    frames = [W.small_frame(rng, M, N, 5, (0, 12), (-5, 5), qam=16, snr_db=25.0, max_iters=ITERS,
                            tol=0.0) for _ in range(n)]
    say("trace with refresh", M, N, n)
    y = np.concatenate([O.received_frame(f)[2] for f in frames]).astype(np.complex64)
    tx = torch.from_numpy(np.concatenate([f.sym for f in frames]).astype(np.uint8)).cuda()
    plan = otfs.Plan([f.spec for f in frames], max_iters=ITERS, rel_tol=0.0, refresh_every=EVERY,
                     tune=False)
    assert plan.info().lds_bytes == TILE_LDS and plan.info().launches == 1
    sym = torch.zeros(plan.total_elems, dtype=torch.uint8, device="cuda")
    stats, tstats = plan.new_stats(), plan.new_stats()
    x = plan.lmmse_cg(to_dev(y), sym=sym, stats=stats)
    # the solve before left its own partial norms in the workspace: another right-hand side
    plan.lmmse_cg(to_dev(-3 * y[::-1].copy()))
    xt, st, errs = plan.lmmse_cg_trace(to_dev(y), tx, stats=tstats)
    torch.cuda.synchronize()
    assert np.array_equal(xt.cpu().numpy().view(np.uint32), x.cpu().numpy().view(np.uint32))
    assert np.array_equal(st.cpu().numpy(), sym.cpu().numpy())
    assert np.array_equal(tstats.cpu().numpy(), stats.cpu().numpy())
    sg = split(sym.cpu().numpy(), frames)
    assert list(errs[-1].cpu().numpy()) == [O.bit_errors(s, f.sym, 16) for s, f in zip(sg, frames)]
