"""The built-in kinds under capture: solves on register-resident tiles through the library's graph
(OTFS_USE_GRAPH) and through a capture of the caller's, with and without the FP64 refresh, replayed
several times with eager work in between, bit for bit as without a graph; the switch to the
streaming kinds when a pilot's paths replace the host's, after which the old graph must not run,
and back with the next binding; applications and transforms in a capture of the caller's."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from helpers import say, to_dev

pytestmark = pytest.mark.gpu

ITERS = 12
TILE_LDS = 159 * 1024
REPLAYS = 4


@pytest.fixture(scope="module")
def otfs():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_02266_amd as m
    m.lib()
    return m


def _frames(seed, shapes):
    rng = np.random.default_rng(seed)
    return [W.small_frame(rng, M, N, 6, (0, 12), (-5, 5), qam=16, snr_db=25.0, max_iters=ITERS,
                          tol=0.0) for M, N in shapes]


def _plan(otfs, frames, refresh, flags=0):
    p = otfs.Plan([f.spec for f in frames], max_iters=ITERS, rel_tol=0.0, refresh_every=refresh,
                  flags=flags, tune=False)
    assert p.info().lds_bytes == TILE_LDS, "the register-resident kind"
    return p


def _y(frames):
    return np.concatenate([O.received_frame(f)[2] for f in frames]).astype(np.complex64)


def _outputs(plan):
    import torch
    return (torch.empty(plan.total_elems, dtype=torch.complex64, device="cuda"),
            torch.empty(plan.total_elems, dtype=torch.uint8, device="cuda"), plan.new_stats())


def _numpy(o):
    return o[0].cpu().numpy().view(np.uint32), o[1].cpu().numpy(), o[2].cpu().numpy()


def _spoil(o):
    import torch
    o[0].fill_(float("nan"))
    o[1].fill_(255)
    o[2].fill_(-1)
    torch.rand(1000, device="cuda").sort()      # unrelated eager work between the replays


def _same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(_numpy(a), b))


SHAPES = {"uniform": [(512, 64)] * 5, "mixed": [(128, 64), (64, 16), (257, 35), (37, 11), (512, 96)]}


@pytest.mark.parametrize("refresh", [0, 5])
@pytest.mark.parametrize("shapes", sorted(SHAPES))
def test_solve_through_the_librarys_graph(otfs, shapes, refresh):
    import torch
    frames = _frames(61, SHAPES[shapes])
    say("tiles through the library's graph", shapes, refresh)
    y = _y(frames)
    direct = _plan(otfs, frames, refresh)
    o = _outputs(direct)
    direct.lmmse_cg(to_dev(y), *o)
    torch.cuda.synchronize()
    want = _numpy(o)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        plan = _plan(otfs, frames, refresh, otfs.USE_GRAPH)
        yd, o = to_dev(y), _outputs(plan)
        for rep in range(REPLAYS):
            _spoil(o)
            plan.lmmse_cg(yd, *o)
            side.synchronize()
            assert _same(o, want), rep
        # other buffers: captured again
        o2 = _outputs(plan)
        _spoil(o2)
        plan.lmmse_cg(yd, *o2)
        side.synchronize()
        assert _same(o2, want)


@pytest.mark.parametrize("refresh", [0, 5])
def test_graph_is_dropped_when_the_paths_change(otfs, refresh):
    import torch
    frames = _frames(62, [(128, 64)] * 3)
    say("graph and paths from a pilot", refresh)
    y = to_dev(_y(frames))
    # pilots of other channels than the ones given to the plan
    rng = np.random.default_rng(63)
    pilots = []
    for f in frames:
        s = f.spec
        tau, nu = rng.integers(0, 20, 5), rng.integers(-6, 7, 5)
        h = 0.3 * np.exp(2j * np.pi * rng.random(5))
        x = np.zeros((s.N, s.M), np.complex128)
        x[s.N // 2, s.M // 2] = 1.0
        pilots.append(O.TwistedConvChannel(s.M, s.N, h, tau, nu).apply(x.reshape(-1)))
    yp = to_dev(np.concatenate(pilots).astype(np.complex64))
    direct = _plan(otfs, frames, refresh)
    o = _outputs(direct)
    direct.lmmse_cg(y, *o)
    host = _numpy(o)
    direct.paths_from_pilot(yp)
    direct.lmmse_cg(y, *o)
    dev = _numpy(o)
    assert not np.array_equal(host[0], dev[0])
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        plan = _plan(otfs, frames, refresh, otfs.USE_GRAPH)
        o = _outputs(plan)
        for want, step in ((host, lambda: None), (dev, lambda: plan.paths_from_pilot(yp)),
                           (host, plan.bind), (dev, lambda: plan.paths_from_pilot(yp))):
            step()
            for rep in range(2):
                _spoil(o)
                plan.lmmse_cg(y, *o)
                side.synchronize()
                assert _same(o, want), rep


@pytest.mark.parametrize("refresh", [0, 5])
def test_a_capture_of_the_callers(otfs, refresh):
    import torch
    frames = _frames(64, [(512, 128)] * 24)
    say("a capture of the caller's", refresh)
    y = to_dev(_y(frames))
    plan = _plan(otfs, frames, refresh)
    o, hx, hy, td = _outputs(plan), torch.empty_like(y), torch.empty_like(y), torch.empty_like(y)

    def work():
        plan.lmmse_cg(y, *o)
        plan.apply_H(y, hx)
        plan.apply_HH(y, hy)
        otfs.dzt(y, 512, 128, out=td)

    work()
    torch.cuda.synchronize()
    want, also = _numpy(o), [t.clone() for t in (hx, hy, td)]
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=side):
        work()
    for rep in range(REPLAYS):
        _spoil(o)
        for t in (hx, hy, td):
            t.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert _same(o, want), rep
        for t, w in zip((hx, hy, td), also):
            assert torch.equal(torch.view_as_real(t), torch.view_as_real(w)), rep
