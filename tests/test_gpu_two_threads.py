"""Two threads with a plan and a stream of their own, whose applications (and transforms) take
LDS windows of different sizes: neither's launches may depend on what the other thread last
asked for.  Every result equals the one computed before the threads started, bit for bit."""
import threading

import numpy as np
import pytest

import workloads as W
from helpers import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def otfs():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_02266_amd as m
    m.lib()
    return m


def _both(jobs, rounds):
    import torch
    errors = []

    def loop(job):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for i in range(rounds):
                    job(i)
        except Exception as e:   # (shown by the test)
            errors.append(repr(e))

    threads = [threading.Thread(target=loop, args=(j,)) for j in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors


def test_applications_of_two_threads(otfs):
    import torch
    rng = np.random.default_rng(88)
    jobs = []
    for tr, vr in (((0, 32), (-8, 8)), ((0, 200), (-20, 20))):   # small and large windows
        specs = [W.small_frame(rng, 512, 128, 8, tr, vr).spec for _ in range(4)]
        plan = otfs.Plan(specs, tune=False)
        x = torch.view_as_complex(torch.randn(plan.total_elems, 2, device="cuda"))
        want = plan.apply_H(x).clone(), plan.apply_HH(x).clone()
        torch.cuda.synchronize()

        def job(i, plan=plan, x=x, want=want):
            got = plan.apply_H(x), plan.apply_HH(x)
            assert all(torch.equal(torch.view_as_real(a), torch.view_as_real(b)) for a, b in zip(got, want)), i
        jobs.append(job)
    say("applications of two threads")
    _both(jobs, 100)


def test_transforms_of_two_threads(otfs):
    import torch
    jobs = []
    for M, N in ((64, 72), (64, 2048)):
        x = torch.view_as_complex(torch.randn(3 * M * N, 2, device="cuda"))
        want = otfs.dzt(x, M, N).clone()
        torch.cuda.synchronize()

        def job(i, M=M, N=N, x=x, want=want):
            got = otfs.dzt(x, M, N)
            assert torch.equal(torch.view_as_real(got), torch.view_as_real(want)), i
        jobs.append(job)
    say("transforms of two threads")
    _both(jobs, 100)
