"""The XCD layout is found once per process, by the first binding.  A first binding after a graph's
replay, or beside a busy stream, finds the workgroups dealt round robin from another XCD than the
first one: the XCD-local kinds and the register-resident tiles have to run there too, with the bits
of a process that did nothing before.  (Each case is a process of its own.)"""
import os
import subprocess
import sys

import pytest

from helpers import say

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CHILD = r'''
import sys
sys.path.insert(0, %r)
import hashlib
import numpy as np
import torch
import paper_2604_02266_amd as otfs
import workloads as W
before = sys.argv[1]
a = torch.ones(1000, 1000, device="cuda")
torch.cuda.synchronize()
if before == "graph":
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        b = a + 1
    g.replay()
    torch.cuda.synchronize()
elif before == "busy":
    with torch.cuda.stream(torch.cuda.Stream()):
        for _ in range(200):
            a = a @ a * 1e-6
rng = np.random.default_rng(4)
h = hashlib.sha256()
for te in (0, 4096):
    specs = [W.small_frame(rng, 512, 128, 6, (0, 20), (-6, 6)).spec for _ in range(3)]
    plan = otfs.Plan(specs, max_iters=8, rel_tol=0.0, tune=False, tile_elems=te)
    i = plan.info()
    y = rng.standard_normal((plan.total_elems, 2)).astype(np.float32)
    x = plan.lmmse_cg(torch.view_as_complex(torch.from_numpy(y).cuda()))
    torch.cuda.synchronize()
    h.update(x.cpu().numpy().tobytes())
    print("info", i.xcd_local, i.groups, i.lds_bytes)
print("bits", h.hexdigest())
''' % ROOT


def _run(before):
    say("first binding of a process", before)
    r = subprocess.run([sys.executable, "-c", CHILD, before], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    return [l for l in r.stdout.splitlines() if l.startswith(("info", "bits"))]


def test_first_binding_of_a_process():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    fresh = _run("nothing")
    assert fresh[0].split()[1] == "1" and int(fresh[0].split()[3]) == 159 * 1024
    assert fresh[1].split()[1] == "1"
    assert _run("graph") == fresh
    assert _run("busy") == fresh
