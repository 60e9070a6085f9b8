"""The workgroups that a run reports are those of the kernel it launched, as the
profiler sees it: GPU alone and beside the host, every payload's kernels, the
engine's own choice and a caller's. In a process of its own, since the profiler
stays loaded."""
import json
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = r"""
import json, sys, tempfile
import torch
from torch.profiler import ProfilerActivity, profile
import paper_1805_02755_amd as ce

STATIC, DYNAMIC = dict(kind=ce.CE_SCHED_STATIC), dict(kind=ce.CE_SCHED_DYNAMIC, n_packages=5)
runs = []
for w, h in ((64, 64), (1024, 1024), (1920, 1080), (2560, 2001), (100, 30000), (5700, 5800)):
    runs.append((ce.CE_KERNEL_ESCAPE, ce.ce_escape_params(w, h, -2.0, -1.5, 3.0 / w, 3.0 / h, 64), [w, h], None, [],
                 w * h, 0, STATIC))
for w, h, g in ((2560, 2001, 5000), (700, 300, 4096), (700, 300, 3)):
    for sched in (STATIC, DYNAMIC):
        runs.append((ce.CE_KERNEL_ESCAPE, ce.ce_escape_params(w, h, -2.0, -1.5, 3.0 / w, 3.0 / h, 64), [w, h], None,
                     [], w * h, g, sched))
for w, h in ((640, 480), (4096, 8192)):
    runs.append((ce.CE_KERNEL_BLUR5, ce.ce_blur5_params(w, h), [w, h], None, [w * h, 25], w * h, 0, STATIC))
for n, strict in ((3000, 1), (12000, 1), (40000, 0), (100000, 1)):
    for sched in (STATIC, DYNAMIC):
        runs.append((ce.CE_KERNEL_NBODY_ACC, ce.ce_nbody_params(n, 1e-6, strict), [n], [256], [4 * n], 4 * n, 0, sched))
f = tempfile.NamedTemporaryFile(suffix=".json")
said = []
zeros = torch.zeros(1 << 26, device="cuda")
with ce.Engine() as e, profile(activities=[ProfilerActivity.CUDA]) as prof:
    for kid, prm, gws, lws, ins, n_out, g, sched in runs:
        e.use(ce.CE_DEV_GPU, 0, 0)
        e.gpu_workgroups(g)
        e.work_items(gws, lws)
        e.scheduler(**sched)
        e.program_kernel(kid, prm)
        for s, n in enumerate(ins):
            e.program_in(s, dev=zeros, nbytes=4 * n)
        out = torch.empty(n_out, device="cuda")
        e.program_out(0, dev=out, nbytes=4 * n_out)
        e.run()
        said.append(e.stats().gpu_workgroups)
    torch.cuda.synchronize()
prof.export_chrome_trace(f.name)
launched = []
for ev in sorted((x for x in json.load(open(f.name))["traceEvents"] if x.get("cat") == "kernel"), key=lambda x: x["ts"]):
    if any(k in ev["name"] for k in ("k_sweep", "k_direct", "k_wide", "k_feed", "k_persistent")):
        launched.append([ev["name"], ev["args"]["grid"][0]])
print("GRIDS " + json.dumps([said, launched]))
"""


def test_reported_workgroups_are_the_launched_ones():
    p = subprocess.run([sys.executable, "-c", CHILD], cwd=ROOT, capture_output=True, text=True, timeout=100)
    line = [x for x in p.stdout.splitlines() if x.startswith("GRIDS ")]
    assert p.returncode == 0 and line, p.stdout[-2000:] + p.stderr[-2000:]
    said, launched = json.loads(line[0][6:])
    if not launched:
        pytest.skip("the profiler recorded no kernels")
    assert [g for _, g in launched] == said, list(zip(said, launched))
