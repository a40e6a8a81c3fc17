"""A device without memory for the grid of a split transform, but with memory
for the staged one (the refusal is forced on the host: MILS_WORKSPACE_LIMIT):
the call falls back once, and later calls keep the workspace they have."""
import os
import re
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# nf: split grid 1310720 cells, staged about 1.07e6
PROBE = """
import os, sys
sys.path.insert(0, {root!r})
import numpy as np, torch
from paper_2409_08090_amd import mils
nd, nf = 9000, 850_001
g = torch.Generator(device="cuda")
g.manual_seed(1)
t = torch.sort(torch.rand(nd, generator=g, device="cuda", dtype=torch.float64) * 500.0).values
y = torch.randn(nd, generator=g, device="cuda", dtype=torch.float64)
args = (t, y, None, 0.001, 0.0004, nf)
ref = mils.periodogram(*args)
need = mils.plan_info(nd, nf, 1e-9)["workspace_bytes"]
os.environ["MILS_WORKSPACE_LIMIT"] = str(int(need * 0.92))
ctx = mils.Context(0)
def check(p):
    assert float((p - ref).abs().max() / ref.abs().max()) <= 1e-8
for i in range(3):
    print("call", i, file=sys.stderr, flush=True)
    check(mils.periodogram(*args, ctx=ctx))
print("capture", file=sys.stderr, flush=True)
out = torch.empty(nf, dtype=torch.float64, device="cuda")
s = torch.cuda.Stream()
s.wait_stream(torch.cuda.current_stream())
graph = torch.cuda.CUDAGraph()
with torch.cuda.graph(graph, stream=s):
    mils.periodogram(*args, out=out, ctx=ctx, sync=False, stream=torch.cuda.current_stream())
for i in range(2):
    out.zero_()
    graph.replay()
    torch.cuda.synchronize()
    check(out)
print("shared", file=sys.stderr, flush=True)
y2 = torch.stack([y, y * y])
limit = mils.plan_info(nd, nf, 1e-9)["workspace_bytes"] + 32 * nf + (1 << 20)
os.environ["MILS_WORKSPACE_LIMIT"] = str(int(limit * 0.92))
ctx2 = mils.Context(0)
for i in range(3):
    check(mils.periodogram_shared_t(t, y2, None, 0.001, 0.0004, nf, ctx=ctx2)[0])
del graph
ctx.close()
ctx2.close()
print("ok")
"""


def test_fallback_is_remembered():
    env = dict(os.environ, MILS_LOG_LEVEL="2")
    env.pop("MILS_WORKSPACE_LIMIT", None)
    r = subprocess.run([sys.executable, "-c", PROBE.format(root=ROOT)], capture_output=True,
                       text=True, timeout=110, env=env)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stderr[-3000:]
    single, shared = r.stderr[r.stderr.index("call 0"):].split("shared")
    for part in (single, shared):
        assert len(re.findall("hipMalloc of the workspace failed", part)) == 1, part
        assert len(re.findall("workspace grown", part)) == 1, part
