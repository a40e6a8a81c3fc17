"""Batches whose staged grids the context's budget has no room for, while the
16 bytes a point that sub-grids in LDS need fit."""
import os
import subprocess
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

import oracle  # noqa: E402
from paper_2409_08090_amd import mils, workloads  # noqa: E402


# enough series of a size for the tuner to try staged candidates (16), and fewer
@pytest.mark.parametrize("count", [20, 6])
def test_batch_on_sub_grids_where_staged_grids_do_not_fit(count):
    rng = np.random.default_rng(count)
    curves = [workloads.batch_curve(rng, 6000 + i) for i in range(count)]
    t, y, dy, nd_off, nf_off, f0, df = mils.pack_curves(curves)
    # one staged series takes 4.5 MB of grids, more than the half of the budget
    # that a chunk may
    ctx = mils.Context(0, hbm_budget_bytes=6 << 20)
    try:
        p = mils.periodogram_batch(t, y, dy, nd_off, nf_off, f0, df, ctx=ctx)
        again = mils.periodogram_batch(t, y, dy, nd_off, nf_off, f0, df, ctx=ctx)
        p, again = p.cpu().numpy(), again.cpu().numpy()
        for c in (0, count - 1):
            k = np.unique(np.concatenate([np.arange(40), rng.integers(0, curves[c].nf, 200)]))
            ref = oracle.periodogram(curves[c].t, curves[c].y, curves[c].dy, curves[c].f0,
                                     curves[c].df, k=k)
            for q in (p, again):
                assert np.max(np.abs(q[nf_off[c] + k] - ref)) <= 1e-8 * np.max(np.abs(ref))
    finally:
        ctx.close()


REPEAT = """
import sys
sys.path.insert(0, {root!r})
import numpy as np
from paper_2409_08090_amd import mils, workloads
rng = np.random.default_rng(20)
t, y, dy, nd_off, nf_off, f0, df = mils.pack_curves([workloads.batch_curve(rng, 6000) for _ in range(20)])
ctx = mils.Context(0, hbm_budget_bytes=6 << 20)
for i in range(3):
    print("call", i, file=sys.stderr, flush=True)
    mils.periodogram_batch(t, y, dy, nd_off, nf_off, f0, df, ctx=ctx)
ctx.close()
print("ok")
"""


def test_refused_candidates_are_tried_once():
    """The tuner tries a band's candidates on the first call only, also when
    there was memory for none."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    env = dict(os.environ, MILS_LOG_LEVEL="2")
    env.pop("MILS_TUNE_CACHE", None)
    r = subprocess.run([sys.executable, "-c", REPEAT.format(root=root)], capture_output=True,
                       text=True, timeout=110, env=env)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stderr[-2000:]
    first, second, third = r.stderr.split("call ")[1:]
    assert "HBM budget" in first, first
    assert "HBM budget" not in second + third, second + third
