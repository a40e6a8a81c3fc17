"""The allocation-free call with one path's tables after the other's in its
scratch: sub-grids in LDS, the split transform, LDS passes and the
register-tile FFT in turn, at two tolerances, each call made twice and against
mils_periodogram (same grid and kernel: rounding only)."""
import os
import re
import subprocess
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_2409_08090_amd import mils, workloads  # noqa: E402

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)).cuda()


def test_tables_of_every_path_in_turn():
    small, sub = workloads.single_small(seed=1, nd=60, nf=700), workloads.single_small(seed=2, nd=900, nf=9000)
    mid, big = workloads.single_large(seed=3, nd=9000, span_years=1), workloads.single_large(seed=4, nd=30_000, span_years=2)
    calls = [(sub, "fp64", 1e-9), (sub, "fp64", 1e-6), (mid, "fp64", 1e-9), (sub, "fp64", 1e-9),
             (big, "fp64", 1e-9), (small, "fp64", 1e-9), (mid, "fp32", 1e-5), (sub, "fp64", 1e-6),
             (big, "fp64", 1e-6), (sub, "fp64", 1e-6), (sub, "fp32", 1e-5), (big, "fp64", 1e-9)]
    a, b = mils.Context(0), mils.Context(0)
    for i, (c, prec, eps) in enumerate(calls):
        args = (dev(c.t), dev(c.y), dev(c.dy), c.f0, c.df, c.nf)
        ref = mils.periodogram(*args, eps=eps, precision=prec, ctx=a).cpu().numpy()
        for ctx in (a, b):  # the scratch is the GPU's, not the context's
            p = mils.periodogram_noalloc(*args, eps=eps, precision=prec, ctx=ctx).cpu().numpy()
            tol = 1e-12 if prec == "fp64" else 1e-6
            assert np.max(np.abs(p - ref)) <= tol * np.max(np.abs(ref)), (i, c.nd, prec, eps)
    a.close()
    b.close()


def test_budget_without_room_for_the_sub_grid_tables():
    """A short series in a context whose budget holds its staged workspace but
    not the tables of the sub-grids runs staged, call after call."""
    c = workloads.single_small(seed=5, nd=900, nf=9000)
    args = (dev(c.t), dev(c.y), dev(c.dy), c.f0, c.df, c.nf)
    ref = mils.periodogram(*args).cpu().numpy()
    need = mils.plan_info(c.nd, c.nf, 1e-9)["workspace_bytes"]
    ctx = mils.Context(0, hbm_budget_bytes=need + (96 << 10))
    for _ in range(3):
        p = mils.periodogram(*args, ctx=ctx).cpu().numpy()
        assert np.max(np.abs(p - ref)) <= 1e-8 * np.max(np.abs(ref))
    ctx.close()


# (the grids of the last two fit the scratch only as staged ones, or not split)
PROBE = """
import sys
sys.path.insert(0, {root!r})
import torch
from paper_2409_08090_amd import mils
for nf in (170_003, 480_011, 700_001, 770_001):
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    t = torch.sort(torch.rand(9000, generator=g, device="cuda", dtype=torch.float64) * 500.0).values
    y = torch.randn(9000, generator=g, device="cuda", dtype=torch.float64)
    p = mils.periodogram_noalloc(t, y, None, 0.001, 0.0004, nf)
    q = mils.periodogram(t, y, None, 0.001, 0.0004, nf)
    print("rel", nf, float((p - q).abs().max() / q.abs().max()))
"""


def test_grids_of_a_split_transform_take_it():
    """A grid that the planner chose for the split transform runs its two
    passes (the staged ones gain nothing from its size)."""
    env = dict(os.environ, MILS_LOG_LEVEL="2")
    r = subprocess.run([sys.executable, "-c", PROBE.format(root=ROOT)], capture_output=True,
                       text=True, timeout=110, env=env)
    assert r.returncode == 0, r.stderr[-2000:]
    tables = re.findall(r"scratch tables nf=(\d+) .*? n=(\d+) passes=(\d+)(.*)", r.stderr)
    assert [int(x[0]) for x in tables] == [170_003, 480_011, 700_001, 770_001], r.stderr[-2000:]
    assert all(x[2] == "2" and "split" in x[3] for x in tables[:2]), tables
    rel = [float(x) for x in re.findall(r"rel \d+ (\S+)", r.stdout)]
    assert max(rel[:2]) <= 1e-12 and max(rel) <= 1e-8, rel


def test_sub_grid_tables_make_room_for_a_larger_call():
    """A budget that holds a short and then a longer call on their staged grids
    holds them too when the short one ran on sub-grids and left their tables:
    every way through an entry point that allocates."""
    c = workloads.single_small(seed=6, nd=400, nf=4000)
    short = (dev(c.t), dev(c.y), dev(c.dy), c.f0, c.df, c.nf)
    rng = np.random.default_rng(1)
    nd, nf = 20_000, 60_000
    t, y = dev(np.sort(rng.uniform(0.0, 100.0, nd))), dev(rng.normal(0.0, 1.0, nd))
    y2 = torch.stack([y, y * y])

    def long_call(kind, ctx):
        if kind == "periodogram":
            return mils.periodogram(t, y, None, 0.002, 0.002, nf, ctx=ctx)
        if kind == "sums":
            return mils.trig_sums(t, y, 0.002, 0.002, nf, ctx=ctx).abs()
        if kind == "shared":
            return mils.periodogram_shared_t(t, y2, None, 0.002, 0.002, nf, ctx=ctx)[0]
        off, foff = np.array([0, nd], dtype=np.int64), np.array([0, nf], dtype=np.int64)
        one = np.array([0.002])
        return mils.periodogram_batch(t, y, None, off, foff, one, one, ctx=ctx)

    def fits(kind, budget, staged):
        ctx = mils.Context(0, hbm_budget_bytes=budget)
        try:
            mils.periodogram(*short, deterministic=staged, ctx=ctx)
            p = long_call(kind, ctx)
            mils.periodogram(*short, ctx=ctx)
            return p
        except mils.MilsError as e:
            assert e.status == mils.MILS_ERR_OOM
            return None
        finally:
            ctx.close()

    for kind in ("periodogram", "sums", "shared", "batch"):
        ref = long_call(kind, mils.default_context(0))
        lo, hi = 1 << 20, 1 << 26  # refused, held
        assert fits(kind, lo, True) is None and fits(kind, hi, True) is not None
        while hi - lo > 4096:
            mid = (lo + hi) // 2
            if fits(kind, mid, True) is None:
                lo = mid
            else:
                hi = mid
        p = fits(kind, hi, False)
        assert p is not None, (kind, hi)
        assert float((p - ref).abs().max() / ref.abs().max()) <= 1e-8


REFUSED = """
import sys
sys.path.insert(0, {root!r})
import torch
from paper_2409_08090_amd import mils
g = torch.Generator(device="cuda")
g.manual_seed(1)
t = torch.sort(torch.rand(400, generator=g, device="cuda", dtype=torch.float64) * 50.0).values
y = torch.randn(400, generator=g, device="cuda", dtype=torch.float64)
ctx = mils.Context(0, hbm_budget_bytes=32 << 20)
ref = mils.periodogram(t, y, None, 0.002, 0.002, 4000, ctx=ctx)
for i in range(2):
    print("refused", i, file=sys.stderr, flush=True)
    try:
        mils.periodogram(t, y, None, 0.002, 0.002, 4_000_000, ctx=ctx)
        print("not refused")
    except mils.MilsError as e:
        assert e.status == mils.MILS_ERR_OOM
    for k in range(2):
        p = mils.periodogram(t, y, None, 0.002, 0.002, 4000, ctx=ctx)
        assert float((p - ref).abs().max() / ref.abs().max()) <= 1e-12
ctx.close()
print("ok")
"""


def test_a_call_larger_than_the_budget_leaves_sub_grids_on():
    """One that the budget has no room for at all is refused; short calls after
    it take the sub-grids as before it."""
    env = dict(os.environ, MILS_LOG_LEVEL="2")
    r = subprocess.run([sys.executable, "-c", REFUSED.format(root=ROOT)], capture_output=True,
                       text=True, timeout=110, env=env)
    assert r.returncode == 0 and r.stdout.strip() == "ok", (r.stdout, r.stderr[-2000:])
    parts = r.stderr.split("refused ")
    assert [len(re.findall("on-chip tables", x)) for x in parts] == [1, 1, 1], r.stderr[-3000:]
