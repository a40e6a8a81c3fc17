"""Series on sub-grids in LDS (one workgroup per residue of the frequency
index): single calls, raw sums, shared times and batches at the sizes where
the split can go wrong, against the CPU oracle and against the staged kernels
(the reproducible mode and batches with the on-chip path off stay on them)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

import oracle  # noqa: E402
from paper_2409_08090_amd import mils, workloads  # noqa: E402


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)).cuda()


def rel(p, ref):
    return float(np.max(np.abs(p - ref)) / np.max(np.abs(ref)))


# the transform's tolerance on the power, as for the other FP64 paths: 10 eps
def tol(eps):
    return max(10 * eps, 1e-11)


@pytest.mark.parametrize("nd,nf", [(5, 1), (5, 2), (63, 200), (64, 201), (65, 399), (129, 801),
                                   (1000, 12001), (2047, 47_999), (2049, 24_599), (4096, 49_150),
                                   (100, 150_001)])
@pytest.mark.parametrize("sorted_t", [True, False])
def test_residues_match_oracle_and_staged_path(nd, nf, sorted_t):
    c = workloads.uniform_series(seed=nd + nf, nd=nd, nf=nf, span=30.0, sorted_t=sorted_t)
    p = mils.periodogram(dev(c.t), dev(c.y), dev(c.dy), c.f0, c.df, c.nf).cpu().numpy()
    q = mils.periodogram(dev(c.t), dev(c.y), dev(c.dy), c.f0, c.df, c.nf,
                         deterministic=True).cpu().numpy()
    k = np.unique(np.concatenate([np.arange(min(nf, 300)), np.arange(max(0, nf - 300), nf)]))
    ref = oracle.periodogram(c.t, c.y, c.dy, c.f0, c.df, k=k)
    assert rel(p[k], ref) <= tol(1e-9)
    assert rel(p, q) <= 2 * tol(1e-9)


@pytest.mark.parametrize("eps", [1e-13, 1e-11, 1e-10, 1e-6, 1e-2])  # widths 15 .. 20, 10, 4
def test_kernel_widths(eps):
    c = workloads.uniform_series(seed=3, nd=700, nf=9001, span=30.0)
    p = mils.periodogram(dev(c.t), dev(c.y), dev(c.dy), c.f0, c.df, c.nf, eps=eps).cpu().numpy()
    ref = oracle.periodogram(c.t, c.y, c.dy, c.f0, c.df, nf=c.nf)
    assert rel(p, ref) <= tol(eps)


@pytest.mark.parametrize("normalization", ["standard", "model", "log", "psd"])
@pytest.mark.parametrize("center,mean,dy", [(True, True, False), (False, True, True),
                                            (True, False, True), (False, False, False)])
def test_forms_match_staged_path(normalization, center, mean, dy):
    c = workloads.uniform_series(seed=5, nd=900, nf=10_007, span=30.0)
    c.y = c.y + 2.3
    kw = dict(normalization=normalization, center_data=center, fit_mean=mean)
    d = dev(c.dy) if dy else None
    f0 = -c.df * 5000  # across f = 0
    p = mils.periodogram(dev(c.t), dev(c.y), d, f0, c.df, c.nf, **kw).cpu().numpy()
    q = mils.periodogram(dev(c.t), dev(c.y), d, f0, c.df, c.nf, deterministic=True,
                         **kw).cpu().numpy()
    assert p[5000] == 0.0 and np.array_equal(np.isnan(p), np.isnan(q))
    assert rel(p, q) <= 2 * tol(1e-9)


@pytest.mark.parametrize("nd,nf", [(1, 1), (64, 200), (777, 4801), (4000, 50_001)])
def test_raw_sums(nd, nf):
    rng = np.random.default_rng(nd)
    t, h = rng.uniform(-50.0, 900.0, nd), rng.normal(0.0, 1.0, nd)
    g = mils.trig_sums(dev(t), dev(h), -1.7, 0.00113, nf).cpu().numpy()
    k = np.unique(np.concatenate([np.arange(min(nf, 300)), np.arange(max(0, nf - 300), nf)]))
    ref = oracle.trig_sums(t, h, -1.7, 0.00113, k=k)
    assert np.max(np.abs(g[k] - ref)) <= 1e-9 * np.sum(np.abs(h))


def test_shared_times_in_chunks_with_a_bad_series():
    s = workloads.shared_times(seed=6, nd=200, nseries=131, span_years=1, shared_dy=False)
    s.y[70] = 3.0
    s.y[5, 17] = np.nan
    p, st = mils.periodogram_shared_t(dev(s.t), dev(s.y), dev(s.dy), s.f0, s.df, s.nf,
                                      return_status=True)
    p = p.cpu().numpy()
    assert st[70] == mils.MILS_ERR_DEGENERATE and st[5] == mils.MILS_ERR_INVALID_ARG
    assert np.count_nonzero(st) == 2
    for i in (0, 63, 64, 130):
        ref = oracle.periodogram(s.t, s.y[i], s.dy[i], s.f0, s.df, nf=s.nf)
        assert rel(p[i], ref) <= tol(1e-9)


@pytest.mark.parametrize("count,nd", [(3, 60), (40, 700), (500, 900), (900, 2600)])
def test_batches_of_every_grid_size(count, nd):
    """Few short series take small sub-grids, many long ones the largest."""
    rng = np.random.default_rng(count)
    curves = [workloads.batch_curve(rng, int(n)) for n in rng.integers(nd // 2, nd + 1, count)]
    t, y, dy, nd_off, nf_off, f0, df = mils.pack_curves(curves)
    ctx = mils.Context(0)
    try:
        on = mils.periodogram_batch(t, y, dy, nd_off, nf_off, f0, df, ctx=ctx).cpu().numpy()
        ctx.set_batch_onchip(False)
        off = mils.periodogram_batch(t, y, dy, nd_off, nf_off, f0, df, ctx=ctx).cpu().numpy()
    finally:
        ctx.close()
    for i in range(count):
        a, b = on[nf_off[i]:nf_off[i + 1]], off[nf_off[i]:nf_off[i + 1]]
        assert rel(a, b) <= 2 * tol(1e-9), i
    c = curves[-1]
    ref = oracle.periodogram(c.t, c.y, c.dy, c.f0, c.df, nf=c.nf)
    assert rel(on[nf_off[-2]:], ref) <= tol(1e-9)


def test_captured_call_replays():
    """A short call captured in the caller's graph, replayed with eager work
    and other calls between the replays; its status comes from the replay."""
    c = workloads.single_small(seed=4, nd=300, nf=3600)
    o = workloads.single_small(seed=5, nd=900, nf=9000)
    t, y, dy = dev(c.t), dev(c.y), dev(c.dy)
    ctx = mils.Context(0)
    eager = mils.periodogram(t, y, dy, c.f0, c.df, c.nf, ctx=ctx).cpu().numpy()
    out = torch.empty(c.nf, dtype=torch.float64, device="cuda")
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        mils.periodogram(t, y, dy, c.f0, c.df, c.nf, out=out, ctx=ctx, sync=False,
                         stream=torch.cuda.current_stream())
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert rel(out.cpu().numpy(), eager) <= 1e-13
        other = mils.periodogram(dev(o.t), dev(o.y), dev(o.dy), o.f0, o.df, o.nf, ctx=ctx)
        assert np.isfinite(other.cpu().numpy()).all()
    del g
    ctx.close()
