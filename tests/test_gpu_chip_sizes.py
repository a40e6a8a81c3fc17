"""Batches on every size of sub-grid (asserted from the log) and with kernels of
one and two sets of lanes, and a captured short call whose replay meets invalid
data."""
import re

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

import oracle  # noqa: E402
from paper_2409_08090_amd import mils, workloads  # noqa: E402


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)).cuda()


@pytest.fixture
def logged(monkeypatch):
    monkeypatch.setenv("MILS_LOG_LEVEL", "2")
    ctx = mils.Context(0)
    yield ctx
    ctx.close()
    monkeypatch.delenv("MILS_LOG_LEVEL")
    mils.Context(0).close()


SIZES = (256, 1024, 2048, 4096, 8192)


# layouts of `count` series of nd points, and the sub-grid that most of them take
@pytest.mark.parametrize("count,nd,n", [(4, 300, 256), (10, 900, 1024), (16, 2000, 2048),
                                        (64, 1000, 4096), (200, 1900, 8192)])
@pytest.mark.parametrize("eps", [1e-9, 1e-11, 1e-13])
def test_batches_on_every_size(count, nd, n, eps, logged, capfd):
    rng = np.random.default_rng(count)
    curves = [workloads.batch_curve(rng, nd - i % 7) for i in range(count)]
    t, y, dy, nd_off, nf_off, f0, df = mils.pack_curves(curves)
    args = (t, y, dy, nd_off, nf_off, f0, df)
    on = mils.periodogram_batch(*args, eps=eps, ctx=logged).cpu().numpy()
    log = capfd.readouterr().err
    logged.set_batch_onchip(False)
    off = mils.periodogram_batch(*args, eps=eps, ctx=logged).cpu().numpy()
    took = [int(x) for x in re.search(r"batch of \d+: (\d+) staged, on sub-grids of 256 (\d+), "
                                      r"1024 (\d+), 2048 (\d+), 4096 (\d+), 8192 (\d+)",
                                      log).groups()]
    if eps == 1e-9:
        assert took[1 + SIZES.index(n)] > count // 2, (took, log[-500:])
    assert took[0] == 0 and sum(took) == count
    tol = max(10 * eps, 1e-11)
    for i in range(count):
        a, b = on[nf_off[i]:nf_off[i + 1]], off[nf_off[i]:nf_off[i + 1]]
        assert np.max(np.abs(a - b)) <= 2 * tol * np.max(np.abs(b)), i
    c = curves[-1]
    k = np.unique(np.concatenate([np.arange(300), rng.integers(0, c.nf, 300)]))
    ref = oracle.periodogram(c.t, c.y, c.dy, c.f0, c.df, k=k)
    assert np.max(np.abs(on[nf_off[-2]:][k] - ref)) <= tol * np.max(np.abs(ref))


@pytest.mark.parametrize("nd,nf", [(300, 3600), (9000, 90_000)])
def test_status_of_a_captured_call_is_the_replays(nd, nf):
    """Valid data at the capture, then a value that is not finite, then valid
    data again: the status word that the replay's kernels leave."""
    c = workloads.uniform_series(seed=nd, nd=nd, nf=nf, span=30.0)
    t, y, dy = dev(c.t), dev(c.y), dev(c.dy)
    ctx = mils.Context(0)
    try:
        eager = mils.periodogram(t, y, dy, c.f0, c.df, c.nf, ctx=ctx).cpu().numpy()
        out = torch.empty(c.nf, dtype=torch.float64, device="cuda")
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            mils.periodogram(t, y, dy, c.f0, c.df, c.nf, out=out, ctx=ctx, sync=False,
                             stream=torch.cuda.current_stream())
        y[nd // 2] = float("inf")
        g.replay()
        torch.cuda.synchronize()
        assert mils.context_status(ctx) == mils.MILS_ERR_INVALID_ARG
        y[nd // 2] = float(c.y[nd // 2])
        for _ in range(2):
            out.zero_()
            g.replay()
            torch.cuda.synchronize()
            p = out.cpu().numpy()
            assert np.max(np.abs(p - eager)) <= 1e-12 * np.max(np.abs(eager))
        del g
    finally:
        ctx.close()
