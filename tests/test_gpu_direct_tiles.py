"""The direct sums at the edges of their tiles (4096 frequencies, 32 points)
and slices of the points, against the CPU oracle to the direct path's own
tolerance (1e-10 of the power, 1e-12 of the strengths' sum), and with a memory
budget that leaves no room for slices."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

import oracle  # noqa: E402
from paper_2409_08090_amd import mils, workloads  # noqa: E402


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)).cuda()


@pytest.mark.parametrize("nd", [31, 32, 33, 64, 65, 1023])
@pytest.mark.parametrize("nf", [63, 4095, 4096, 4097, 20_001])
def test_tiles_and_slices(nd, nf):
    c = workloads.uniform_series(seed=nd + nf, nd=nd, nf=nf, span=20.0, sorted_t=False)
    p = mils.direct_periodogram(dev(c.t), dev(c.y), dev(c.dy), c.f0, c.df, c.nf).cpu().numpy()
    k = np.unique(np.concatenate([np.arange(min(nf, 150)), np.arange(max(0, nf - 150), nf)]))
    ref = oracle.periodogram(c.t, c.y, c.dy, c.f0, c.df, k=k)
    assert np.max(np.abs(p[k] - ref)) <= 1e-10 * np.max(np.abs(ref))
    g = mils.direct_trig_sums(dev(c.t), dev(c.y), -2.5, 0.01, nf).cpu().numpy()
    gr = oracle.trig_sums(c.t, c.y, -2.5, 0.01, k=k)
    assert np.max(np.abs(g[k] - gr)) <= 1e-12 * np.sum(np.abs(c.y))


def test_small_budget_takes_one_slice():
    c = workloads.uniform_series(seed=9, nd=3000, nf=30_000, span=20.0)
    full = mils.direct_periodogram(dev(c.t), dev(c.y), dev(c.dy), c.f0, c.df, c.nf).cpu().numpy()
    ctx = mils.Context(0, hbm_budget_bytes=1 << 20)
    try:
        one = mils.direct_periodogram(dev(c.t), dev(c.y), dev(c.dy), c.f0, c.df, c.nf,
                                      ctx=ctx).cpu().numpy()
    finally:
        ctx.close()
    assert np.max(np.abs(one - full)) <= 1e-12 * np.max(np.abs(full))
