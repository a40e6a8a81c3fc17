"""The FP64 transform in two passes split by residue: every shape of its lines
and residue counts up to the largest, all rows reached and few, the three
kinds of last pass, against the staged passes of the same grid (the
allocation-free call, and stage timing) and the CPU oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

import oracle  # noqa: E402
from paper_2409_08090_amd import mils  # noqa: E402


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)).cuda()


def rel(p, ref):
    return float(np.max(np.abs(p - ref)) / np.max(np.abs(ref)))


# (nf: grids of 2^17 R cells for R = 2, 3, 4, 5, 6, 8, 9, 10, 12, 15, 16, and
# the two register-tile grids that the split transform takes over)
NF = [200_003, 300_007, 400_009, 500_009, 600_011, 800_011, 940_001, 1_020_001, 1_200_007,
      1_530_011, 1_630_003, 2_900_003, 3_100_001, 6_100_003]


@pytest.mark.parametrize("nf", NF)
@pytest.mark.parametrize("oversampling", [1.0, 5.0])
def test_power_against_staged_passes_and_oracle(nf, oversampling):
    rng = np.random.default_rng(nf)
    nd, span = 9000, 700.0
    t = rng.uniform(0.0, span, nd)
    if nf % 2:
        t.sort()
    y, dy = rng.normal(0.0, 1.0, nd), rng.uniform(0.5, 1.0, nd)
    df = 1.0 / (oversampling * span)
    ctx = mils.Context(0)
    args = (dev(t), dev(y), dev(dy), df, df, nf)
    p = mils.periodogram(*args, ctx=ctx).cpu().numpy()
    ctx.profile_enable(True)  # the staged passes
    q = mils.periodogram(*args, ctx=ctx).cpu().numpy()
    # the same kernel values on the same grid: FFT and spread roundings only
    assert rel(p, q) <= 1e-12
    k = np.unique(np.concatenate([np.arange(30), np.arange(nf - 30, nf),
                                  np.arange(nf // 2 - 30, nf // 2 + 30),
                                  rng.integers(0, nf, 200), np.argsort(p)[-10:]]))
    ref = oracle.periodogram(t, y, dy, df, df, k=k)
    assert np.max(np.abs(p[k] - ref)) <= 1e-8 * np.max(np.abs(ref))
    ctx.close()


@pytest.mark.parametrize("nf", [200_003, 600_011, 1_530_011])
@pytest.mark.parametrize("nseries", [1, 2, 3, 5])
def test_shared_times_match_single_calls(nf, nseries):
    rng = np.random.default_rng(nf + nseries)
    nd = 7000
    t, y = np.sort(rng.uniform(0.0, 500.0, nd)), rng.normal(0.0, 1.0, (nseries, nd))
    y[nseries // 2] += 1.0
    s = mils.periodogram_shared_t(dev(t), dev(y), None, 0.0, 0.0004, nf).cpu().numpy()
    for i in range(nseries):
        p = mils.periodogram(dev(t), dev(y[i]), None, 0.0, 0.0004, nf).cpu().numpy()
        assert rel(s[i], p) <= 1e-11


@pytest.mark.parametrize("nf", [200_003, 400_009, 1_530_011, 3_100_001])
def test_raw_sums(nf):
    rng = np.random.default_rng(nf)
    nd = 6000
    t, h = rng.uniform(-50.0, 900.0, nd), rng.normal(0.0, 1.0, nd)
    g = mils.trig_sums(dev(t), dev(h), -1.7, 0.000213, nf).cpu().numpy()
    k = np.unique(np.concatenate([np.arange(50), np.arange(nf - 50, nf), rng.integers(0, nf, 200)]))
    ref = oracle.trig_sums(t, h, -1.7, 0.000213, k=k)
    assert np.max(np.abs(g[k] - ref)) <= 1e-9 * np.sum(np.abs(h))


def test_budget_that_only_the_staged_grid_fits():
    rng = np.random.default_rng(1)
    nd, nf = 9000, 850_001  # split grid 1310720 cells, staged about 1.07e6
    t, y = np.sort(rng.uniform(0.0, 500.0, nd)), rng.normal(0.0, 1.0, nd)
    args = (dev(t), dev(y), None, 0.001, 0.0004, nf)
    need = mils.plan_info(nd, nf, 1e-9)["workspace_bytes"]
    p = mils.periodogram(*args).cpu().numpy()
    ctx = mils.Context(0, hbm_budget_bytes=int(need * 0.92) + (8 << 20))
    q = mils.periodogram(*args, ctx=ctx).cpu().numpy()
    assert rel(q, p) <= 1e-8
    ctx.close()
