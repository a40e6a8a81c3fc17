"""Statistics, binning, row flags and the fused spread of one staged series, at
the sizes where a branch changes: sorted points, points out of order, sorted
points whose bins descend, gaps, histograms scanned by one block and by many,
direct sums inside the spread's launch and beside the FFT.  Against the
reproducible mode (its own binning and unfused kernels) and the CPU oracle."""
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


# the paths' tolerances on the power against the oracle; both sides of a
# comparison carry one
TOL = {"fp64": 1e-8, "fp32": 1e-4}
EPS = {"fp64": 1e-9, "fp32": 1e-5}


def order_points(t, order, rng):
    """t in one of the orders the binning tells apart."""
    t = np.sort(t)
    if order == "gap":  # two stretches of points with empty bins between them
        s = t - t[0]
        span = s[-1]
        t = np.sort(np.where(s < span / 2, 0.6 * s, 0.7 * span + 0.6 * (s - span / 2)))
    elif order == "shuffled":
        rng.shuffle(t)
    elif order == "one_swap":  # one pair out of order, across workgroups
        t[[1, -2]] = t[[-2, 1]]
    return t


@pytest.mark.parametrize("nd,nf", [(6000, 6001), (6000, 30_011), (16_385, 200_003),
                                   (40_000, 700_001), (200_000, 100_003), (200_001, 100_003)])
@pytest.mark.parametrize("order", ["sorted", "gap", "shuffled", "one_swap"])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_single(nd, nf, order, precision):
    rng = np.random.default_rng(nd + nf)
    c = workloads.uniform_series(seed=nd + nf, nd=nd, nf=nf, span=30.0)
    t = order_points(c.t.copy(), order, rng)
    args = (dev(t), dev(c.y), dev(c.dy), c.f0, c.df, c.nf)
    p = mils.periodogram(*args, eps=EPS[precision], precision=precision).cpu().numpy()
    q = mils.periodogram(*args, eps=EPS[precision], precision=precision,
                         deterministic=True).cpu().numpy()
    k = np.unique(np.concatenate([np.arange(20), rng.integers(0, nf, 20), [nf - 1]]))
    ref = oracle.periodogram(t, c.y, c.dy, c.f0, c.df, k=k)
    scale = np.max(np.abs(q))
    assert rel(p, q) <= 2 * TOL[precision]
    assert np.max(np.abs(p[k] - ref)) <= TOL[precision] * scale


@pytest.mark.parametrize("nd,df,nf", [(7000, 1.0, 9001), (7000, 0.7, 120_001)])
def test_sorted_points_whose_bins_descend(nd, df, nf):
    # a span of many periods of 1 / df: the bins wrap round while t ascends
    rng = np.random.default_rng(nd)
    t = np.sort(rng.uniform(0.0, 40.0, nd))
    y = rng.normal(0.0, 1.0, nd)
    p = mils.periodogram(dev(t), dev(y), None, 0.3, df, nf).cpu().numpy()
    q = mils.periodogram(dev(t), dev(y), None, 0.3, df, nf, deterministic=True).cpu().numpy()
    assert rel(p, q) <= 2 * TOL["fp64"]
    h = mils.trig_sums(dev(t), dev(y), 0.3, df, nf).cpu().numpy()
    k = rng.integers(0, nf, 40)
    assert np.max(np.abs(h[k] - oracle.trig_sums(t, y, 0.3, df, k=k))) <= 1e-9 * np.sum(np.abs(y))


def test_status_and_ill_posed_counts_between_calls():
    # the words that a call leaves on the host belong to that call alone
    ctx = mils.Context()
    rng = np.random.default_rng(9)
    nd, nf = 6000, 12_001
    t, y = np.sort(rng.uniform(0.0, 400.0, nd)), rng.normal(0.0, 1.0, nd)

    def call(t, y, f0, df):
        p = mils.periodogram(dev(t), dev(y), None, f0, df, nf, ctx=ctx).cpu().numpy()
        assert mils.context_illposed(ctx) == int(np.isnan(p).sum())
        return p

    good = call(t, y, 0.01, 0.0007)
    assert not np.isnan(good).any()
    # evenly spaced times: the sine vanishes at multiples of the Nyquist frequency
    comb = call(np.arange(nd) / nd, y, 0.5, 0.5)
    assert np.isnan(comb).any()
    bad = y.copy()
    bad[nd // 2] = np.nan
    with pytest.raises(mils.MilsError, match="non-finite"):
        call(t, bad, 0.01, 0.0007)
    again = call(t, y, 0.01, 0.0007)
    assert not np.isnan(again).any() and rel(again, good) <= 2 * TOL["fp64"]
    with pytest.raises(mils.MilsError, match="constant"):
        call(t, np.full(nd, 2.0), 0.01, 0.0007)
