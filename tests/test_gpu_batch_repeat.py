"""A batch layout's first call (launched), its repeats (captured, replayed) and
layouts that alternate give the same powers and statuses; sizes grow and shrink
between calls, so that the descriptor buffers are reused and replaced."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_2409_08090_amd import mils  # noqa: E402


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)).cuda()


def layout(seed, sizes):
    rng = np.random.default_rng(seed)
    nd = np.array(sizes)
    off = np.concatenate([[0], np.cumsum(nd)])
    foff = np.concatenate([[0], np.cumsum(12 * nd + 1)])
    t = np.concatenate([np.sort(rng.uniform(0.0, 100.0, n)) for n in nd])
    y = rng.normal(0.0, 1.0, off[-1])
    y[off[1]:off[2]] = 3.0  # one constant series
    df = np.full(nd.size, 0.002)
    return dev(t), dev(y), None, off, foff, df, df


# 1500 frequencies take the in-LDS FP32 kernel, 20000 points the staged phases
@pytest.mark.parametrize("precision,eps", [("fp64", 1e-9), ("fp32", 1e-5)])
def test_first_call_repeats_and_alternation(precision, eps):
    ctx = mils.Context(0)
    calls = [layout(1, [100, 60, 5000]), layout(2, [90, 70, 20_000] + [300] * 40),
             layout(3, [128, 50])]
    first = {}
    for i in (0, 0, 0, 1, 0, 2, 1, 1, 2, 2, 0):
        p, st = mils.periodogram_batch(*calls[i], eps=eps, precision=precision, ctx=ctx,
                                       return_status=True)
        p = p.cpu().numpy()
        foff = calls[i][4]
        assert st[1] != 0 and not st[0] and not st[2:].any()
        keep = np.ones(p.size, bool)
        keep[foff[1]:foff[2]] = False  # the constant series has no power
        if i not in first:
            first[i] = p
        # the spread's order of additions may differ between calls
        tol = 1e-11 if precision == "fp64" else 1e-5
        assert np.max(np.abs(p[keep] - first[i][keep])) <= tol * np.max(np.abs(first[i][keep]))
    ctx.close()
