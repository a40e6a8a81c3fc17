"""Batches whose staged grids the context's budget has no room for, while the
16 bytes a point that sub-grids in LDS need fit."""
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
