"""A served FP64 request gets the same grid whatever it is batched with: the
requests of a burst against the same requests one at a time, at a tolerance
whose transform error (1e-7 and more) would show another grid.  What is left
is the order of the atomic additions in LDS."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_2409_08090_amd import mils, workloads  # noqa: E402

EPS = 1e-5


# short series on sub-grids, on the edge between them and the staged phases,
# and staged ones whose grids lie within 6 % of each other
@pytest.mark.parametrize("sizes", [(60, 200, 700, 1000, 1100), (3000, 3900, 4300, 5200, 6100),
                                   (7000, 7300, 7600, 8000, 16000), (90, 1000, 5000, 9000, 12000)])
def test_alone_and_in_a_burst(sizes):
    rng = np.random.default_rng(sum(sizes))
    curves = [workloads.batch_curve(rng, int(n)) for n in sizes]
    srv = mils.Server(0, lanes=1)

    def submit(c):
        rc, tk = srv.submit(c.t, c.y, c.dy, c.f0, c.df, c.nf, eps=EPS)
        assert rc == mils.MILS_OK
        return tk

    def take(tk, c):
        assert srv.wait(tk, 60_000_000) == mils.MILS_OK
        rc, p, st = srv.take(tk, c.nf)
        assert rc == mils.MILS_OK
        return p, st["batch_size"]

    alone = [take(submit(c), c)[0] for c in curves]
    burst = curves * 8
    got = [take(tk, c) for tk, c in [(submit(c), c) for c in burst]]
    assert max(n for _, n in got) > 1
    for i, (p, _) in enumerate(got):
        a = alone[i % len(curves)]
        assert np.max(np.abs(p - a)) <= 1e-11 * np.max(np.abs(a)), sizes[i % len(curves)]
    srv.close()
