"""Series that share their times, in groups (one spread and one set of direct
sums for up to three series), against single calls: group sizes, a bad and a
constant series in a group, few and many points (the number of partial sums
of the direct frequencies), both precisions, centred or not."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_2409_08090_amd import mils  # noqa: E402


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)).cuda()


# both sides take the same grid and kernel: the order of additions differs
TOL = {"fp64": 1e-11, "fp32": 1e-4}


@pytest.mark.parametrize("precision,eps", [("fp64", 1e-9), ("fp32", 1e-5)])
@pytest.mark.parametrize("nd,nf", [(3000, 40_001), (6000, 90_001), (150_000, 200_003),
                                   (300_000, 100_003)])
@pytest.mark.parametrize("nseries", [1, 2, 3, 4])
def test_groups_match_single_calls(precision, eps, nd, nf, nseries):
    rng = np.random.default_rng(nd + nseries)
    t = np.sort(rng.uniform(0.0, 900.0, nd))
    y = rng.normal(2.0, 1.0, (nseries, nd))
    dy = rng.uniform(0.5, 1.0, nd)
    kw = dict(eps=eps, precision=precision, center_data=nseries != 2)
    f0, df = 1.0 / 4500.0, 1.0 / 4500.0
    s = mils.periodogram_shared_t(dev(t), dev(y), dev(dy), f0, df, nf, **kw).cpu().numpy()
    for i in range(nseries):
        p = mils.periodogram(dev(t), dev(y[i]), dev(dy), f0, df, nf, **kw).cpu().numpy()
        assert np.max(np.abs(s[i] - p)) <= TOL[precision] * np.max(np.abs(p))


@pytest.mark.parametrize("first", [0, 1, 2])
def test_bad_series_leave_the_others_of_their_group(first):
    rng = np.random.default_rng(first)
    nd, nf = 9000, 90_001
    t, y = np.sort(rng.uniform(0.0, 300.0, nd)), rng.normal(0.0, 1.0, (3, nd))
    y[first] = 1.5
    y[(first + 1) % 3, 77] = np.inf
    p, st = mils.periodogram_shared_t(dev(t), dev(y), None, 0.001, 0.0007, nf, return_status=True)
    good = (first + 2) % 3
    assert st[good] == 0 and st[first] != 0 and st[(first + 1) % 3] != 0
    q = mils.periodogram(dev(t), dev(y[good]), None, 0.001, 0.0007, nf).cpu().numpy()
    assert np.max(np.abs(p.cpu().numpy()[good] - q)) <= 1e-11 * np.max(np.abs(q))
