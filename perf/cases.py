"""The work that a user of this package has it do, as cases that can be timed.

Every case is a call of the public Python entry points on seeded inputs of the
package's own workload recipes (workloads.py), drawn here on the GPU so that
making them is quick:

  single   mils.periodogram: one series, FP64 or FP32 form, with or without dy,
           sorted or not
  sums     mils.trig_sums: the raw sums of one series
  shared   mils.periodogram_shared_t: several series on the same times
  batch    mils.periodogram_batch: many independent series
  direct   mils.direct_periodogram: term-by-term sums (the brute-force check)
  serve    mils.Server: a burst of host requests, submitted and taken back

The FP32 batches stay small enough that no band of sizes reaches the count at
which the batch autotuner times candidates: its choice of sigma would change
the FP32 rounding from one process to the next.  For the same reason the
served requests are FP64 (which requests share a batch depends on timing).
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2409_08090_amd import mils

EPS = {"fp64": 1e-9, "fp32": 1e-5}
SEASON, YEAR = 245.0, 365.0


def listed():
    return [
        # the shortest series of the paper's range: launch latency
        dict(name="tiny_fp64", kind="single", nd=100, nf=1200, precision="fp64", dy=True,
             sorted=True, norm="standard", fit_mean=True),
        # the interactive call: one ordinary light curve
        dict(name="small_fp64", kind="single", nd=1000, nf=12000, precision="fp64", dy=True,
             sorted=True, norm="standard", fit_mean=True),
        # an ordinary curve without errors at odd sizes, FP32 form
        dict(name="odd_fp32", kind="single", nd=3001, nf=36011, precision="fp32", dy=False,
             sorted=True, norm="standard", fit_mean=True),
        # a long survey light curve
        dict(name="medium_fp64", kind="single", nd=100_003, nf=1_200_037, precision="fp64",
             dy=True, sorted=True, norm="standard", fit_mean=True),
        # the headline: the longest series of the paper's range, both forms
        dict(name="large_fp64", kind="single", nd=1_000_000, nf=12_000_000, precision="fp64",
             dy=True, sorted=True, norm="standard", fit_mean=True),
        dict(name="large_fp32", kind="single", nd=1_000_000, nf=12_000_000, precision="fp32",
             dy=True, sorted=True, norm="standard", fit_mean=True),
        # raw sums of unordered points (event lists are not sorted)
        dict(name="sums_unsorted", kind="sums", nd=30_011, nf=360_137, precision="fp64",
             sorted=False),
        # the paper's batched mode: several bands or targets of one cadence
        dict(name="shared_fp64", kind="shared", nd=400_000, nf=4_800_000, nseries=8,
             precision="fp64"),
        # a survey batch: 10^4 series of 10^2 .. 10^4 points
        dict(name="batch_fp64", kind="batch", ncurves=10_000, nd_min=100, nd_max=10_000,
             precision="fp64", dy=True),
        # one field of a survey in the FP32 form
        dict(name="batch_fp32", kind="batch", ncurves=64, nd_min=100, nd_max=10_000,
             precision="fp32", dy=True),
        # the brute-force check of an ordinary curve
        dict(name="direct", kind="direct", nd=10_000, nf=120_000, dy=True),
        # a burst of requests to the serving loop
        dict(name="serve_burst", kind="serve", nreq=40, nd_min=50, nd_max=5000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: sizes log-uniform, N_f about 12 N_d
    and mostly odd."""
    kind = rng.choice(["single"] * 5 + ["sums", "shared", "batch", "direct", "serve"])
    if kind == "single":
        nd = _log_int(rng, 100, 1_000_000)
        return dict(kind=kind, nd=nd, nf=12 * nd - rng.randrange(nd // 8),
                    precision=rng.choice(["fp64", "fp64", "fp32"]), dy=rng.random() < 0.8,
                    sorted=rng.random() < 0.8,
                    norm=rng.choice(["standard", "standard", "model", "log", "psd"]),
                    fit_mean=rng.random() < 0.8)
    if kind == "sums":
        nd = _log_int(rng, 100, 500_000)
        return dict(kind=kind, nd=nd, nf=12 * nd - rng.randrange(nd // 8), precision="fp64",
                    sorted=rng.random() < 0.5)
    if kind == "shared":
        nd = _log_int(rng, 1000, 400_000)
        return dict(kind=kind, nd=nd, nf=12 * nd - rng.randrange(nd // 8),
                    nseries=rng.randrange(2, 9), precision="fp64")
    if kind == "batch":
        prec = rng.choice(["fp64", "fp32"])
        return dict(kind=kind, ncurves=_log_int(rng, 8, 2000 if prec == "fp64" else 64),
                    nd_min=100, nd_max=_log_int(rng, 1000, 10_000), precision=prec,
                    dy=rng.random() < 0.8)
    if kind == "direct":
        nd = _log_int(rng, 500, 10_000)
        return dict(kind=kind, nd=nd, nf=12 * nd - rng.randrange(nd // 8), dy=rng.random() < 0.8)
    return dict(kind=kind, nreq=rng.randrange(8, 41), nd_min=50, nd_max=_log_int(rng, 500, 5000))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _device():
    return torch.device("cuda", torch.cuda.current_device())


def _gen(seed):
    g = torch.Generator(device=_device())
    g.manual_seed(int(seed))
    return g


def _u(g, n, lo=0.0, hi=1.0):
    return torch.rand(n, generator=g, device=g.device, dtype=torch.float64) * (hi - lo) + lo


def _normal(g, n, sd):
    return torch.randn(n, generator=g, device=g.device, dtype=torch.float64) * sd


def _season_times(g, nd, years, in_order=True):
    """Times uniform on `years` observing seasons of 245 days in a year of 365."""
    t = torch.floor(_u(g, nd, 0.0, years)) * YEAR + _u(g, nd, 0.0, SEASON)
    return torch.sort(t).values if in_order else t


def _three_sines(g, t, noise):
    y = _normal(g, t.numel(), noise)
    f, a, ph = _u(g, 3, 0.01, 5.0), _u(g, 3, 0.1, 1.0), _u(g, 3, 0.0, 2 * math.pi)
    for i in range(3):
        y += a[i] * torch.sin(2 * math.pi * f[i] * t + ph[i])
    return y


def _batch_sizes(case):
    """Sizes, spans and grids of the series: the case's own (a seed changes the
    data, not the layout)."""
    n = case["ncurves"] if case["kind"] == "batch" else case["nreq"]
    rng = np.random.default_rng([n, case["nd_min"], case["nd_max"]])
    nd = np.floor(np.exp(rng.uniform(np.log(case["nd_min"]), np.log(case["nd_max"]), n)))
    nd = nd.astype(np.int64)
    span = np.exp(rng.uniform(np.log(10.0), np.log(1000.0), n))
    return nd, span, 12 * nd, 1.0 / (5.0 * span)


def _batch_series(case, seed):
    """Concatenated t, y, dy on the GPU: sorted uniform times on each series'
    span, one sinusoid + N(0, 0.5^2), dy = 0.5; f0 = df = 1 / (5 span)."""
    nd, span, nf, df = _batch_sizes(case)
    g = _gen(seed)
    dev = _device()
    seg = torch.repeat_interleave(torch.arange(len(nd), device=dev), torch.from_numpy(nd).to(dev))
    x = torch.sort(seg.double() + _u(g, int(nd.sum()))).values - seg.double()
    t = x * torch.from_numpy(span).to(dev)[seg]
    lo = torch.from_numpy(20 * df).to(dev)
    hi = torch.from_numpy(0.8 * nf * df).to(dev)
    f = lo + _u(g, len(nd)) * (hi - lo)
    ph = _u(g, len(nd), 0.0, 2 * math.pi)
    y = torch.sin(2 * math.pi * f[seg] * t + ph[seg]) + _normal(g, t.numel(), 0.5)
    return nd, nf, df, t, y, torch.full_like(t, 0.5)


def _inputs(case, seed):
    kind = case["kind"]
    if kind in ("batch", "serve"):
        nd, nf, df, t, y, dy = _batch_series(case, seed)
        return dict(t=t, y=y, dy=dy, df=df,
                    nd_off=np.concatenate([[0], np.cumsum(nd)]).astype(np.int64),
                    nf_off=np.concatenate([[0], np.cumsum(nf)]).astype(np.int64))
    g = _gen(seed)
    nd = case["nd"]
    years = 10 if nd >= 20_000 else 1
    s = dict(df=1.0 / (5.0 * YEAR * years))
    s["t"] = _season_times(g, nd, years, case.get("sorted", True))
    if kind == "sums":
        s["h"] = _normal(g, nd, 1.0)
        return s
    ns = case.get("nseries")
    if ns:
        s["y"] = torch.stack([_three_sines(g, s["t"], 0.2) for _ in range(ns)])
    else:
        s["y"] = _three_sines(g, s["t"], 0.2)
    s["dy"] = _u(g, nd, 0.1, 0.3) if case.get("dy", True) else None
    return s


@functools.lru_cache(maxsize=None)
def _server(nf_max):
    """The program's one server, its plan classes built ahead of traffic."""
    srv = mils.Server(lanes=2)
    if srv.warm(nf_max) != mils.MILS_OK:
        raise RuntimeError("server warm-up failed")
    return srv


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    kind = case["kind"]
    if kind == "serve":
        host = [None if s[k] is None else s[k].cpu().numpy() for k in ("t", "y", "dy")]
        s["requests"] = []
        for i in range(case["nreq"]):
            j = slice(int(s["nd_off"][i]), int(s["nd_off"][i + 1]))
            nf = int(s["nf_off"][i + 1] - s["nf_off"][i])
            s["requests"].append((*(np.ascontiguousarray(h[j]) for h in host), float(s["df"][i]), nf))
        s["server"] = _server(12 * 5000)
    elif kind == "batch":
        if not case["dy"]:
            s["dy"] = None
        s["out"] = torch.empty(int(s["nf_off"][-1]), dtype=torch.float64, device=_device())
    elif kind == "shared":
        s["out"] = torch.empty((case["nseries"], case["nf"]), dtype=torch.float64, device=_device())
    elif kind in ("single", "direct"):
        s["out"] = torch.empty(case["nf"], dtype=torch.float64, device=_device())
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(s):
    c = s["case"]
    kind, df = c["kind"], s["df"]
    if kind == "single":
        return mils.periodogram(s["t"], s["y"], s["dy"], df, df, c["nf"], eps=EPS[c["precision"]],
                                precision=c["precision"], normalization=c["norm"],
                                fit_mean=c["fit_mean"], out=s["out"])
    if kind == "sums":
        return mils.trig_sums(s["t"], s["h"], df, df, c["nf"], eps=EPS[c["precision"]],
                              precision=c["precision"])
    if kind == "shared":
        return mils.periodogram_shared_t(s["t"], s["y"], s["dy"], df, df, c["nf"],
                                         eps=EPS[c["precision"]], precision=c["precision"],
                                         out=s["out"])
    if kind == "batch":
        return mils.periodogram_batch(s["t"], s["y"], s["dy"], s["nd_off"], s["nf_off"], df, df,
                                      eps=EPS[c["precision"]], precision=c["precision"],
                                      out=s["out"])
    if kind == "direct":
        return mils.direct_periodogram(s["t"], s["y"], s["dy"], df, df, c["nf"], out=s["out"])
    srv, tickets, got = s["server"], [], []
    for t, y, dy, d, nf in s["requests"]:
        rc, ticket = srv.submit(t, y, dy, d, d, nf)
        if rc != mils.MILS_OK:
            raise RuntimeError(mils.status_str(rc))
        tickets.append((ticket, nf))
    for ticket, nf in tickets:
        srv.wait(ticket)
        rc, power, _ = srv.take(ticket, nf)
        if rc != mils.MILS_OK:
            raise RuntimeError(mils.status_str(rc))
        got.append(power)
    return got


def work(case):
    """Each input read and each output written once; the arithmetic of the
    method: three transforms of 1.25 N_f cells (one for raw sums, and for each
    series of a shared cadence after the first two) and the kernel-weighted
    additions of every point; the direct form takes the three sums at 12
    operations for each point and frequency (products of two phase factors
    that a pair of frequencies shares)."""
    kind = case["kind"]

    def transform(nf):
        n = max(16.0, 1.25 * nf)
        return 5.0 * n * math.log2(n)

    w = 8 if case.get("precision") == "fp32" else 14
    if kind in ("batch", "serve"):
        m = case["ncurves"] if kind == "batch" else case["nreq"]
        lo, hi = case["nd_min"], case["nd_max"]
        mean = (hi - lo) / math.log(hi / lo) if hi > lo else lo
        return {"bytes": m * mean * (24 + 8 * 12),
                "flops": m * (3 * transform(12 * mean) + 12 * w * mean)}
    nd, nf = case["nd"], case["nf"]
    if kind == "sums":
        return {"bytes": 16.0 * nd + 16.0 * nf, "flops": transform(nf) + 4.0 * w * nd}
    if kind == "shared":
        m = case["nseries"]
        return {"bytes": (16.0 + 8 * m) * nd + 8.0 * m * nf,
                "flops": (2 + m) * (transform(nf) + 4.0 * w * nd)}
    read = (24.0 if case["dy"] else 16.0) * nd
    if kind == "direct":
        return {"bytes": read + 8.0 * nf, "flops": 12.0 * nd * nf}
    return {"bytes": read + 8.0 * nf, "flops": 3 * transform(nf) + 12.0 * w * nd}


# ---------------------------------------------------------------------------
# the same in 64 bits with plain torch
# ---------------------------------------------------------------------------
def _two_sum(a, b):
    s = a + b
    x = s - a
    return s, (a - (s - x)) + (b - x)


def _two_prod(a, b):
    """a * b as an exact pair (Dekker's splitting)."""
    p = a * b

    def halves(x):
        y = x * 134217729.0
        hi = y - (y - x)
        return hi, x - hi

    ah, al = halves(a)
    bh, bl = halves(b)
    return p, ((ah * bh - p) + ah * bl + al * bh) + al * bl


def _phase(fh, fl, t):
    """exp(2 pi i (fh + fl) t), the product reduced mod 1 before it is rounded."""
    p, e = _two_prod(fh, t)
    r = (p - torch.floor(p)) + (e + fl * t)
    x = 2 * math.pi * (r - torch.round(r))
    return torch.complex(torch.cos(x), torch.sin(x))


def _sums(t, f0, df, nf, strengths, twice):
    """sum_j h_j exp(2 pi i f_k t_j), f_k = f0 + k df, for each h of strengths
    (and at 2 f_k for those of twice), as one product of matrices: with
    k = q R + r the phase factor is that of f0 + q R df times that of r df."""
    dev = t.device
    R = max(1, int(math.isqrt(nf)))
    Q = -(-nf // R)
    q = torch.arange(Q, device=dev, dtype=torch.float64)[:, None]
    r = torch.arange(R, device=dev, dtype=torch.float64)[None, :]
    d = torch.tensor(df, device=dev, dtype=torch.float64)
    kh, kl = _two_prod(q * R, d)
    fh, fe = _two_sum(torch.full_like(kh, f0), kh)
    rh, rl = _two_prod(r, d)
    out = [torch.zeros((Q, R), dtype=torch.complex128, device=dev) for _ in strengths + twice]
    step = max(256, 60_000_000 // max(Q, R))
    for j in range(0, t.numel(), step):
        tj = t[j:j + step]
        a = _phase(fh, fe + kl, tj[None, :])
        b = _phase(rh, rl, tj[:, None])
        for i, h in enumerate(strengths):
            out[i] += torch.mm(a * h[None, j:j + step], b)
        if twice:
            a, b = a * a, b * b
            for i, h in enumerate(twice):
                out[len(strengths) + i] += torch.mm(a * h[None, j:j + step], b)
    return [o.reshape(-1)[:nf] for o in out]


def _powers(t, ys, dy, df, nf, norm="standard", fit_mean=True):
    """The least-squares power of each series of ys at f_k = (k + 1) df."""
    w = torch.ones_like(t) if dy is None else 1.0 / (dy * dy)
    W = w.sum()
    wh = w / W
    ys = [y - (wh * y).sum() for y in ys]
    *As, B, B2 = _sums(t, df, df, nf, [wh * y for y in ys] + [wh], [wh])
    CC, SS, CS = 0.5 * (1 + B2.real), 0.5 * (1 - B2.real), 0.5 * B2.imag
    if fit_mean:
        CC, SS, CS = CC - B.real ** 2, SS - B.imag ** 2, CS - B.real * B.imag
    D = CC * SS - CS * CS
    got = []
    for y, A in zip(ys, As):
        N = SS * A.real ** 2 + CC * A.imag ** 2 - 2 * CS * A.real * A.imag
        YY = (wh * y * y).sum()
        got.append({"standard": lambda: N / (YY * D), "model": lambda: N / (YY * D - N),
                    "log": lambda: -torch.log1p(-N / (YY * D)),
                    "psd": lambda: 0.5 * W * N / D}[norm]())
    return got


def exact(case, seed):
    kind = case["kind"]
    s = _inputs(case, seed)
    if kind in ("batch", "serve"):
        if kind == "batch" and not case["dy"]:
            s["dy"] = None
        got = []
        for i in range(len(s["df"])):
            j = slice(int(s["nd_off"][i]), int(s["nd_off"][i + 1]))
            dy = None if s["dy"] is None else s["dy"][j]
            nf = int(s["nf_off"][i + 1] - s["nf_off"][i])
            got += _powers(s["t"][j], [s["y"][j]], dy, float(s["df"][i]), nf)
        return torch.cat(got) if kind == "batch" else [p.cpu().numpy() for p in got]
    if kind == "sums":
        return _sums(s["t"], s["df"], s["df"], case["nf"], [s["h"]], [])[0]
    if kind == "shared":
        return torch.stack(_powers(s["t"], list(s["y"]), s["dy"], s["df"], case["nf"]))
    return _powers(s["t"], [s["y"]], s["dy"], s["df"], case["nf"], case.get("norm", "standard"),
                   case.get("fit_mean", True))[0]
