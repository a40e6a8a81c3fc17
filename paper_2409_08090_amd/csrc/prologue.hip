// prologue.hip -- statistics, binning and row classes of one series (gfx950),
// in as few launches as their dependences allow: a short call is bound by the
// launches and the gaps between them, not by any kernel.
//   k_pro_stats  one pass over the points: block partials of the moments, the
//                time range, validity, and whether the bins of consecutive
//                points descend (then the points need the counting sort); the
//                histogram of the sort is cleared
//   k_pro_bins   every block combines the partials (in one fixed order, so all
//                of them hold the same statistics; block 0 writes them out);
//                sorted points: the bin starts; others: the histogram, and
//                for fewer than kScanOne bins the last block to finish scans it
//   k_scan1/3    the scan of more bins
//   k_pro_rows   the points into bin order (only when they need it) and the
//                row flags of both geometries
// With the spreads and the direct sums in one launch, all grids in each FFT
// pass, and the status in pinned host memory, a periodogram of 3000 points
// takes 6 kernels instead of 17 and a copy (143 us -> 61 in FP32), one of
// 100 000 in FP64 212 us -> 154.  The bound is the 5 us from one dependent
// kernel to the next.
#include <hip/hip_runtime.h>

#include "device_math.h"
#include "kernels.h"
#include "mils_internal.h"
#include "path_device.h"

namespace mils {

namespace {

constexpr int kStatsCap = 512;      // blocks of k_pro_stats
// Bins that one block scans: 4 us per 16 k against the 10 us of two launches
// more, and up to four times that only to keep the sorted points' call short.
constexpr int kScanOne = 1 << 16;

enum { kBad = 1, kUnsorted = 2, kDescends = 4 };

struct Part {
  Moments m;
  double lo, hi;
  int flags;
};

__device__ __forceinline__ void part_merge(Part& x, const Part& y) {
  moments_merge(x.m, y.m.W, y.m.mu, y.m.M2);
  x.lo = fmin(x.lo, y.lo);
  x.hi = fmax(x.hi, y.hi);
  x.flags |= y.flags;
}

// Total of one Part per thread, in a fixed order; every thread gets it.
__device__ __forceinline__ Part block_part(Part x, Part* sh /* kThreads / 64 */) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    Part y;
    y.m.W = __shfl_down(x.m.W, off, 64);
    y.m.mu = __shfl_down(x.m.mu, off, 64);
    y.m.M2 = __shfl_down(x.m.M2, off, 64);
    y.lo = __shfl_down(x.lo, off, 64);
    y.hi = __shfl_down(x.hi, off, 64);
    y.flags = __shfl_down(x.flags, off, 64);
    part_merge(x, y);
  }
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = x;
  __syncthreads();
  x = sh[0];
#pragma unroll
  for (int i = 1; i < kThreads / 64; ++i) part_merge(x, sh[i]);
  return x;
}

__global__ __launch_bounds__(kThreads) void k_pro_stats(CallArgs a, Plan p, Work w) {
  __shared__ Part sh[kThreads / 64];
  const int64_t gtid = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  for (int64_t i = gtid; i <= p.nbins; i += stride) w.bin_count[i] = 0;
  if (gtid == 0) w.done[0] = 0;
  Part x = {{0.0, 0.0, 0.0}, INFINITY, -INFINITY, 0};
  const double* yv = a.periodogram ? a.y : a.h;
  // the time origin if the points are sorted (else the bins do not matter)
  const double tau = a.periodogram ? a.t[0] : 0.0;
  // four consecutive points a thread, so that few bins are worked out twice
  for (int64_t j0 = 4 * gtid; j0 < a.nd; j0 += 4 * stride) {
    double t[4], y[4], d[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t j = j0 + q < a.nd ? j0 + q : a.nd - 1;
      t[q] = a.t[j];
      y[q] = yv ? yv[j] : 0.0;
      d[q] = a.dy ? a.dy[j] : 1.0;
    }
    double tp = a.t[j0 > 0 ? j0 - 1 : 0];
    int bp = point_bin(tp, tau, a.df, p);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (j0 + q >= a.nd) break;
      if (!(d[q] > 0.0) || !isfinite(d[q])) x.flags |= kBad;
      const double wj = 1.0 / (d[q] * d[q]);
      if (!isfinite(t[q]) || !isfinite(y[q]) || !isfinite(wj)) x.flags |= kBad;
      const int b = point_bin(t[q], tau, a.df, p);
      if (t[q] < tp) x.flags |= kUnsorted;
      else if (b < bp) x.flags |= kDescends;
      tp = t[q];
      bp = b;
      x.lo = fmin(x.lo, t[q]);
      x.hi = fmax(x.hi, t[q]);
      moments_merge(x.m, wj, y[q], 0.0);
    }
  }
  const Part r = block_part(x, sh);
  if (threadIdx.x == 0) {
    double* o = w.partials + 8 * blockIdx.x;
    o[0] = r.m.W;
    o[1] = r.m.mu;
    o[2] = r.m.M2;
    o[3] = r.lo;
    o[4] = r.hi;
    o[5] = (double)r.flags;
  }
}

// ONE: the last block scans (its registers would cost the others occupancy).
template <bool ONE>
__global__ __launch_bounds__(kThreads) void k_pro_bins(CallArgs a, Plan p, Work w, int nparts) {
  __shared__ Part sh[kThreads / 64];
  __shared__ int scan[kThreads / 64];
  __shared__ int last;
  const int tid = threadIdx.x;
  Part x = {{0.0, 0.0, 0.0}, INFINITY, -INFINITY, 0};
  for (int i = tid; i < nparts; i += kThreads) {
    const double* q = w.partials + 8 * i;
    part_merge(x, Part{{q[0], q[1], q[2]}, q[3], q[4], (int)q[5]});
  }
  x = block_part(x, sh);
  DevStats st;
  st.W = x.m.W;
  st.mu = x.m.mu;
  st.M2 = x.m.M2;
  st.tmin = x.lo;
  st.tmax = x.hi;
  st.invalid = x.flags & kBad ? 1 : 0;
  st.unsorted = x.flags & kUnsorted ? 1 : 0;
  st.need_sort = x.flags & (kUnsorted | kDescends) ? 1 : 0;
  st.tau = a.periodogram ? x.lo : 0.0;
  st.ysub = a.center ? x.m.mu : 0.0;
  st.Ybar = a.center ? 0.0 : x.m.mu;
  st.YY = x.m.M2 / x.m.W;
  if (!a.fit_mean && !a.center) st.YY += x.m.mu * x.m.mu;
  st.status = st.invalid ? -1 : (a.periodogram && a.y && !(st.YY > 0.0)) ? -2 : 0;
  st.nill = 0;
  st.nlow = 0;
  st.k_lo = 0;
  if (blockIdx.x == 0 && tid == 0) {
    if (st.status == 0 && a.periodogram) low_band(st, a.f0, a.df, a.nf, st.k_lo, st.nlow);
    *w.stats = st;
    if (a.host_words) {
      a.host_words[0] = st.status;
      a.host_words[1] = 0;
    }
  }
  if (st.status != 0) return;
  const int nd = (int)a.nd;
  const int nb = (int)p.nbins;
  const double tau = st.tau;
  const int64_t gtid = (int64_t)blockIdx.x * kThreads + tid;
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  if (st.need_sort) {
    for (int64_t j = gtid; j < nd; j += stride)
      atomicAdd(&w.bin_count[point_bin(a.t[j], tau, a.df, p)], 1);
    if constexpr (ONE) {
      // the last block to finish scans the histogram
      __threadfence();
      __syncthreads();
      if (tid == 0) last = atomicAdd(&w.done[0], 1) == (int)gridDim.x - 1;
      __syncthreads();
      if (!last) return;
      __threadfence();
      // 16 pieces of 256 bins a wave in one round, their loads all in flight
      // (8 bins a thread and round took 31 us for 16 k bins, this 8)
      constexpr int kPieces = 16, kWaveBins = kPieces * 256, kRound = kWaveBins * kThreads / 64;
      const int lane = tid & 63, wave = tid >> 6;
      int carry = 0;
      for (int base = 0; base <= nb; base += kRound) {
        const int first = base + wave * kWaveBins + 4 * lane;
        int4 v[kPieces];
        int inc[kPieces];  // inclusive over the piece
#pragma unroll
        for (int q = 0; q < kPieces; ++q) {
          const int i = first + 256 * q;
          v[q] = make_int4(0, 0, 0, 0);
          if (i + 3 <= nb) {
            v[q] = *reinterpret_cast<const int4*>(w.bin_count + i);
          } else {
            if (i <= nb) v[q].x = w.bin_count[i];
            if (i + 1 <= nb) v[q].y = w.bin_count[i + 1];
            if (i + 2 <= nb) v[q].z = w.bin_count[i + 2];
          }
        }
#pragma unroll
        for (int q = 0; q < kPieces; ++q) {
          v[q].y += v[q].x;
          v[q].z += v[q].y;
          v[q].w += v[q].z;
          inc[q] = v[q].w;
        }
#pragma unroll
        for (int off = 1; off < 64; off <<= 1)
#pragma unroll
          for (int q = 0; q < kPieces; ++q) {
            const int y = __shfl_up(inc[q], off, 64);
            if (lane >= off) inc[q] += y;
          }
        int total = 0;  // of the wave's pieces
#pragma unroll
        for (int q = 0; q < kPieces; ++q) total += __shfl(inc[q], 63, 64);
        if (lane == 0) scan[wave] = total;
        __syncthreads();
        int run = carry;
#pragma unroll
        for (int i = 0; i < kThreads / 64; ++i) {
          if (i < wave) run += scan[i];
          carry += scan[i];
        }
#pragma unroll
        for (int q = 0; q < kPieces; ++q) {
          const int i = first + 256 * q, e = run + inc[q] - v[q].w;
          const int4 o = make_int4(e, e + v[q].x, e + v[q].y, e + v[q].z);
          if (i + 3 <= nb) {
            *reinterpret_cast<int4*>(w.bin_start + i) = o;
          } else {
            if (i <= nb) w.bin_start[i] = o.x;
            if (i + 1 <= nb) w.bin_start[i + 1] = o.y;
            if (i + 2 <= nb) w.bin_start[i + 2] = o.z;
          }
          run += __shfl(inc[q], 63, 64);
        }
        __syncthreads();
      }
    }
    return;
  }
  // Sorted points: bin_start[b] is the first point whose bin is >= b.  The
  // bins up to the first point's all start at point 0 and those after the
  // last point's at nd: the whole grid writes them (they can be most of the
  // grid: the frequency step makes the grid's period several times the time
  // span).  Every other point j starts the bins (bin(j-1), bin(j)]: each bin
  // is written by one point, and a run of 8 or more (a gap in the data) by the
  // whole wave.
  const int b_first = point_bin(a.t[0], tau, a.df, p);
  const int b_last = point_bin(a.t[nd - 1], tau, a.df, p);
  for (int64_t b = gtid; b <= nb; b += stride) {
    if (b <= b_first) w.bin_start[b] = 0;
    else if (b > b_last) w.bin_start[b] = nd;
  }
  const int lane = tid & 63;
  // wave-uniform loop over points 1 .. nd-1: every lane takes part in the
  // ballot and the shuffles
  for (int64_t j0 = 1 + (int64_t)blockIdx.x * kThreads + (tid - lane); j0 < nd; j0 += stride) {
    const int64_t j = j0 + lane;
    int lo = 0, hi = -1;  // the bins [lo, hi] that start at point j
    if (j < nd) {
      lo = point_bin(a.t[j - 1], tau, a.df, p) + 1;
      hi = point_bin(a.t[j], tau, a.df, p);
    }
    const bool run = hi - lo >= 8;
    if (!run)
      for (int b = lo; b <= hi; ++b) w.bin_start[b] = (int)j;
    unsigned long long runs = __ballot(run);
    while (runs) {
      const int src = __ffsll(runs) - 1;
      runs &= runs - 1;
      const int l = __shfl(lo, src, 64), h = __shfl(hi, src, 64);
      const int v = (int)(j0 + src);
      for (int b = l + lane; b <= h; b += 64) w.bin_start[b] = v;
    }
  }
}

// Exclusive scan of bin_count[0..nbins] into bin_start for more than kScanOne
// bins: per-chunk scans, then the offsets.
__global__ __launch_bounds__(kThreads) void k_scan1(Plan p, Work w) {
  const DevStats* st = w.stats;
  if (st->status != 0 || !st->need_sort) return;
  __shared__ int s[kThreads];
  const int64_t base = (int64_t)blockIdx.x * kScanChunk;
  const int64_t cnt = p.nbins + 1;
  int v[8];
  int sum = 0;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    int64_t i = base + threadIdx.x * 8 + q;
    v[q] = i < cnt ? w.bin_count[i] : 0;
    sum += v[q];
  }
  s[threadIdx.x] = sum;
  __syncthreads();
  for (int off = 1; off < kThreads; off <<= 1) {
    int x = threadIdx.x >= off ? s[threadIdx.x - off] : 0;
    __syncthreads();
    s[threadIdx.x] += x;
    __syncthreads();
  }
  int run = s[threadIdx.x] - sum;  // exclusive prefix of this thread
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    int64_t i = base + threadIdx.x * 8 + q;
    if (i < cnt) w.bin_start[i] = run;
    run += v[q];
  }
  if (threadIdx.x == kThreads - 1) w.scan_part[blockIdx.x] = s[kThreads - 1];
}

// Offsets of the per-chunk scans: block b adds the totals of chunks 0..b-1
// (a few hundred values) to its chunk.
__global__ __launch_bounds__(kThreads) void k_scan3(Plan p, Work w) {
  const DevStats* st = w.stats;
  if (st->status != 0 || !st->need_sort) return;
  __shared__ int red[kThreads];
  int part = 0;
  for (unsigned b = threadIdx.x; b < blockIdx.x; b += kThreads) part += w.scan_part[b];
  red[threadIdx.x] = part;
  __syncthreads();
  for (int sft = kThreads / 2; sft > 0; sft >>= 1) {
    if ((int)threadIdx.x < sft) red[threadIdx.x] += red[threadIdx.x + sft];
    __syncthreads();
  }
  const int add = red[0];
  const int64_t cnt = p.nbins + 1;
  for (int q = 0; q < 8; ++q) {
    int64_t i = (int64_t)blockIdx.x * kScanChunk + q * kThreads + threadIdx.x;
    if (i < cnt) w.bin_start[i] += add;
  }
}

// Row flags (whether any kernel support of a geometry reaches a row of the
// [nrows][S1] view; ngeo geometries) and, with scatter, the points into bin
// order where they need it.
__global__ __launch_bounds__(kThreads) void k_pro_rows(CallArgs a, Plan p, Work w, int ngeo,
                                                       int scatter) {
  const DevStats* st = w.stats;
  if (st->status != 0) return;
  const int64_t gtid = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  const int nd = (int)a.nd;
  const int h = (int)ceil(p.hw) + 1;
  for (int64_t i = gtid; i < ngeo * p.nrows; i += stride) {
    const bool two = i >= p.nrows;
    const int64_t r = two ? i - p.nrows : i;
    const bool active = two ? row_active<2>(r, h, p, w.bin_start, nd)
                            : row_active<1>(r, h, p, w.bin_start, nd);
    (two ? w.rowflag_2f : w.rowflag_f)[r] = (unsigned char)active;
  }
  if (!scatter || !st->need_sort) return;
  const double tau = st->tau;
  for (int64_t j = gtid; j < nd; j += stride) {
    const double t = a.t[j];
    // the histogram counts down: each bin's points fill it from its end
    const int b = point_bin(t, tau, a.df, p);
    const int pos = w.bin_start[b] + atomicSub(&w.bin_count[b], 1) - 1;
    if (pos < 0 || pos >= nd) continue;  // cannot happen with a consistent histogram
    w.ts[pos] = t;
    if (a.periodogram) {
      w.ys[pos] = a.y ? a.y[j] : 0.0;
      w.dys[pos] = a.dy ? a.dy[j] : 1.0;
    } else {
      w.hs[pos] = a.h[j];
    }
  }
}

unsigned blocks_for(int64_t work, int64_t cap) {
  const int64_t b = (work + kThreads - 1) / kThreads;
  return (unsigned)(b < 1 ? 1 : b > cap ? cap : b);
}

}  // namespace

// 4 points a thread and up: the partials stay few enough for every block of
// k_pro_bins to combine them.
static unsigned stats_blocks(int64_t nd) { return blocks_for((nd + 3) / 4, kStatsCap); }

void enqueue_pro_stats(const CallArgs& a, const Plan& p, const Work& w, hipStream_t s) {
  hipLaunchKernelGGL(k_pro_stats, dim3(stats_blocks(a.nd)), dim3(kThreads), 0, s, a, p, w);
}

void enqueue_bins(const CallArgs& a, const Plan& p, const Work& w, hipStream_t s) {
  const unsigned np = stats_blocks(a.nd);
  const int64_t work = a.nd > p.nbins + 1 ? a.nd : p.nbins + 1;
  const dim3 grid(blocks_for(work, 1024));
  if (p.nbins < kScanOne) {
    hipLaunchKernelGGL(k_pro_bins<true>, grid, dim3(kThreads), 0, s, a, p, w, (int)np);
  } else {
    hipLaunchKernelGGL(k_pro_bins<false>, grid, dim3(kThreads), 0, s, a, p, w, (int)np);
    const unsigned nc = (unsigned)((p.nbins + 1 + kScanChunk - 1) / kScanChunk);
    hipLaunchKernelGGL(k_scan1, dim3(nc), dim3(kThreads), 0, s, p, w);
    hipLaunchKernelGGL(k_scan3, dim3(nc), dim3(kThreads), 0, s, p, w);
  }
}

void enqueue_rows(const CallArgs& a, const Plan& p, const Work& w, int ngeo, bool scatter,
                  hipStream_t s) {
  const int64_t work = scatter && a.nd > 2 * p.nrows ? a.nd : 2 * p.nrows;
  hipLaunchKernelGGL(k_pro_rows, dim3(blocks_for(work, 512)), dim3(kThreads), 0, s, a, p, w, ngeo,
                     scatter ? 1 : 0);
}

}  // namespace mils
