// spread.hip -- exponential-of-semicircle spreading of one series onto the
// upsampled grids (gfx950): tiles of the active rows, accumulated in LDS.
//
// Built without the compiler's hoisting of constants out of loops: it keeps
// some 20 FP64 literals of sincospi in registers (124 VGPRs instead of 94 with
// two grids, 108 instead of 80 with one), and these kernels live on the waves
// that hide each other's loads.
#include <hip/hip_runtime.h>

#include "device_math.h"
#include "kernels.h"
#include "mils_internal.h"
#include "path_device.h"

namespace mils {

// Whether any kernel support reaches row r (through scalar loads).
__device__ __forceinline__ bool row_set(const unsigned char* flags, int r) {
  const unsigned word = ((ConstPtr<unsigned>)(const unsigned*)flags)[r >> 2];
  return (word >> (8 * (r & 3))) & 255u;
}

// Spreading over the tiles of the rows whose flag is set: a fixed grid of
// workgroups takes tiles b, b + nb, ...; every tile is written by exactly one
// workgroup, so the result does not depend on scheduling.  T divides the row
// length S1 here.
template <typename Real, int GEO, int NG, int SETS>
__device__ __forceinline__ void spread_tiles(int b, int nb, int T, int tcap, const CallArgs& a,
                                             const Plan& p, const Work& w, const DevStats& st,
                                             void* out0, void* out1, double* acc) {
  const unsigned char* flags = GEO == 1 ? w.rowflag_f : w.rowflag_2f;
  const int tpr = (int)p.S1 / T;
  const int ntile = (int)p.nrows * tpr;
  for (int t = b; t < ntile; t += nb)
    if (row_set(flags, t / tpr))
      spread_tile<Real, GEO, NG, kThreads, SETS>(t, T, tcap, a, p, w, st, out0, out1, acc);
}

template <typename Real, int GEO, int NG, int SETS>
__global__ __launch_bounds__(kThreads) void k_spread_rows(CallArgs a, Plan p, Work w, void* out0,
                                                          void* out1) {
  __shared__ double acc[NG * 2 * kTileMax];
  const DevStats st = load_stats(w.stats);
  if (st.status != 0) return;
  spread_tiles<Real, GEO, NG, SETS>(blockIdx.x, gridDim.x, p.T, kTileMax, a, p, w, st, out0, out1,
                                    acc);
}

// Direct sums A, B, B2 at four of the frequencies near f = 0 (group g: k_lo +
// 4 g ..) over slice r of nr of the points, into row r of lowfix, in a fixed
// order.
__device__ __forceinline__ void low_slice(const CallArgs& a, const DevStats& st, int g, int r,
                                          int nr, double* lowfix, double* red) {
  constexpr int NV = 24;
  const int tid = threadIdx.x;
  const int ng = st.nlow - 4 * g < 4 ? st.nlow - 4 * g : 4;
  if (ng <= 0) return;
  double v[NV];
  low_accumulate<4>(a, st, st.k_lo + 4 * g, ng, (int64_t)r * kThreads + tid,
                    (int64_t)nr * kThreads, v);
  const double sum = block_share_sum<kThreads, NV>(v, red);
  if (tid < NV) lowfix[r * 6 * kLowMax + NV * g + tid] = sum;
}

// A periodogram's spreads and direct sums in one launch: the first 4 lowrows
// workgroups take the direct sums (they run longest), the next nf the tiles of
// geometry f, the others those of geometry 2f, whose one grid lets a tile be
// twice as long (T2).
template <typename Real, int SETS>
__global__ __launch_bounds__(kThreads) void k_spread_pg(CallArgs a, Plan p, Work w, int lowrows,
                                                        int nf, int T2) {
  __shared__ double acc[4 * kTileMax];
  const DevStats st = load_stats(w.stats);
  if (st.status != 0) return;
  int b = (int)blockIdx.x;
  if (b < 4 * lowrows) {
    low_slice(a, st, b & 3, b >> 2, lowrows, w.lowfix, acc);
    return;
  }
  b -= 4 * lowrows;
  if (b < nf)
    spread_tiles<Real, 1, 2, SETS>(b, nf, p.T, kTileMax, a, p, w, st, w.grid[0], w.grid[1], acc);
  else
    spread_tiles<Real, 2, 1, SETS>(b - nf, (int)gridDim.x - 4 * lowrows - nf, T2, 2 * kTileMax, a,
                                   p, w, st, w.grid[2], w.grid[2], acc);
}

// The A spreads of NG series that share their times and weights, with their
// direct sums (the first 4 lowrows NG workgroups; their statistics are there).
// One launch instead of a spread and two kernels of direct sums a series: 160
// us -> 82 for three series of 4e5 points, statistics included.
template <typename Real, int NG, int SETS>
__global__ __launch_bounds__(kThreads) void k_spread_series(CallArgs a, Plan p, Work w,
                                                            int lowrows) {
  __shared__ double acc[2 * NG * kTileMax];
  const DevStats st = load_stats(a.wstats);
  if (st.status != 0) return;
  int b = (int)blockIdx.x;
  if (b < 4 * lowrows * NG) {
    const int g = b / (4 * lowrows);
    b -= g * 4 * lowrows;
    CallArgs ag = a;
    ag.y = g == 0 ? a.sy[0] : g == 1 ? a.sy[1] : a.sy[2];
    const DevStats* sp = g == 0 ? a.sst[0] : g == 1 ? a.sst[1] : a.sst[2];
    double* low = g == 0 ? a.slow[0] : g == 1 ? a.slow[1] : a.slow[2];
    const DevStats sg = load_stats(sp);
    if (sg.status == 0) low_slice(ag, sg, b & 3, b >> 2, lowrows, low, acc);
    return;
  }
  b -= 4 * lowrows * NG;
  const int nb = (int)gridDim.x - 4 * lowrows * NG;
  const int tpr = (int)p.S1 / p.T;
  const int ntile = (int)p.nrows * tpr;
  for (int t = b; t < ntile; t += nb)
    if (row_set(w.rowflag_f, t / tpr))
      spread_tile<Real, 1, NG, kThreads, SETS, true>(t, p.T, kTileMax, a, p, w, st, w.grid[0],
                                                     w.grid[1], acc, w.grid[2]);
}

// k_spread_rows with fixed summation orders.
template <typename Real, int GEO, int NG>
__global__ __launch_bounds__(kThreads) void k_spread_det(CallArgs a, Plan p, Work w, void* out0,
                                                         void* out1) {
  __shared__ double acc[NG * 2 * kTileMax];
  __shared__ int rb[8], re[8], sv[1];
  __shared__ SpreadRecords<Real, NG, kThreads> rec;
  const DevStats st = *w.stats;
  if (st.status != 0) return;
  const unsigned char* flags = GEO == 1 ? w.rowflag_f : w.rowflag_2f;
  const int tpr = (int)(p.S1 / p.T);
  const int ntile = (int)p.nrows * tpr;
  for (int t = blockIdx.x; t < ntile; t += gridDim.x)
    if (row_set(flags, t / tpr))
      spread_tile_det<Real, GEO, NG, kThreads>(t, p.T, kTileMax, a, p, w, st, out0, out1, acc, rb,
                                               re, sv, rec);
}

namespace {

template <typename Real, int GEO, int NG>
void enqueue(const CallArgs& a, const Plan& p, const Work& w, int gbase, hipStream_t s) {
  const int64_t ntiles = (p.S1 / p.T) * p.nrows;
  const dim3 grid((unsigned)(ntiles < kSpreadGrid ? ntiles : kSpreadGrid));
  void* out0 = w.grid[gbase];
  void* out1 = w.grid[gbase + NG - 1];
  if (a.deterministic)
    hipLaunchKernelGGL((k_spread_det<Real, GEO, NG>), grid, dim3(kThreads), 0, s, a, p, w, out0,
                       out1);
  else if (p.w <= 16)
    hipLaunchKernelGGL((k_spread_rows<Real, GEO, NG, 1>), grid, dim3(kThreads), 0, s, a, p, w,
                       out0, out1);
  else
    hipLaunchKernelGGL((k_spread_rows<Real, GEO, NG, 2>), grid, dim3(kThreads), 0, s, a, p, w,
                       out0, out1);
}

template <typename Real, int NG>
void enqueue_series(const CallArgs& a, const Plan& p, const Work& w, int lowrows, hipStream_t s) {
  const int64_t n = (p.S1 / p.T) * p.nrows;
  const dim3 grid((unsigned)(4 * lowrows * NG + (n < kSpreadGrid ? n : kSpreadGrid)));
  if (p.w <= 16)
    hipLaunchKernelGGL((k_spread_series<Real, NG, 1>), grid, dim3(kThreads), 0, s, a, p, w,
                       lowrows);
  else
    hipLaunchKernelGGL((k_spread_series<Real, NG, 2>), grid, dim3(kThreads), 0, s, a, p, w,
                       lowrows);
}

template <typename Real>
void enqueue_pg(const CallArgs& a, const Plan& p, const Work& w, int lowrows, bool f, bool f2,
                hipStream_t s) {
  const int T2 = p.S1 % (2 * p.T) == 0 ? 2 * p.T : p.T;
  auto blocks = [&](int T) {
    const int64_t n = (p.S1 / T) * p.nrows;
    return (int)(n < kSpreadGrid ? n : kSpreadGrid);
  };
  const int nf = f ? blocks(p.T) : 0, n2 = f2 ? blocks(T2) : 0;
  const dim3 grid((unsigned)(4 * lowrows + nf + n2));
  if (p.w <= 16)
    hipLaunchKernelGGL((k_spread_pg<Real, 1>), grid, dim3(kThreads), 0, s, a, p, w, lowrows, nf,
                       T2);
  else
    hipLaunchKernelGGL((k_spread_pg<Real, 2>), grid, dim3(kThreads), 0, s, a, p, w, lowrows, nf,
                       T2);
}

template <typename Real>
void enqueue_real(const CallArgs& a, const Plan& p, const Work& w, int geo, int ng, int gbase,
                  hipStream_t s) {
  if (geo == 2) enqueue<Real, 2, 1>(a, p, w, gbase, s);
  else if (ng == 2) enqueue<Real, 1, 2>(a, p, w, gbase, s);
  else enqueue<Real, 1, 1>(a, p, w, gbase, s);
}

}  // namespace

void enqueue_spread(const CallArgs& a, const Plan& p, const Work& w, int geo, int ng, int gbase,
                    hipStream_t s) {
  if (p.prec == 1) enqueue_real<float>(a, p, w, geo, ng, gbase, s);
  else enqueue_real<double>(a, p, w, geo, ng, gbase, s);
}

void enqueue_spread_pg(const CallArgs& a, const Plan& p, const Work& w, int lowrows, bool f,
                       bool f2, hipStream_t s) {
  if (p.prec == 1) enqueue_pg<float>(a, p, w, lowrows, f, f2, s);
  else enqueue_pg<double>(a, p, w, lowrows, f, f2, s);
}

void enqueue_spread_series(const CallArgs& a, const Plan& p, const Work& w, int lowrows,
                           hipStream_t s) {
  if (p.prec == 1) {
    if (a.nser == 1) enqueue_series<float, 1>(a, p, w, lowrows, s);
    else if (a.nser == 2) enqueue_series<float, 2>(a, p, w, lowrows, s);
    else enqueue_series<float, 3>(a, p, w, lowrows, s);
  } else {
    if (a.nser == 1) enqueue_series<double, 1>(a, p, w, lowrows, s);
    else if (a.nser == 2) enqueue_series<double, 2>(a, p, w, lowrows, s);
    else enqueue_series<double, 3>(a, p, w, lowrows, s);
  }
}

}  // namespace mils
