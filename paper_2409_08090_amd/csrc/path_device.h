// path_device.h -- device-side building blocks of the NUFFT Lomb-Scargle
// path, shared by the single-series kernels (kernels.hip) and the persistent
// batched kernel (batch.hip): moment merging, point binning, tile spreading,
// one workgroup's share of an FFT pass, and the power assembly.
#pragma once

#include <hip/hip_runtime.h>

#include "device_math.h"
#include "fft_core.h"
#include "mils_internal.h"

namespace mils {

struct Moments {
  double W, mu, M2;
};

__device__ __forceinline__ void moments_merge(Moments& a, double Wb, double mub, double M2b) {
  double W = a.W + Wb;
  if (W == 0.0) return;
  double d = mub - a.mu;
  double fb = Wb / W;
  a.mu += d * fb;
  a.M2 += M2b + d * d * a.W * fb;
  a.W = W;
}


__device__ __forceinline__ int point_bin(double t, double tau, double df, const Plan& p) {
  int cell;
  double frac;
  grid_coord32(t, tau, df, (double)p.n, (int)p.n, cell, frac);
  return cell >> p.Tb_shift;
}


constexpr int kScanChunk = 2048;  // 256 threads x 8


__device__ __forceinline__ int64_t floordiv2(int64_t x) { return x >= 0 ? x / 2 : -((-x + 1) / 2); }
__device__ __forceinline__ int64_t ceildiv2(int64_t x) { return x >= 0 ? (x + 1) / 2 : -((-x) / 2); }

// Append the point ranges of the cyclic cell interval [c0, c1) (of the
// binning geometry) to rb/re (LDS arrays), at most two ranges.
__device__ __forceinline__ void add_cell_range(int* rb, int* re, int& cnt, int64_t c0, int64_t c1,
                                               const Plan& p, const int* bs, int nd) {
  const int64_t n = p.n;
  if (c1 - c0 >= n) {
    rb[cnt] = 0;
    re[cnt] = nd;
    ++cnt;
    return;
  }
  // (c0 is within one period of [0, n): no division)
  int64_t x0 = c0;
  if (x0 < 0) x0 += n;
  else if (x0 >= n) x0 -= n;
  const int64_t x1 = x0 + (c1 - c0);
  const int64_t e1 = x1 <= n ? x1 : n;
  rb[cnt] = bs[x0 >> p.Tb_shift];
  re[cnt] = bs[((e1 - 1) >> p.Tb_shift) + 1];
  ++cnt;
  if (x1 > n) {
    rb[cnt] = bs[0];
    re[cnt] = bs[((x1 - n - 1) >> p.Tb_shift) + 1];
    ++cnt;
  }
}

// Points whose geometry-GEO coordinate may fall in the cyclic interval
// [c0, c1); returns the number of ranges written (<= 4).
template <int GEO>
__device__ __forceinline__ int gather_ranges(int* rb, int* re, int64_t c0, int64_t c1,
                                             const Plan& p, const int* bs, int nd) {
  int cnt = 0;
  if (GEO == 1) {
    add_cell_range(rb, re, cnt, c0, c1, p, bs, nd);
  } else {
    // u_2f = 2 u_f mod n: the cyclic interval [c0, c1) has the two pre-images
    // [c0/2, c1/2) and [(c0+n)/2, (c1+n)/2) in u_f (one cell of slack each side).
    if (c1 - c0 + 8 >= p.n) {
      rb[0] = 0;
      re[0] = nd;
      return 1;
    }
    add_cell_range(rb, re, cnt, floordiv2(c0) - 1, ceildiv2(c1) + 1, p, bs, nd);
    add_cell_range(rb, re, cnt, floordiv2(c0 + p.n) - 1, ceildiv2(c1 + p.n) + 1, p, bs, nd);
  }
  return cnt;
}

// The plan's kernel table is read-only for the whole launch: reading it
// through the constant address space lets the compiler use scalar loads (one
// per wave, not per lane) and feed the coefficients to the FMAs from SGPRs.
template <typename Real>
using ConstPtr = const __attribute__((address_space(4))) Real*;

// Whether any kernel support of geometry GEO reaches row r of the
// [nrows][S1] view of the grid (h: half-width in cells, rounded up, plus one).
template <int GEO>
__device__ __forceinline__ bool row_active(int64_t r, int h, const Plan& p, const int* bs, int nd) {
  int rb[4], re[4];
  const int cnt = gather_ranges<GEO>(rb, re, r * p.S1 - h, (r + 1) * p.S1 + h, p, bs, nd);
  int tot = 0;
  for (int i = 0; i < cnt; ++i) tot += re[i] - rb[i];
  return tot > 0;
}

// Lane I of every row of 16 lanes, broadcast to its row (one DPP move).
template <int I, typename V>
__device__ __forceinline__ V row_lane(V x) {
  return __builtin_amdgcn_update_dpp((V)0, x, 0x150 + I, 0xf, 0xf, true);
}

// A lane's kernel polynomials: cell lane mod 16 of a support and, for kernels
// wider than 16 cells (SETS = 2), cell 16 + lane mod 16 (zero past the
// kernel's width).
template <typename Real, int SETS>
struct LaneKernel {
  static constexpr int N = sizeof(Real) == 8 ? kHornerN64 : kHornerN32;
  Real c[SETS][N];
};
template <typename Real, int SETS>
__device__ __forceinline__ void load_kernel(LaneKernel<Real, SETS>& lk, const Real* tab) {
  const int cell = threadIdx.x & 15;
#pragma unroll
  for (int s = 0; s < SETS; ++s)
#pragma unroll
    for (int j = 0; j < LaneKernel<Real, SETS>::N; ++j)
      lk.c[s][j] = cell + 16 * s < kHornerK ? tab[j * kHornerK + cell + 16 * s] : (Real)0;
}
template <typename Real, int SETS>
__device__ __forceinline__ Real kernel_value(const LaneKernel<Real, SETS>& lk, int s, Real u) {
  Real v = lk.c[s][0];
#pragma unroll
  for (int j = 1; j < LaneKernel<Real, SETS>::N; ++j) v = v * u + lk.c[s][j];
  return v;
}

// Statistics of the call through the constant address space (they do not
// change during the kernels that use this): scalar loads.
__device__ __forceinline__ DevStats load_stats(const DevStats* src) {
  static_assert(sizeof(DevStats) % 4 == 0, "whole words");
  DevStats st;
  const ConstPtr<int> q = (ConstPtr<int>)(const int*)src;
  int* d = reinterpret_cast<int*>(&st);
#pragma unroll
  for (int i = 0; i < (int)(sizeof(DevStats) / 4); ++i) d[i] = q[i];
  return st;
}

// Where the spread reads the points: the caller's arrays or, after a sort, the
// sorted copies.
struct PointSource {
  const double* t;
  const double* y;   // y, or the raw strengths
  const double* dy;  // NULL: unit weights
};
__device__ __forceinline__ PointSource point_source(const CallArgs& a, const Work& w,
                                                    const DevStats& st) {
  PointSource s;
  if (st.need_sort) {
    s.t = w.ts;
    s.y = a.periodogram ? w.ys : w.hs;
    s.dy = a.periodogram ? w.dys : nullptr;
  } else {
    s.t = a.t;
    s.y = a.periodogram ? a.y : a.h;
    s.dy = a.periodogram ? a.dy : nullptr;
  }
  return s;
}

// First cell of a point's support relative to cell a0 (mod n, in (-n, n - w])
// and its kernel argument u.
template <typename Real, int GEO>
__device__ __forceinline__ void point_cell(double t, const DevStats& st, const CallArgs& a,
                                           const Plan& p, int64_t a0, int& lb, Real& u) {
  int cell;
  double frac;
  const int n = (int)p.n;
  grid_coord32(t, st.tau, GEO * a.df, (double)p.n, n, cell, frac);
  const int o0 = (int)ceil(frac - p.hw);
  lb = cell + o0 - (int)a0;  // in (-2n, n)
  if (lb < 0) lb += n;
  if (lb < 0) lb += n;
  if (lb > n - p.w) lb -= n;
  // u = 2t - 1, t = o0 + hw - frac in [0, 1)
  u = (Real)(2.0 * ((double)o0 + p.hw - frac) - 1.0);
}

// The complex strengths of a point: component c of grid g at h[2 g + c].
template <typename Real, int GEO, int NG>
__device__ __forceinline__ void point_strengths(double t, double y, double dv,
                                                const DevStats& st, const CallArgs& a,
                                                double invW, Real* h) {
  double pc, ps;
  prephase(t, st.tau, a.fch, a.fcl, pc, ps);
  if (a.periodogram) {
    const double wj = 1.0 / (dv * dv);
    const double wh = wj * invW;
    if (GEO == 1) {
      const double yt = a.unit_y ? 1.0 : y - st.ysub;
      h[0] = (Real)(wh * yt * pc);
      h[1] = (Real)(wh * yt * ps);
      if (NG > 1) {
        h[2 * NG - 2] = (Real)(wh * pc);
        h[2 * NG - 1] = (Real)(wh * ps);
      }
    } else {
      // exp(2 i theta) from exp(i theta)
      h[0] = (Real)(wh * (pc * pc - ps * ps));
      h[1] = (Real)(wh * (2.0 * pc * ps));
    }
  } else {
    h[0] = (Real)(y * pc);
    h[1] = (Real)(y * ps);
  }
}

// Value and error of point j as far as geometry GEO needs them (0 and 1 else).
template <int GEO>
__device__ __forceinline__ void point_values(const PointSource& src, const CallArgs& a, int j,
                                             double& y, double& dv) {
  y = GEO == 1 && !a.unit_y ? src.y[j] : 0.0;
  dv = src.dy ? src.dy[j] : 1.0;
}

// The point ranges of the cyclic cell interval [c0, c1), c0 within one period
// of [0, n): b0..e0 and, past the period's end, b1..e1.  Every lane of the
// workgroup computes them alike, so the loads are scalar ones.
struct CellRanges {
  int b0, e0, b1, e1;
};
__device__ __forceinline__ CellRanges cell_ranges(int c0, int c1, const Plan& p, const int* bin_start,
                                                  int nd) {
  const ConstPtr<int> bs = (ConstPtr<int>)bin_start;
  const int n = (int)p.n;
  CellRanges r = {0, nd, 0, 0};
  if (c1 - c0 >= n) return r;
  int x0 = c0 < 0 ? c0 + n : c0 >= n ? c0 - n : c0;
  const int x1 = x0 + (c1 - c0);
  const int e1 = x1 <= n ? x1 : n;
  r.b0 = bs[x0 >> p.Tb_shift];
  r.e0 = bs[((e1 - 1) >> p.Tb_shift) + 1];
  if (x1 > n) {
    r.b1 = bs[0];
    r.e1 = bs[((x1 - n - 1) >> p.Tb_shift) + 1];
  }
  return r;
}

constexpr int kSpreadNone = -(1 << 30);  // first cell of a point that misses the tile

// Four points of the wave at a time (lanes I .. of the four rows of 16), every
// lane its cell of the support: see spread_tile.
template <typename Real, int NG, int SETS, int I>
__device__ __forceinline__ void add_wave_points(double* acc, int tcap, int T, int n, int w,
                                                const LaneKernel<Real, SETS>& lk, int cnt, int lb,
                                                Real u, const Real* h) {
  if constexpr (I < 16) {
    // (cnt is the same for the whole wave; lanes without a point miss the tile)
    if (I % 4 == 0 && I >= cnt) return;
    const Real ui = row_lane<I>(u);
    const int first = row_lane<I>(lb) + (int)(threadIdx.x & 15);
    Real hi[2 * NG];
#pragma unroll
    for (int c = 0; c < 2 * NG; ++c) hi[c] = row_lane<I>(h[c]);
#pragma unroll
    for (int s = 0; s < SETS; ++s) {
      const Real v = kernel_value(lk, s, ui);
      int x = first + 16 * s;
      if (x < 0) x += n;
      else if (x >= n) x -= n;
      if ((unsigned)x < (unsigned)T && (s == 0 || (int)(threadIdx.x & 15) + 16 < w)) {
#pragma unroll
        for (int c = 0; c < 2 * NG; ++c) atomicAdd(&acc[c * tcap + x], (double)(v * hi[c]));
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    add_wave_points<Real, NG, SETS, I + 1>(acc, tcap, T, n, w, lk, cnt, lb, u, h);
  }
}

// Spread one tile of geometry GEO into NG grids: cells [tile*T, tile*T + T)
// of the flat grid, where T either divides the row length S1 of the
// [nrows][S1] view or is a whole number of rows; the caller knows that the
// tile lies in an active row.  out0, out1: the grids (passed apart: an index
// into w.grid known only at run time puts the kernel's whole argument into
// scratch memory).  acc: LDS accumulator of NG*2*tcap doubles
// (T <= tcap; doubles for FP32 grids too: on gfx950 the LDS atomic add of
// doubles runs at full rate while that of floats waits ~50x longer per
// instruction).  Called by every thread of the workgroup (it contains
// barriers).
//
// Each wave takes 64 points of the tile's ranges at a time, one per lane, and
// adds them four at a time: 16 lanes take one point's cells, each with its
// own polynomial in registers and the point's values by DPP broadcast from
// its lane, so that a row's adds are one run of cells and the waves need
// neither records in LDS nor barriers between the clearing and the store.
// Bound by the latency of a tile's loads and by FP64 arithmetic (both
// geometries of the 1e6-point curve: 47 us of it).  Against records in LDS, a
// barrier per 256 points and arguments in scratch: both spreads of that curve,
// side by side, 115 -> 73 us (FP32 100 -> 55), 1e5 points 27 -> 17 us.
//
// SER: the A grids of NG series that share their times and weights (a.sy,
// a.sst; st the weights-only call's statistics): one evaluation of the kernel
// and the phase of a point for all of them.
template <typename Real, int GEO, int NG, int NT, int SETS, bool SER = false>
__device__ __forceinline__ void spread_tile(int tile, int Tt, int tcap, const CallArgs& a,
                                            const Plan& p, const Work& w, const DevStats& st,
                                            void* out0, void* out1, double* acc,
                                            void* out2 = nullptr) {
  using T2 = typename cplx<Real>::T;
  const int tid = threadIdx.x;
  const int n = (int)p.n, nd = (int)a.nd;
  const int a0 = tile * Tt;
  const int T = n - a0 < Tt ? n - a0 : Tt;
  const int h = (int)ceil(p.hw) + 1;
  CellRanges ra, rb = {0, 0, 0, 0};
  if constexpr (GEO == 1) {
    ra = cell_ranges(a0 - h, a0 + T + h, p, w.bin_start, nd);
  } else {
    // u_2f = 2 u_f mod n: the cyclic interval [c0, c1) has the two pre-images
    // [c0/2, c1/2) and [(c0+n)/2, (c1+n)/2) in u_f (one cell of slack each side)
    const int c0 = a0 - h, c1 = a0 + T + h;
    if (c1 - c0 + 8 >= n) {
      ra = {0, nd, 0, 0};
    } else {
      ra = cell_ranges((int)floordiv2(c0) - 1, (int)ceildiv2(c1) + 1, p, w.bin_start, nd);
      rb = cell_ranges((int)floordiv2((int64_t)c0 + n) - 1, (int)ceildiv2((int64_t)c1 + n) + 1, p,
                       w.bin_start, nd);
    }
  }
  for (int x = tid; x < T; x += NT) {
#pragma unroll
    for (int c = 0; c < 2 * NG; ++c) acc[c * tcap + x] = 0.0;
  }
  LaneKernel<Real, SETS> lk;
  load_kernel(lk, (const Real*)p.hcoef);
  __syncthreads();
  const PointSource src = point_source(a, w, st);
  const double invW = 1.0 / st.W;
  double ysub[NG] = {};
  if constexpr (SER) {
    ysub[0] = ((ConstPtr<double>)&a.sst[0]->ysub)[0];
    if constexpr (NG > 1) ysub[1] = ((ConstPtr<double>)&a.sst[1]->ysub)[0];
    if constexpr (NG > 2) ysub[2] = ((ConstPtr<double>)&a.sst[2]->ysub)[0];
  }
  // a kernel support can meet the tile at most once unless the tile spans
  // nearly the whole periodic grid
  const bool wrap_free = T <= n - p.w;
  const int lane = tid & 63;
#pragma unroll 1
  for (int r = 0; r < 2 * GEO; ++r) {
    const int jbeg = r == 0 ? ra.b0 : r == 1 ? ra.b1 : r == 2 ? rb.b0 : rb.b1;
    const int jend = r == 0 ? ra.e0 : r == 1 ? ra.e1 : r == 2 ? rb.e0 : rb.e1;
    for (int j0 = jbeg + (tid - lane); j0 < jend; j0 += NT) {
      const int j = j0 + lane;
      int lb = kSpreadNone;
      Real u = 0, hs[2 * NG] = {};
      if (j < jend) {
        // (all three loads at once: few points of the ranges miss the tile)
        const double t = src.t[j];
        double y[SER ? NG : 1], dv;
        if constexpr (SER) {
          dv = src.dy ? src.dy[j] : 1.0;
          y[0] = a.sy[0][j];
          if constexpr (NG > 1) y[1] = a.sy[1][j];
          if constexpr (NG > 2) y[2] = a.sy[2][j];
        } else {
          point_values<GEO>(src, a, j, y[0], dv);
        }
        point_cell<Real, GEO>(t, st, a, p, a0, lb, u);
        if (wrap_free && (lb >= T || lb + p.w <= 0)) lb = kSpreadNone;
        if constexpr (SER) {
          double pc, ps;
          prephase(t, st.tau, a.fch, a.fcl, pc, ps);
          const double wh = 1.0 / (dv * dv) * invW;
#pragma unroll
          for (int g = 0; g < NG; ++g) {
            const double yt = y[g] - ysub[g];
            hs[2 * g] = (Real)(wh * yt * pc);
            hs[2 * g + 1] = (Real)(wh * yt * ps);
          }
        } else {
          point_strengths<Real, GEO, NG>(t, y[0], dv, st, a, invW, hs);
        }
      }
      add_wave_points<Real, NG, SETS, 0>(acc, tcap, T, n, p.w, lk, jend - j0, lb, u, hs);
    }
  }
  __syncthreads();
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    T2* out = reinterpret_cast<T2*>(g == 0 ? out0 : g == 1 ? out1 : out2) + a0;
    for (int x = tid; x < T; x += NT) {
      T2 v;
      v.x = (Real)acc[(2 * g) * tcap + x];
      v.y = (Real)acc[(2 * g + 1) * tcap + x];
      out[x] = v;
    }
  }
  __syncthreads();  // acc is reused by the next tile
}

// The same in a fixed order (bitwise-reproducible sums): a chunk of NT points
// at a time leaves its records in LDS, and each thread adds them one after
// another to the cells x = tid, tid + NT, ... that it owns.
template <typename Real, int NG, int NT>
struct SpreadRecords {
  int lb[NT];
  Real u[NT];
  Real h[2 * NG * NT];
};
template <typename Real, int GEO, int NG, int NT>
__device__ void spread_tile_det(int tile, int Tt, int tcap, const CallArgs& a, const Plan& p,
                                const Work& w, const DevStats& st, void* out0, void* out1,
                                double* acc, int* rb, int* re, int* sv,
                                SpreadRecords<Real, NG, NT>& rec) {
  using T2 = typename cplx<Real>::T;
  const int tid = threadIdx.x;
  const int64_t a0 = (int64_t)tile * Tt;
  const int T = (int)((p.n - a0) < Tt ? (p.n - a0) : Tt);
  const int nd = (int)a.nd;
  if (tid == 0) {
    const int h = (int)ceil(p.hw) + 1;
    sv[0] = gather_ranges<GEO>(rb, re, a0 - h, a0 + T + h, p, w.bin_start, nd);
  }
  for (int x = tid; x < T; x += NT) {
#pragma unroll
    for (int c = 0; c < 2 * NG; ++c) acc[c * tcap + x] = 0.0;
  }
  __syncthreads();
  const int nr = sv[0];
  const PointSource src = point_source(a, w, st);
  const double invW = 1.0 / st.W;
  const int n = (int)p.n;
  const bool wrap_free = T <= n - p.w;
  constexpr int NC = LaneKernel<Real, 1>::N;
  const ConstPtr<Real> hc = (ConstPtr<Real>)(p.hcoef);
  for (int r = 0; r < nr; ++r) {
    const int jend = re[r];
    for (int base = rb[r]; base < jend; base += NT) {
      const int j = base + tid;
      int lb = kSpreadNone;
      if (j < jend) {
        const double t = src.t[j];
        Real u, h[2 * NG];
        point_cell<Real, GEO>(t, st, a, p, a0, lb, u);
        if (wrap_free && (lb >= T || lb + p.w <= 0)) lb = kSpreadNone;
        else {
          double y, dv;
          point_values<GEO>(src, a, j, y, dv);
          point_strengths<Real, GEO, NG>(t, y, dv, st, a, invW, h);
          rec.u[tid] = u;
#pragma unroll
          for (int c = 0; c < 2 * NG; ++c) rec.h[c * NT + tid] = h[c];
        }
      }
      rec.lb[tid] = lb;
      __syncthreads();
      const int cnt = jend - base < NT ? jend - base : NT;
      for (int i = 0; i < cnt; ++i) {
        const int lbi = rec.lb[i];
        if (lbi == kSpreadNone) continue;
        const Real u = rec.u[i];
        for (int x = tid; x < T; x += NT) {
          int off = x - lbi;  // cell offset within the point's support, mod n
          if (off < 0) off += n;
          else if (off >= n) off -= n;
          if (off >= p.w) continue;
          Real v = hc[off];
          for (int jc = 1; jc < NC; ++jc) v = v * u + hc[jc * kHornerK + off];
#pragma unroll
          for (int c = 0; c < 2 * NG; ++c)
            acc[c * tcap + x] += (double)(v * rec.h[c * NT + i]);
        }
      }
      __syncthreads();
    }
  }
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    T2* out = reinterpret_cast<T2*>(g == 0 ? out0 : out1);
    for (int x = tid; x < T; x += NT) {
      T2 v;
      v.x = (Real)acc[(2 * g) * tcap + x];
      v.y = (Real)acc[(2 * g + 1) * tcap + x];
      out[a0 + x] = v;
    }
  }
  __syncthreads();
}

template <typename Real>
struct PassBufs {
  typename cplx<Real>::T* in[3];
  typename cplx<Real>::T* out[3];
  const unsigned char* rowflag[3];
};

// A first/middle pass: workgroup = C consecutive columns s of one outer index
// p; loads L x C elements (C contiguous per row, 128-256 B segments),
// transforms along L in LDS, applies the inter-pass twiddle and stores with
// the outer index and k transposed.  One workgroup's share of the pass is the
// logical block blk.  smem: L*C elements + the twiddle table (L entries, or
// tw2_count(L) for TW2) + L row flags; rflag (NULL: every row) marks the
// input rows that are not all zero.  C is a power of two that divides NT,
// so a thread keeps one column c = tid mod C and visits rows l0, l0 + NT/C,
// ... (l0 = tid / C): its global addresses are a base plus uniform strides.
template <typename Real, int EMAX, int NT, bool TW2 = false>
__device__ void fft_pass_block(int64_t blk, const typename cplx<Real>::T* in,
                               typename cplx<Real>::T* out, const unsigned char* rflag,
                               const FftPass& ps, const typename cplx<Real>::T* tw,
                               unsigned char* smem) {
  using T2 = typename cplx<Real>::T;
  const int tid = threadIdx.x;
  const int L = ps.L, C = ps.C, csh = ps.cshift;
  const int ntw = TW2 ? tw2_count(L) : L;
  T2* buf = reinterpret_cast<T2*>(smem);
  T2* twL = buf + L * C;
  const int64_t S = ps.S, P = ps.P;
  const uint32_t nsb = (uint32_t)((S + C - 1) / C);
  const uint32_t pidx32 = (uint32_t)blk / nsb;
  const int64_t pidx = pidx32;
  const int64_t s0 = (int64_t)((uint32_t)blk - pidx32 * nsb) * C;
  const int ceff = (int)((S - s0) < C ? (S - s0) : C);
  const int c = tid & (C - 1);
  const int l0 = tid >> csh;
  const int LS = NT >> csh;  // rows between a thread's consecutive elements
  const bool cok = c < ceff;
  constexpr int PER = (EMAX + NT - 1) / NT;
  const T2* pin = in + pidx * (int64_t)L * S + s0 + (int64_t)l0 * S + c;
  const int64_t istep = (int64_t)LS * S;
  T2 v[PER];
  if (rflag) {
    // first pass: the row flags (and the twiddle table) into LDS, then the
    // loads of the rows that are not all zero
    unsigned char* rf = reinterpret_cast<unsigned char*>(twL + ntw);
    for (int x = tid; x < ntw; x += NT) twL[x] = tw[ps.twL_off + x];
    for (int x = tid; x < L; x += NT) rf[x] = rflag[x];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int l = l0 + i * LS;
      v[i] = czero<T2>();
      if (l < L && cok && rf[l]) v[i] = pin[i * istep];
    }
  } else {
    // later passes: the tile's loads first, then the twiddle table, whose
    // loads and LDS stores overlap the data's latency
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int l = l0 + i * LS;
      v[i] = czero<T2>();
      if (l < L && cok) v[i] = pin[i * istep];
    }
    for (int x = tid; x < ntw; x += NT) twL[x] = tw[ps.twL_off + x];
  }
#pragma unroll
  for (int i = 0; i < PER; ++i)
    if (l0 + i * LS < L) buf[tid + i * NT] = v[i];
  // Inter-pass twiddles exp(2 pi i s k / N), N = L S, of this thread's
  // outputs (column s = s0 + c, rows k = l0 + i LS), fetched before the
  // transform so that their latency overlaps it: the first from the table,
  // the others by repeated multiplication with the step exp(2 pi i s LS / N).
  // Threads without outputs (l0 >= L or c >= ceff) and threads with a single
  // output (LS >= L) take index 0 for what they do not use, so every index is
  // below N.
  const int64_t mask = ((int64_t)1 << ps.bshift) - 1;
  const T2* tlo = tw + ps.twlo_off;
  const T2* thi = tw + ps.twhi_off;
  const int64_t scol = s0 + c;
  const int64_t q0 = (cok && l0 < L) ? scol * (int64_t)l0 : 0;
  const int64_t qs = (cok && LS < L) ? scol * (int64_t)LS : 0;
  const T2 w0 = cmul(thi[q0 >> ps.bshift], tlo[q0 & mask]);
  const T2 ws = cmul(thi[qs >> ps.bshift], tlo[qs & mask]);
  __syncthreads();
  lds_fft<EMAX, NT, TW2>(buf, L, C, C, ps.rad, ps.nrad, twL);
  const int64_t PS = P * S;
  T2* pout = out + (int64_t)l0 * PS + pidx * S + s0 + c;
  const int64_t ostep = (int64_t)LS * PS;
  T2 tk = w0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    if (l0 + i * LS < L && cok) pout[i * ostep] = cmul(buf[tid + i * NT], tk);
    tk = cmul(tk, ws);
  }
  __syncthreads();
}

// Power of the floating-mean Lomb-Scargle fit from the three normalised sums
// A = sum w^ y~ e^{iwt}, B = sum w^ e^{iwt}, B2 = sum w^ e^{2iwt}
// (w^ = w / W).  cos^2 and sin^2 sums follow from B2 by the double-angle
// identities; the 2x2 fit is solved in closed form (tau-free form).
__device__ __forceinline__ double ls_power(double Ar, double Ai, double Br, double Bi, double B2r,
                                           double B2i, const DevStats& st, int norm,
                                           int fit_mean, double dmin) {
  double CC = 0.5 * (1.0 + B2r);
  double SS = 0.5 * (1.0 - B2r);
  double CS = 0.5 * B2i;
  double YC = Ar, YS = Ai;
  if (fit_mean) {
    CC -= Br * Br;
    SS -= Bi * Bi;
    CS -= Br * Bi;
    YC -= st.Ybar * Br;
    YS -= st.Ybar * Bi;
  }
  const double D = CC * SS - CS * CS;
  // ill-posed: D below the accuracy of the sums, or below 1e-12 of CC SS
  if (!(D > dmin) || !(D > 1e-12 * CC * SS)) return __builtin_nan("");
  const double N = SS * YC * YC + CC * YS * YS - 2.0 * CS * YC * YS;
  const double YYD = st.YY * D;
  switch (norm) {
    case 1:
      return N / (YYD - N);
    case 2:
      return -log1p(-N / YYD);
    case 3:
      return 0.5 * st.W * N / D;
    default:
      return N / YYD;
  }
}

// Counts ill-posed outputs (power NaN) and tells the host that there are some.
__device__ __forceinline__ void count_nan(const CallArgs& a, int* nill, int n) {
  atomicAdd(nill, n);
  if (a.host_words) a.host_words[1] = 1;
}

// Last pass: D rows of length L per workgroup for the G grids, transformed in
// LDS; output k of row p is the mode m = p + P k.  Deconvolution, crop to the
// nf requested modes and (G = 3) the power are fused into the store.
// One workgroup's share of the last pass: D rows starting at p0 = blk*D.
// The G*D rows are interleaved in LDS, element l of row r at l*R + r with
// R = G*D: every wave access of a stage (and of the power readout) is then a
// run of consecutive elements, which the LDS serves without bank conflicts.
// The global loads take the row index fastest (lanes (l, d), D rows of one
// grid), so that their LDS stores are contiguous runs too while each row is
// still read in contiguous 16-element pieces.  smem: L*R elements + the
// twiddle table (L entries, or tw2_count(L) for TW2).  nf and K are those of
// the series (a batched series may use fewer frequencies than its grid's
// plan).
template <typename Real, int G, int EMAX, int NT, bool TW2 = false, bool SER = false>
__device__ void fft_last_block(int64_t blk, const PassBufs<Real>& b, const FftPass& ps,
                               int64_t n, int64_t nf, int64_t K, const CallArgs& a,
                               const typename cplx<Real>::T* tw, const double* inv_phihat,
                               const DevStats& st, unsigned char* smem,
                               const double* lowfix = nullptr, int lowparts = 1,
                               int* nill = nullptr) {
  using T2 = typename cplx<Real>::T;
  const int tid = threadIdx.x;
  const int L = ps.L, D = ps.C;
  const int R = G * D;
  T2* buf = reinterpret_cast<T2*>(smem);
  T2* twL = buf + L * R;
  const int64_t P = ps.P;
  const int64_t p0 = blk * D;
  const int deff = (int)((P - p0) < D ? (P - p0) : D);
  const int E = D * L;
  const int dsh = __builtin_ctz(D);  // D is a power of two
  constexpr int PER = (EMAX / G + NT - 1) / NT;
  // element e = l D + d of the block's rows (row d, position l)
  const int d0 = tid & (D - 1);
  const int l0 = tid >> dsh;
  const int LS = NT >> dsh;  // NT is a multiple of D
  // the rows' loads first, then the twiddle table (its latency hides behind
  // theirs), then the rows into LDS
  T2 v[G][PER];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const T2* in = b.in[g] + (p0 + d0) * (int64_t)L + l0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      v[g][i] = czero<T2>();
      if (l0 + i * LS < L && d0 < deff) v[g][i] = in[i * LS];
    }
  }
  for (int x = tid; x < (TW2 ? tw2_count(L) : L); x += NT) twL[x] = tw[ps.twL_off + x];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int l = l0 + i * LS;
      if (l < L) buf[__mul24(l, R) + g * D + d0] = v[g][i];
    }
  __syncthreads();
  // kernel-transform factors of this thread's outputs, fetched before the
  // transform so that their latency overlaps it (-1: output cropped)
  constexpr int PO = (EMAX / G + NT - 1) / NT;
  double ipv[PO];
  int64_t kov[PO];
#pragma unroll
  for (int i = 0; i < PO; ++i) {
    const int e = tid + i * NT;
    const int d = e & (D - 1);
    const int k = e >> dsh;
    kov[i] = -1;
    ipv[i] = 0.0;
    if (e < E && d < deff) {
      const int64_t m = p0 + d + P * (int64_t)k;
      const int64_t mm = (m <= nf - 1 - K) ? m : m - n;
      const int64_t kout = mm + K;
      if (kout >= 0 && kout < nf) {
        kov[i] = kout;
        ipv[i] = inv_phihat[mm < 0 ? -mm : mm];
      }
    }
  }
  // statistics of the series of a shared-weights group, once per workgroup
  // (uniform loads; the power stores below cannot then force reloads)
  DevStats ser[SER ? G : 1];
  if constexpr (SER) {
#pragma unroll
    for (int g = 0; g < G; ++g)
      if (g < a.nser) ser[g] = *a.sst[g];
  }
  lds_fft<EMAX, NT, TW2>(buf, L, G * D, R, ps.rad, ps.nrad, twL);
#pragma unroll
  for (int i = 0; i < PO; ++i) {
    const int64_t kout = kov[i];
    if (kout < 0) continue;
    const int e = tid + i * NT;
    const int d = e & (D - 1);
    const int k = e >> dsh;
    const double ip = ipv[i];
    if constexpr (SER) {
      // series sharing their weights: grid g holds series g's A; B and B2
      // were computed once for all
      const double2 B = reinterpret_cast<const double2*>(a.bsum_b)[kout];
      const double2 B2 = reinterpret_cast<const double2*>(a.bsum_b2)[kout];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if (g >= a.nser) continue;
        const DevStats& sg = ser[g];
        if (sg.status != 0) continue;
        const T2 A = buf[k * R + g * D + d];
        double s6[6] = {(double)A.x * ip, (double)A.y * ip, B.x, B.y, B2.x, B2.y};
        const int64_t q = kout - sg.k_lo;
        const bool low = q >= 0 && q < sg.nlow;
        if (low) {
          const double* lf = a.slow[g];
          for (int j = 0; j < 6; ++j) s6[j] = lf[6 * q + j];
          for (int r = 1; r < lowparts; ++r)
            for (int j = 0; j < 6; ++j) s6[j] += lf[r * 6 * kLowMax + 6 * q + j];
        }
        double pw = ls_power(s6[0], s6[1], s6[2], s6[3], s6[4], s6[5], sg, a.norm, a.fit_mean,
                             low ? 0.0 : a.dmin);
        if (kout == a.kzero) pw = 0.0;
        a.spow[g][kout] = pw;
      }
    } else if (G == 3) {
      const T2 A = buf[k * R + d];
      const T2 B = buf[k * R + D + d];
      const T2 B2 = buf[k * R + 2 * D + d];
      double s6[6] = {(double)A.x * ip,  (double)A.y * ip,  (double)B.x * ip,
                      (double)B.y * ip,  (double)B2.x * ip, (double)B2.y * ip};
      const int64_t q = kout - st.k_lo;
      const bool low = lowfix && q >= 0 && q < st.nlow;
      if (low) {
        for (int j = 0; j < 6; ++j) s6[j] = lowfix[6 * q + j];
        for (int r = 1; r < lowparts; ++r)
          for (int j = 0; j < 6; ++j) s6[j] += lowfix[r * 6 * kLowMax + 6 * q + j];
      }
      double pw = ls_power(s6[0], s6[1], s6[2], s6[3], s6[4], s6[5], st, a.norm, a.fit_mean,
                           low ? 0.0 : a.dmin);
      if (kout == a.kzero) pw = 0.0;
      else if (nill && pw != pw) count_nan(a, nill, 1);
      a.power[kout] = pw;
    } else {
      const T2 A = buf[k * R + d];
      double2 v = make_double2((double)A.x * ip, (double)A.y * ip);
      reinterpret_cast<double2*>(a.sums)[kout] = v;
    }
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------
// Direct sums near f = 0.
// ---------------------------------------------------------------------------
// The frequencies k in [k_lo, k_lo + nlow) with |f_k| (tmax - tmin) < 2,
// at most kLowMax of them, the ones closest to f = 0.
__device__ __forceinline__ void low_band(const DevStats& st, double f0, double df, int64_t nf,
                                         int64_t& k_lo, int& nlow) {
  nlow = 0;
  k_lo = 0;
  const double span = st.tmax - st.tmin;
  if (!(span > 0.0)) return;
  const double fl = 2.0 / span;
  double ka = ceil((-fl - f0) / df);
  double kb = floor((fl - f0) / df);
  if (ka < 0.0) ka = 0.0;
  if (kb > (double)(nf - 1)) kb = (double)(nf - 1);
  if (kb < ka) return;
  double lo = ka;
  if (kb - ka + 1.0 > (double)kLowMax) {
    double centre = rint(-f0 / df);
    lo = centre - kLowMax / 2;
    if (lo < ka) lo = ka;
    if (lo > kb - kLowMax + 1) lo = kb - kLowMax + 1;
  }
  k_lo = (int64_t)lo;
  nlow = (int)fmin(kb - lo + 1.0, (double)kLowMax);
}

// Extra workgroups of a first pass (the last lr.n of x, y = 0): the rows of
// direct sums into the first.  True for them.
__device__ __forceinline__ bool low_rows_block(const LowRows& lr) {
  const int i = (int)blockIdx.x - ((int)gridDim.x - lr.n);
  if (i < 0) return false;
  const int x = threadIdx.x;
  if (blockIdx.y == 0 && x < 6 * kLowMax) {
    double* low = i == 0 ? lr.low[0] : i == 1 ? lr.low[1] : lr.low[2];
    double sum = 0.0;
#pragma unroll 8
    for (int r = 0; r < lr.rows; ++r) sum += low[r * 6 * kLowMax + x];
    low[x] = sum;
  }
  return true;
}

// This thread's contributions to A, B, B2 at frequencies k_lo + g0 + q,
// q < kLowGroup, summed over points j = j0, j0 + stride, ... < nd.  The phase
// at the first frequency is reduced in double-double; the others follow by
// the exact angle-sum recurrence with the step exp(i 2 pi df t).
template <int GRP>
__device__ __forceinline__ void low_accumulate(const CallArgs& a, const DevStats& st, int64_t k_first,
                                               int ng, int64_t j0, int64_t stride,
                                               double* acc /* 6 * GRP */) {
#pragma unroll
  for (int i = 0; i < 6 * GRP; ++i) acc[i] = 0.0;
  // f_first = f0 + k_first df as a double-double
  double kp, ke;
  dd_two_prod((double)k_first, a.df, kp, ke);
  double fh, fe;
  dd_two_sum(a.f0, kp, fh, fe);
  const double fl = fe + ke;
  const double invW = 1.0 / st.W;
  for (int64_t j = j0; j < a.nd; j += stride) {
    const double t = a.t[j];
    double wj = 1.0;
    if (a.dy) {
      const double dv = a.dy[j];
      wj = 1.0 / (dv * dv);
    }
    const double wh = wj * invW;
    const double wy = wh * (a.y[j] - st.ysub);
    double pc, ps, sc, ss;
    prephase(t, st.tau, fh, fl, pc, ps);
    prephase(t, st.tau, a.df, 0.0, sc, ss);
#pragma unroll
    for (int q = 0; q < GRP; ++q) {
      if (q < ng) {
        const double c2 = pc * pc - ps * ps, s2 = 2.0 * pc * ps;
        acc[6 * q + 0] += wy * pc;
        acc[6 * q + 1] += wy * ps;
        acc[6 * q + 2] += wh * pc;
        acc[6 * q + 3] += wh * ps;
        acc[6 * q + 4] += wh * c2;
        acc[6 * q + 5] += wh * s2;
      }
      const double nc = pc * sc - ps * ss;
      ps = pc * ss + ps * sc;
      pc = nc;
    }
  }
}

// Sums of NV = 3 2^k values over the lanes of a wave, in a fixed order: the
// lanes exchange halves k times, each then holding three values of fewer lanes,
// and add those up.  Returns the first of the three; lanes that are multiples
// of 64 / 2^k have the totals.  (NV + 3 log2 exchanges instead of 6 NV: they go
// through the LDS, whose rate they were bound by.)
template <int NV>
__device__ __forceinline__ int wave_share_sum(double* v) {
  const int lane = threadIdx.x & 63;
  int base = 0, off = 32;
#pragma unroll
  for (int half = NV / 2; half >= 3; half /= 2, off /= 2) {
    const bool up = lane & off;
    if (up) base += half;
#pragma unroll
    for (int i = 0; i < half; ++i) {
      const double keep = up ? v[i + half] : v[i];
      const double give = up ? v[i] : v[i + half];
      v[i] = keep + __shfl_xor(give, off, 64);
    }
  }
#pragma unroll
  for (; off > 0; off /= 2)
#pragma unroll
    for (int i = 0; i < 3; ++i) v[i] += __shfl_xor(v[i], off, 64);
  return base;
}

// The same over a workgroup of NT threads: thread i < NV gets total i.  red:
// NT / 64 * NV doubles of LDS.
template <int NT, int NV>
__device__ __forceinline__ double block_share_sum(double* v, double* red) {
  constexpr int kStep = 64 * 3 / NV;
  static_assert(kStep >= 1 && NV == 3 * 64 / kStep, "three values a lane");
  const int tid = threadIdx.x, lane = tid & 63;
  const int base = wave_share_sum<NV>(v);
  if ((lane & (kStep - 1)) == 0)
#pragma unroll
    for (int i = 0; i < 3; ++i) red[(tid >> 6) * NV + base + i] = v[i];
  __syncthreads();
  double sum = 0.0;
  if (tid < NV)
    for (int i = 0; i < NT / 64; ++i) sum += red[i * NV + tid];
  return sum;
}

// Sum `cnt` doubles of every thread of the workgroup; thread i < cnt gets the
// total of value i.  red: LDS of (NT / 64) * cnt doubles.
template <int NT, int CNT>
__device__ __forceinline__ void block_sum(const double* v, double* red, double* out) {
  constexpr int cnt = CNT;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < cnt; ++i) {
    double x = v[i];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
    if (lane == 0) red[wave * cnt + i] = x;
  }
  __syncthreads();
  if ((int)threadIdx.x < cnt) {
    double s = 0.0;
    for (int w = 0; w < NT / 64; ++w) s += red[w * cnt + threadIdx.x];
    out[threadIdx.x] = s;
  }
  __syncthreads();
}

}  // namespace mils
