// split.hip -- the FP64 transform of a mid-size grid in two passes (gfx950).
//
// n = R La L1 cells, cell l = l0 L1 + s, l0 = a + La r: the first pass takes
// the transforms down the columns s, split by the residue rho of their output
// digit m0 = rho + R kappa,
//   Y(s, rho + R kappa) = sum_a e(a kappa / La) [ e(a rho / (R La))
//                                 sum_r e(r rho / R) x(a + La r, s) ],
// a fold of the column to La cells and one transform of that length per
// residue, so that R may be any number (up to kSplitMax) while the lines stay powers of two in
// registers (fft2.h: 16 cells a thread).  The fold only reads the rows that a
// kernel support reaches: with the usual frequency step of 1/5 of the inverse
// time span those are a fifth (geometry f) and two fifths (2f) of the rows, so
// the R workgroups of a column block read about as much as one that reads all
// of it, from the L2 of the XCD they share.
//   The last pass takes the transforms along the rows m0, D rows side by side
// so that neighbouring lanes write neighbouring frequencies, m = m0 + L0 m1.
// A thread keeps its 16 modes of every grid in registers, so the power needs
// no exchange, and all its loads are issued before the first transform.
//
// The three-pass plans that this replaces move the grids through memory once
// more each way and hold lines of about 120 cells, with LDS traffic for every
// radix stage: 38 + 34 + 35 us for the three grids of 1.57e6 cells, here 21 +
// 37 (75 MB written and read: 15 us each at the rate of a fill).  Both passes
// are bound by their workgroups' latency, which load, exchange and store in
// turn, four (first) and two (last) waves a SIMD.
#include <hip/hip_runtime.h>

#include "fft2.h"
#include "kernels.h"
#include "path_device.h"

namespace mils {

namespace {

// exp(2 pi i x / n) from the plan's two-level table, 0 <= x < n.
struct Roots {
  const double2* lo;
  const double2* hi;
  int shift;
  __device__ __forceinline__ double2 operator()(int64_t x) const {
    return cmul(hi[x >> shift], lo[x & (((int64_t)1 << shift) - 1)]);
  }
};

// First pass of residue rho and the C columns of one column block of grid
// blockIdx.y: LA / 16 threads a column, the columns fastest.
template <int LA, int NT>
__global__ __launch_bounds__(NT, 4) void k_split_first(Fft2Bufs<double> b, FftPass ps, int R,
                                                       const double2* tw, const DevStats* st,
                                                       LowRows lr) {
  extern __shared__ __align__(16) unsigned char smem[];
  if (((ConstPtr<int>)&st->status)[0] != 0 || low_rows_block(lr)) return;
  constexpr int TL = LA / 16, C = NT / TL, LP = fft2::line_pitch_c(LA, C);
  constexpr int WR = 64 / C;  // rows that one load of a wave covers
  static_assert(C >= 4 && C <= 16 && WR >= 4, "rows of a wave in whole words of flags");
  const int tid = threadIdx.x;
  const int c = tid & (C - 1), t = tid / C;
  const int tw0 = __builtin_amdgcn_readfirstlane(t);  // a multiple of WR
  const int g = blockIdx.y;
  const int blk = (int)xcd_remap(blockIdx.x, (int64_t)gridDim.x - lr.n);
  const int rho = blk % R, s = (blk / R) * C + c;
  const int L1 = (int)ps.S;
  double* ex = reinterpret_cast<double*>(smem);
  double2* twl = reinterpret_cast<double2*>(smem + (size_t)C * LP * sizeof(double));
  for (int x = tid; x < tw2_count(LA); x += NT) twl[x] = tw[ps.twL_off + x];
  const Roots root{tw + ps.twlo_off, tw + ps.twhi_off, ps.bshift};
  const int sub = t - tw0;  // row of the thread among the WR
  const int lane = tid & 63;
  // Row flags, one load for four r: lane 16 i + q holds those of the wave's
  // rows of element q, a bit a row.
  constexpr int kFlags = (kSplitMax + 3) / 4;
  unsigned fl[kFlags];
#pragma unroll
  for (int i = 0; i < kFlags; ++i) {
    fl[i] = 0;
    const int r = 4 * i + (lane >> 4);
    if (r < R) {
      const unsigned* f = reinterpret_cast<const unsigned*>(b.rowflag[g] + tw0 +
                                                            TL * (lane & 15) + LA * r);
#pragma unroll
      for (int k = 0; k < WR / 4; ++k)
        fl[i] |= ((f[k] & 0x01010101u) * 0x10204080u >> 28) << (4 * k);
    }
  }
  // lane r: e(r rho / R)
  const double2 wl = root((int64_t)((lane < R ? lane : 0) * rho % R) * LA * L1);
  auto wl_of = [&](int r) {
    auto half = [&](double x) {
      const long long u = __double_as_longlong(x);
      const unsigned lo = __builtin_amdgcn_readlane((int)u, r);
      const unsigned hi = __builtin_amdgcn_readlane((int)(u >> 32), r);
      return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
    };
    return make_double2(half(wl.x), half(wl.y));
  };
  // r = 0 (factor 1) straight into the registers of the transform, the others
  // on top of it, eight at a time; elements none of whose rows is reached cost
  // a scalar branch
  double2 v[16];
  const double2* in = b.grid[g] + (int64_t)t * L1 + s;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    v[q] = make_double2(0.0, 0.0);
    if ((__builtin_amdgcn_readlane(fl[0], q) >> sub) & 1u) v[q] = in[(int64_t)(TL * q) * L1];
  }
  for (int r = 1; r < R; ++r) {
    unsigned f = fl[0];
#pragma unroll
    for (int i = 1; i < kFlags; ++i)
      if (r >= 4 * i) f = fl[i];
    const int r4 = 16 * (r & 3);
    const unsigned qm = (unsigned)(__ballot(f != 0) >> r4) & 0xffffu;
    if (!qm) continue;
    in = b.grid[g] + (int64_t)(r * LA + t) * L1 + s;
    const double2 wr = wl_of(r);
#pragma unroll
    for (int h = 0; h < 16; h += 8) {
      if (!((qm >> h) & 255u)) continue;
      double2 x[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        x[q] = make_double2(0.0, 0.0);
        if ((__builtin_amdgcn_readlane(f, r4 + h + q) >> sub) & 1u)
          x[q] = in[(int64_t)(TL * (h + q)) * L1];
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) v[h + q] = cadd(v[h + q], cmul(x[q], wr));
    }
  }
  // a = t + TL q: e(a rho / L0), from the first and the step
  if (rho > 0) {
    const double2 step = root((int64_t)TL * rho * L1);
    double2 w = root((int64_t)t * rho * L1);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      v[q] = cmul(v[q], w);
      if (q < 15) w = cmul(w, step);
    }
  }
  // e(s m0 / n) of the outputs m0 = rho + R (t + TL j), fetched before the
  // transform
  double2 tk = root((int64_t)s * (rho + R * t));
  const double2 ts = root((int64_t)s * R * TL);
  __syncthreads();
  f2_line<LA, true>(v, t, ex + c * LP, twl);
  double2* out = b.mid[g] + s;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    out[(int64_t)(rho + R * (t + TL * j)) * L1] = cmul(v[f2_reg_of<LA>(j)], tk);
    if (j < 15) tk = cmul(tk, ts);
  }
}

enum { kSplitPower, kSplitSums, kSplitSeries };

// Last pass of D rows.  NG grids a thread: the power of a series (three), raw
// sums (one; blockIdx.y the grid, whose sums go to sums[blockIdx.y]), or the
// powers of up to three series that share B and B2.
template <int L1, int NT, int NG, int MODE>
__global__ __launch_bounds__(NT, NG == 1 ? 4 : 2) void k_split_last(Fft2Bufs<double> b, FftPass ps,
                                                                  Plan pl, CallArgs a,
                                                                  const double2* tw,
                                                                  const double* inv_phihat,
                                                                  const DevStats* stp,
                                                                  const double* lowfix,
                                                                  int lowrows, double2* sums0,
                                                                  double2* sums1) {
  extern __shared__ __align__(16) unsigned char smem[];
  if (((ConstPtr<int>)&stp->status)[0] != 0) return;
  constexpr int TL = L1 / 16, D = NT / TL, LP = fft2::line_pitch_c(L1, D);
  const int tid = threadIdx.x;
  const int d = tid & (D - 1), t = tid / D;
  const int64_t L0 = ps.P;
  const int64_t m0 = xcd_remap(blockIdx.x, (int64_t)gridDim.x) * D + d;
  double* ex = reinterpret_cast<double*>(smem) + d * LP;
  double2* twl = reinterpret_cast<double2*>(smem + (size_t)D * LP * sizeof(double));
  double2 v[NG][16];
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    const double2* in = b.mid[MODE == kSplitSums ? blockIdx.y : g] + m0 * L1 + t;
#pragma unroll
    for (int q = 0; q < 16; ++q) v[g][q] = ld_stream(&in[TL * q]);
  }
  for (int x = tid; x < tw2_count(L1); x += NT) twl[x] = tw[ps.twL_off + x];
  __syncthreads();
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    // (the positions of each grid's exchanges are worked out anew: kept for
    // all of them, they would not fit beside the modes)
    int tg = t;
    asm volatile("" : "+v"(tg));
    f2_line<L1, true>(v[g], tg, ex, twl);
    // (all of it here: sunk into the branches of the outputs, the last stage
    // would keep more registers alive than it saves work)
#pragma unroll
    for (int q = 0; q < 16; ++q) asm volatile("" : "+v"(v[g][q].x), "+v"(v[g][q].y));
  }
  // The outputs four at a time, the next four's deconvolution factors on
  // their way; the barriers to the scheduler keep it from holding the factors
  // and addresses of all sixteen beside the modes' registers.
  const int n = (int)pl.n, nf = (int)a.nf, K = (int)pl.K, rows = (int)L0;
  int mb = (int)m0 + rows * t;
  auto output = [&](int j) {  // frequency of mode j, -1: cropped
    const int m = mb + rows * TL * j;
    const int k = (m <= nf - 1 - K ? m : m - n) + K;
    return k < nf ? k : -1;
  };
  auto factor = [&](int k) { return inv_phihat[k < 0 ? 0 : k < K ? K - k : k - K]; };
  DevStats st[MODE == kSplitSums ? 1 : MODE == kSplitPower ? 1 : NG];
  if constexpr (MODE == kSplitPower) st[0] = load_stats(stp);
  if constexpr (MODE == kSplitSeries)
#pragma unroll
    for (int g = 0; g < NG; ++g) st[g] = load_stats(a.sst[g]);
  // power of series g from its A and the shared or its own B and B2
  auto power = [&](int k, double2 A, double2 B, double2 B2, const DevStats& sg,
                   const double* lf) {
    double s6[6] = {A.x, A.y, B.x, B.y, B2.x, B2.y};
    const int q = k - (int)sg.k_lo;
    const bool low = q >= 0 && q < sg.nlow;
    if (low) {
      for (int i = 0; i < 6; ++i) s6[i] = lf[6 * q + i];
      for (int p = 1; p < lowrows; ++p)
        for (int i = 0; i < 6; ++i) s6[i] += lf[p * 6 * kLowMax + 6 * q + i];
    }
    const double p = ls_power(s6[0], s6[1], s6[2], s6[3], s6[4], s6[5], sg, a.norm, a.fit_mean,
                              low ? 0.0 : a.dmin);
    return k == a.kzero ? 0.0 : p;
  };
  int nan_count = 0;
  int k[4];
  double ip[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    k[i] = output(i);
    ip[i] = factor(k[i]);
  }
#pragma unroll
  for (int j0 = 0; j0 < 16; j0 += 4) {
    int kn[4];
    double nx[4];
    asm volatile("" : "+v"(mb));
    if (j0 < 12)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        kn[i] = output(j0 + 4 + i);
        nx[i] = factor(kn[i]);
      }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = f2_reg_of<L1>(j0 + i);
      auto mode = [&](int g) { return make_double2(v[g][r].x * ip[i], v[g][r].y * ip[i]); };
      const bool in = k[i] >= 0;
      if constexpr (MODE == kSplitSums) {
        const double2 A = mode(0);
        if (in) (blockIdx.y ? sums1 : sums0)[k[i]] = A;
      } else if constexpr (MODE == kSplitPower) {
        const double p = power(k[i], mode(0), mode(1), mode(2), st[0], lowfix);
        if (in) {
          if (p != p) ++nan_count;
          a.power[k[i]] = p;
        }
      } else {
        const int kk = in ? k[i] : 0;
        const double2 B = reinterpret_cast<const double2*>(a.bsum_b)[kk];
        const double2 B2 = reinterpret_cast<const double2*>(a.bsum_b2)[kk];
        double p[NG];
        p[0] = power(k[i], mode(0), B, B2, st[0], a.slow[0]);
        if constexpr (NG > 1) p[1] = power(k[i], mode(1), B, B2, st[1], a.slow[1]);
        if constexpr (NG > 2) p[2] = power(k[i], mode(2), B, B2, st[2], a.slow[2]);
        if (in) {
          if (st[0].status == 0) a.spow[0][k[i]] = p[0];
          if constexpr (NG > 1)
            if (st[1].status == 0) a.spow[1][k[i]] = p[1];
          if constexpr (NG > 2)
            if (st[2].status == 0) a.spow[2][k[i]] = p[2];
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (j0 < 12)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        k[i] = kn[i];
        ip[i] = nx[i];
      }
  }
  if (MODE == kSplitPower && nan_count) count_nan(a, const_cast<int*>(&stp->nill), nan_count);
}

template <int L, int NT>
constexpr size_t split_lds() {
  constexpr int C = NT / (L / 16);
  return (size_t)C * fft2::line_pitch_c(L, C) * sizeof(double) + tw2_count(L) * sizeof(double2);
}

Fft2Bufs<double> bufs(const Work& w, int g0, int ng, int grid_2f) {
  Fft2Bufs<double> b;
  for (int i = 0; i < 3; ++i) {
    const int g = g0 + (i < ng ? i : ng - 1);
    b.grid[i] = reinterpret_cast<double2*>(w.grid[g]);
    b.mid[i] = reinterpret_cast<double2*>(w.grid2[g]);
    b.rowflag[i] = g == grid_2f ? w.rowflag_2f : w.rowflag_f;
  }
  return b;
}

// (a workgroup's LDS above 64 KB must be allowed for its kernel)
template <int LA, int NT>
void first(const Plan& p, const Fft2Bufs<double>& b, int ng, const Work& w, const LowRows& lr,
           hipStream_t s) {
  constexpr int C = NT / (LA / 16);
  constexpr size_t lds = split_lds<LA, NT>();
  const FftPass& ps = p.pass[0];
  auto kern = k_split_first<LA, NT>;
  big_lds(reinterpret_cast<const void*>(kern), lds);
  hipLaunchKernelGGL(kern, dim3((unsigned)(ps.S / C * p.split) + lr.n, ng), dim3(NT), lds, s, b,
                     ps, p.split, reinterpret_cast<const double2*>(w.tw), w.stats, lr);
}

template <int L1, int NT, int NG, int MODE>
void last(const CallArgs& a, const Plan& p, const Fft2Bufs<double>& b, int ny, const Work& w,
          int lowrows, double* s0, double* s1, hipStream_t s) {
  constexpr int D = NT / (L1 / 16);
  const FftPass& ps = p.pass[1];
  hipLaunchKernelGGL((k_split_last<L1, NT, NG, MODE>), dim3((unsigned)(ps.P / D), ny), dim3(NT),
                     (split_lds<L1, NT>()), s, b, ps, p, a, reinterpret_cast<const double2*>(w.tw),
                     w.inv_phihat, w.stats, w.lowfix, lowrows, reinterpret_cast<double2*>(s0),
                     reinterpret_cast<double2*>(s1));
}

template <int L1, int NT, int NTS>
void last_l(const CallArgs& a, const Plan& p, const Fft2Bufs<double>& b, int ng, const Work& w,
            int lowrows, double* s0, double* s1, hipStream_t s) {
  if (s0) last<L1, NT, 1, kSplitSums>(a, p, b, s1 ? 2 : 1, w, lowrows, s0, s1, s);
  else if (!a.nser) last<L1, NT, 3, kSplitPower>(a, p, b, 1, w, lowrows, s0, s1, s);
  else if (ng == 3) last<L1, NTS, 3, kSplitSeries>(a, p, b, 1, w, lowrows, s0, s1, s);
  else if (ng == 2) last<L1, NTS, 2, kSplitSeries>(a, p, b, 1, w, lowrows, s0, s1, s);
  else last<L1, NTS, 1, kSplitSeries>(a, p, b, 1, w, lowrows, s0, s1, s);
}

}  // namespace

void enqueue_split_first(const Plan& p, const Work& w, int g0, int ng, int grid_2f,
                         const LowRows& lr, hipStream_t s) {
  const Fft2Bufs<double> b = bufs(w, g0, ng, grid_2f);
  // 8 columns (128-byte pieces) a workgroup: with 4, lines of 1024 took 320 us
  // instead of 297 in all at n = 6.3e6
  switch (p.la) {
    case 256: first<256, 256>(p, b, ng, w, lr, s); break;
    case 512: first<512, 256>(p, b, ng, w, lr, s); break;
    default: first<1024, 512>(p, b, ng, w, lr, s); break;
  }
}

void enqueue_split_last(const CallArgs& a, const Plan& p, const Work& w, int g0, int ng,
                        int lowrows, double* s0, double* s1, hipStream_t s) {
  const Fft2Bufs<double> b = bufs(w, g0, ng, -1);
  // As many workgroups as give every CU some at n ~ 1e6; the powers of series
  // that share B and B2 want rows side by side for the reads of those (1797 us
  // -> 1578 for eight series at n = 6.3e6), lines of 2048 for the power's stores
  switch (p.pass[1].L) {
    case 512: last_l<512, 128, 256>(a, p, b, ng, w, lowrows, s0, s1, s); break;
    case 1024: last_l<1024, 128, 256>(a, p, b, ng, w, lowrows, s0, s1, s); break;
    default: last_l<2048, 256, 256>(a, p, b, ng, w, lowrows, s0, s1, s); break;
  }
}

}  // namespace mils
