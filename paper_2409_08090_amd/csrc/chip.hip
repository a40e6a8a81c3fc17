// chip.hip -- periodograms on grids in LDS, one workgroup per residue of the
// frequency index (gfx950); see chip.h.
//
// What bounds it: every point is visited by all D workgroups of its series, and
// HBM sees only the points and the power, so the time is FP64 arithmetic and LDS
// adds.  A lane works out the coordinate and phase of one point; then 16 lanes
// take one point's cells, each lane with the polynomial of its own cell in
// registers (a second set for kernels of 17 to 20 cells), so that four points
// of the wave cost one evaluation by Horner's rule, two products and two LDS
// adds a grid.  A row's adds are one run of cells; with a point per lane the
// 64 runs of a wave's add collide in the banks (9 LDS cycles against 26).
#include <hip/hip_runtime.h>

#include <mutex>

#include "batch.h"
#include "chip.h"
#include "chip_index.h"
#include "device_math.h"
#include "fft_core.h"
#include "path_device.h"

namespace mils {

namespace {

// Cells past the end of a grid that a kernel support may run into; they are
// folded onto the start after the spread.
constexpr int kGhost = 32;

// ---- statistics -------------------------------------------------------------
struct Part {
  Moments m;
  double lo, hi;
  int bad;
};

__device__ __forceinline__ void part_add(Part& x, const CallArgs& a, int64_t j) {
  const double t = a.t[j];
  const double y = a.periodogram ? a.y[j] : a.h[j];
  double wj = 1.0;
  if (a.dy) {
    const double d = a.dy[j];
    if (!(d > 0.0) || !isfinite(d)) x.bad = 1;
    wj = 1.0 / (d * d);
  }
  if (!isfinite(t) || !isfinite(y) || !isfinite(wj)) x.bad = 1;
  x.lo = fmin(x.lo, t);
  x.hi = fmax(x.hi, t);
  moments_merge(x.m, wj, y, 0.0);
}

__device__ __forceinline__ void part_merge(Part& x, const Part& y) {
  moments_merge(x.m, y.m.W, y.m.mu, y.m.M2);
  x.lo = fmin(x.lo, y.lo);
  x.hi = fmax(x.hi, y.hi);
  x.bad |= y.bad;
}

// Statistics of the series by one workgroup, in a fixed order; every thread
// gets them.  sh: LDS, NT / 64 Parts.
template <int NT>
__device__ __forceinline__ DevStats chip_stats(const CallArgs& a, Part* sh) {
  const int tid = threadIdx.x;
  Part x = {{0.0, 0.0, 0.0}, INFINITY, -INFINITY, 0};
  for (int64_t j = tid; j < a.nd; j += NT) part_add(x, a, j);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    Part y;
    y.m.W = __shfl_down(x.m.W, off, 64);
    y.m.mu = __shfl_down(x.m.mu, off, 64);
    y.m.M2 = __shfl_down(x.m.M2, off, 64);
    y.lo = __shfl_down(x.lo, off, 64);
    y.hi = __shfl_down(x.hi, off, 64);
    y.bad = __shfl_down(x.bad, off, 64);
    part_merge(x, y);
  }
  if ((tid & 63) == 0) sh[tid >> 6] = x;
  __syncthreads();
  x = sh[0];
#pragma unroll
  for (int i = 1; i < NT / 64; ++i) part_merge(x, sh[i]);
  DevStats st;
  st.W = x.m.W;
  st.mu = x.m.mu;
  st.M2 = x.m.M2;
  st.tmin = x.lo;
  st.tmax = x.hi;
  st.invalid = x.bad;
  st.unsorted = 0;
  st.need_sort = 0;
  st.tau = a.periodogram ? x.lo : 0.0;
  st.ysub = a.center ? x.m.mu : 0.0;
  st.Ybar = a.center ? 0.0 : x.m.mu;
  double YY = x.m.M2 / x.m.W;
  if (!a.fit_mean && !a.center) YY += x.m.mu * x.m.mu;
  st.YY = YY;
  st.status = x.bad ? -1 : (a.periodogram && !(YY > 0.0)) ? -2 : 0;
  st.nill = 0;
  st.nlow = 0;
  st.k_lo = 0;
  return st;
}

// ---- spread -----------------------------------------------------------------
template <int NG, int AP, int SETS, int I>
__device__ __forceinline__ void add_points(double* acc, const LaneKernel<double, SETS>& lk, int w,
                                           int cnt, int lb, double u, const double* h) {
  if constexpr (I < 16) {
    // (four points a step; cnt is the same for the whole wave, and lanes
    // without a point have zero strengths)
    if (I % 4 == 0 && I >= cnt) return;
    const double ui = row_lane<I>(u);
    double* cell = acc + row_lane<I>(lb) + (threadIdx.x & 15);
    double v[SETS];
#pragma unroll
    for (int s = 0; s < SETS; ++s) v[s] = kernel_value(lk, s, ui);
#pragma unroll
    for (int c = 0; c < 2 * NG; ++c) {
      const double hi = row_lane<I>(h[c]);
      atomicAdd(&cell[c * AP], v[0] * hi);
      if constexpr (SETS == 2)
        if ((int)(threadIdx.x & 15) + 16 < w) atomicAdd(&cell[c * AP + 16], v[1] * hi);
    }
    add_points<NG, AP, SETS, I + 1>(acc, lk, w, cnt, lb, u, h);
  }
}

// The wave's points (one per lane, cnt of them in its first lanes; grid phase
// fh + pl cycles, fh in [0, 1)) onto NG grids: component c of cell x is
// acc[c AP + x], h the strengths (0 for lanes without a point).  16 lanes take
// one point's cells at a time, each with its own polynomial in registers, so
// that the adds of a row are one run of cells (9 LDS cycles for the wave's
// add, against 26 with a point per lane, whose 64 runs collide in the banks);
// the points' values come from their lanes by DPP broadcasts, with no LDS and
// no barrier.
template <int N, int NG, int AP, int SETS>
__device__ __forceinline__ void chip_add(double* acc, const LaneKernel<double, SETS>& lk,
                                         const ChipPlan& cp, int cnt, double fh, double pl,
                                         const double* h) {
  const double uh = (double)N * fh, ul = (double)N * pl;  // exact: N is a power of two
  double ci = floor(uh);
  double d = (uh - ci) + ul;
  const double fl = floor(d);
  ci += fl;
  d -= fl;
  if (d >= 1.0) {
    d -= 1.0;
    ci += 1.0;
  }
  const double o = ceil(d - cp.hw);
  const int lb = ((int)ci + (int)o) & (N - 1);
  const double u = 2.0 * (o + cp.hw - d) - 1.0;
  add_points<NG, AP, SETS, 0>(acc, lk, cp.w, cnt, lb, u, h);
}

// Phases of a point: f geometry grid phase (fh, pl) for the step g = gh + gl,
// and exp(2 pi i fc (t - tau)).
struct PointPhase {
  double fh, pl, pc, ps;
};
__device__ __forceinline__ PointPhase point_phase(double t, double tau, double gh, double gl,
                                                  double fch, double fcl) {
  PointPhase r;
  double th, tl, ph;
  dd_two_sum(t, -tau, th, tl);
  dd_two_prod(gh, th, ph, r.pl);
  r.pl = __builtin_fma(gh, tl, r.pl);
  r.pl = __builtin_fma(gl, th, r.pl);
  r.fh = ph - floor(ph);
  prephase(t, tau, fch, fcl, r.pc, r.ps);
  return r;
}

// One sweep over the points: geometry f strengths A and B and geometry 2f
// strengths B2 onto three grids (ALL), or one of them (which = 0, 1, 2), or
// the raw strengths (which = 0).  fetch(j, t, ha, hb): point j's time and real
// strengths.
template <int N, int NT, bool ALL, int AP, int SETS, typename Fetch>
__device__ __forceinline__ void chip_spread(double* acc, const LaneKernel<double, SETS>& lk,
                                            const ChipPlan& cp, int nd, double tau, double gh,
                                            double gl, double fch, double fcl, int which,
                                            const Fetch& fetch) {
  const int lane = threadIdx.x & 63;
  double tn = tau, hn[2] = {0.0, 0.0};
  int j0 = threadIdx.x - lane;
  if (j0 + lane < nd) fetch(j0 + lane, tn, hn[0], hn[1]);
  for (; j0 < nd; j0 += NT) {
    const int cnt = nd - j0;
    const double t = tn, ha = hn[0], hb = hn[1];
    // the next points' loads are in flight while these are added
    hn[0] = hn[1] = 0.0;
    if (j0 + NT + lane < nd) fetch(j0 + NT + lane, tn, hn[0], hn[1]);
    PointPhase p = point_phase(t, tau, gh, gl, fch, fcl);
    if constexpr (ALL) {
      const double h[4] = {ha * p.pc, ha * p.ps, hb * p.pc, hb * p.ps};
      chip_add<N, 2, AP, SETS>(acc, lk, cp, cnt, p.fh, p.pl, h);
    }
    if (ALL || which == 2) {
      // geometry 2f: twice the phase, the square of the factor
      const double c = p.pc, s = p.ps;
      p.pc = c * c - s * s;
      p.ps = 2.0 * c * s;
      p.fh += p.fh;
      p.fh = p.fh >= 1.0 ? p.fh - 1.0 : p.fh;
      p.pl *= 2.0;
    }
    const double hr = ALL || which != 0 ? hb : ha;
    const double h[2] = {hr * p.pc, hr * p.ps};
    chip_add<N, 1, AP, SETS>(acc + (ALL ? 4 * AP : 0), lk, cp, cnt, p.fh, p.pl, h);
  }
}

// ---- transforms -----------------------------------------------------------------
// exp(2 pi i x / L), two-level table in LDS
__device__ __forceinline__ double2 chip_tw(const double2* t, int x) {
  return cmul(t[kTwLo + (x >> 6)], t[x & (kTwLo - 1)]);
}

template <int L, int S>
__device__ __forceinline__ void chip_stage(double2 (&v)[chipfft::elems(L)], int t,
                                           const double2* twl) {
  constexpr int E = chipfft::elems(L);
  constexpr int R = chipfft::radix(L, S), NS = chipfft::ns(L, S), TL = chipfft::threads(L);
  constexpr int step = L / (NS * R);
#pragma unroll
  for (int k = 0; k < E / R; ++k) {
    if constexpr (NS > 1) {
      const int kb = (t + TL * k) & (NS - 1);
      const double2 w1 = chip_tw(twl, kb * step);
      double2 w = w1;
#pragma unroll
      for (int q = 1; q < R; ++q) {
        v[k * R + q] = cmul(v[k * R + q], w);
        if (q + 1 < R) w = cmul(w, w1);
      }
    }
    dft<R>(&v[k * R]);
  }
}

template <int L, int S>
__device__ __forceinline__ void chip_exchange(double2 (&v)[chipfft::elems(L)], int t,
                                              double2* line, bool act) {
  constexpr int E = chipfft::elems(L);
  constexpr int R = chipfft::radix(L, S), R2 = chipfft::radix(L, S + 1);
  constexpr int TL = chipfft::threads(L);
  if (act) {
#pragma unroll
    for (int k = 0; k < E / R; ++k)
#pragma unroll
      for (int q = 0; q < R; ++q)
        line[chipfft::pad(L, chipfft::out_pos(L, S, t + TL * k, q))] = v[k * R + q];
  }
  __syncthreads();
  if (act) {
#pragma unroll
    for (int k = 0; k < E / R2; ++k)
#pragma unroll
      for (int q = 0; q < R2; ++q)
        v[k * R2 + q] = line[chipfft::pad(L, chipfft::in_pos(L, S + 1, t + TL * k, q))];
  }
  __syncthreads();
}

// All stages of the line (act: this thread holds a part of one; every thread
// of the workgroup takes the barriers).
template <int L, int S = 0>
__device__ __forceinline__ void chip_line(double2 (&v)[chipfft::elems(L)], int t, double2* line,
                                          const double2* twl, bool act) {
  if (act) chip_stage<L, S>(v, t, twl);
  if constexpr (S + 1 < chipfft::nstages(L)) {
    chip_exchange<L, S>(v, t, line, act);
    chip_line<L, S + 1>(v, t, line, twl, act);
  }
}

// Writes the power of output k from its sums (deconvolved) or, near f = 0,
// from the direct ones (low; NULL: another workgroup writes those outputs).
__device__ __forceinline__ void chip_power(const CallArgs& a, const DevStats& st, int64_t k,
                                           double* s6, const double* low, int& nan_count) {
  const int64_t q = k - st.k_lo;
  const bool is_low = q >= 0 && q < st.nlow;
  if (is_low) {
    if (!low) return;
    for (int j = 0; j < 6; ++j) s6[j] = low[6 * q + j];
  }
  double pw = ls_power(s6[0], s6[1], s6[2], s6[3], s6[4], s6[5], st, a.norm, a.fit_mean,
                       is_low ? 0.0 : a.dmin);
  if (k == a.kzero) pw = 0.0;
  else if (pw != pw) ++nan_count;
  a.power[k] = pw;
}

// Shape of a workgroup for grids of N cells: the three grids at once up to
// 2048 cells (transform threads: N / E per grid), beyond that one after another
// (their spectra kept in registers, which hold the same modes for every grid).
template <int N>
struct ChipShape {
  static constexpr bool seq = N > 2048;
  static constexpr int E = chipfft::elems(N);           // elements of a thread
  static constexpr int NT = seq ? N / E : (N == 2048 ? 1024 : N == 1024 ? 512 : 256);
  // threads of a single call: one workgroup on a CU of its own, so more waves
  static constexpr int NT1 = 1024;
  static constexpr int G = seq ? 1 : 3;
  static constexpr int AP = N + kGhost;                 // doubles per component
  static constexpr int LP = chipfft::line_pitch(N);     // complex per exchange line
  static constexpr size_t acc_bytes = sizeof(double) * 2 * G * AP;
  static constexpr size_t line_bytes = 16 * (size_t)G * LP;
  static constexpr size_t buf_bytes = acc_bytes > line_bytes ? acc_bytes : line_bytes;
  static constexpr size_t coef_bytes = sizeof(double) * kHornerN64 * kHornerK;
  static constexpr size_t lds = buf_bytes + 16 * (size_t)tw2_count(N) + coef_bytes;
};

// One residue of one series: grids, transforms, power (or raw sums, PG
// false).  low: direct sums of the outputs k_lo .. k_lo + nlow - 1.
template <int N, int NT, bool PG, int SETS, typename Fetch>
__device__ __forceinline__ int chip_residue(const CallArgs& a, const DevStats& st,
                                            const ChipPlan& cp, int D, int rho,
                                            const Fetch& fetch, const double* low,
                                            unsigned char* smem) {
  using S = ChipShape<N>;
  constexpr int E = S::E, AP = S::AP, TL = chipfft::threads(N), LP = S::LP;
  constexpr int G = PG ? S::G : 1;
  const int tid = threadIdx.x;
  double* acc = reinterpret_cast<double*>(smem);
  double2* line = reinterpret_cast<double2*>(smem);
  double2* twl = reinterpret_cast<double2*>(smem + S::buf_bytes);
  const double2* tw = reinterpret_cast<const double2*>(cp.tw);
  for (int x = tid; x < tw2_count(N); x += NT) twl[x] = tw[x];
  double* coef = reinterpret_cast<double*>(twl + tw2_count(N));
  for (int x = tid; x < kHornerN64 * kHornerK; x += NT) coef[x] = cp.hcoef[x];
  __syncthreads();
  const int nd = (int)a.nd;
  const int nfr = (int)((a.nf - rho + D - 1) / D);  // frequencies of this residue
  const int K = nfr / 2;
  // step D df and centre f0 + (rho + D K) df as double-doubles
  double gh, gl, ph, pe, fch, fe;
  dd_two_prod((double)D, a.df, gh, gl);
  dd_two_prod((double)rho + (double)D * (double)K, a.df, ph, pe);
  dd_two_sum(a.f0, ph, fch, fe);
  const double fcl = fe + pe;
  auto clear = [&]() {
    for (int x = tid; x < 2 * G * AP; x += NT) acc[x] = 0.0;
    __syncthreads();
  };
  auto fold = [&]() {  // the cells past the end onto the start
    __syncthreads();
    constexpr int F = 2 * G * kGhost;
    for (int x = tid; x < F; x += NT) {
      double* c = acc + (x / kGhost) * AP;
      c[x % kGhost] += c[N + x % kGhost];
    }
    __syncthreads();
  };
  auto load = [&](double2(&v)[E], int g, int t) {
    const double* re = acc + 2 * g * AP;
#pragma unroll
    for (int q = 0; q < E; ++q) v[q] = make_double2(re[t + q * TL], re[AP + t + q * TL]);
  };
  int nan_count = 0;
  if constexpr (!PG || !S::seq) {
    LaneKernel<double, SETS> lk;
    load_kernel(lk, coef);
    clear();
    chip_spread<N, NT, PG, AP, SETS>(acc, lk, cp, nd, st.tau, gh, gl, fch, fcl, 0, fetch);
    fold();
    const int g = tid / TL, t = tid - g * TL;
    const bool act = g < G;
    double2 v[E];
    if (act) load(v, g, t);
    __syncthreads();
    chip_line<N>(v, t, line + (act ? g * LP : 0), twl, act);
    if (act) {
#pragma unroll
      for (int j = 0; j < E; ++j) line[g * N + t + TL * j] = v[chipfft::reg_of(N, j)];
    }
    __syncthreads();
    for (int kap = tid; kap < nfr; kap += NT) {
      const int mm = kap - K;
      const int m = mm & (N - 1);
      const double ip = cp.iph[mm < 0 ? -mm : mm];
      const int64_t k = rho + (int64_t)D * kap;
      const double2 A = line[m];
      if constexpr (PG) {
        const double2 B = line[N + m], B2 = line[2 * N + m];
        double s6[6] = {A.x * ip, A.y * ip, B.x * ip, B.y * ip, B2.x * ip, B2.y * ip};
        chip_power(a, st, k, s6, low, nan_count);
      } else {
        reinterpret_cast<double2*>(a.sums)[k] = make_double2(A.x * ip, A.y * ip);
      }
    }
  } else {
    static_assert(TL == NT, "one line of N / E threads");
    // one grid after another (t is opaque in each, so that the transform's LDS
    // addresses are not kept in registers from one grid to the next)
    auto one_grid = [&](double2(&v)[E], int g) {
      int t = tid;
      asm volatile("" : "+v"(t));
      clear();
      LaneKernel<double, SETS> lk;
      load_kernel(lk, coef);
      chip_spread<N, NT, false, AP, SETS>(acc, lk, cp, nd, st.tau, gh, gl, fch, fcl, g, fetch);
      fold();
      load(v, 0, t);
      __syncthreads();
      chip_line<N>(v, t, line, twl, true);
    };
    double2 va[E], vb[E], vc[E];
    one_grid(va, 0);
    one_grid(vb, 1);
    one_grid(vc, 2);
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const int m = tid + TL * j;
      const int mm = m <= nfr - 1 - K ? m : m - N;
      const int kap = mm + K;
      if (kap < 0 || kap >= nfr) continue;
      const double ip = cp.iph[mm < 0 ? -mm : mm];
      const int64_t k = rho + (int64_t)D * kap;
      const int r = chipfft::reg_of(N, j);
      double s6[6] = {va[r].x * ip, va[r].y * ip, vb[r].x * ip,
                      vb[r].y * ip, vc[r].x * ip, vc[r].y * ip};
      chip_power(a, st, k, s6, low, nan_count);
    }
  }
  return nan_count;
}

// ---- one series in one launch ---------------------------------------------------
// Workgroups 0 .. D - 1 take the residues; workgroup D + q writes the output
// k_lo + q near f = 0 from its direct sums.  Each forms the statistics itself
// (the same sums in the same order in all of them), and the one that finishes
// last leaves the status in host memory, so that a call is one launch and one
// wait.  The time is the latency of one workgroup that visits every point.
template <int N, bool PG, int SETS>
__global__ __launch_bounds__(ChipShape<N>::NT1) void k_chip_single(CallArgs a, ChipPlan cp, int D,
                                                                   DevStats* stp, ChipDone* done,
                                                                   int* host_status,
                                                                   int64_t dy_stride) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int NT = ChipShape<N>::NT1;
  __shared__ Part parts[NT / 64];
  __shared__ int nan_block;
  const int tid = threadIdx.x;
  const int rho = blockIdx.x;
  const int64_t series = blockIdx.y;  // of those sharing their times
  if (PG) a.y += series * a.nd;
  if (a.dy) a.dy += series * dy_stride;
  a.power += series * a.nf;
  stp += series;
  done += series;
  if (tid == 0) nan_block = 0;
  DevStats st = chip_stats<NT>(a, parts);
  if (st.status != 0) {
    if (rho == 0 && tid == 0) {
      stp->status = st.status;
      stp->nill = 0;
      if (series == 0) {
        host_status[0] = st.status;
        host_status[1] = 0;
      }
    }
    return;
  }
  if constexpr (PG) low_band(st, a.f0, a.df, a.nf, st.k_lo, st.nlow);
  int nan_count = 0;
  if (rho < D) {
    const double invW = 1.0 / st.W, ysub = st.ysub;
    auto fetch = [&](int j, double& t, double& ha, double& hb) {
      t = a.t[j];
      if constexpr (PG) {
        double wj = 1.0;
        if (a.dy) {
          const double dv = a.dy[j];
          wj = 1.0 / (dv * dv);
        }
        hb = wj * invW;
        ha = hb * (a.y[j] - ysub);
      } else {
        ha = a.h[j];
        hb = 0.0;
      }
    };
    nan_count = chip_residue<N, NT, PG, SETS>(a, st, cp, D, rho, fetch, nullptr, smem);
  } else if (rho - D < st.nlow) {
    const int64_t k = st.k_lo + (rho - D);
    double acc[6];
    low_accumulate<1>(a, st, k, 1, tid, NT, acc);
    double* red = reinterpret_cast<double*>(smem);
    double* sum = red + 6 * (NT / 64);
    block_sum<NT, 6>(acc, red, sum);
    if (tid == 0) {
      double s6[6];
      for (int i = 0; i < 6; ++i) s6[i] = sum[i];
      st.k_lo = k;
      chip_power(a, st, k, s6, s6, nan_count);
    }
  }
  if (PG && nan_count) atomicAdd(&nan_block, nan_count);
  __syncthreads();
  if (tid == 0) {
    // finished workgroups in the low word, their ill-posed outputs in the high
    const unsigned long long mine = 1ull + ((unsigned long long)nan_block << 32);
    const unsigned long long all = atomicAdd(&done->count, mine) + mine;
    if ((unsigned)all == gridDim.x) {
      const int nill = (int)(all >> 32);
      done->count = 0;
      stp->status = 0;
      stp->nill = nill;
      if (series == 0) {
        host_status[0] = 0;
        host_status[1] = nill;
      }
    }
  }
}

// ---- batches --------------------------------------------------------------------

__device__ __forceinline__ CallArgs chip_args(const BatchArgs& ba, const BatchCurve& c) {
  CallArgs a{};
  a.t = ba.t + c.t_off;
  a.y = ba.y + c.t_off;
  a.dy = ba.dy ? ba.dy + c.t_off : nullptr;
  a.nd = c.nd;
  a.nf = c.nf;
  a.f0 = c.f0;
  a.df = c.df;
  a.kzero = c.kzero;
  a.norm = ba.norm;
  a.dmin = ba.dmin;
  a.center = ba.center;
  a.fit_mean = ba.fit_mean;
  a.periodogram = 1;
  a.power = ba.power + c.out_off;
  return a;
}

// Statistics, point records (w^ y~, w^: the visits then need no division) and
// the direct sums near f = 0 of one series.
template <int NT>
__global__ __launch_bounds__(NT) void k_chip_pro(BatchArgs ba, const BatchItem* series) {
  constexpr int NV = 6 * kLowMax;
  __shared__ Part parts[NT / 64];
  __shared__ double red[NT / 64 * NV];
  const int tid = threadIdx.x;
  const int ci = series[blockIdx.x].curve;
  const BatchCurve& c = ba.curves[ci];
  const Work& w = ba.works[ci];
  const CallArgs a = chip_args(ba, c);
  DevStats st = chip_stats<NT>(a, parts);
  if (tid == 0) ba.status[c.index] = st.status;
  if (st.status != 0) {
    if (tid == 0) *w.stats = st;
    return;
  }
  const double invW = 1.0 / st.W;
  double2* rec = reinterpret_cast<double2*>(w.rec);
  for (int j = tid; j < (int)a.nd; j += NT) {
    double wj = 1.0;
    if (a.dy) {
      const double dv = a.dy[j];
      wj = 1.0 / (dv * dv);
    }
    const double wh = wj * invW;
    rec[j] = make_double2(wh * (a.y[j] - st.ysub), wh);
  }
  low_band(st, a.f0, a.df, a.nf, st.k_lo, st.nlow);
  if (st.nlow > 0) {
    double acc[NV];
    low_accumulate<kLowMax>(a, st, st.k_lo, st.nlow, tid, NT, acc);
    const double sum = block_share_sum<NT, NV>(acc, red);
    if (tid < 6 * st.nlow) w.lowfix[tid] = sum;
  }
  if (tid == 0) *w.stats = st;
}

template <int N, int SETS>
__global__ __launch_bounds__(ChipShape<N>::NT, ChipShape<N>::NT / 256) void k_chip_item(BatchArgs ba, ChipPlan cp,
                                                                const BatchItem* items) {
  extern __shared__ __align__(16) unsigned char smem[];
  // the items of a series on one XCD: its points and the lines of its power
  // that the residues fill together stay in that XCD's L2
  const BatchItem it = items[xcd_remap(blockIdx.x, gridDim.x)];
  const BatchCurve& c = ba.curves[it.curve];
  const Work& w = ba.works[it.curve];
  const DevStats st = *w.stats;
  if (st.status != 0) return;
  const CallArgs a = chip_args(ba, c);
  const double2* rec = reinterpret_cast<const double2*>(w.rec);
  auto fetch = [&](int j, double& t, double& ha, double& hb) {
    t = a.t[j];
    const double2 r = rec[j];
    ha = r.x;
    hb = r.y;
  };
  chip_residue<N, ChipShape<N>::NT, true, SETS>(a, st, cp, it.plan, it.sub, fetch, w.lowfix, smem);
}

template <int N, int SETS>
hipError_t allow_lds() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(k_chip_item<N, SETS>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)ChipShape<N>::lds);
}

template <int SETS>
hipError_t allow_all() {
  hipError_t e = allow_lds<2048, SETS>();
  if (e == hipSuccess) e = allow_lds<4096, SETS>();
  if (e == hipSuccess) e = allow_lds<8192, SETS>();
  return e;
}

template <int N, int SETS>
void launch_items(const BatchArgs& ba, const ChipPlan& cp, const BatchItem* items, int n,
                  hipStream_t s) {
  using S = ChipShape<N>;
  hipLaunchKernelGGL((k_chip_item<N, SETS>), dim3((unsigned)n), dim3(S::NT), S::lds, s, ba, cp,
                     items);
}

template <int SETS>
hipError_t launch_items_of(const BatchArgs& ba, const ChipPlan& cp, const BatchItem* items,
                           int n, hipStream_t s) {
  switch (cp.N) {
    case 256: launch_items<256, SETS>(ba, cp, items, n, s); break;
    case 1024: launch_items<1024, SETS>(ba, cp, items, n, s); break;
    case 2048: launch_items<2048, SETS>(ba, cp, items, n, s); break;
    case 4096: launch_items<4096, SETS>(ba, cp, items, n, s); break;
    case 8192: launch_items<8192, SETS>(ba, cp, items, n, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <bool PG, int SETS>
void launch_single(const CallArgs& a, const ChipPlan& cp, int D, DevStats* st, ChipDone* done,
                   int* host_status, int nseries, int64_t dy_stride, hipStream_t s) {
  const dim3 grid((unsigned)(D + (PG ? kLowMax : 0)), (unsigned)nseries);
  if (cp.N == 1024) {
    using S = ChipShape<1024>;
    hipLaunchKernelGGL((k_chip_single<1024, PG, SETS>), grid, dim3(S::NT1), S::lds, s, a, cp, D,
                       st, done, host_status, dy_stride);
  } else {
    using S = ChipShape<256>;
    hipLaunchKernelGGL((k_chip_single<256, PG, SETS>), grid, dim3(S::NT1), S::lds, s, a, cp, D,
                       st, done, host_status, dy_stride);
  }
}

}  // namespace

hipError_t chip_prepare() {
  static std::mutex mu;
  static uint64_t done = 0;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lk(mu);
  const uint64_t bit = dev < 64 ? (uint64_t)1 << dev : 0;
  if (bit && (done & bit)) return hipSuccess;
  e = allow_all<1>();
  if (e == hipSuccess) e = allow_all<2>();
  if (e == hipSuccess) done |= bit;
  return e;
}

hipError_t launch_chip_single(const CallArgs& a, const ChipPlan& cp, int D, DevStats* st,
                              ChipDone* done, int* host_status, int nseries, int64_t dy_stride,
                              hipStream_t s) {
  (void)hipGetLastError();
  const bool wide = cp.w > 16;
  if (a.periodogram) {
    if (wide) launch_single<true, 2>(a, cp, D, st, done, host_status, nseries, dy_stride, s);
    else launch_single<true, 1>(a, cp, D, st, done, host_status, nseries, dy_stride, s);
  } else {
    if (wide) launch_single<false, 2>(a, cp, D, st, done, host_status, nseries, dy_stride, s);
    else launch_single<false, 1>(a, cp, D, st, done, host_status, nseries, dy_stride, s);
  }
  return hipGetLastError();
}

constexpr int kProWide = 512;
hipError_t launch_chip_prologue(const BatchArgs& ba, const BatchItem* series, int n,
                                hipStream_t s) {
  (void)hipGetLastError();
  // Few series: eight waves each, as the call waits for the longest (32 us for
  // up to 5000 points against 46 with four).  Many: four, of which a CU holds
  // two workgroups (10 000 series: 0.8 ms against 1.0).
  if (n < kProWide) hipLaunchKernelGGL(k_chip_pro<512>, dim3((unsigned)n), dim3(512), 0, s, ba, series);
  else hipLaunchKernelGGL(k_chip_pro<256>, dim3((unsigned)n), dim3(256), 0, s, ba, series);
  return hipGetLastError();
}

hipError_t launch_chip_items(const BatchArgs& ba, const ChipPlan& cp, const BatchItem* items,
                             int n, hipStream_t s) {
  (void)hipGetLastError();
  return cp.w > 16 ? launch_items_of<2>(ba, cp, items, n, s)
                   : launch_items_of<1>(ba, cp, items, n, s);
}

}  // namespace mils
