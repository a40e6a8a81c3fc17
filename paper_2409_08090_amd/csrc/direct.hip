// direct.hip -- direct sums: the three sums of every frequency evaluated term
// by term (Sec. 1, Eq. 1), O(N_d N_f), FP64 throughout (gfx950); a check of
// the transform at any size and the paper's brute-force comparison.
//
// The sums as a contraction: with a frequency written as f_q +- (r + 1/2) df,
// f_q the centre of 64 consecutive ones, the phase factor of point j is the
// product of one that depends on (j, q) and one that depends on (j, r):
//   cos(a +- b) = cos a cos b -+ sin a sin b,  sin(a +- b) = sin a cos b +- ...
// so four products summed over the points, cc, ss, sc and cs, give both
// frequencies: six FP64 multiply-adds for the three complex sums of a
// frequency and point.  They run on the matrix cores
// (v_mfma_f64_16x16x4_f64): a workgroup takes 64 centres x 32 offsets = 4096
// frequencies, a wave 16 centres x 32 offsets (24 accumulators), and the
// factors of 32 points at a time come from LDS.  The factors themselves are
// products of a coarse and a fine one (28 sincospi a point for the 96), each
// reduced in double-double.  The points are split into slices until there are
// two workgroups per CU.
//
// Bound: the rate of the FP64 matrix instruction, 44 TFLOP/s measured (the
// vector units do 69, but not at the same time, and the same tile on them, 2 x
// 4 a thread, waits for its LDS operands: 446 us where this takes 336).  At
// N_d = 1e4, N_f = 1.2e5 the call takes 0.36 ms, 12 frequencies a thread by
// recurrence (40 workgroups) 4.45 ms; at N_d = 1e6, N_f = 1.2e7 2.7 s
// instead of 8.6 s.
#include <hip/hip_runtime.h>

#include "device_math.h"
#include "kernels.h"
#include "mils_internal.h"
#include "path_device.h"

namespace mils {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int kNT = 256;        // 4 waves
constexpr int kPts = 32;        // points of a chunk
constexpr int kQ = 64;          // centres of a workgroup (16 per wave)
constexpr int kR = 32;          // offsets on either side of a centre
constexpr int kTile = kDirectTile;
static_assert(kTile == kQ * 2 * kR, "frequencies of a workgroup");

struct Chunk {
  double2 e1[kPts][kQ];         // exp(2 pi i f_q t): (cos, sin)
  double2 e2[kPts][kR];         // exp(2 pi i (r + 1/2) df t)
  double2 e4[kPts][kR];         // its square
  double2 w[kPts];              // (w^ y~, w^), 0 for slots without a point
};

// fh + fl = f0 + m df
__device__ __forceinline__ void dd_freq(double f0, double m, double df, double& fh, double& fl) {
  double p, e, s;
  dd_two_prod(m, df, p, e);
  dd_two_sum(f0, p, fh, s);
  fl = s + e;
}

__device__ __forceinline__ double2 phase(double t, double tau, double fh, double fl) {
  double2 z;
  prephase(t, tau, fh, fl, z.x, z.y);
  return z;
}

__device__ __forceinline__ v4d mfma(double a, double b, v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// One slice of the points (blockIdx.y) for one tile of frequencies
// (blockIdx.x).  part == NULL (a single slice): the power or the raw sums;
// else the sums of the slice, value v of frequency k at
// part[(slice nv + v) npad + k] (nv = 6, or 2 for raw sums).
template <bool PG>
__global__ __launch_bounds__(kNT, 2) void k_direct(CallArgs a, Work w, int64_t per, double* part,
                                                   int64_t npad) {
  extern __shared__ __align__(16) unsigned char smem[];
  Chunk& c = *reinterpret_cast<Chunk*>(smem);
  const DevStats st = *w.stats;
  if (st.status != 0) return;
  const int tid = threadIdx.x;
  const int64_t k0 = (int64_t)blockIdx.x * kTile;
  const int64_t jb = (int64_t)blockIdx.y * per;
  const int64_t je = jb + per < a.nd ? jb + per : a.nd;
  const double invW = 1.0 / st.W;
  // this thread's share of the factors of point tid / 8: i = tid % 8 is the
  // coarse index (centre 8 i, offset 8 i) and the fine one (centre or offset i
  // beyond a coarse one)
  const int i = tid & 7, p = tid >> 3;
  double f1h, f1l, f2h, f2l, f3h, f3l, f4h, f4l;
  dd_freq(a.f0, (double)k0 + (2 * kR) * 8.0 * i + (kR - 0.5), a.df, f1h, f1l);
  dd_freq(0.0, (2 * kR) * (double)i, a.df, f2h, f2l);
  dd_freq(0.0, 8.0 * (i & 3) + 0.5, a.df, f3h, f3l);
  dd_freq(0.0, (double)i, a.df, f4h, f4l);
  const int lane = tid & 63, wave = tid >> 6;
  const int row = lane & 15, kk = lane >> 4;  // operand element: (row, point kk) of a step
  constexpr int NACC = PG ? 12 : 4;
  v4d acc[2][NACC];
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int x = 0; x < NACC; ++x) acc[b][x] = (v4d){0.0, 0.0, 0.0, 0.0};
  for (int64_t j0 = jb; j0 < je; j0 += kPts) {
    const int64_t j = j0 + p;
    double t = st.tau, wy = 0.0, wh = 0.0;
    if (j < je) {
      t = a.t[j];
      if constexpr (PG) {
        double wj = 1.0;
        if (a.dy) {
          const double dv = a.dy[j];
          wj = 1.0 / (dv * dv);
        }
        wh = wj * invW;
        wy = wh * (a.y[j] - st.ysub);
      } else {
        wy = a.h[j];
      }
    }
    const double2 x1 = phase(t, st.tau, f1h, f1l), y1 = phase(t, st.tau, f2h, f2l);
    const double2 x2 = phase(t, st.tau, f3h, f3l), y2 = phase(t, st.tau, f4h, f4l);
    __syncthreads();  // the last chunk's factors have been read
    if (i == 0) c.w[p] = make_double2(wy, wh);
    const int g = lane & ~7;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const double2 y = make_double2(__shfl(y1.x, g + b, 64), __shfl(y1.y, g + b, 64));
      c.e1[p][8 * i + b] = cmul(x1, y);
    }
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      // offsets 8 (i & 3) + b, b = 4 (i >> 2) + h
      const int b = 4 * (i >> 2) + h;
      const double2 y = make_double2(__shfl(y2.x, g + b, 64), __shfl(y2.y, g + b, 64));
      const double2 z = cmul(x2, y);
      c.e2[p][8 * (i & 3) + b] = z;
      if constexpr (PG)
        c.e4[p][8 * (i & 3) + b] = make_double2(z.x * z.x - z.y * z.y, 2.0 * z.x * z.y);
    }
    __syncthreads();
#pragma unroll 2
    for (int s = 0; s < kPts / 4; ++s) {
      const int q = 4 * s + kk;
      const double2 wv = c.w[q], e = c.e1[q][16 * wave + row];
      const double ac = wv.x * e.x, as = wv.x * e.y;
      const double bc = wv.y * e.x, bs = wv.y * e.y;
      const double dc = bc * e.x - bs * e.y, ds = 2.0 * bc * e.y;
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const double2 z = c.e2[q][16 * b + row];
        acc[b][0] = mfma(ac, z.x, acc[b][0]);
        acc[b][1] = mfma(as, z.y, acc[b][1]);
        acc[b][2] = mfma(as, z.x, acc[b][2]);
        acc[b][3] = mfma(ac, z.y, acc[b][3]);
        if constexpr (PG) {
          acc[b][4] = mfma(bc, z.x, acc[b][4]);
          acc[b][5] = mfma(bs, z.y, acc[b][5]);
          acc[b][6] = mfma(bs, z.x, acc[b][6]);
          acc[b][7] = mfma(bc, z.y, acc[b][7]);
          const double2 z2 = c.e4[q][16 * b + row];
          acc[b][8] = mfma(dc, z2.x, acc[b][8]);
          acc[b][9] = mfma(ds, z2.y, acc[b][9]);
          acc[b][10] = mfma(ds, z2.x, acc[b][10]);
          acc[b][11] = mfma(dc, z2.y, acc[b][11]);
        }
      }
    }
  }
  // element v of an accumulator: centre 4 v + lane / 16 of the wave's 16,
  // offset lane % 16 of the block's 16
  constexpr int NV = PG ? 6 : 2;
  int nan_count = 0;
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int sgn = 0; sgn < 2; ++sgn) {
        const int q = 16 * wave + 4 * v + kk, r = 16 * b + row;
        const int64_t k = k0 + (2 * kR) * q + (sgn ? kR - 1 - r : kR + r);
        double s6[6];
#pragma unroll
        for (int x = 0; x < NACC / 4; ++x) {
          const double cc = acc[b][4 * x][v], ss = acc[b][4 * x + 1][v];
          const double sc = acc[b][4 * x + 2][v], cs = acc[b][4 * x + 3][v];
          s6[2 * x] = sgn ? cc + ss : cc - ss;
          s6[2 * x + 1] = sgn ? sc - cs : sc + cs;
        }
        if (k >= a.nf) continue;
        if (part) {
#pragma unroll
          for (int x = 0; x < NV; ++x) part[((int64_t)blockIdx.y * NV + x) * npad + k] = s6[x];
        } else if constexpr (PG) {
          double pw = ls_power(s6[0], s6[1], s6[2], s6[3], s6[4], s6[5], st, a.norm, a.fit_mean,
                               0.0);
          if (k == a.kzero) pw = 0.0;
          else if (pw != pw) ++nan_count;
          a.power[k] = pw;
        } else {
          reinterpret_cast<double2*>(a.sums)[k] = make_double2(s6[0], s6[1]);
        }
      }
  if (PG && nan_count) atomicAdd(&w.stats->nill, nan_count);
}

// Sums of the slices, in order, and the power.
template <bool PG>
__global__ __launch_bounds__(kNT) void k_direct_final(CallArgs a, Work w, const double* part,
                                                      int64_t npad, int nslice) {
  const DevStats st = *w.stats;
  if (st.status != 0) return;
  const int64_t k = (int64_t)blockIdx.x * kNT + threadIdx.x;
  if (k >= a.nf) return;
  constexpr int NV = PG ? 6 : 2;
  double s[NV];
#pragma unroll
  for (int x = 0; x < NV; ++x) s[x] = 0.0;
#pragma unroll 4
  for (int i = 0; i < nslice; ++i)
#pragma unroll
    for (int x = 0; x < NV; ++x) s[x] += part[((int64_t)i * NV + x) * npad + k];
  if constexpr (PG) {
    double pw = ls_power(s[0], s[1], s[2], s[3], s[4], s[5], st, a.norm, a.fit_mean, 0.0);
    if (k == a.kzero) pw = 0.0;
    else if (pw != pw) atomicAdd(&w.stats->nill, 1);
    a.power[k] = pw;
  } else {
    reinterpret_cast<double2*>(a.sums)[k] = make_double2(s[0], s[1]);
  }
}

template <bool PG>
hipError_t launch_t(const CallArgs& a, const Work& w, int nslice, double* part, hipStream_t s) {
  const int64_t ntile = (a.nf + kTile - 1) / kTile, npad = ntile * kTile;
  const int64_t per = ((a.nd + nslice - 1) / nslice + kPts - 1) / kPts * kPts;
  const dim3 grid((unsigned)ntile, (unsigned)nslice);
  hipLaunchKernelGGL(k_direct<PG>, grid, dim3(kNT), sizeof(Chunk), s, a, w, per,
                     nslice > 1 ? part : nullptr, npad);
  if (nslice > 1)
    hipLaunchKernelGGL(k_direct_final<PG>, dim3((unsigned)((a.nf + kNT - 1) / kNT)), dim3(kNT), 0,
                       s, a, w, part, npad, nslice);
  return hipGetLastError();
}

}  // namespace

hipError_t direct_prepare() {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_direct<true>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)sizeof(Chunk));
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_direct<false>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(Chunk));
  return e;
}

hipError_t launch_direct(const CallArgs& a, const Work& w, int nslice, double* part,
                         hipStream_t s) {
  (void)hipGetLastError();
  enqueue_stats(a, w, s);
  return a.periodogram ? launch_t<true>(a, w, nslice, part, s)
                       : launch_t<false>(a, w, nslice, part, s);
}

}  // namespace mils
