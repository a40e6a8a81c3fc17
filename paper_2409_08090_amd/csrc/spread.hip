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

// Spreading over the tiles of the active rows only (their list and count come
// from k_row_compact): a fixed grid of workgroups takes tiles blk, blk + grid,
// ...; every tile is written by exactly one workgroup, so the result does not
// depend on scheduling.  T divides the row length S1 here.
template <typename Real, int GEO, int NG, int SETS>
__global__ __launch_bounds__(kThreads) void k_spread_rows(CallArgs a, Plan p, Work w, void* out0,
                                                          void* out1, const int* act_rows,
                                                          int slot) {
  __shared__ double acc[NG * 2 * kTileMax];
  const DevStats st = load_stats(w.stats);
  if (st.status != 0) return;
  const int tpr = (int)(p.S1 / p.T);
  const int ntile = *(ConstPtr<int>)(w.nact + slot) * tpr;
  for (int t = blockIdx.x; t < ntile; t += gridDim.x) {
    const int q = t / tpr;
    const int tile = ((ConstPtr<int>)act_rows)[q] * tpr + (t - q * tpr);
    spread_tile<Real, GEO, NG, kThreads, SETS>(tile, p.T, kTileMax, a, p, w, st, out0, out1,
                                               acc);
  }
}

// The same with fixed summation orders.
template <typename Real, int GEO, int NG>
__global__ __launch_bounds__(kThreads) void k_spread_det(CallArgs a, Plan p, Work w, void* out0,
                                                         void* out1, const int* act_rows,
                                                         int slot) {
  __shared__ double acc[NG * 2 * kTileMax];
  __shared__ int rb[8], re[8], sv[1];
  __shared__ SpreadRecords<Real, NG, kThreads> rec;
  const DevStats st = *w.stats;
  if (st.status != 0) return;
  const int tpr = (int)(p.S1 / p.T);
  const int ntile = w.nact[slot] * tpr;
  for (int t = blockIdx.x; t < ntile; t += gridDim.x) {
    const int q = t / tpr;
    const int tile = act_rows[q] * tpr + (t - q * tpr);
    spread_tile_det<Real, GEO, NG, kThreads>(tile, p.T, kTileMax, a, p, w, st, out0, out1, acc,
                                             rb, re, sv, rec);
  }
}

namespace {

template <typename Real, int GEO, int NG>
void enqueue(const CallArgs& a, const Plan& p, const Work& w, int gbase, hipStream_t s) {
  const int64_t ntiles = (p.S1 / p.T) * p.nrows;
  const dim3 grid((unsigned)(ntiles < kSpreadGrid ? ntiles : kSpreadGrid));
  void* out0 = w.grid[gbase];
  void* out1 = w.grid[gbase + NG - 1];
  const int* rows = GEO == 1 ? w.act_rows_f : w.act_rows_2f;
  if (a.deterministic)
    hipLaunchKernelGGL((k_spread_det<Real, GEO, NG>), grid, dim3(kThreads), 0, s, a, p, w, out0,
                       out1, rows, GEO - 1);
  else if (p.w <= 16)
    hipLaunchKernelGGL((k_spread_rows<Real, GEO, NG, 1>), grid, dim3(kThreads), 0, s, a, p, w,
                       out0, out1, rows, GEO - 1);
  else
    hipLaunchKernelGGL((k_spread_rows<Real, GEO, NG, 2>), grid, dim3(kThreads), 0, s, a, p, w,
                       out0, out1, rows, GEO - 1);
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

}  // namespace mils
