// kernels.h -- host-side launchers of the HIP kernels (kernels.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "mils_internal.h"

namespace mils {

// Stages of the single-series path, for per-stage event timing.
enum Stage {
  kStageStats = 0,
  kStageBin = 1,
  kStageSpreadF = 2,
  kStageSpread2F = 3,
  kStagePass0 = 4,  // first FFT pass (pruned), then 5, 6 for later middle passes
  kStageLast = 7,   // last FFT pass + deconvolution + power
  kStageLow = 8,    // direct sums near f = 0
  kStageRows = 9,   // row classes of both geometries (two-pass plans)
  kStageOut = 10,   // transpose into frequency order (two-pass plans)
  kNumStages = 11
};

// A second stream for the 2f geometry of a periodogram, with the events
// that fork it from and join it back to the call's stream.
struct AuxStream {
  hipStream_t s;
  hipEvent_t fork, join;
};

// Optional hook called before (begin = 1) and after (begin = 0) each stage is
// enqueued; used to record HIP events around the stage's kernels.
struct StageHook {
  void (*fn)(void* ud, int stage, int begin, hipStream_t s);
  void* ud;
};

// Enqueue the whole single-series path (statistics, binning, spread, FFT
// passes, deconvolution and power or raw sums) on stream s.
hipError_t launch_path(const CallArgs& a, const Plan& p, const Work& w, hipStream_t s,
                       const StageHook* hook = nullptr, const AuxStream* aux = nullptr);

// 1 / phihat(m) for m = 0..K by Gauss-Legendre quadrature of the kernel.
// Series that share their observation times and weights: the weights-only
// call aw (y == NULL, unit_y set; statistics into w.stats) leaves the
// deconvolved sums B and B2 of every output frequency in bsum_b and bsum_b2
// (interleaved re/im), and the binning and row lists in w.
hipError_t launch_weight_sums(const CallArgs& aw, const Plan& p, const Work& w, double* bsum_b,
                              double* bsum_b2, hipStream_t s);

// Up to three such series at once: series g has values y[g], writes power[g]
// and keeps its statistics in stats[g] and its direct sums near f = 0 in
// lowfix[g]; its A sums go through grid g of the workspace.
struct SeriesGroup {
  int m;
  int need_sort;  // the weights-only call's sort decision (read back by the host)
  const double* y[3];
  double* power[3];
  DevStats* stats[3];
  double* lowfix[3];
};
// a: the call's arguments with bsum_b, bsum_b2 and wstats set; w: the
// workspace of the weights-only call (w.stats its statistics).
hipError_t launch_series_group(const CallArgs& a, const Plan& p, const Work& w,
                               const SeriesGroup& sg, hipStream_t s);

// prologue.hip: the block partials of the statistics; then the statistics, the
// bins and the histogram of points that need the sort; then the row flags of
// ngeo geometries (0: none) and, with scatter, those points in bin order.
void enqueue_pro_stats(const CallArgs& a, const Plan& p, const Work& w, hipStream_t s);
void enqueue_bins(const CallArgs& a, const Plan& p, const Work& w, hipStream_t s);
void enqueue_rows(const CallArgs& a, const Plan& p, const Work& w, int ngeo, bool scatter,
                  hipStream_t s);

// Spread of geometry geo (1: f, 2: 2f) into grids gbase .. gbase + ng - 1 of w
// (spread.hip), over the tiles of rows whose flag is set.
void enqueue_spread(const CallArgs& a, const Plan& p, const Work& w, int geo, int ng, int gbase,
                    hipStream_t s);
// Allows a kernel more than 64 KB of dynamic LDS a workgroup.
void big_lds(const void* kern, size_t bytes);

// split.hip: the first pass of a split plan over grids g0 .. g0 + ng - 1 of w
// (grid grid_2f of geometry 2f); then the last: into sums s0 (grid g0) and s1
// (the next, or NULL) if given, else the power of a (three grids), or the
// powers of the a.nser series that share their weights.
void enqueue_split_first(const Plan& p, const Work& w, int g0, int ng, int grid_2f,
                         const LowRows& lr, hipStream_t s);
void enqueue_split_last(const CallArgs& a, const Plan& p, const Work& w, int g0, int ng,
                        int lowrows, double* s0, double* s1, hipStream_t s);

// In one launch: lowrows rows of direct sums near f = 0 (0: none), geometry f
// into grids 0 and 1, and geometry 2f into grid 2.
void enqueue_spread_pg(const CallArgs& a, const Plan& p, const Work& w, int lowrows, bool f,
                       bool f2, hipStream_t s);

// In one launch: the A spreads of the a.nser series into grids 0 .. of w, and
// lowrows rows of each one's direct sums.
void enqueue_spread_series(const CallArgs& a, const Plan& p, const Work& w, int lowrows,
                           hipStream_t s);

// Statistics of the call into w.stats (a.nser > 0: of each series).
void enqueue_stats(const CallArgs& a, const Work& w, hipStream_t s);

// Direct sums at every frequency, term by term, FP64 (direct.hip; statistics
// into w.stats, which with w.partials is all of w it uses): the power
// (a.power) or, with a.periodogram == 0, the raw sums of a.h (a.sums,
// interleaved re/im).  The points are split into nslice slices; more than one
// leaves its sums in part (direct_part_bytes).
constexpr int kDirectTile = 4096;  // frequencies of a workgroup
inline size_t direct_part_bytes(int64_t nf, bool periodogram, int nslice) {
  return nslice > 1 ? sizeof(double) * (periodogram ? 6 : 2) * (size_t)nslice *
                          (size_t)((nf + kDirectTile - 1) / kDirectTile * kDirectTile)
                    : 0;
}
hipError_t launch_direct(const CallArgs& a, const Work& w, int nslice, double* part,
                         hipStream_t s);
// Allows the kernels their LDS (before their first launch on a device).
hipError_t direct_prepare();

// 1 / phihat in the order of the two-pass FFT's last pass (see k_phihat2).
hipError_t launch_phihat2(double* iphi2, const double* inv_phihat, int L0, int L1, int64_t n,
                          int64_t nf, int64_t K, hipStream_t s);

hipError_t launch_phihat(double* inv_phihat, int64_t K, double w, double n, const double* z,
                         const double* gphi, int q, hipStream_t s);

}  // namespace mils
