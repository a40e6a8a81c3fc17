// chip.h -- periodograms whose grids never leave the chip (chip.hip).
//
// The frequencies of a series are split by residue: k = rho + D kappa, rho <
// D.  The sums over kappa for one rho are the same transform again (first
// frequency f0 + rho df, step D df, about nf / D frequencies), on a grid of
// N >= 1.36 nf / D cells.  With D chosen so that N is one of a few powers of
// two, one workgroup takes one rho: it spreads all points of the series onto
// its grids in LDS, transforms them there and writes its share of the power.
// Nothing but the points and the power crosses HBM, the tables serve every
// number of frequencies, and a series is spread over D workgroups.  (A single
// call and one of shared times still make the staged plan of their size, which
// profiled, reproducible and refused calls fall back on.)  Every point is
// visited by D workgroups: the cheaper way for short series (chip_rule.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "chip_rule.h"
#include "mils_internal.h"

namespace mils {

// One sub-grid size: the kernel (shared by every size of a tolerance), the
// factors 1 / phihat(m) and the two-level table of exp(2 pi i x / N).
struct ChipPlan {
  int N;                // grid cells (a power of two)
  int nfmax;            // most frequencies of a sub-transform
  int w;                // kernel width (even)
  double hw;            // w / 2
  const double* hcoef;  // kernel polynomials (see kHornerK), FP64
  const double* iph;    // 1 / phihat(m), m = 0 .. nfmax / 2
  const double* tw;     // tw2_count(N) complex
};

// Status of a single call in host memory (written by the call's last
// workgroup) and the counter that finds that workgroup; zero between calls.
struct ChipDone {
  unsigned long long count;
};

// The whole periodogram (or, without a.periodogram, the raw sums) of one
// series on grids of cp.N cells, one workgroup per residue of D.
// host_status: device address of two pinned ints (status, ill-posed count).
// nseries > 1: series i of the same times has its values at a.y + i nd, its
// errors at a.dy + i dy_stride, its power at a.power + i nf, its statistics in
// st[i] and its counter in done[i] (at most kChipMaxSeries; host_status is
// series 0's).
constexpr int kChipMaxSeries = 64;
hipError_t launch_chip_single(const CallArgs& a, const ChipPlan& cp, int D, DevStats* st,
                              ChipDone* done, int* host_status, int nseries, int64_t dy_stride,
                              hipStream_t s);

// Batch: the statistics of the on-chip series and their point records
// (prologue, one workgroup per series), then one workgroup per item (series,
// residue) and grid size.
struct BatchArgs;
struct BatchItem;
hipError_t launch_chip_prologue(const BatchArgs& ba, const BatchItem* series, int n,
                                hipStream_t s);
hipError_t launch_chip_items(const BatchArgs& ba, const ChipPlan& cp, const BatchItem* items,
                             int n, hipStream_t s);

// Allows the kernels their dynamic LDS (once per device, before any launch).
hipError_t chip_prepare();

}  // namespace mils
