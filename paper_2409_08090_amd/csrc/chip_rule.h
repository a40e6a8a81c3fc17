// chip_rule.h -- which FP64 series run on sub-grids in LDS (chip.h) and on which
// size, by estimated time (host only, no HIP: a host build checks it).
//
// The estimates for batches are fits to batches of 1 to 1000 equal series of 100 to 25000
// points at 1 to 100 frequencies a point, every size of sub-grid and the staged
// phases timed at each (270 layouts; eps = 1e-9): a workgroup takes a + b nd us
// (of a full chip's time, or alone, when the call waits for it), and a call of
// more workgroups than CUs ends about half a workgroup's time after the mean.
// The fits are within 6 % of the throughput, and the choice by them takes 1.5 %
// longer than the fastest choice in the mean and at most 20 %.  A limit on nd
// alone does not do: at 12 frequencies a point the staged phases are the
// faster ones from 6600 points (1000 series of 8000: 6.4 ms against 9.3), at
// 100 the sub-grids are up to 6000 (250 series of 4000: 6.1 ms against 8.3).
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <vector>

namespace mils {

// Sub-grid sizes; single calls take one of the first two.
constexpr int kChipBatchN[] = {256, 1024, 2048, 4096, 8192};
constexpr int kChipBatchSizes = 5;
// kinds of a batch's items: a grid size with the tolerance's kernel, or with
// the widest one
constexpr int kChipKinds = 2 * kChipBatchSizes;
// most frequencies of a series that takes the widest kernel (its whole grid
// fits one pass of the staged path, which does the same), and of a series
// whose three grids would fit one workgroup's LDS whole
constexpr int64_t kChipWideNf = 800, kChipOneNf = 2400;
// Most points of a series on sub-grids (the range of the fits), unless it has
// at most kChipOneNf frequencies.
constexpr int64_t kChipBatchNd = 16384;

// Residues (workgroups) of a series on sub-grids of at most nfmax frequencies.
inline int64_t chip_residues(int64_t nf, int nfmax) { return (nf + nfmax - 1) / nfmax; }

namespace chiprule {

struct Line {
  double a, b;  // us, us a point
  double at(int64_t nd) const { return a + b * (double)nd; }
};
constexpr Line kFull[kChipBatchSizes] = {
    {1.0, 8.0e-3}, {4.4, 7.8e-3}, {9.8, 8.2e-3}, {18.7, 12.5e-3}, {42.4, 13.0e-3}};
constexpr Line kAlone[kChipBatchSizes] = {
    {9.6, 13.0e-3}, {11.8, 10.8e-3}, {13.6, 10.4e-3}, {21.9, 14.6e-3}, {42.3, 14.9e-3}};
// kernels wider than 16 cells take two sets of lanes a point (eps = 1e-11)
constexpr double kTwoSets[kChipBatchSizes] = {1.8, 1.8, 1.55, 1.55, 1.55};
// a call on sub-grids alone, and what staged series add to it or take alone
constexpr double kCallUs = 60.0, kStagedCallUs = 105.0, kBothUs = 125.0;

// Staged series: its share of a full chip's time (grids of more than 104 000
// frequencies take three FFT passes, the others two), with the host's work on
// its items in a layout not seen before (1e-5 us a frequency); and the
// prologue's one workgroup, which the call waits for.
inline double staged_us(int64_t nd, int64_t nf) {
  return 0.066 + 8.3e-5 * (double)nd +
         (nf <= 104000 ? 7.7e-5 * (double)nf : 3.2 + 8.5e-5 * (double)nf);
}
inline double staged_alone_us(int64_t nd) { return 3.5e-3 * (double)nd; }

struct Rule {
  const int* nfmax;  // most frequencies of a residue, by size
  int num_cu;
  bool two_sets;     // the tolerance's kernel is wider than 16 cells

  // Size of sub-grid of a series where `top` is the largest: the smallest up
  // to it that holds the series whole.
  int size(int64_t nf, int top) const {
    int i = 0;
    while (i < top && nf > nfmax[i]) ++i;
    return i;
  }
  double full(int i, int64_t nd) const {
    return kFull[i].a + kFull[i].b * (two_sets ? kTwoSets[i] : 1.0) * (double)nd;
  }
  double alone(int i, int64_t nd) const {
    return kAlone[i].at(nd) * (two_sets ? 1.35 : 1.0);
  }
  bool takes(int64_t nd, int64_t nf) const { return nd <= kChipBatchNd || nf <= kChipOneNf; }
};

// Time of a batch's series on sub-grids: work is the sum of the items' time on
// a full chip (us of one CU).
struct ChipTime {
  double work = 0.0, items = 0.0, longest = 0.0;
  void add(const Rule& r, int i, int64_t nd, int64_t nf) {
    const double D = (double)chip_residues(nf, r.nfmax[i]);
    work += D * r.full(i, nd);
    items += D;
    longest = std::max(longest, r.alone(i, nd));
  }
  double us(const Rule& r) const {
    return items <= r.num_cu ? longest
                             : std::max(longest, work / r.num_cu + 0.5 * longest);
  }
};
struct StagedTime {
  double work = 0.0, longest = 0.0;
  int64_t n = 0;
  void add(int64_t nd, int64_t nf) {
    work += staged_us(nd, nf);
    longest = std::max(longest, staged_alone_us(nd));
    ++n;
  }
  double us(const Rule& r) const { return longest + work * 256.0 / r.num_cu; }
};
inline double call_us(const Rule& r, const ChipTime& c, const StagedTime& s) {
  return (c.items > 0.0 ? (s.n ? kBothUs : kCallUs) + c.us(r) : kStagedCallUs) +
         (s.n ? s.us(r) : 0.0);
}

// Size of sub-grid (index) of every series of a batch, -1: staged.  The batch's
// largest sub-grid is the one with which the call is estimated shortest: larger
// ones visit every point from fewer workgroups, smaller ones spread few series
// over the chip.  With it, every series on sub-grids, or only those that take
// less of the chip there than staged; or none.  Series of at most kChipOneNf
// frequencies always are on sub-grids.  all: staged only what cannot be.
inline void choose_batch(const Rule& r, const std::vector<int64_t>& nd,
                         const std::vector<int64_t>& nf, bool all, std::vector<int>* size) {
  const size_t m = nd.size();
  enum { kEvery, kCheaper, kNone };
  auto on = [&](int how, int i, size_t j) {
    if (nf[j] <= kChipOneNf) return true;
    if (how == kNone || !r.takes(nd[j], nf[j])) return false;
    return how == kEvery || r.full(i, nd[j]) * (double)chip_residues(nf[j], r.nfmax[i]) <=
                                256.0 * staged_us(nd[j], nf[j]);
  };
  double best = 1e300;
  int best_top = 0, best_how = kEvery;
  for (int top = 0; top < kChipBatchSizes; ++top)
    for (int how = kEvery; how <= (all ? kEvery : kNone); ++how) {
      ChipTime c;
      StagedTime s;
      for (size_t j = 0; j < m; ++j) {
        const int i = r.size(nf[j], top);
        if (on(how, i, j)) c.add(r, i, nd[j], nf[j]);
        else s.add(nd[j], nf[j]);
      }
      const double us = call_us(r, c, s);
      if (us < 0.97 * best) {
        best = us;
        best_top = top;
        best_how = how;
      }
    }
  size->assign(m, -1);
  for (size_t j = 0; j < m; ++j) {
    const int i = r.size(nf[j], best_top);
    if (on(best_how, i, j)) (*size)[j] = i;
  }
}

// The same for a series of the serving loop, from the series alone, so that its
// result does not depend on the requests it shares a batch with: the size that
// serves one such series and sixteen of them in the shortest time, or the
// staged phases where that takes 15 % more (a batch with staged series has
// their launches too).
inline int choose_alone(const Rule& r, int64_t nd, int64_t nf) {
  if (!r.takes(nd, nf)) return -1;
  double best = 1e300;
  int size = -1;
  for (int top = 0; top < kChipBatchSizes; ++top) {
    const int i = r.size(nf, top);
    ChipTime one, many;
    one.add(r, i, nd, nf);
    for (int k = 0; k < 16; ++k) many.add(r, i, nd, nf);
    const double us = call_us(r, one, {}) + call_us(r, many, {});
    if (us < 0.97 * best) {
      best = us;
      size = i;
    }
  }
  if (nf <= kChipOneNf) return size;
  StagedTime one, many;
  one.add(nd, nf);
  for (int k = 0; k < 16; ++k) many.add(nd, nf);
  return best <= 1.05 * (call_us(r, {}, one) + call_us(r, {}, many)) ? size : -1;
}

// ---- single calls ---------------------------------------------------------------
// A single call (pg false: of raw sums), on the first two sizes; series that
// share their times take the same, so that their results are the single calls'.
// Fits to 2 to 8000 points at 100 to 6e6 frequencies, within 8 %: a call takes
// 27 us and a round of workgroups, one a CU, `first` alone or `each` with more
// behind it, and `b` a point.  The staged kernels take 60 us of launches, a
// share a frequency (two passes; the split transform beyond 1.6e5) and, where
// few frequencies leave the spread few tiles, a share a point.  At 3e6
// frequencies and 100 points: 16 rounds 286 us, staged 195; at 1.2e4 and 1000
// 41 and 59.
struct Round {
  double first, each, b;
};
constexpr Round kRound[2] = {{7.5, 13.0, 7.5e-3}, {10.0, 15.5, 6.8e-3}};
constexpr Round kRoundSums[2] = {{7.0, 9.8, 3.8e-3}, {7.8, 11.0, 3.8e-3}};

inline double single_us(const Rule& r, int i, bool pg, int64_t nd, int64_t nf) {
  const Round& q = pg ? kRound[i] : kRoundSums[i];
  // (a periodogram has one more workgroup for each frequency near f = 0)
  const double blocks = (double)(chip_residues(nf, r.nfmax[i]) + (pg ? 16 : 0));
  const double rounds = std::ceil(blocks / r.num_cu);
  const double b = q.b * (r.two_sets ? (pg ? 1.75 : 1.55) : 1.0);
  return 27.0 + rounds * ((rounds > 1.0 ? q.each : q.first) + b * (double)nd);
}
inline double single_staged_us(bool pg, int64_t nd, int64_t nf) {
  const double share = pg ? 4.5e-5 : 2.2e-5;
  const double tiles = (double)nd * (pg ? std::min(16.5e-3, 10.0 / (double)nf)
                                        : std::min(14e-3, 25.0 / (double)nf));
  return (pg && nf > 160000 ? 68.0 : 60.0) + share * (double)nf + tiles;
}
// Size (0 or 1) of the sub-grids of such a call, -1: staged.
inline int choose_single(const Rule& r, bool pg, int64_t nd, int64_t nf) {
  double best = single_staged_us(pg, nd, nf);
  int size = -1;
  for (int i = 0; i < 2; ++i) {
    const double us = single_us(r, i, pg, nd, nf);
    if (us < best) {
      best = us;
      size = i;
    }
  }
  return size;
}

}  // namespace chiprule
}  // namespace mils
