// Host checks of the sub-grids in LDS (plan.cpp, chip_rule.h, chip_tables.cpp), built and run by
// tests/test_subgrid_host.py.  Prints "ok" at the end.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "../paper_2409_08090_amd/csrc/chip_rule.h"
#include "../paper_2409_08090_amd/csrc/chip_tables.h"
#include "../paper_2409_08090_amd/csrc/plan.h"

using namespace mils;

// Transform at mode m of n cells of the kernel of width w and shape beta: the
// trapezoidal rule in theta, z = sin theta.
static double phihat(int w, double beta, double m, double n) {
  constexpr int kSteps = 2000;
  double s = 0.0;
  for (int i = 1; i < kSteps; ++i) {
    const double th = M_PI * ((double)i / kSteps - 0.5), c = std::cos(th);
    s += std::exp(beta * (c - 1.0)) * c * std::cos(M_PI * w * std::sin(th) * m / n);
  }
  return 0.5 * w * s * M_PI / kSteps;
}

// Aliasing error of the sums at mode m, relative to the strengths: the worst
// a point can do.
static double aliasing(int w, double beta, double m, double n) {
  double s = 0.0;
  for (int j : {-2, -1, 1, 2}) s += std::fabs(phihat(w, beta, m + j * n, n));
  return s / std::fabs(phihat(w, beta, m, n));
}

// Sub-grids are as accurate at the edge of their residues' bands as the staged
// plans of grid classes are in the middle of their range: the aliasing of
// every size of sub-grid over the classes' frequencies against the staged
// plans' median.
static int accuracy() {
  int bad = 0;
  for (double eps : {1e-2, 1e-3, 1e-4, 1e-5, 1e-6, 1e-7, 1e-8, 1e-9, 1e-10, 1e-11, 1e-12}) {
    double sigma, beta;
    int w;
    chip_kernel(eps, false, &sigma, &w, &beta);
    const double s0 = planner_sigma(eps, 0, true);
    std::vector<double> staged, on;
    for (int j = 0; j < 190; ++j) {
      const int64_t nf = (int64_t)std::ceil(64.0 * std::pow(2.0, j / 16.0));
      if (nf <= kChipWideNf || nf > 200000) continue;
      PlanRequest r{nf, eps, 0, 3};
      r.batch = true;
      Plan own, cls;
      std::string err;
      if (!make_plan(r, &own, &err)) return 1;
      PlanRequest rc{(int64_t)std::floor((double)own.n / s0), eps, 0, 3};
      rc.batch = true;
      rc.n_fixed = own.n;
      if (!make_plan(rc, &cls, &err)) return 1;
      staged.push_back(aliasing(cls.w, cls.beta, 0.5 * (double)nf, (double)own.n));
      for (int N : kChipBatchN) {
        const int nfmax = (int)std::floor((double)N / sigma);
        const int64_t D = chip_residues(nf, nfmax);
        on.push_back(aliasing(w, beta, 0.5 * (double)((nf + D - 1) / D), (double)N));
      }
    }
    std::sort(staged.begin(), staged.end());
    std::sort(on.begin(), on.end());
    const double median = staged[staged.size() / 2];
    if (on.back() > median) {
      std::printf("eps %g, width %d: sub-grids up to %.2e, staged %.2e .. %.2e, median %.2e\n", eps,
                  w, on.back(), staged.front(), staged.back(), median);
      ++bad;
    }
  }
  return bad;
}

// The sizes that choose_batch gives, eps = 1e-9 on 256 CUs.
struct Sizes {
  int nfmax[kChipBatchSizes];
  chiprule::Rule rule(bool two_sets = false) const { return {nfmax, 256, two_sets}; }
  Sizes() {
    double sigma, beta;
    int w;
    chip_kernel(1e-9, false, &sigma, &w, &beta);
    for (int i = 0; i < kChipBatchSizes; ++i) nfmax[i] = (int)((double)kChipBatchN[i] / sigma);
  }
};

// Layouts of `count` series of nd points at nd ratio frequencies, timed both
// ways (us, replayed; the sub-grids at their best size): the rule takes the
// shorter.
static int choice() {
  const struct {
    int count, nd;
    double ratio;
    int staged_us, on_us;
  } timed[] = {
      {1, 100, 12, 106, 63},       {1, 4000, 12, 118, 99},      {1, 13000, 12, 167, 195},
      {1, 10000, 3, 129, 169},     {4, 13000, 1, 149, 200},     {4, 13000, 30, 247, 484},
      {4, 8000, 100, 362, 498},    {15, 2000, 12, 139, 88},     {15, 4000, 100, 604, 433},
      {15, 13000, 12, 359, 490},   {60, 1000, 12, 165, 92},     {60, 8000, 12, 477, 647},
      {60, 2000, 100, 1216, 599},  {60, 13000, 12, 1060, 1489}, {250, 4000, 30, 3277, 1909},
      {250, 4000, 3, 392, 270},    {250, 8000, 12, 1671, 2356}, {250, 13000, 12, 4074, 5322},
      {1000, 300, 30, 1005, 420},  {1000, 1000, 3, 514, 252},   {1000, 2000, 12, 1629, 1210},
      {1000, 8000, 12, 6382, 9251}, {1000, 13000, 3, 3274, 6070}};
  const Sizes s;
  int bad = 0;
  for (const auto& x : timed) {
    std::vector<int64_t> nd(x.count, x.nd), nf(x.count, (int64_t)(x.nd * x.ratio));
    std::vector<int> size;
    chiprule::choose_batch(s.rule(), nd, nf, false, &size);
    for (int z : size)
      if ((z < 0) != (x.staged_us < x.on_us)) {
        std::printf("%d x %d, ratio %g: size %d, staged %d us, sub-grids %d us\n", x.count, x.nd,
                    x.ratio, z, x.staged_us, x.on_us);
        ++bad;
        break;
      }
  }
  return bad;
}

// Single calls and raw sums, timed staged and on either size (us): the rule
// takes one within 12 % of the shortest.
static int single() {
  const struct {
    bool pg;
    int nd, nf;
    double us[3];  // staged, 256 cells, 1024 cells
  } timed[] = {
      {true, 100, 1200, {57.4, 34.5, 36.4}},       {true, 1000, 12000, {58.6, 39.7, 41.5}},
      {true, 3000, 48000, {60.8, 71.6, 56.6}},     {true, 5000, 30000, {61.0, 75.3, 71.6}},
      {true, 6000, 72000, {62.7, 140.3, 79.3}},    {true, 8000, 12000, {62.4, 100.3, 100.3}},
      {true, 8000, 100, {189.7, 157.1, 158.4}},    {true, 2, 200000, {89.6, 95.8, 56.0}},
      {true, 100, 500000, {99.4, 180.7, 73.9}},    {true, 100, 2000000, {154.0, 604.8, 204.0}},
      {true, 100, 3000000, {194.9, 893.4, 286.0}}, {true, 2, 6000000, {358.4, 1792.0, 560.8}},
      {true, 3000, 200000, {76.8, 203.1, 96.0}},   {false, 100, 12000, {60.2, 34.5, 35.4}},
      {false, 8000, 3000, {128.8, 63.6, 63.5}},    {false, 3000, 100000, {63.4, 87.6, 46.3}},
      {false, 100, 2000000, {104.3, 462.3, 153.5}}, {false, 100, 3000000, {125.7, 680.2, 211.6}},
      {false, 1000, 500000, {69.9, 170.8, 70.2}}};
  const Sizes s;
  int bad = 0;
  for (const auto& x : timed) {
    const int i = chiprule::choose_single(s.rule(), x.pg, x.nd, x.nf);
    const double best = std::min(x.us[0], std::min(x.us[1], x.us[2]));
    if (x.us[i + 1] > 1.12 * best) {
      std::printf("%s %d points, %d frequencies: size %d takes %.1f us, best %.1f\n",
                  x.pg ? "power" : "sums", x.nd, x.nf, i, x.us[i + 1], best);
      ++bad;
    }
  }
  return bad;
}

// Every choice is one that the kernels can take: a size whose residues hold the
// series, staged beyond the range of the rule unless the series is short enough
// for one workgroup, and with `all` whatever can be is on sub-grids.
static int forms() {
  const Sizes s;
  int bad = 0;
  unsigned x = 12345;
  auto rnd = [&]() { return (double)((x = x * 1664525u + 1013904223u) >> 8) / 16777216.0; };
  for (int trial = 0; trial < 300; ++trial) {
    const int m = 1 + (int)(rnd() * rnd() * 200);
    std::vector<int64_t> nd, nf;
    for (int i = 0; i < m; ++i) {
      nd.push_back((int64_t)std::exp(rnd() * std::log(1e6)));
      nf.push_back((int64_t)std::exp(rnd() * std::log((double)(1 << 28))));
      if (trial % 4 == 0) nf.back() = 1 + (int64_t)(rnd() * 3000);
    }
    for (bool all : {false, true})
      for (bool two : {false, true}) {
        std::vector<int> size;
        chiprule::choose_batch(s.rule(two), nd, nf, all, &size);
        for (int i = 0; i < m; ++i) {
          const bool can = nd[i] <= kChipBatchNd || nf[i] <= kChipOneNf;
          bool ok = size[i] >= -1 && size[i] < kChipBatchSizes;
          if (size[i] < 0) ok = ok && !(all && can) && nf[i] > kChipOneNf;
          else {
            const int64_t D = chip_residues(nf[i], s.nfmax[size[i]]);
            ok = ok && can && D * s.nfmax[size[i]] >= nf[i] && D <= 0x7fffffff &&
                 (nf[i] + D - 1) / D <= s.nfmax[size[i]];
          }
          if (!ok) {
            std::printf("nd %lld nf %lld: size %d\n", (long long)nd[i], (long long)nf[i], size[i]);
            ++bad;
          }
        }
      }
    // (a served series, from itself alone)
    for (int i = 0; i < m; ++i) {
      const int z = chiprule::choose_alone(s.rule(), nd[i], nf[i]);
      if (z < -1 || z >= kChipBatchSizes || (z < 0 && nf[i] <= kChipOneNf) ||
          (z >= 0 && nd[i] > kChipBatchNd && nf[i] > kChipOneNf)) {
        std::printf("served nd %lld nf %lld: size %d\n", (long long)nd[i], (long long)nf[i], z);
        ++bad;
      }
    }
  }
  return bad;
}

// A context's first call on sub-grids at a tolerance makes two kernel tables on
// the host beside the plan's own: together less than 0.5 ms (they took 1.2).
static int host_time() {
  double best = 1e9;
  for (int rep = 0; rep < 50; ++rep) {
    const auto t0 = std::chrono::steady_clock::now();
    std::vector<double> coef;
    for (bool wide : {false, true}) {
      Plan p{};
      chip_kernel(1e-9, wide, &p.sigma, &p.w, &p.beta);
      make_horner(p, &coef);
    }
    best = std::min(best, 1e3 * std::chrono::duration<double>(std::chrono::steady_clock::now() - t0)
                                    .count());
  }
  std::printf("two kernel tables %.3f ms\n", best);
  return best > 0.5;
}

// The tables of a tolerance: the layout, which every call without tables of its
// own asks for, costs next to nothing; what is made lies where it says, in
// pieces that do not overlap, and is what the kernels and sizes need.
static int tables() {
  int bad = 0;
  for (double eps : {1e-14, 1e-12, 1e-9, 1e-5, 1e-2}) {
    double best = 1e9;
    ChipTables t;
    for (int rep = 0; rep < 50; ++rep) {
      const auto t0 = std::chrono::steady_clock::now();
      t = layout_chip_tables(eps);
      best = std::min(best, std::chrono::duration<double>(std::chrono::steady_clock::now() - t0)
                                .count());
    }
    if (best > 50e-6) bad += std::printf("layout takes %.0f us\n", 1e6 * best) > 0;
    const std::vector<double> made = make_chip_tables(t);
    std::vector<std::pair<size_t, size_t>> used;  // [from, to)
    auto same = [&](const std::vector<double>& v, size_t at, const char* what) {
      used.push_back({at, at + v.size()});
      if (at + v.size() > t.host || std::memcmp(&made[at], v.data(), 8 * v.size()) != 0)
        bad += std::printf("eps %g: %s\n", eps, what) > 0;
    };
    std::vector<double> v, g;
    for (bool wide : {false, true}) {
      Plan p{};
      chip_kernel(eps, wide, &p.sigma, &p.w, &p.beta);
      make_horner(p, &v);
      same(v, t.hcoef[wide], "kernel polynomials");
      phihat_nodes(p, &v, &g);
      if ((int)v.size() != t.nnodes[wide]) bad += std::printf("nodes\n") > 0;
      v.insert(v.end(), g.begin(), g.end());
      same(v, t.nodes[wide], "quadrature nodes");
      for (int i = 0; i < kChipBatchSizes; ++i) {
        const ChipTables::Kind& k = t.kind[i + (wide ? kChipBatchSizes : 0)];
        if (k.w != p.w || k.N != kChipBatchN[i] || (double)k.nfmax * p.sigma > k.N || k.w % 2)
          bad += std::printf("eps %g: kind of %d cells\n", eps, k.N) > 0;
        used.push_back({k.iph, k.iph + (size_t)k.nfmax / 2 + 1});
      }
    }
    for (int i = 0; i < kChipBatchSizes; ++i) {
      make_twiddle2(kChipBatchN[i], &v);
      same(v, t.tw[i], "roots");
    }
    std::sort(used.begin(), used.end());
    for (size_t i = 0; i + 1 < used.size(); ++i)
      if (used[i].second > used[i + 1].first) bad += std::printf("pieces overlap\n") > 0;
    if (made.size() != t.host || 8 * used.back().second > t.bytes)
      bad += std::printf("sizes\n") > 0;
  }
  return bad;
}

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  const int bad = what == "accuracy" ? accuracy()
                  : what == "choice" ? choice()
                  : what == "single" ? single()
                  : what == "forms"  ? forms()
                  : what == "time"   ? host_time()
                  : what == "tables" ? tables()
                                     : 1;
  if (bad) return 1;
  std::printf("ok\n");
  return 0;
}
