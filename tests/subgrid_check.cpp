// Host checks of the sub-grids in LDS (plan.cpp, chip.h), built and run by
// tests/test_subgrid_host.py.  Prints "ok" at the end.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "../paper_2409_08090_amd/csrc/chip.h"
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

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  const int bad = what == "accuracy" ? accuracy() : 1;
  if (bad) return 1;
  std::printf("ok\n");
  return 0;
}
