// chip_tables.cpp -- see chip_tables.h.
#include "chip_tables.h"

#include <algorithm>
#include <cmath>

#include "plan.h"

namespace mils {

namespace {

Plan kernel_plan(double eps, bool wide) {
  Plan p{};
  chip_kernel(eps, wide, &p.sigma, &p.w, &p.beta);
  return p;
}

}  // namespace

ChipTables layout_chip_tables(double eps) {
  ChipTables t;
  t.eps = eps;
  size_t off = 0;
  auto take = [&](size_t n) {  // 256-byte pieces
    const size_t at = off;
    off += (n + 31) & ~(size_t)31;
    return at;
  };
  for (int wide = 0; wide < 2; ++wide) {
    t.hcoef[wide] = take((size_t)kHornerN64 * kHornerK);
    t.nnodes[wide] = phihat_node_count(kernel_plan(eps, wide != 0).w);
    t.nodes[wide] = take(2 * (size_t)t.nnodes[wide]);
  }
  for (int i = 0; i < kChipBatchSizes; ++i) t.tw[i] = take(2 * (size_t)tw2_count(kChipBatchN[i]));
  t.host = off;
  for (int k = 0; k < kChipKinds; ++k) {
    const Plan p = kernel_plan(eps, k >= kChipBatchSizes);
    ChipTables::Kind& c = t.kind[k];
    c.N = kChipBatchN[k % kChipBatchSizes];
    c.nfmax = (int)std::floor((double)c.N / p.sigma);
    c.w = p.w;
    c.iph = take((size_t)(c.nfmax / 2 + 1));
  }
  t.bytes = sizeof(double) * off;
  return t;
}

std::vector<double> make_chip_tables(const ChipTables& t) {
  std::vector<double> out(t.host, 0.0), v, g;
  auto put = [&](const std::vector<double>& x, size_t at) {
    std::copy(x.begin(), x.end(), out.begin() + (std::ptrdiff_t)at);
  };
  for (int wide = 0; wide < 2; ++wide) {
    const Plan p = kernel_plan(t.eps, wide != 0);
    make_horner(p, &v);
    put(v, t.hcoef[wide]);
    phihat_nodes(p, &v, &g);
    put(v, t.nodes[wide]);
    put(g, t.nodes[wide] + (size_t)t.nnodes[wide]);
  }
  for (int i = 0; i < kChipBatchSizes; ++i) {
    make_twiddle2(kChipBatchN[i], &v);
    put(v, t.tw[i]);
  }
  return out;
}

}  // namespace mils
