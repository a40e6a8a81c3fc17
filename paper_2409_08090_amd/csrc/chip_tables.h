// chip_tables.h -- the tables of the sub-grids in LDS (chip.h) for a tolerance,
// every size and kernel together (host only): two kernel polynomial tables, the
// nodes of their transforms, the roots of every size, and room for the factors
// 1 / phihat, which the device fills.
#pragma once

#include <cstddef>
#include <vector>

#include "chip_rule.h"

namespace mils {

// Where everything lies, in doubles from the start of the tables.
struct ChipTables {
  struct Kind {
    int N, nfmax, w;
    size_t iph;  // nfmax / 2 + 1
  };
  double eps = 0.0;
  size_t hcoef[2] = {}, nodes[2] = {}, tw[kChipBatchSizes] = {};
  int nnodes[2] = {};
  Kind kind[kChipKinds] = {};
  size_t host = 0;   // doubles that the host makes, from the start
  size_t bytes = 0;  // of everything
};

// The layout alone: a few divisions, so that a caller can see whether the
// tables fit, or are there already, before they are made.
ChipTables layout_chip_tables(double eps);

// The host's part of the tables (t.host doubles; about 0.3 ms).
std::vector<double> make_chip_tables(const ChipTables& t);

}  // namespace mils
