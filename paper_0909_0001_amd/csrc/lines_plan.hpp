// Planner of the line kernel (lines.hpp, lines_fp32.hip).
#pragma once

#include <stddef.h>

#include <vector>

#include "lines.hpp"

namespace omni {

constexpr int kLineMaxBatch = 16;  // samples transformed together at most

struct LineSetup {
  LineP P{};                  // F, fmt, time_block and xcd_groups are set by the launch
  std::vector<uint16_t> tab;  // the passes' line offsets and twiddle steps
  std::vector<int32_t> kmap;  // [n_split][cells] -> natural frequency index
  std::vector<int> order;     // axis of each pass
  int threads = 0;
  int per_cu = 1;             // work-groups that fit a CU
  size_t lds = 0;
};

// Schedule for d axes of n[k] antennas and transform lengths m[k] (2 n[k], or n[k] for a beam axis), batches of at
// most max_batch samples.  False where no schedule exists: a prime factor above 13, or a grid whose cells cannot
// be divided along axis 0 into shares that fit LDS.
bool plan_lines(int d, const int* n, const int* m, int max_batch, LineSetup& out);

}  // namespace omni
