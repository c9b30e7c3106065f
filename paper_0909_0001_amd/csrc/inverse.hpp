// Schedule of the grouped inverse transform (inverse.hip), shared with the planner.
//
// The inverse runs along groups of consecutive axes.  A group sees its source as [outer][M_g][inner], M_g the product
// of its axes' lengths m_k, and gives [outer][N_g][inner], N_g the product of their 2 n_k - 1 valid lags.  A
// work-group transforms a few (outer, inner) columns in LDS as complex float64 (stages as in lines.hpp, all plain: in
// place, one thread a line); the first pass takes its lines straight from HBM, the last one writes the valid lags
// straight to it.  The first axis' last stage comes last, so that neighbouring lines of that pass are neighbouring
// lags of the inner axes.  The axes of a group need no round trip through HBM between them, and all their sums and
// intermediates are float64; only the values between two groups are stored as complex float32.  Arrays beyond the
// last-level cache take their axes of 8, 16 and 32 one by one instead, a thread a line (InvGroup::line).
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <vector>

namespace omni {

constexpr int kInvMaxPass = 16;
constexpr int kInvPlain[] = {2, 3, 4, 5, 6, 7, 8, 11, 13};  // register transforms of the passes
constexpr uint32_t kInvNoLag = 0xffff;

struct InvPass {
  int32_t f;       // values per line
  int32_t stride;  // double2 elements between a line's values
  int32_t lines;   // lines per column
  uint32_t magic;  // division by lines
  int32_t tab;     // first entry of the lines' offsets in the table
  int32_t tj;      // first entry of the lines' twiddle steps (-1: none)
  int32_t tw;      // offset of the axis' exp(+2 pi i q / m) table
};

struct InvP {
  int32_t n_pass;
  int32_t cols;        // columns per work-group (a power of two)
  int32_t lg_cols;
  int32_t col_fast;    // 1: neighbouring threads take neighbouring columns (inner > 1); 0: neighbouring cells
  int32_t col_stride;  // double2 elements between columns
  int32_t Mg, Ng;      // cells and valid lags per column
  int32_t out_tab;     // last pass: lag of value k of each line at out_tab + k * lines + line (kInvNoLag: none)
  InvPass pass[kInvMaxPass];
};

struct InvGroup {
  int axis0 = 0, axes = 0;    // the axes it covers
  bool direct = false;        // one axis without a register transform: plain sums (finalize.hip)
  bool line = false;          // one axis, a thread a line (arrays beyond the caches)
  InvP P{};
  std::vector<uint16_t> tab;
  size_t tab_off = 0;         // first entry in the plan's device table
  size_t lds = 0;
};

// Groups for d axes of n[k] antennas and lengths m[k] = 2 n[k], `channels` independent transforms, `inner` values
// behind the last axis.  tw_off[k]: offset of axis k's table.
std::vector<InvGroup> plan_inverse(int d, const int* n, const int* m, int64_t channels, int64_t inner,
                                   const int* tw_off);

}  // namespace omni
