// Schedule of the line kernel (lines_fp32.hip), shared with the planner.
//
// Every axis is written as a chain of stages (decimation in frequency): a transform of length m = f_1 f_2 ... f_s
// contracts the input's highest digit first.  Stage 1 of a zero-padded axis takes n f_1 / m = f_1 / 2 inputs per
// line and gives f_1 outputs (the padding never exists), the later stages f_i inputs and outputs; after stage i
// the output kappa_i of a line is multiplied by w^{kappa_i j'}, j' the index formed by the digits still to come.
// The frequency is kappa = kappa_1 + f_1 kappa_2 + f_1 f_2 kappa_3 + ...  Axes whose length has a register
// transform (line_padded, line_plain) are one stage.
//
// The LDS working array has one extent per stage (its outputs; the stage of the last pass its inputs), all strides
// padded to odd numbers of float2, so that lanes on neighbouring lines of any pass fall on different banks.
// Passes run in place: a line's inputs lie inside its outputs' slots, and one thread transforms a whole line.
// Two short zero-padded axes (n1 n2 <= 16) are one pass: its "line" is the n1 x n2 block of both, 4 n1 n2 outputs.
#pragma once

#include <stdint.h>

namespace omni {

constexpr int kLineMaxPass = 16;

struct LinePass {
  int32_t type;    // inputs per line | 32 if zero-padded (twice as many outputs); two axes: 256 + 16 n1 + n2
  int32_t stride;  // float2 elements between a line's consecutive values (two axes: along the first)
  int32_t stride2; // along the second axis
  int32_t lines;   // lines per sample
  uint32_t magic;  // ceil(2^32 / lines): exact division of q < 2^16 by `lines`
  int32_t tab;     // first entry of the lines' offsets in the table
  int32_t tj;      // first entry of the lines' twiddle steps in the table (-1: no twiddle after this pass)
  int32_t tw;      // offset of the axis' w_m^q table
};

struct LineP {
  int32_t n_pass;       // passes; the last one is squared
  int32_t F, N;         // channels and samples per (t, channel) tile of the source
  int32_t fmt;          // sample format
  int32_t batch;        // samples transformed together
  int32_t groups;       // copies of the power array (lines of several samples summed by different threads)
  int32_t w_size;       // float2 elements of one sample's working array
  int32_t cells;        // Fourier cells of one work-group
  int32_t n_split;      // work-groups that share a channel's cells (residues of stage 1 of axis 0)
  int32_t n_tab;        // entries of the offset table
  int32_t n_tw;         // twiddles kept in LDS (0: read from global memory)
  int32_t time_block;   // samples summed in float32 before the float64 add
  int32_t xcd_groups;   // 1: XCD-aware block mapping is valid
  int32_t load_lines;   // N / n_in of stage 0: sample i is value i / load_lines of load line i % load_lines
  uint32_t load_magic;  // division by load_lines
  int32_t load_tab;     // first entry of the load lines' offsets in the table
  int32_t load_stride;  // float2 elements between a load line's values
  int32_t load_tj;      // split form: the load lines' twiddle steps (-1: none)
  uint32_t n_magic;     // division by N
  int32_t f1, n1, m0;   // split form: stage 1 of axis 0 has f1 outputs of n1 inputs; length m0 of axis 0
  int32_t k_out;        // split form: outputs kappa_1 of this work-group, f1 / n_split
  uint32_t k_magic;     // division by load_lines * k_out
  LinePass pass[kLineMaxPass];
};

// Lengths with a register transform, as the first stage of a zero-padded axis (n inputs, 2n outputs) or plain.
constexpr int kLinePadded[] = {1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 16};
constexpr int kLinePlain[] = {2, 3, 4, 5, 6, 7, 8, 11, 13, 16};
// Pairs of zero-padded axes that are one pass, n1 >= n2.
constexpr bool line_pair_ok(int n1, int n2) { return n1 >= n2 && n2 >= 2 && n1 <= 8 && n1 * n2 <= 16; }

}  // namespace omni
