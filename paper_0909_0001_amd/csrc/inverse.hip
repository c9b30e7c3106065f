// Inverse transform along a group of axes (gfx950); schedule in inverse.hpp.
//
//   V[Delta] = (1/M) sum_kappa A[kappa] exp(+2 pi i sum_k kappa_k Delta_k / m_k)    (Sec. II.A "inverse FFT")
//
// The stages are the forward register transforms (dftn.hpp) on values with real and imaginary parts exchanged,
// which turns a forward transform into an inverse one.  Bound by the barriers between its passes: a group moves about
// 2 TB/s, so that arrays beyond the caches take their axes of 8, 16 and 32 one by one (inverse_line_kernel).  Passes
// of 2 to 8 values leave three work-groups a CU their registers; with passes of 16 (fewer passes, four waves a SIMD and
// spills) 64 channels of 64x64 took 23 us instead of 19, of 12x12/5x5 (32) 45 instead of 35.  Loading a tile's lines
// while the tile before is transformed (one persistent work-group a slot) was slower: 1269 for 745 us at 6 x 2^24 cells.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include "dftn.hpp"
#include "inverse.hpp"
#include "plan.hpp"

namespace omni {
namespace {

__device__ __forceinline__ uint32_t fast_div(uint32_t q, uint32_t magic) {
  return magic ? __umulhi(q, magic) : q;
}

struct Ctx {
  double2* W;
  const double2* __restrict__ twi;
  const uint16_t* __restrict__ tab;
  const void* __restrict__ src;
  float2* __restrict__ dst;
  int64_t src0, dst0, inner;  // of this thread's column (interleaved columns) or of the tile (whole columns)
  double scale;
  int n_cols;                 // columns of this tile
  bool mine;                  // this thread's column exists (interleaved columns)
  const uint16_t* __restrict__ pair_tab;  // SRC 3: p P + q of every tile pair p <= q
  uint32_t col0, n_pairs, n_tiles;        // SRC 3: first column, pairs per channel, tiles
};

// One pass' lines: FIRST reads them from HBM, otherwise from LDS; LAST writes the valid lags to HBM.
// SRC: 0 = real float64, 1 = complex float32, 2 = complex float64, 3 = complex float64 of the tile pairs p <= q,
// [channel][cell][pair]: a column is one pair, written as C_pq[Delta] and as C_qp[-Delta] = conj C_pq[Delta].
template <int N, int SRC, bool FIRST, bool LAST>
__device__ __forceinline__ void inv_pass(const InvPass& p, const InvP& P, const Ctx& x) {
  const uint32_t jobs = (uint32_t)(p.lines * (P.col_fast ? P.cols : x.n_cols));
  for (uint32_t q = threadIdx.x; q < jobs; q += blockDim.x) {
    uint32_t c, line;
    if (P.col_fast && !(SRC == 3 && LAST)) {
      c = q & (uint32_t)(P.cols - 1);
      line = q >> P.lg_cols;
    } else {  // (a pair's lags are one run: neighbouring threads write neighbouring lags)
      c = fast_div(q, p.magic);
      line = q - c * p.lines;
    }
    double2 v[N];
    if constexpr (FIRST) {
      const int64_t at = x.src0 + (P.col_fast ? (int64_t)line * x.inner : (int64_t)(c * P.Mg + line));
      const int64_t step = P.col_fast ? (int64_t)p.lines * x.inner : (int64_t)p.lines;
#pragma unroll
      for (int j = 0; j < N; ++j) {
        if (!x.mine) {
          v[j] = make_double2(0.0, 0.0);
        } else if constexpr (SRC == 0) {
          v[j] = make_double2(0.0, static_cast<const double*>(x.src)[at + j * step]);
        } else if constexpr (SRC == 1) {
          const float2 t = static_cast<const float2*>(x.src)[at + j * step];
          v[j] = make_double2(t.y, t.x);
        } else {
          const double2 t = static_cast<const double2*>(x.src)[at + j * step];
          v[j] = make_double2(t.y, t.x);
        }
      }
    }
    double2* w = x.W + (FIRST && LAST ? 0 : c * P.col_stride + x.tab[p.tab + line]);
    if constexpr (!FIRST) {
#pragma unroll
      for (int j = 0; j < N; ++j) v[j] = w[j * p.stride];
    }
    dn::dft<N>(v);
    if constexpr (!LAST) {
      if (p.tj >= 0) {
        const int step = x.tab[p.tj + line];
#pragma unroll
        for (int k = 1; k < N; ++k) {
          const double2 t = x.twi[p.tw + k * step];
          v[k] = dn::mul(v[k], make_double2(t.x, -t.y));
        }
      }
#pragma unroll
      for (int k = 0; k < N; ++k) w[k * p.stride] = v[k];
    } else if constexpr (SRC == 3) {
      if ((int)c >= x.n_cols) continue;
      const uint32_t col = x.col0 + c, f = col / x.n_pairs, pq = x.pair_tab[col - f * x.n_pairs];
      const uint32_t tp = pq / x.n_tiles, tq = pq - tp * x.n_tiles;
      float2* d = x.dst + ((int64_t)f * x.n_tiles * x.n_tiles + pq) * P.Ng;
      float2* m = x.dst + ((int64_t)f * x.n_tiles * x.n_tiles + tq * x.n_tiles + tp) * P.Ng + (P.Ng - 1);
#pragma unroll
      for (int k = 0; k < N; ++k) {
        const uint32_t o = x.tab[P.out_tab + k * p.lines + line];
        if (o == kInvNoLag) continue;
        const float a = (float)(v[k].y * x.scale), b = (float)(v[k].x * x.scale);
        d[o] = make_float2(a, b);
        if (tp != tq) m[-(int64_t)o] = make_float2(a, -b);
      }
    } else if (x.mine) {
#pragma unroll
      for (int k = 0; k < N; ++k) {
        const uint32_t o = x.tab[P.out_tab + k * p.lines + line];
        if (o == kInvNoLag) continue;
        x.dst[x.dst0 + (P.col_fast ? (int64_t)o * x.inner : (int64_t)(c * P.Ng + o))] =
            make_float2((float)(v[k].y * x.scale), (float)(v[k].x * x.scale));
      }
    }
  }
}

template <int SRC, bool WIDE, bool FIRST, bool LAST>
__device__ __forceinline__ void inv_any(const InvPass& p, const InvP& P, const Ctx& x) {
  switch (p.f) {
    case 2: inv_pass<2, SRC, FIRST, LAST>(p, P, x); break;
    case 3: inv_pass<3, SRC, FIRST, LAST>(p, P, x); break;
    case 4: inv_pass<4, SRC, FIRST, LAST>(p, P, x); break;
    case 5: inv_pass<5, SRC, FIRST, LAST>(p, P, x); break;
    case 6: inv_pass<6, SRC, FIRST, LAST>(p, P, x); break;
    case 7: inv_pass<7, SRC, FIRST, LAST>(p, P, x); break;
    case 8: inv_pass<8, SRC, FIRST, LAST>(p, P, x); break;
    case 11:
      if constexpr (WIDE) inv_pass<11, SRC, FIRST, LAST>(p, P, x);
      break;
    case 13:
      if constexpr (WIDE) inv_pass<13, SRC, FIRST, LAST>(p, P, x);
      break;
    default: break;
  }
}

// WIDE: a pass of 11 or 13 values, which need the registers of four waves a SIMD.
template <int SRC, bool WIDE>
__global__ __launch_bounds__(512, WIDE ? 4 : 6) void inverse_group_kernel(
    const void* __restrict__ src, float2* __restrict__ dst, const double2* __restrict__ twi,
    const uint16_t* __restrict__ tab, int64_t columns, int64_t inner, double scale, InvP P,
    const uint16_t* __restrict__ pair_tab, int n_tiles) {
  extern __shared__ double2 W[];
  // consecutive column tiles on one XCD: where the columns are interleaved, tiles share cache lines
  int64_t blk = blockIdx.x;
  if (gridDim.x % 8 == 0) blk = (blk & 7) * (gridDim.x >> 3) + (blk >> 3);
  const int64_t col0 = blk * P.cols;
  // interleaved columns: this thread's column is fixed (the thread count is a multiple of cols); whole columns: the
  // tile is one contiguous run
  const int64_t col = col0 + (threadIdx.x & (uint32_t)(P.cols - 1)), ou = P.col_fast ? col / inner : 0;
  const Ctx x{W,
              twi,
              tab,
              src,
              dst,
              P.col_fast ? ou * P.Mg * inner + (col - ou * inner) : col0 * P.Mg,
              P.col_fast ? ou * P.Ng * inner + (col - ou * inner) : col0 * P.Ng,
              inner,
              scale,
              (int)min<int64_t>(P.cols, columns - col0),
              !P.col_fast || col < columns,
              pair_tab,
              (uint32_t)col0,
              (uint32_t)inner,
              (uint32_t)n_tiles};
  if (SRC != 3 && P.n_pass == 1) {
    inv_any<SRC == 3 ? 1 : SRC, WIDE, true, true>(P.pass[0], P, x);
    return;
  }
  inv_any<SRC, WIDE, true, false>(P.pass[0], P, x);
  for (int i = 1; i + 1 < P.n_pass; ++i) {
    __syncthreads();
    inv_any<1, WIDE, false, false>(P.pass[i], P, x);
  }
  __syncthreads();
  inv_any<SRC == 3 ? 3 : 1, WIDE, false, true>(P.pass[P.n_pass - 1], P, x);
}

// One axis of an array beyond the caches, a thread a line, transformed in registers: neighbouring threads take
// neighbouring columns.  One read and one write of the array at HBM's rate: axes
// of 32, 32, 16, 16 of 6 x 2^24 cells 411, 284, 266 and 244 us (3.7 to 5.5 TB/s), the same axes in two groups 745 and 689 us.
template <int M, int SRC>
__global__ __launch_bounds__(256) void inverse_line_kernel(const void* __restrict__ src, float2* __restrict__ dst,
                                                           int64_t columns, int64_t inner) {
  const int64_t col = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (col >= columns) return;
  const int64_t ou = col / inner, in = col - ou * inner;
  double2 v[M];
#pragma unroll
  for (int j = 0; j < M; ++j) {
    const int64_t at = (ou * M + j) * inner + in;
    if constexpr (SRC == 0) {
      v[j] = make_double2(0.0, static_cast<const double*>(src)[at]);
    } else {
      const float2 t = static_cast<const float2*>(src)[at];
      v[j] = make_double2(t.y, t.x);
    }
  }
  dn::dft<M>(v);
#pragma unroll
  for (int o = 0; o < M - 1; ++o) {
    const int k = (o + M / 2 + 1) % M;  // lag o - (M / 2 - 1)
    dst[(ou * (M - 1) + o) * inner + in] = make_float2((float)v[k].y, (float)v[k].x);
  }
}

}  // namespace

// One axis of length 8, 16 or 32 that is not the last one: [outer][m][inner] -> [outer][m - 1][inner].
hipError_t launch_inverse_line(int src_kind, const void* src, void* dst, int64_t outer, int m, int64_t inner,
                               hipStream_t st) {
  const int64_t columns = outer * inner, blocks = (columns + 255) / 256;
  if (blocks < 1 || blocks > INT32_MAX || src_kind < 0 || src_kind > 1) return hipErrorInvalidValue;
  const auto go = [&](auto* kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(256), 0, st, src, static_cast<float2*>(dst), columns, inner);
    return hipGetLastError();
  };
  switch (m) {
    case 8: return src_kind ? go(inverse_line_kernel<8, 1>) : go(inverse_line_kernel<8, 0>);
    case 16: return src_kind ? go(inverse_line_kernel<16, 1>) : go(inverse_line_kernel<16, 0>);
    case 32: return src_kind ? go(inverse_line_kernel<32, 1>) : go(inverse_line_kernel<32, 0>);
    default: return hipErrorInvalidValue;
  }
}

// src_kind: 0 = real float64, 1 = complex float32, 2 = complex float64; outer x inner columns.  3 = the tile pairs
// p <= q of n_tiles tiles (inner = their number, pair_tab = p n_tiles + q of each), both orders written.
hipError_t launch_inverse_group(int src_kind, const void* src, void* dst, const double2* twi, const uint16_t* tab,
                                int64_t outer, int64_t inner, double scale, const InvP& P, size_t lds, hipStream_t st,
                                const uint16_t* pair_tab, int n_tiles) {
  const int64_t columns = outer * inner, blocks = (columns + P.cols - 1) / P.cols;
  const int threads = P.cols * P.Mg > 2048 ? 512 : 256;
  if (threads % P.cols) return hipErrorInvalidValue;
  if (blocks < 1 || blocks > INT32_MAX || P.n_pass < 1 || P.n_pass > kInvMaxPass || (inner > 1) != (P.col_fast != 0))
    return hipErrorInvalidValue;
  if (src_kind == 3 && (!pair_tab || P.n_pass < 2 || !P.col_fast || n_tiles < 2 || columns >= INT32_MAX ||
                        inner != (int64_t)n_tiles * (n_tiles + 1) / 2))
    return hipErrorInvalidValue;
  const auto go = [&](auto* kernel) {
    // (always the largest: the limit belongs to the process, and another thread may be launching another plan)
    hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3((unsigned)threads), lds, st, src, static_cast<float2*>(dst), twi,
                       tab, columns, inner, scale, P, pair_tab, n_tiles);
    return hipGetLastError();
  };
  bool wide = false;
  for (int i = 0; i < P.n_pass; ++i) wide = wide || P.pass[i].f > 8;
  switch (src_kind) {
    case 0: return wide ? go(inverse_group_kernel<0, true>) : go(inverse_group_kernel<0, false>);
    case 1: return wide ? go(inverse_group_kernel<1, true>) : go(inverse_group_kernel<1, false>);
    case 2: return wide ? go(inverse_group_kernel<2, true>) : go(inverse_group_kernel<2, false>);
    case 3: return wide ? go(inverse_group_kernel<3, true>) : go(inverse_group_kernel<3, false>);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace omni
