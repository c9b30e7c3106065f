// Inverse transform along a group of axes (gfx950); schedule in inverse.hpp.
//
//   V[Delta] = (1/M) sum_kappa A[kappa] exp(+2 pi i sum_k kappa_k Delta_k / m_k)    (Sec. II.A "inverse FFT")
//
// The stages are the forward register transforms (dftn.hpp) on values with real and imaginary parts exchanged,
// which turns a forward transform into an inverse one.  Bound by HBM where the array is large (each group reads and
// writes it once), by its barriers where it is small.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include "dftn.hpp"
#include "inverse.hpp"

namespace omni {
namespace {

constexpr int kInvUnroll = 8;  // cells a thread has in flight while it loads and stores

__device__ __forceinline__ uint32_t fast_div(uint32_t q, uint32_t magic) {
  return magic ? __umulhi(q, magic) : q;
}

template <int N>
__device__ __forceinline__ void inv_pass(const InvPass& p, const InvP& P, double2* W, const uint16_t* __restrict__ tab,
                                         const double2* __restrict__ twi) {
  const uint32_t jobs = (uint32_t)(p.lines * P.cols);
  for (uint32_t q = threadIdx.x; q < jobs; q += blockDim.x) {
    uint32_t c, line;
    if (P.col_fast) {
      c = q & (uint32_t)(P.cols - 1);
      line = q >> P.lg_cols;
    } else {
      c = fast_div(q, p.magic);
      line = q - c * p.lines;
    }
    double2* w = W + c * P.col_stride + tab[p.tab + line];
    double2 x[N];
#pragma unroll
    for (int j = 0; j < N; ++j) x[j] = w[j * p.stride];
    dn::dft<N>(x);
    if (p.tj >= 0) {
      const int step = tab[p.tj + line];
#pragma unroll
      for (int k = 1; k < N; ++k) {
        const double2 t = twi[p.tw + k * step];
        x[k] = dn::mul(x[k], make_double2(t.x, -t.y));
      }
    }
#pragma unroll
    for (int k = 0; k < N; ++k) w[k * p.stride] = x[k];
  }
}

// SRC: 0 = real float64, 1 = complex float32, 2 = complex float64.
template <int SRC>
__global__ __launch_bounds__(512) void inverse_group_kernel(const void* __restrict__ src, float2* __restrict__ dst,
                                                            const double2* __restrict__ twi,
                                                            const uint16_t* __restrict__ tab, int64_t columns,
                                                            int64_t inner, double scale, InvP P) {
  extern __shared__ double2 W[];
  const uint32_t tid = threadIdx.x, nt = blockDim.x;
  // consecutive column tiles on one XCD: where the columns are interleaved, tiles share cache lines
  int64_t blk = blockIdx.x;
  if (gridDim.x % 8 == 0) blk = (blk & 7) * (gridDim.x >> 3) + (blk >> 3);
  const int64_t col0 = blk * P.cols;
  // interleaved columns: this thread's column is fixed (the thread count is a multiple of cols), cells step through
  // the source; whole columns: the tile is one contiguous run
  const uint32_t tc = tid & (uint32_t)(P.cols - 1);
  const int64_t col = col0 + tc, ou = P.col_fast ? col / inner : 0;
  const int64_t src0 = P.col_fast ? ou * P.Mg * inner + (col - ou * inner) : col0 * P.Mg;
  const int64_t dst0 = P.col_fast ? ou * P.Ng * inner + (col - ou * inner) : col0 * P.Ng;
  const bool mine = !P.col_fast || col < columns;
  const uint32_t n_in = (uint32_t)(P.col_fast ? P.cols : min<int64_t>(P.cols, columns - col0)) * P.Mg;
  const uint32_t n_out = (uint32_t)(P.col_fast ? P.cols : min<int64_t>(P.cols, columns - col0)) * P.Ng;
  for (uint32_t e0 = tid; e0 < n_in; e0 += kInvUnroll * nt) {
    double2 v[kInvUnroll];
#pragma unroll
    for (int u = 0; u < kInvUnroll; ++u) {
      const uint32_t e = e0 + u * nt;
      v[u] = make_double2(0.0, 0.0);
      if (e >= n_in || !mine) continue;
      const int64_t at = src0 + (P.col_fast ? (int64_t)(e >> P.lg_cols) * inner : (int64_t)e);
      if constexpr (SRC == 0) {
        v[u].y = static_cast<const double*>(src)[at];
      } else if constexpr (SRC == 1) {
        const float2 t = static_cast<const float2*>(src)[at];
        v[u] = make_double2(t.y, t.x);
      } else {
        const double2 t = static_cast<const double2*>(src)[at];
        v[u] = make_double2(t.y, t.x);
      }
    }
#pragma unroll
    for (int u = 0; u < kInvUnroll; ++u) {
      const uint32_t e = e0 + u * nt;
      if (e >= n_in) continue;
      const uint32_t c = P.col_fast ? tc : fast_div(e, P.m_magic);
      const uint32_t cell = P.col_fast ? e >> P.lg_cols : e - c * P.Mg;
      const uint32_t j = fast_div(cell, P.load_magic), line = cell - j * P.load_lines;
      W[c * P.col_stride + tab[P.pass[0].tab + line] + j * P.pass[0].stride] = v[u];
    }
  }
  __syncthreads();
  for (int i = 0; i < P.n_pass; ++i) {
    const InvPass& p = P.pass[i];
    switch (p.f) {
      case 2: inv_pass<2>(p, P, W, tab, twi); break;
      case 3: inv_pass<3>(p, P, W, tab, twi); break;
      case 4: inv_pass<4>(p, P, W, tab, twi); break;
      case 5: inv_pass<5>(p, P, W, tab, twi); break;
      case 6: inv_pass<6>(p, P, W, tab, twi); break;
      case 7: inv_pass<7>(p, P, W, tab, twi); break;
      case 8: inv_pass<8>(p, P, W, tab, twi); break;
      case 11: inv_pass<11>(p, P, W, tab, twi); break;
      case 13: inv_pass<13>(p, P, W, tab, twi); break;
      case 16: inv_pass<16>(p, P, W, tab, twi); break;
      default: break;
    }
    __syncthreads();
  }
  for (uint32_t e0 = tid; e0 < n_out; e0 += kInvUnroll * nt) {
    uint32_t off[kInvUnroll];
#pragma unroll
    for (int u = 0; u < kInvUnroll; ++u) {
      const uint32_t e = min(e0 + u * nt, n_out - 1);
      const uint32_t c = P.col_fast ? tc : fast_div(e, P.g_magic);
      const uint32_t o = P.col_fast ? e >> P.lg_cols : e - c * P.Ng;
      off[u] = c * P.col_stride + tab[P.out_tab + o];
    }
#pragma unroll
    for (int u = 0; u < kInvUnroll; ++u) {
      const uint32_t e = e0 + u * nt;
      if (e >= n_out || !mine) continue;
      const double2 v = W[off[u]];
      dst[dst0 + (P.col_fast ? (int64_t)(e >> P.lg_cols) * inner : (int64_t)e)] =
          make_float2((float)(v.y * scale), (float)(v.x * scale));
    }
  }
}

}  // namespace

// src_kind: 0 = real float64, 1 = complex float32, 2 = complex float64; outer x inner columns.
hipError_t launch_inverse_group(int src_kind, const void* src, void* dst, const double2* twi, const uint16_t* tab,
                                int64_t outer, int64_t inner, double scale, const InvP& P, size_t lds,
                                hipStream_t st) {
  const int64_t columns = outer * inner, blocks = (columns + P.cols - 1) / P.cols;
  const int threads = P.cols * P.Mg > 2048 ? 512 : 256;
  if (threads % P.cols) return hipErrorInvalidValue;
  if (blocks < 1 || blocks > INT32_MAX || P.n_pass < 1 || P.n_pass > kInvMaxPass || (inner > 1) != (P.col_fast != 0))
    return hipErrorInvalidValue;
  const auto go = [&](auto* kernel) {
    hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3((unsigned)threads), lds, st, src, static_cast<float2*>(dst), twi,
                       tab, columns, inner, scale, P);
    return hipGetLastError();
  };
  switch (src_kind) {
    case 0: return go(inverse_group_kernel<0>);
    case 1: return go(inverse_group_kernel<1>);
    case 2: return go(inverse_group_kernel<2>);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace omni
