// General float32 correlator for gfx950: any grid whose axes factor into short register transforms.
//
// One work-group owns (time slice, channel, split residue).  It takes `batch` time samples at a time:
//   load   the samples' tiles from HBM, decoded into the LDS working array (split form: stage 1 of axis 0 summed
//          directly for the work-group's own outputs, straight from HBM);
//   passes one per stage of every axis: a thread reads one line (n values), transforms it in registers with
//          compile-time twiddles (dftn.hpp) and writes its outputs in place;
//   last   the last pass' thread squares its line's outputs for every sample of the batch, sums them in registers
//          and adds the sums to the float32 power array in LDS (Sec. II.A: square modulus, time integration).
// Every time_block samples the power array is added to the float64 partial sums in HBM.
//
// What bounds it: latency.  The short lines leave few jobs per sample (a 16 x 16 grid has 16 and 32), so samples are
// batched until a pass fills the work-group; job addresses come from a table in LDS (one 2-byte read) instead of a
// chain of divisions per job and sample.  A pass costs about 1000 cycles of waiting (table, line, barrier) besides its
// instructions, which is why short axes are transformed two by two (n1 n2 values a thread): 5x3 / 3x3 / 3x3, 12
// channels, T = 333: 635 -> 390 us, 2x2 / 16x16, 16 channels, T = 250: 130 -> 72 us, together with one round of
// work-groups instead of a fixed count.  Vector units issue 30 to 40% of the cycles.  Eight waves a SIMD instead of four
// (64 registers, for schedules of short transforms only) made most grids slower, for the schedules that the planner then
// chose: 36x18, 8 channels, T = 500: 59 us for 46; 15x6, 32 channels, T = 1500: 45 for 38; 5x3/3x3/3x3: 418 for 400;
// at best 126 for 135 (5x8/7x7, 8 channels, T = 200).
#include <hip/hip_runtime.h>

#include <stdint.h>

#include "dftn.hpp"
#include "lines.hpp"
#include "plan.hpp"

namespace omni {
namespace {

using dn::dft;

// Lambdas are called from several unrolled places: always inlined.  A pass' schedule is handed on by value: captured
// by reference it would make the compiler copy the kernel's whole argument structure into scratch memory.
#define OMNI_INLINE __attribute__((always_inline))

// q / d for q < 2^16, magic = ceil(2^32 / d) (exact: the excess q (d - 1) / 2^32 stays below 1 / d); d = 1 has
// magic 0.
__device__ __forceinline__ uint32_t fast_div(uint32_t q, uint32_t magic) {
  return magic ? __umulhi(q, magic) : q;
}

__device__ __forceinline__ float2 sample_at(const void* __restrict__ src, int64_t i, int fmt) {
  if (fmt == 0) return static_cast<const float2*>(src)[i];
  if (fmt == 1) {
    const char2 v = static_cast<const char2*>(src)[i];
    return make_float2((float)v.x, (float)v.y);
  }
  const int8_t v = static_cast<const int8_t*>(src)[i];
  return make_float2((float)(v >> 4), (float)((int8_t)(v << 4) >> 4));
}

// Inputs of the odd outputs of a zero-padded transform (2N outputs of N values): the even ones are DFT_N(x), output
// 2q + 1 is DFT_N(x_j w_2N^j)[q], and for odd N output 2q + N mod 2N is DFT_N((-1)^j x_j)[q], without rotations.
template <int N>
__device__ __forceinline__ float2 odd_input(float2 v, int j) {
  if constexpr (N % 2) return j & 1 ? make_float2(-v.x, -v.y) : v;
  return dn::rot<2 * N>(v, j);
}
template <int N>
constexpr int odd_output(int q) {
  return N % 2 ? (2 * q + N) % (2 * N) : 2 * q + 1;
}

// Outputs of one line: N values transformed (plain), or zero-padded to 2N.
template <int N, bool PAD, class Put>
__device__ __forceinline__ void line_dft(const float2 (&x)[N], Put put) {
  float2 z[N];
#pragma unroll
  for (int j = 0; j < N; ++j) z[j] = x[j];
  dft<N>(z);
#pragma unroll
  for (int q = 0; q < N; ++q) put(PAD ? 2 * q : q, z[q]);
  if constexpr (PAD) {
#pragma unroll
    for (int j = 0; j < N; ++j) z[j] = odd_input<N>(x[j], j);
    dft<N>(z);
#pragma unroll
    for (int q = 0; q < N; ++q) put(odd_output<N>(q), z[q]);
  }
}

struct Ctx {
  float2* W;
  float* Pw;
  const uint16_t* tab;
  const float2* tw_lds;
  const float2* tw_glob;
  int w_size, cells, nb, groups, tid, nt;
  bool lds_tw;
};

template <int N, bool PAD>
__device__ __forceinline__ void mid_pass(const LinePass p, const Ctx& c) {
  const uint32_t jobs = (uint32_t)(c.nb * p.lines);
  for (uint32_t q = c.tid; q < jobs; q += c.nt) {
    const uint32_t b = fast_div(q, p.magic), line = q - b * p.lines;
    float2* w = c.W + b * c.w_size + c.tab[p.tab + line];
    float2 x[N];
#pragma unroll
    for (int j = 0; j < N; ++j) x[j] = w[j * p.stride];
    if (p.tj < 0) {
      line_dft<N, PAD>(x, [&](int k, float2 v) OMNI_INLINE { w[k * p.stride] = v; });
    } else {
      const int step = c.tab[p.tj + line];
      if (c.lds_tw)
        line_dft<N, PAD>(x, [&](int k, float2 v) OMNI_INLINE { w[k * p.stride] = k ? dn::mul(v, c.tw_lds[p.tw + k * step]) : v; });
      else
        line_dft<N, PAD>(x, [&](int k, float2 v) OMNI_INLINE { w[k * p.stride] = k ? dn::mul(v, c.tw_glob[p.tw + k * step]) : v; });
    }
  }
}

template <int N, bool PAD>
__device__ __forceinline__ void last_pass(const LinePass p, const Ctx& c) {
  constexpr int OUT = PAD ? 2 * N : N;
  const uint32_t jobs = (uint32_t)(c.groups * p.lines);
  for (uint32_t q = c.tid; q < jobs; q += c.nt) {
    const uint32_t g = fast_div(q, p.magic), line = q - g * p.lines;
    if ((int)g >= c.nb) continue;
    const float2* w = c.W + c.tab[p.tab + line];
    float acc[OUT];
#pragma unroll
    for (int k = 0; k < OUT; ++k) acc[k] = 0.f;
    for (int b = (int)g; b < c.nb; b += c.groups) {
      float2 x[N];
#pragma unroll
      for (int j = 0; j < N; ++j) x[j] = w[b * c.w_size + j * p.stride];
      line_dft<N, PAD>(x, [&](int k, float2 v) OMNI_INLINE { acc[k] = fmaf(v.x, v.x, fmaf(v.y, v.y, acc[k])); });
    }
    float* pw = c.Pw + g * c.cells + line;
#pragma unroll
    for (int k = 0; k < OUT; ++k) pw[k * p.lines] += acc[k];
  }
}

// Two zero-padded axes at once: N1 x N2 values in, 2 N1 x 2 N2 out.  The second axis' even outputs and odd outputs are
// formed one after the other, each followed by the first axis' lines, so that N1 N2 values are live besides the inputs.
template <int N1, int N2, int HALF, class Get, class Put>
__device__ __forceinline__ void block_dft(Get get, Put put) {
  float2 z[N1 * N2];
#pragma unroll
  for (int i = 0; i < N1; ++i) {
    float2 t[N2];
#pragma unroll
    for (int j = 0; j < N2; ++j) t[j] = HALF ? odd_input<N2>(get(i, j), j) : get(i, j);
    dft<N2>(t);
#pragma unroll
    for (int j = 0; j < N2; ++j) z[i * N2 + j] = t[j];
  }
#pragma unroll
  for (int q = 0; q < N2; ++q) {
    float2 v[N1];
#pragma unroll
    for (int i = 0; i < N1; ++i) v[i] = z[i * N2 + q];
    line_dft<N1, true>(v, [&](int k1, float2 y) OMNI_INLINE { put(k1, HALF ? odd_output<N2>(q) : 2 * q, y); });
  }
}

template <int N1, int N2>
__device__ __forceinline__ void mid_pass2(const LinePass p, const Ctx& c) {
  const uint32_t jobs = (uint32_t)(c.nb * p.lines);
  for (uint32_t q = c.tid; q < jobs; q += c.nt) {
    const uint32_t b = fast_div(q, p.magic), line = q - b * p.lines;
    float2* w = c.W + b * c.w_size + c.tab[p.tab + line];
    float2 x[N1 * N2];
#pragma unroll
    for (int i = 0; i < N1; ++i)
#pragma unroll
      for (int j = 0; j < N2; ++j) x[i * N2 + j] = w[i * p.stride + j * p.stride2];
    const auto get = [&](int i, int j) OMNI_INLINE { return x[i * N2 + j]; };
    const auto put = [&](int k1, int k2, float2 y) OMNI_INLINE { w[k1 * p.stride + k2 * p.stride2] = y; };
    block_dft<N1, N2, 0>(get, put);
    block_dft<N1, N2, 1>(get, put);
  }
}

// Output (k1, k2) of a block is cell (k1 2 N2 + k2) lines + line.  The inputs are read again for the odd outputs:
// the sums of one half are what the registers hold.
template <int N1, int N2, int HALF>
__device__ __forceinline__ void last_half(const LinePass p, const Ctx& c, const float2* w, float* pw, int g) {
  float acc[N2 * 2 * N1];
#pragma unroll
  for (int k = 0; k < N2 * 2 * N1; ++k) acc[k] = 0.f;
#pragma unroll 1
  for (int b = g; b < c.nb; b += c.groups) {
    block_dft<N1, N2, HALF>([&](int i, int j) OMNI_INLINE { return w[b * c.w_size + i * p.stride + j * p.stride2]; },
                            [&](int k1, int k2, float2 y) OMNI_INLINE {
                              float& a = acc[(k2 / 2) * 2 * N1 + k1];
                              a = fmaf(y.x, y.x, fmaf(y.y, y.y, a));
                            });
  }
#pragma unroll
  for (int q = 0; q < N2; ++q)
#pragma unroll
    for (int k = 0; k < 2 * N1; ++k) pw[(k * 2 * N2 + 2 * q + HALF) * p.lines] += acc[q * 2 * N1 + k];
}

template <int N1, int N2>
__device__ __forceinline__ void last_pass2(const LinePass p, const Ctx& c) {
  const uint32_t jobs = (uint32_t)(c.groups * p.lines);
  for (uint32_t q = c.tid; q < jobs; q += c.nt) {
    const uint32_t g = fast_div(q, p.magic), line = q - g * p.lines;
    if ((int)g >= c.nb) continue;
    const float2* w = c.W + c.tab[p.tab + line];
    float* pw = c.Pw + g * c.cells + line;
    last_half<N1, N2, 0>(p, c, w, pw, (int)g);
    last_half<N1, N2, 1>(p, c, w, pw, (int)g);
  }
}

// Every type.
#define OMNI_LINE_TYPES(PASS, PASS2) \
  switch (p.type) {                  \
    case 32 + 1: PASS(1, true);      \
    case 32 + 2: PASS(2, true);      \
    case 32 + 3: PASS(3, true);      \
    case 32 + 4: PASS(4, true);      \
    case 32 + 5: PASS(5, true);      \
    case 32 + 6: PASS(6, true);      \
    case 32 + 7: PASS(7, true);      \
    case 32 + 8: PASS(8, true);      \
    case 32 + 9: PASS(9, true);      \
    case 32 + 10: PASS(10, true);    \
    case 32 + 11: PASS(11, true);    \
    case 32 + 12: PASS(12, true);    \
    case 32 + 13: PASS(13, true);    \
    case 32 + 16: PASS(16, true);    \
    case 2: PASS(2, false);          \
    case 3: PASS(3, false);          \
    case 4: PASS(4, false);          \
    case 5: PASS(5, false);          \
    case 6: PASS(6, false);          \
    case 7: PASS(7, false);          \
    case 8: PASS(8, false);          \
    case 11: PASS(11, false);        \
    case 13: PASS(13, false);        \
    case 16: PASS(16, false);        \
    case 256 + 34: PASS2(2, 2);      \
    case 256 + 50: PASS2(3, 2);      \
    case 256 + 66: PASS2(4, 2);      \
    case 256 + 51: PASS2(3, 3);      \
    case 256 + 82: PASS2(5, 2);      \
    case 256 + 98: PASS2(6, 2);      \
    case 256 + 114: PASS2(7, 2);     \
    case 256 + 130: PASS2(8, 2);     \
    case 256 + 67: PASS2(4, 3);      \
    case 256 + 83: PASS2(5, 3);      \
    case 256 + 68: PASS2(4, 4);      \
    default: break;                  \
  }

__device__ __forceinline__ void run_mid(const LinePass p, const Ctx& c) {
#define OMNI_MID(N_, PAD_)  \
  mid_pass<N_, PAD_>(p, c); \
  break
#define OMNI_MID2(N1_, N2_)   \
  mid_pass2<N1_, N2_>(p, c); \
  break
  OMNI_LINE_TYPES(OMNI_MID, OMNI_MID2)
#undef OMNI_MID
#undef OMNI_MID2
}

__device__ __forceinline__ void run_last(const LinePass p, const Ctx& c) {
#define OMNI_LAST(N_, PAD_)  \
  last_pass<N_, PAD_>(p, c); \
  break
#define OMNI_LAST2(N1_, N2_)   \
  last_pass2<N1_, N2_>(p, c); \
  break
  OMNI_LINE_TYPES(OMNI_LAST, OMNI_LAST2)
#undef OMNI_LAST
#undef OMNI_LAST2
}

// Dynamic LDS: W [batch][w_size] float2, twiddles [n_tw] float2, power [groups][cells] float, table [n_tab] uint16.
__global__ __launch_bounds__(1024, 4) void lines_fp32_kernel(const void* __restrict__ src, int64_t T, int64_t tps,
                                                             const float2* __restrict__ tw_glob,
                                                             const uint16_t* __restrict__ tab_glob,
                                                             double* __restrict__ partial, LineP P) {
  extern __shared__ float2 smem[];
  Ctx c;
  c.W = smem;
  float2* const tw = smem + P.batch * P.w_size;
  c.Pw = reinterpret_cast<float*>(tw + P.n_tw);
  uint16_t* const tab = reinterpret_cast<uint16_t*>(c.Pw + P.groups * P.cells);
  c.tab = tab;
  c.tw_lds = tw;
  c.tw_glob = tw_glob;
  c.lds_tw = P.n_tw > 0;
  c.w_size = P.w_size;
  c.cells = P.cells;
  c.groups = P.groups;
  c.tid = threadIdx.x;
  c.nt = blockDim.x;

  // block -> (slice, channel, split residue); the n_split work-groups of a (slice, channel) share an XCD's L2
  const int bid = blockIdx.x;
  int grp, s;
  if (P.xcd_groups) {
    const int j = bid >> 3;
    grp = (bid & 7) + 8 * (j / P.n_split);
    s = j % P.n_split;
  } else {
    grp = bid / P.n_split;
    s = bid % P.n_split;
  }
  const int f = grp % P.F;
  const int64_t t0 = (int64_t)(grp / P.F) * tps;
  const int64_t t1 = min(T, t0 + tps);

  for (int i = c.tid; i < P.n_tab; i += c.nt) tab[i] = tab_glob[i];
  for (int i = c.tid; i < P.n_tw; i += c.nt) tw[i] = tw_glob[i];
  for (int i = c.tid; i < P.groups * P.cells; i += c.nt) c.Pw[i] = 0.f;
  double* const out = partial + ((int64_t)grp * P.n_split + s) * P.cells;
  bool first = true;
  int held = 0;  // samples in the power array
  for (int64_t t = t0; t < t1; t += P.batch) {
    c.nb = (int)min<int64_t>(P.batch, t1 - t);
    __syncthreads();  // W free, tables and power array ready
    const int64_t tile = (t * P.F + f) * (int64_t)P.N, next = (int64_t)P.F * P.N;
    if (P.n_split == 1) {
      const uint32_t total = (uint32_t)(c.nb * P.N);
      for (uint32_t e = c.tid; e < total; e += c.nt) {
        const uint32_t b = fast_div(e, P.n_magic), i = e - b * P.N;
        const uint32_t j = fast_div(i, P.load_magic), line = i - j * P.load_lines;
        c.W[b * P.w_size + tab[P.load_tab + line] + j * P.load_stride] = sample_at(src, tile + b * next + i, P.fmt);
      }
    } else {
      // stage 1 of axis 0 for the outputs kappa_1 = s + n_split k, k < k_out, by direct sums
      const uint32_t per = (uint32_t)(P.load_lines * P.k_out), jobs = per * (uint32_t)c.nb;
      const int step0 = P.m0 / P.f1;
      for (uint32_t q = c.tid; q < jobs; q += c.nt) {
        const uint32_t b = fast_div(q, P.k_magic), r = q - b * per;
        const uint32_t k = fast_div(r, P.load_magic), line = r - k * P.load_lines;
        const int kap = s + P.n_split * (int)k;
        const int64_t base = tile + b * next + line;
        float2 z = make_float2(0.f, 0.f);
        int e = 0;  // kappa_1 j mod f1
        for (int j = 0; j < P.n1; ++j) {
          const float2 v = sample_at(src, base + (int64_t)j * P.load_lines, P.fmt);
          const float2 w = c.lds_tw ? tw[e * step0] : tw_glob[e * step0];
          z.x = fmaf(v.x, w.x, fmaf(-v.y, w.y, z.x));
          z.y = fmaf(v.x, w.y, fmaf(v.y, w.x, z.y));
          e += kap;
          if (e >= P.f1) e -= P.f1;
        }
        if (P.load_tj >= 0) {
          const int at = kap * (int)tab[P.load_tj + line];
          z = dn::mul(z, c.lds_tw ? tw[at] : tw_glob[at]);
        }
        c.W[b * P.w_size + tab[P.load_tab + line] + (int)k * P.load_stride] = z;
      }
    }
    __syncthreads();
    for (int pass = 0; pass < P.n_pass - 1; ++pass) {
      run_mid(P.pass[pass], c);
      __syncthreads();
    }
    run_last(P.pass[P.n_pass - 1], c);
    held += c.nb;
    if (held + P.batch > P.time_block || t + P.batch >= t1) {
      __syncthreads();
      for (int i = c.tid; i < P.cells; i += c.nt) {
        double v = first ? 0.0 : out[i];
        for (int g = 0; g < P.groups; ++g) {
          v += (double)c.Pw[g * P.cells + i];
          c.Pw[g * P.cells + i] = 0.f;
        }
        out[i] = v;
      }
      first = false;
      held = 0;
    }
  }
}

}  // namespace

hipError_t launch_lines_fp32(const void* src, int64_t T, int64_t tps, const float2* tw, const uint16_t* tab,
                             double* partial, const LineP& P, int grid, int threads, size_t lds, hipStream_t st) {
  if (P.n_pass < 1 || P.n_pass > kLineMaxPass || threads > 1024) return hipErrorInvalidValue;
  // (always the largest: the limit belongs to the process, and another thread may be launching another plan)
  hipError_t e = hipFuncSetAttribute((const void*)lines_fp32_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(lines_fp32_kernel, dim3((unsigned)grid), dim3((unsigned)threads), lds, st, src, T, tps, tw, tab,
                     partial, P);
  return hipGetLastError();
}

}  // namespace omni
