// Short complex DFTs of any small length with compile-time twiddles, in registers (gfx950).
//
// dft<N> transforms N float2 or double2 values in place, natural order, w_N = exp(-2 pi i / N): composite lengths by
// Cooley-Tukey (factor 4, then 2, then the smallest odd prime; without rotations between coprime factors), odd primes
// p by the sums and differences of the pairs (j, p - j), which need (p - 1)^2 real multiplications instead of
// 4 (p - 1)^2.  The twiddles are constants of the instruction stream, evaluated in float64 at compile time (a Taylor series after exact reduction of the
// angle to [0, pi/4]) and rounded to the values' precision once.  In float32 a rounded twiddle is not of length one, and
// a short transform uses few of them, so that the powers of all its outputs are off the same way (-2.1e-8 an axis of 3,
// -4.1e-8 of 16).  Rotations therefore keep the smaller of cosine and sine in 24 bits and the other one, from it, in
// 48: the angle is off by at most 2^-25, the length by nothing; the 3- and 5-point transforms' constants have 48 bits too.
// 12 x 12, 32 channels: error against 64 bits 7.2e-8 -> 2.7e-8 of the visibilities' norm (direct sums with a rounded
// table: 5.4e-8).
#pragma once

#include <hip/hip_runtime.h>

namespace omni {
namespace dn {

constexpr double kPi = 3.141592653589793238462643383279502884;

constexpr double taylor_sin(double x) {
  double term = x, sum = x;
  for (int k = 1; k < 14; ++k) {
    term *= -x * x / ((2.0 * k) * (2.0 * k + 1.0));
    sum += term;
  }
  return sum;
}
constexpr double taylor_cos(double x) {
  double term = 1.0, sum = 1.0;
  for (int k = 1; k < 14; ++k) {
    term *= -x * x / ((2.0 * k - 1.0) * (2.0 * k));
    sum += term;
  }
  return sum;
}

// cos(pi u / n), sin(pi u / n) for 0 <= u <= n / 2
constexpr double cos_q(int u, int n) {
  return 4 * u <= n ? taylor_cos(kPi * u / n) : taylor_sin(kPi * (n - 2 * u) / (2.0 * n));
}
constexpr double sin_q(int u, int n) {
  return 4 * u <= n ? taylor_sin(kPi * u / n) : taylor_cos(kPi * (n - 2 * u) / (2.0 * n));
}
// cos(2 pi q / n), sin(2 pi q / n)
constexpr double cos2pi(int q, int n) {
  int u = 2 * (q % n);
  if (u > n) u = 2 * n - u;
  return 2 * u > n ? -cos_q(n - u, n) : cos_q(u, n);
}
constexpr double sin2pi(int q, int n) {
  int u = 2 * (q % n);
  const bool neg = u > n;
  if (neg) u = 2 * n - u;
  const double s = 2 * u > n ? sin_q(n - u, n) : sin_q(u, n);
  return neg ? -s : s;
}

// w_N^q = (c[q], -s[q])
template <int N>
struct Roots {
  double c[N] = {}, s[N] = {};
  constexpr Roots() {
    for (int q = 0; q < N; ++q) {
      c[q] = cos2pi(q, N);
      s[q] = sin2pi(q, N);
    }
  }
};
template <int N>
constexpr Roots<N> kRoots{};

constexpr double root(double v) {  // square root of 0.5 <= v <= 1 (Newton's iteration)
  double r = v;
  for (int k = 0; k < 8; ++k) r = 0.5 * (r + v / r);
  return r;
}
// The rotation by -2 pi q / N in float32: c - i s with c = c1 + c2, s = s1 + s2; one of c2 and s2 is zero.
struct Turn {
  float c1 = 0, c2 = 0, s1 = 0, s2 = 0;
  constexpr Turn(double c, double s) {
    c1 = (float)c;
    s1 = (float)s;
    if ((s < 0 ? -s : s) < (c < 0 ? -c : c)) {
      const double e = root(1.0 - (double)s1 * s1) * (c < 0 ? -1.0 : 1.0);
      c1 = (float)e;
      c2 = (float)(e - c1);
    } else {
      const double e = root(1.0 - (double)c1 * c1) * (s < 0 ? -1.0 : 1.0);
      s1 = (float)e;
      s2 = (float)(e - s1);
    }
  }
};

__device__ __forceinline__ float2 pair(float x, float y) { return make_float2(x, y); }
__device__ __forceinline__ double2 pair(double x, double y) { return make_double2(x, y); }
__device__ __forceinline__ float mad(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double mad(double a, double b, double c) { return fma(a, b, c); }
template <class V>
__device__ __forceinline__ V add(V a, V b) {
  return pair(a.x + b.x, a.y + b.y);
}
template <class V>
__device__ __forceinline__ V sub(V a, V b) {
  return pair(a.x - b.x, a.y - b.y);
}
template <class V>
__device__ __forceinline__ V mul(V a, V b) {
  return pair(mad(a.x, b.x, -a.y * b.y), mad(a.x, b.y, a.y * b.x));
}

// v * w_N^q, q a constant after unrolling: multiples of a quarter turn cost nothing
template <int N, class V>
__device__ __forceinline__ V rot(V v, int q) {
  using S = decltype(v.x);
  constexpr Roots<N> R = kRoots<N>;
  q %= N;
  if (q == 0) return v;
  if (4 * q == N) return pair(v.y, -v.x);
  if (2 * q == N) return pair(-v.x, -v.y);
  if (4 * q == 3 * N) return pair(-v.y, v.x);
  if constexpr (sizeof(S) == sizeof(float)) {
    // (the small part goes with its own product: added to the other one, which may be exact, rounding would drop it)
    const Turn t(R.c[q], R.s[q]);
    if (t.s2 == 0.f) return pair(mad(v.y, t.s1, mad(v.x, t.c1, v.x * t.c2)), mad(-v.x, t.s1, mad(v.y, t.c1, v.y * t.c2)));
    return pair(mad(v.x, t.c1, mad(v.y, t.s1, v.y * t.s2)), mad(v.y, t.c1, mad(-v.x, t.s1, -v.x * t.s2)));
  } else {
    const S c = R.c[q], s = R.s[q];
    return pair(mad(v.x, c, v.y * s), mad(v.y, c, -v.x * s));
  }
}

constexpr int first_factor(int n) {
  if (n % 4 == 0) return 4;
  if (n % 2 == 0) return 2;
  for (int p = 3; p * p <= n; p += 2)
    if (n % p == 0) return p;
  return n;
}

template <int N, class V>
__device__ __forceinline__ void dft(V (&x)[N]) {
  using S = decltype(x[0].x + x[0].x);
  if constexpr (N == 1) {
  } else if constexpr (N == 2) {
    const V a = x[0], b = x[1];
    x[0] = add(a, b);
    x[1] = sub(a, b);
  } else if constexpr (N == 4) {
    const V a = add(x[0], x[2]), b = sub(x[0], x[2]), c = add(x[1], x[3]), d = sub(x[1], x[3]);
    x[0] = add(a, c);
    x[2] = sub(a, c);
    x[1] = pair(b.x + d.y, b.y - d.x);
    x[3] = pair(b.x - d.y, b.y + d.x);
  } else if constexpr (first_factor(N) == N) {  // odd prime
    constexpr Roots<N> R = kRoots<N>;
    constexpr int H = (N - 1) / 2;
    V a[H], b[H];
#pragma unroll
    for (int j = 0; j < H; ++j) {
      a[j] = add(x[j + 1], x[N - 1 - j]);
      b[j] = sub(x[j + 1], x[N - 1 - j]);
    }
    const V x0 = x[0];
    V t = x0;
#pragma unroll
    for (int j = 0; j < H; ++j) t = add(t, a[j]);
    x[0] = t;
#pragma unroll
    for (int k = 1; k <= H; ++k) {
      V r = x0, i = pair((S)0, (S)0);
      if constexpr (N == 5 && sizeof(S) == sizeof(float)) r = i;
      if constexpr (N <= 5 && sizeof(S) == sizeof(float)) {  // what the constants' rounding leaves out
#pragma unroll
        for (int j = 0; j < H; ++j) {
          const double c = R.c[(k * (j + 1)) % N], s = R.s[(k * (j + 1)) % N];
          const S c2 = (S)(c - (S)c), s2 = (S)(s - (S)s);
          if (N == 5) r = pair(mad(a[j].x, c2, r.x), mad(a[j].y, c2, r.y));
          i = pair(mad(b[j].x, s2, i.x), mad(b[j].y, s2, i.y));
        }
      }
#pragma unroll
      for (int j = 0; j < H; ++j) {
        const S c = (S)R.c[(k * (j + 1)) % N], s = (S)R.s[(k * (j + 1)) % N];
        r = pair(mad(a[j].x, c, r.x), mad(a[j].y, c, r.y));
        i = pair(mad(b[j].x, s, i.x), mad(b[j].y, s, i.y));
      }
      if constexpr (N == 5 && sizeof(S) == sizeof(float)) r = add(x0, r);
      x[k] = pair(r.x + i.y, r.y - i.x);
      x[N - k] = pair(r.x - i.y, r.y + i.x);
    }
  } else if constexpr (first_factor(N) % 2 == 0 && (N / first_factor(N)) % 2 == 1) {
    // coprime factors (a power of two and an odd number): j = B j1 + A j2 mod N, kappa = k1 mod A and k2 mod B, no
    // rotations between the two (Good's prime-factor map)
    constexpr int A = first_factor(N), B = N / A;
    V y[A][B];
#pragma unroll
    for (int j1 = 0; j1 < A; ++j1) {
#pragma unroll
      for (int j2 = 0; j2 < B; ++j2) y[j1][j2] = x[(B * j1 + A * j2) % N];
      dft<B>(y[j1]);
    }
#pragma unroll
    for (int k2 = 0; k2 < B; ++k2) {
      V z[A];
#pragma unroll
      for (int j1 = 0; j1 < A; ++j1) z[j1] = y[j1][k2];
      dft<A>(z);
#pragma unroll
      for (int k = 0; k < N; ++k)
        if (k % B == k2) x[k] = z[k % A];
    }
  } else {
    // j = j1 + A j2, kappa = B k1 + k2:  w^{j kappa} = w_A^{j1 k1} w_N^{j1 k2} w_B^{j2 k2}
    constexpr int A = first_factor(N), B = N / A;
    V y[A][B];
#pragma unroll
    for (int j1 = 0; j1 < A; ++j1) {
#pragma unroll
      for (int j2 = 0; j2 < B; ++j2) y[j1][j2] = x[j1 + A * j2];
      dft<B>(y[j1]);
    }
#pragma unroll
    for (int k2 = 0; k2 < B; ++k2) {
      V z[A];
#pragma unroll
      for (int j1 = 0; j1 < A; ++j1) z[j1] = rot<N>(y[j1][k2], j1 * k2);
      dft<A>(z);
#pragma unroll
      for (int k1 = 0; k1 < A; ++k1) x[B * k1 + k2] = z[k1];
    }
  }
}

}  // namespace dn
}  // namespace omni
