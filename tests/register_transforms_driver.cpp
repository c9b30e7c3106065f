// CPU check of the register transforms (dftn.hpp): every length against plain sums in float64, and the mean power of
// the float32 ones (rotations and constants of exact length) against Parseval's sum.
#include "dftn.hpp"

#include <complex>
#include <cstdio>
#include <random>

using namespace omni::dn;

static int bad = 0;

template <int N>
void check() {
  double2 x[N], z[N];
  for (int j = 0; j < N; ++j) z[j] = x[j] = {std::sin(1.3 * j + 1), std::cos(2.1 * j)};
  dft<N>(z);
  double err = 0;
  for (int k = 0; k < N; ++k) {
    std::complex<double> s = 0;
    for (int j = 0; j < N; ++j) s += std::complex<double>(x[j].x, x[j].y) * std::polar(1.0, -2 * M_PI * (j * k % N) / N);
    err = std::max(err, std::abs(s - std::complex<double>(z[k].x, z[k].y)));
  }
  // 2^-53 an operation, values of at most N, at most N additions a value
  if (!(err <= 1.2e-16 * N * N)) ++bad, std::printf("length %d: %.2e\n", N, err);
  std::mt19937 g(N);
  std::normal_distribution<float> u;
  double power[2] = {0, 0}, want = 0;
  for (int it = 0; it < 20000; ++it) {
    float2 a[N], b[N];
    for (int j = 0; j < N; ++j) {
      a[j] = {u(g), u(g)};
      want += (double)a[j].x * a[j].x + (double)a[j].y * a[j].y;
      b[j] = rot<2 * N>(a[j], j);
    }
    dft<N>(a);
    dft<N>(b);
    for (int j = 0; j < N; ++j) {
      power[0] += ((double)a[j].x * a[j].x + (double)a[j].y * a[j].y) / N;
      power[1] += ((double)b[j].x * b[j].x + (double)b[j].y * b[j].y) / N;
    }
  }
  // rounding errors have no sign: 2e-7 / sqrt(20000) at most; constants of 24 bits make 0.9e-8 (7) to 4.1e-8 (16),
  // and are left in the transforms of 7, 11 and 13
  for (int h = 0; h < 2; ++h) {
    const double e = power[h] / want - 1;
    std::printf("length %d%s: mean power %+.1e\n", N, h ? " rotated" : "", e);
    if (!(std::fabs(e) <= (N == 7 || N == 11 || N == 13 ? 1.5e-8 : 3e-9))) ++bad;
  }
}

int main() {
  check<2>(), check<3>(), check<4>(), check<5>(), check<6>(), check<7>(), check<8>(), check<9>(), check<10>();
  check<11>(), check<12>(), check<13>(), check<16>(), check<32>();
  return bad != 0;
}
