// CPU check of the line kernel's schedules and of the inverse's: every table, stride and division of lines.hpp executed on the host in
// float64 with bounds checks, for grids given on stdin ("n_1 ... n_d [b1|b2]", the suffix: that many innermost axes
// unpadded), against plain zero-padded DFTs.  Prints how many schedules were checked and how many
// grids have none.
#include "inverse.hpp"
#include "lines_plan.hpp"

#include <cmath>
#include <complex>
#include <cstdio>
#include <cstdlib>
#include <iostream>
#include <sstream>
#include <string>

using cd = std::complex<double>;
using omni::LinePass;
using omni::LineSetup;

#define CHECK(c)                                                              \
  do {                                                                        \
    if (!(c)) {                                                               \
      std::printf("FAILED %s (line %d) on %s\n", #c, __LINE__, name.c_str()); \
      return 1;                                                               \
    }                                                                         \
  } while (0)

static cd w(long long e, int m) { return std::polar(1.0, -2.0 * M_PI * (double)(e % m) / m); }
static uint32_t fast_div(uint32_t q, uint32_t magic) {
  return magic ? (uint32_t)(((uint64_t)q * magic) >> 32) : q;
}

static int check(const std::string& name, const std::vector<int>& n, const std::vector<int>& m, int max_batch,
                 bool* planned) {
  LineSetup s;
  *planned = omni::plan_lines((int)n.size(), n.data(), m.data(), max_batch, s);
  if (!*planned) return 0;
  const omni::LineP& P = s.P;
  const int d = (int)n.size();
  int64_t N = 1, M = 1;
  for (int k = 0; k < d; ++k) {
    N *= n[(size_t)k];
    M *= m[(size_t)k];
  }
  CHECK(P.N == N && (int64_t)P.cells * P.n_split == M && (int64_t)s.kmap.size() == M);
  CHECK(s.lds <= 160 * 1024 && s.threads >= 64 && s.threads <= 1024 && P.batch >= 1 && P.batch <= max_batch);
  CHECK(P.groups >= 1 && P.groups <= P.batch && P.n_pass >= 1 && P.n_pass <= omni::kLineMaxPass);
  CHECK((size_t)P.n_tab == s.tab.size());
  CHECK(s.lds >= (size_t)P.batch * P.w_size * 8 + P.n_tw * 8 + (size_t)P.groups * P.cells * 4 + P.n_tab * 2);
  std::vector<int> seen((size_t)M, 0);
  for (int32_t k : s.kmap) {
    CHECK(k >= 0 && k < M);
    CHECK(seen[(size_t)k]++ == 0);
  }
  // divisions over every value the kernel forms
  for (uint32_t q = 0; P.n_split == 1 && q < (uint32_t)(P.batch * N); ++q) CHECK(fast_div(q, P.n_magic) == q / N);
  CHECK(P.n_split == 1 ? P.batch * N < 65536 : (int64_t)P.batch * P.load_lines * P.k_out < 65536);
  for (int64_t q = 0; q < (P.n_split == 1 ? N : (int64_t)P.load_lines * P.k_out); ++q)
    CHECK(fast_div((uint32_t)q, P.load_magic) == q / P.load_lines);
  for (int64_t q = 0; P.n_split > 1 && q < (int64_t)P.batch * P.load_lines * P.k_out; ++q)
    CHECK(fast_div((uint32_t)q, P.k_magic) == q / ((int64_t)P.load_lines * P.k_out));
  // twiddle table as the plan lays it out: per axis w_m^q
  std::vector<cd> tw;
  for (int k = 0; k < d; ++k)
    for (int q = 0; q < m[(size_t)k]; ++q) tw.push_back(w(q, m[(size_t)k]));
  // one sample per batch slot, reference transform axis by axis
  std::vector<std::vector<cd>> x((size_t)P.batch);
  std::vector<std::vector<double>> ref((size_t)P.batch);
  unsigned seed = 12345;
  for (int b = 0; b < P.batch; ++b) {
    for (int64_t i = 0; i < N; ++i) {
      seed = seed * 1664525u + 1013904223u;
      x[(size_t)b].push_back(cd((int)(seed >> 28) - 8, (int)((seed >> 24) & 15) - 8));
    }
    std::vector<cd> cur = x[(size_t)b];
    int64_t outer = 1, inner = N;
    for (int k = 0; k < d; ++k) {
      const int nk = n[(size_t)k], mk = m[(size_t)k];
      inner /= nk;
      std::vector<cd> nx((size_t)(outer * mk * inner));
      for (int64_t o = 0; o < outer; ++o)
        for (int q = 0; q < mk; ++q)
          for (int64_t i = 0; i < inner; ++i) {
            cd z = 0;
            for (int j = 0; j < nk; ++j) z += cur[(size_t)((o * nk + j) * inner + i)] * w((long long)j * q, mk);
            nx[(size_t)((o * mk + q) * inner + i)] = z;
          }
      cur.swap(nx);
      outer *= mk;
    }
    for (const cd& v : cur) ref[(size_t)b].push_back(std::norm(v));
  }
  CHECK(P.load_tab + P.load_lines <= P.n_tab && P.load_tj + P.load_lines <= P.n_tab);
  for (int c = 0; c < P.n_split; ++c) {
    std::vector<cd> W((size_t)(P.batch * P.w_size), cd(NAN, NAN));
    std::vector<double> pw((size_t)(P.batch * P.cells), 0.0);
    for (int b = 0; b < P.batch; ++b) {
      if (P.n_split == 1) {
        for (int64_t i = 0; i < N; ++i) {
          const int64_t j = i / P.load_lines, line = i % P.load_lines;
          const int64_t at = s.tab[(size_t)(P.load_tab + line)] + j * P.load_stride;
          CHECK(at < P.w_size);
          W[(size_t)(b * P.w_size + at)] = x[(size_t)b][(size_t)i];
        }
      } else {
        for (int k = 0; k < P.k_out; ++k)
          for (int64_t line = 0; line < P.load_lines; ++line) {
            const int kap = c + P.n_split * k;
            cd z = 0;
            for (int j = 0; j < P.n1; ++j) {
              CHECK(j * P.load_lines + line < N);
              z += x[(size_t)b][(size_t)(j * P.load_lines + line)] * w((long long)kap * j, P.f1);
            }
            if (P.load_tj >= 0) {
              const int e = kap * s.tab[(size_t)(P.load_tj + line)];
              CHECK(e < m[0]);
              z *= tw[(size_t)e];
            }
            const int64_t at = s.tab[(size_t)(P.load_tab + line)] + (int64_t)k * P.load_stride;
            CHECK(at < P.w_size);
            W[(size_t)(b * P.w_size + at)] = z;
          }
      }
    }
    for (int pi = 0; pi < P.n_pass; ++pi) {
      const LinePass& p = P.pass[pi];
      const bool two = (p.type & 256) != 0, last = pi + 1 == P.n_pass;
      const int n1 = two ? (p.type - 256) / 16 : p.type & 31, n2 = two ? p.type & 15 : 1;
      const int o1 = two || (p.type & 32) ? 2 * n1 : n1, o2 = two ? 2 * n2 : 1;
      CHECK(!two || (omni::line_pair_ok(n1, n2) && p.tj < 0));
      CHECK((int64_t)P.batch * p.lines < 65536 && p.tab + p.lines <= P.n_tab);
      for (uint32_t q = 0; q < (uint32_t)(P.batch * p.lines); ++q) CHECK(fast_div(q, p.magic) == q / p.lines);
      std::vector<char> owner(W.size(), 0);
      for (int b = 0; b < P.batch; ++b)
        for (int line = 0; line < p.lines; ++line) {
          const int64_t base = (int64_t)b * P.w_size + s.tab[(size_t)(p.tab + line)];
          std::vector<cd> in, outv;
          for (int i = 0; i < n1; ++i)
            for (int j = 0; j < n2; ++j) {
              const int64_t at = base + (int64_t)i * p.stride + (int64_t)j * p.stride2;
              CHECK(at < (int64_t)(b + 1) * P.w_size);
              CHECK(!owner[(size_t)at]);  // not yet written by another line of this pass
              CHECK(!std::isnan(W[(size_t)at].real()));
              in.push_back(W[(size_t)at]);
            }
          for (int k = 0; k < o1; ++k)
            for (int k2 = 0; k2 < o2; ++k2) {
              cd z = 0;
              for (int i = 0; i < n1; ++i)
                for (int j = 0; j < n2; ++j)
                  z += in[(size_t)(i * n2 + j)] * w((long long)i * k, o1) * w((long long)j * k2, o2);
              if (!last && p.tj >= 0) {
                const int e = k * s.tab[(size_t)(p.tj + line)];
                CHECK(p.tw + e < (int)tw.size());
                z *= tw[(size_t)(p.tw + e)];
              }
              outv.push_back(z);
            }
          CHECK(!last || p.tj < 0);
          for (int k = 0; k < o1; ++k)
            for (int k2 = 0; k2 < o2; ++k2) {
              const cd z = outv[(size_t)(k * o2 + k2)];
              if (last) {
                const int64_t cell = (int64_t)(k * o2 + k2) * p.lines + line;
                CHECK(cell < P.cells);
                pw[(size_t)((int64_t)b * P.cells + cell)] += std::norm(z);
              } else {
                const int64_t at = base + (int64_t)k * p.stride + (int64_t)k2 * p.stride2;
                CHECK(at < (int64_t)(b + 1) * P.w_size);
                CHECK(!owner[(size_t)at]);
                owner[(size_t)at] = 1;
                W[(size_t)at] = z;
              }
            }
        }
    }
    for (int b = 0; b < P.batch; ++b)
      for (int cell = 0; cell < P.cells; ++cell) {
        const double want = ref[(size_t)b][(size_t)s.kmap[(size_t)((int64_t)c * P.cells + cell)]];
        CHECK(std::fabs(pw[(size_t)((int64_t)b * P.cells + cell)] - want) <= 1e-9 * (1.0 + 128.0 * N * N));
      }
  }
  return 0;
}

// The inverse's groups executed on the host: random complex cells [channels][M][inner] against plain sums.
static int check_inverse(const std::string& name, const std::vector<int>& n, int channels, int inner_last) {
  const int d = (int)n.size();
  std::vector<int> m, off;
  int64_t M = 1, at = 0;
  std::vector<cd> tw;
  for (int v : n) {
    m.push_back(2 * v);
    off.push_back((int)at);
    for (int q = 0; q < 2 * v; ++q) tw.push_back(std::conj(w(q, 2 * v)));
    at += 2 * v;
    M *= 2 * v;
  }
  const auto groups = omni::plan_inverse(d, n.data(), m.data(), channels, inner_last, off.data());
  std::vector<cd> cur, ref;
  unsigned seed = 777;
  for (int64_t i = 0; i < channels * M * inner_last; ++i) {
    seed = seed * 1664525u + 1013904223u;
    cur.push_back(cd((int)(seed >> 24) - 128, (int)((seed >> 16) & 255) - 128));
  }
  ref = cur;
  int64_t outer = channels, inner = M * inner_last, axis = 0;
  for (const auto& g : groups) {
    CHECK(g.axis0 == axis && g.axes >= 1);
    // reference: the group's axes one by one
    int64_t o2 = outer, i2 = inner, Mg = 1, Ng = 1;
    for (int k = g.axis0; k < g.axis0 + g.axes; ++k) {
      const int nk = n[(size_t)k], mk = m[(size_t)k], lags = 2 * nk - 1;
      i2 /= mk;
      std::vector<cd> nx((size_t)(o2 * lags * i2));
      for (int64_t o = 0; o < o2; ++o)
        for (int l = 0; l < lags; ++l)
          for (int64_t i = 0; i < i2; ++i) {
            cd z = 0;
            for (int q = 0; q < mk; ++q)
              z += ref[(size_t)((o * mk + q) * i2 + i)] * std::conj(w((long long)q * ((l - (nk - 1) + mk) % mk), mk));
            nx[(size_t)((o * lags + l) * i2 + i)] = z;
          }
      ref.swap(nx);
      o2 *= lags;
      Mg *= mk;
      Ng *= lags;
    }
    inner /= Mg;
    axis += g.axes;
    if (!g.direct) {
      const omni::InvP& P = g.P;
      CHECK(P.Mg == Mg && P.Ng == Ng && P.cols >= 1 && P.cols == 1 << P.lg_cols && (P.col_fast != 0) == (inner > 1));
      CHECK((int64_t)P.cols * Mg <= 4096 && P.cols <= 64 && g.lds <= 160 * 1024 && P.n_pass >= 1 && P.n_pass <= omni::kInvMaxPass);
      const int64_t lds_n = (int64_t)g.lds / 16, columns = outer * inner;
      std::vector<cd> out((size_t)(columns * Ng), cd(NAN, NAN));
      for (int64_t col0 = 0; col0 < columns; col0 += P.cols) {
        std::vector<cd> W((size_t)lds_n, cd(NAN, NAN));
        for (int pi = 0; pi < P.n_pass; ++pi) {
          const omni::InvPass& p = P.pass[pi];
          const bool first = pi == 0, last = pi + 1 == P.n_pass;
          CHECK((int64_t)p.lines * p.f == Mg && p.tab + p.lines <= (int)g.tab.size());
          for (uint32_t q = 0; q < (uint32_t)(p.lines * P.cols); ++q) {
            CHECK(fast_div(q, p.magic) == q / p.lines);
            const int64_t c = q / p.lines, line = q % p.lines, col = col0 + c, ou = col / inner, in = col % inner;
            const int64_t b = c * P.col_stride + g.tab[(size_t)(p.tab + line)];
            std::vector<cd> x;
            for (int j = 0; j < p.f; ++j) {
              if (first) {
                x.push_back(col < columns ? cur[(size_t)((ou * Mg + (int64_t)j * p.lines + line) * inner + in)] : cd(0, 0));
                continue;
              }
              CHECK(b + (int64_t)j * p.stride < lds_n);
              x.push_back(W[(size_t)(b + (int64_t)j * p.stride)]);
              CHECK(!std::isnan(x.back().real()));
            }
            for (int k = 0; k < p.f; ++k) {
              cd z = 0;
              for (int j = 0; j < p.f; ++j) z += x[(size_t)j] * std::conj(w((long long)j * k, p.f));
              if (last) {
                CHECK(p.tj < 0);
                const uint32_t o = g.tab[(size_t)(P.out_tab + k * p.lines + line)];
                if (o == omni::kInvNoLag || col >= columns) continue;
                CHECK(o < Ng && std::isnan(out[(size_t)((ou * Ng + o) * inner + in)].real()));
                out[(size_t)((ou * Ng + o) * inner + in)] = z;
                continue;
              }
              if (p.tj >= 0) {
                const int e = p.tw + k * g.tab[(size_t)(p.tj + line)];
                CHECK(e < (int)tw.size());
                z *= tw[(size_t)e];
              }
              const int64_t a = b + (int64_t)k * p.stride;
              CHECK(a < lds_n && (!first || std::isnan(W[(size_t)a].real())));
              W[(size_t)a] = z;
            }
          }
        }
      }
      CHECK(out.size() == ref.size());
      for (size_t i = 0; i < out.size(); ++i) CHECK(std::abs(out[i] - ref[i]) <= 1e-9 * 256.0 * M);
    }
    cur = ref;
    outer *= Ng;
  }
  CHECK(axis == d && inner == inner_last);
  return 0;
}

// Arrays beyond the caches: one axis of 8, 16 or 32 at a time while whole cache lines lie behind it, every axis once;
// a channel that fits one work-group stays one group however many there are (tile pairs are inverted in one launch).
static int check_large_inverse() {
  const std::string name = "large arrays";
  const int off[8] = {};
  for (const auto& n : std::vector<std::vector<int>>{{16, 16, 8, 8, 4, 4}, {4, 4, 8, 8, 4, 4}, {16, 16, 6, 5, 8, 8}, {128, 128}}) {
    std::vector<int> m;
    int64_t rest = 1;
    for (int v : n) {
      m.push_back(2 * v);
      rest *= 2 * v;
    }
    int axis = 0;
    for (const auto& g : omni::plan_inverse((int)n.size(), n.data(), m.data(), 4096, 1, off)) {
      CHECK(g.axis0 == axis && !g.direct && (!g.line || g.axes == 1));
      const int before = m[(size_t)axis];
      for (int k = 0; k < g.axes; ++k) rest /= m[(size_t)axis++];
      CHECK(g.line == (rest >= 64 && (before == 8 || before == 16 || before == 32)));
    }
    CHECK(axis == (int)n.size());
  }
  for (int x = 1; x <= 32; x *= 2)
    for (int y = 1; y <= 32; y *= 2) {
      const int n[2] = {x, y}, m[2] = {2 * x, 2 * y};
      const auto g = omni::plan_inverse(2, n, m, int64_t(1) << 20, 1, off);
      CHECK(g.size() == 1 && !g[0].line && !g[0].direct && g[0].axes == 2);
    }
  return 0;
}

int main() {
  if (check_large_inverse()) return 1;
  std::string line;
  int done = 0, none = 0;
  while (std::getline(std::cin, line)) {
    std::istringstream is(line);
    std::string tok;
    std::vector<int> n;
    int beams = 0;
    while (is >> tok) {
      if (tok[0] == 'b')
        beams = std::atoi(tok.c_str() + 1);
      else
        n.push_back(std::atoi(tok.c_str()));
    }
    std::vector<int> m;
    for (size_t k = 0; k < n.size(); ++k) m.push_back((int)(n.size() - k) <= beams ? n[k] : 2 * n[k]);
    int64_t M = 1;
    for (int v : n) M *= 2 * v;
    for (int ch : {1, 3, 40})
      for (int inner : {1, 5})
        if (M * ch * inner <= 80000 && check_inverse(line, n, ch, inner)) return 1;
    for (int max_batch : {64, 3}) {
      bool planned = false;
      if (check(line, n, m, max_batch, &planned)) return 1;
      planned ? ++done : ++none;
      if (!planned) std::printf("no schedule: %s\n", line.c_str());
    }
  }
  std::printf("schedules checked: %d\nnot planned: %d\n", done, none);
  return 0;
}
