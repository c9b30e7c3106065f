// Planners of the line kernel and of the grouped inverse (host only): stages of every axis, LDS layout, offset
// tables, split, batch and work-group size.  See lines.hpp and inverse.hpp for the schedules.
#include "lines_plan.hpp"

#include "inverse.hpp"

#include <algorithm>
#include <cmath>
#include <cstring>

namespace omni {
namespace {

constexpr size_t kLds = 160 * 1024;

struct Stage {
  int axis;
  int nin, nout;   // inputs and outputs per line
  bool padded;
  int done;        // product of the axis' earlier stages' outputs (frequency stride of this stage's digit)
  int rem;         // index stride of this stage's digit: length still to come after it
};

template <int K>
bool has(const int (&set)[K], int v) {
  return std::find(set, set + K, v) != set + K;
}

// Factors of a plain transform of length m among the lengths `set`: fewest stages, then the smallest sum.  False if
// m has a prime factor that is not there.
template <int K>
bool plain_chain(int m, std::vector<int>& out, const int (&set)[K]) {
  out.clear();
  if (m == 1) return true;
  if (has(set, m)) {
    out.push_back(m);
    return true;
  }
  std::vector<int> best;
  const auto sum = [](const std::vector<int>& v) {
    int s = 0;
    for (int x : v) s += x;
    return s;
  };
  for (int f : set) {
    if (m % f) continue;
    std::vector<int> rest;
    if (!plain_chain(m / f, rest, set)) continue;
    rest.insert(rest.begin(), f);
    if (best.empty() || rest.size() < best.size() || (rest.size() == best.size() && sum(rest) < sum(best))) best = rest;
  }
  out = best;
  return !best.empty();
}

// Vector instructions of one line's transform, roughly.
double line_cost(int nout) { return nout * (2.5 * std::log2((double)std::max(2, nout)) + 4.0) + 20.0; }

// Stages of one axis, appended to st.  `first` != 0 forces the inputs of a zero-padded axis' first stage (any
// divisor of n); 0 takes the cheapest chain of register transforms.
bool axis_stages(int axis, int n, int m, int first, std::vector<Stage>& st) {
  std::vector<int> rest;
  int done = 1, rem = m;
  if (m == 2 * n) {
    if (first) {
      if (n % first || !plain_chain(n / first, rest, kLinePlain)) return false;
    } else {
      std::vector<int> best;
      double best_cost = 1e300;
      for (int a : kLinePadded) {
        if (n % a || (a == 1 && n > 1) || !plain_chain(n / a, rest, kLinePlain)) continue;
        double cost = (double)m / (2 * a) * line_cost(2 * a);
        for (int f : rest) cost += (double)m / f * (line_cost(f) + 8.0 * f);
        if (cost < best_cost) {
          best_cost = cost;
          first = a;
          best = rest;
        }
      }
      if (!first) return false;
      rest = best;
    }
    rem /= 2 * first;
    st.push_back({axis, first, 2 * first, true, 1, rem});
    done = 2 * first;
  } else if (m == n) {
    if (!plain_chain(m, rest, kLinePlain)) return false;
  } else {
    return false;
  }
  for (int f : rest) {
    rem /= f;
    st.push_back({axis, f, f, false, done, rem});
    done *= f;
  }
  return true;
}

uint32_t magic_of(int64_t d) { return d <= 1 ? 0u : (uint32_t)(((uint64_t(1) << 32) + (uint64_t)d - 1) / (uint64_t)d); }

// One pass: stage a, or the two one-stage zero-padded axes a and b (b >= 0) together.
struct Unit {
  int a, b;
};

int unit_type(const std::vector<Stage>& st, const Unit& u) {
  const Stage& a = st[(size_t)u.a];
  return u.b >= 0 ? 256 + 16 * a.nin + st[(size_t)u.b].nin : a.nin | (a.padded ? 32 : 0);
}

struct Layout {
  std::vector<Unit> order;
  std::vector<int> stride;
  std::vector<int64_t> lines;
  int64_t w_size = 0, cells = 0, tab = 0, load_lines = 0;
};

// Passes: short zero-padded axes two by two where `pairs` allows, everything else stage by stage, long transforms first
// (the later passes see more lines), an axis' stages in order; last a pair, else a zero-padded one-stage axis, else the
// final stage of some axis: the working array holds that pass' inputs, a quarter or half of its outputs.  In the split
// form stage 0 has been summed before the passes.
Layout make_layout(const std::vector<Stage>& st, int split, bool pairs) {
  Layout L;
  const int n = (int)st.size();
  auto alone = [&](int i) {  // the only stage of a zero-padded axis
    return st[(size_t)i].padded && (i + 1 == n || st[(size_t)i + 1].axis != st[(size_t)i].axis);
  };
  std::vector<int> left;  // stages without a unit
  for (int i = split > 1 ? 1 : 0; i < n; ++i) left.push_back(i);
  std::vector<Unit> units;
  if (pairs) {
    std::vector<int> cand;
    for (int i : left)
      if (alone(i)) cand.push_back(i);
    std::stable_sort(cand.begin(), cand.end(), [&](int a, int b) { return st[(size_t)a].nin > st[(size_t)b].nin; });
    while (!cand.empty()) {
      const int a = cand.front();
      cand.erase(cand.begin());
      for (size_t k = 0; k < cand.size(); ++k)
        if (line_pair_ok(st[(size_t)a].nin, st[(size_t)cand[k]].nin)) {
          units.push_back({a, cand[k]});
          left.erase(std::find(left.begin(), left.end(), a));
          left.erase(std::find(left.begin(), left.end(), cand[k]));
          cand.erase(cand.begin() + (std::ptrdiff_t)k);
          break;
        }
    }
    if (units.empty()) return L;
  }
  for (int i : left) units.push_back({i, -1});
  auto in_of = [&](const Unit& u) { return st[(size_t)u.a].nin * (u.b >= 0 ? st[(size_t)u.b].nin : 1); };
  auto out_of = [&](const Unit& u) { return st[(size_t)u.a].nout * (u.b >= 0 ? st[(size_t)u.b].nout : 1); };
  int last = -1;
  for (int k = 0; k < (int)units.size(); ++k) {
    const Unit& u = units[(size_t)k];
    if (u.b < 0 && u.a + 1 < n && st[(size_t)u.a + 1].axis == st[(size_t)u.a].axis) continue;  // not a final stage
    if (last < 0) {
      last = k;
      continue;
    }
    const Unit& v = units[(size_t)last];
    const int gu = out_of(u) / in_of(u), gv = out_of(v) / in_of(v);
    if (gu != gv ? gu > gv : in_of(u) < in_of(v)) last = k;
  }
  if (last < 0) return L;
  const Unit lu = units[(size_t)last];
  units.erase(units.begin() + last);
  std::stable_sort(units.begin(), units.end(), [&](const Unit& u, const Unit& v) {
    const int au = st[(size_t)u.a].axis, av = st[(size_t)v.a].axis;
    if (au == av) return u.a < v.a;
    int mu = out_of(u), mv = out_of(v);  // an axis of several stages sorts as one, by its longest stage
    for (const Stage& s : st) {
      if (s.axis == au) mu = std::max(mu, s.nout);
      if (s.axis == av) mv = std::max(mv, s.nout);
    }
    return mu != mv ? mu > mv : au < av;
  });
  L.order = units;
  L.order.push_back(lu);
  L.stride.assign((size_t)n, 0);
  int64_t s = 1;
  L.cells = 1;
  for (int i = n - 1; i >= 0; --i) {
    const int out = i == 0 ? st[0].nout / split : st[(size_t)i].nout;
    L.stride[(size_t)i] = (int)std::min<int64_t>(s, 1 << 28);
    L.w_size = s * (i == lu.a || i == lu.b ? st[(size_t)i].nin : out);
    s = L.w_size | 1;
    L.cells *= out;
    if (L.cells > (int64_t(1) << 26) || s > (int64_t(1) << 26)) return Layout();
  }
  std::vector<int> cur((size_t)n);
  L.load_lines = 1;
  for (int i = 0; i < n; ++i) {
    cur[(size_t)i] = st[(size_t)i].nin;
    if (i) L.load_lines *= st[(size_t)i].nin;
  }
  L.tab = L.load_lines * (split > 1 && st[0].rem > 1 ? 2 : 1);
  if (split > 1) cur[0] = st[0].nout / split;
  for (const Unit& u : L.order) {
    int64_t lines = 1;
    for (int k = 0; k < n; ++k)
      if (k != u.a && k != u.b) lines *= cur[(size_t)k];
    L.lines.push_back(lines);
    L.tab += lines * (st[(size_t)u.a].rem > 1 ? 2 : 1);
    for (int k : {u.a, u.b})
      if (k >= 0) cur[(size_t)k] = k == 0 ? st[0].nout / split : st[(size_t)k].nout;
  }
  return L;
}

}  // namespace

bool plan_lines(int d, const int* n, const int* m, int max_batch, LineSetup& out) {
  int64_t N = 1;
  int tw_all = 0;
  for (int k = 0; k < d; ++k) {
    N *= n[k];
    tw_all += m[k];
  }
  if (N > (int64_t(1) << 26)) return false;
  std::vector<Stage> tail;  // the stages of axes 1 ... d - 1
  for (int k = 1; k < d; ++k)
    if (!axis_stages(k, n[k], m[k], 0, tail)) return false;

  // Candidates: first stage of axis 0 and its split S (a divisor of the stage's outputs; only a zero-padded
  // stage, which the split form sums directly, so its length is free), pairs of axes or not, threads, batch, copies of
  // the power array.  The cost of one sample of a channel, in cycles of a CU: 1.12 a vector instruction of any wave,
  // plus 3.7 an instruction of the longest wave and 990 a pass (its barrier and LDS latency), shared by the
  // work-groups that fit a CU.  Fitted to 88 schedules of seven grids (measured 940 to 98000 cycles; 12% rms);
  // the last term of the last pass: one wave's LDS latency for each further sample.
  double best = 1e300;
  int bS = 0, bB = 0, bNT = 0, bG = 0, bfit = 1;
  bool bTw = false;
  Layout bL;
  std::vector<Stage> bst, st;
  std::vector<std::pair<int, int>> cands = {{0, 1}};  // (inputs of stage 1 or 0, split)
  if (m[0] == 2 * n[0])
    for (int a = 1; a <= std::min(n[0], 128); ++a)
      for (int S = 2; S <= 2 * a; ++S)
        if (n[0] % a == 0 && (2 * a) % S == 0) cands.push_back({a, S});
  for (const auto& cand : cands) {
    const int S = cand.second;
    st.clear();
    if (!axis_stages(0, n[0], m[0], cand.first, st)) continue;
    st.insert(st.end(), tail.begin(), tail.end());
    if ((int)st.size() > kLineMaxPass || (S > 1 && st.size() < 2)) continue;
    bool twiddled = false;
    for (const Stage& s : st) twiddled = twiddled || s.rem > 1;
    const Stage s0 = st[0];
    for (const bool pairs : {false, true}) {
      const Layout L = make_layout(st, S, pairs);
      if (L.order.empty()) continue;
      const int64_t n_tw = (twiddled || S > 1) && tw_all <= 1024 ? tw_all : 0;
      const int64_t load_lines = N / s0.nin, k_out = s0.nout / S;
      std::vector<double> instr;  // vector instructions of a line of each pass
      double last_sums = 0, last_wait = 0;
      for (const Unit& u : L.order) {
        const Stage& a = st[(size_t)u.a];
        const double one = line_cost(a.nout);
        instr.push_back(one + (a.rem > 1 ? 8.0 * a.nout : 0.0));
        last_sums = 4.0 * a.nout;
        last_wait = 250.0;
        if (u.b >= 0) {
          const Stage& b = st[(size_t)u.b];
          instr.back() = 20.0 + a.nin * (line_cost(b.nout) - 20.0) + b.nout * (one - 20.0);
          last_sums *= b.nout;
          last_wait = 500.0;
        }
      }
      for (int NT = 256; NT <= 1024; NT *= 2) {
        for (int B = 1; B <= std::min(kLineMaxBatch, std::max(1, max_batch)); B *= 2) {
          const int Gmax = (int)std::max<int64_t>(1, std::min<int64_t>(B, NT / L.lines.back()));
          for (int G = Gmax; G >= 1; G = G > 1 ? G / 2 : 0) {
            const size_t lds = (size_t)(B * L.w_size * 8 + n_tw * 8 + G * L.cells * 4 + L.tab * 2);
            if (lds > kLds) continue;
            if (B * N >= 65536 && S == 1) continue;
            if (S > 1 && B * load_lines * k_out >= 65536) continue;
            bool ok = L.w_size < 65536;
            double issue = 0, chain = 0;  // vector instructions of the work-group's waves; of its longest wave, with waits
            auto add = [&](int64_t jobs, double instr) {
              ok = ok && jobs < 65536;
              issue += std::ceil(jobs / 64.0) * instr;
              chain += std::ceil((double)jobs / NT) * instr * 3.7 + 990.0;
            };
            if (S == 1)
              add(B * N, 12.0);
            else
              add(B * load_lines * k_out, 40.0 + 24.0 * s0.nin);  // direct sums with a load from HBM for every input
            for (size_t p = 0; p + 1 < L.order.size(); ++p) add(B * L.lines[p], instr[p]);
            const int64_t jobs = G * L.lines.back();
            ok = ok && jobs < 65536;
            const double each = std::ceil((double)B / G), last = instr.back() * each + last_sums;
            issue += std::ceil(jobs / 64.0) * last;
            chain += std::ceil((double)jobs / NT) * (last * 3.7 + (each - 1.0) * last_wait) + 990.0;
            if (!ok) continue;
            const double fit = std::max(1.0, std::min(std::floor((double)kLds / (double)lds), 1024.0 / NT));
            const double cost = (double)S / B * (1.12 * issue + chain / fit);
            if (cost < best * 0.98) {
              best = cost;
              bS = S;
              bB = B;
              bNT = NT;
              bG = G;
              bfit = (int)fit;
              bL = L;
              bst = st;
              bTw = twiddled || S > 1;
            }
          }
        }
      }
    }
  }
  if (!bS) return false;
  st = bst;
  const Stage& s0 = st[0];
  const int ns = (int)st.size();
  LineP& P = out.P;
  std::memset(&P, 0, sizeof P);
  P.n_pass = (int32_t)bL.order.size();
  P.N = (int32_t)N;
  P.batch = bB;
  P.groups = bG;
  P.w_size = (int32_t)bL.w_size;
  P.cells = (int32_t)bL.cells;
  P.n_split = bS;
  P.n_tw = bTw && tw_all <= 1024 ? tw_all : 0;
  P.load_lines = (int32_t)bL.load_lines;
  P.load_magic = magic_of(P.load_lines);
  P.load_stride = bL.stride[0];
  P.load_tj = -1;
  P.n_magic = magic_of(N);
  P.f1 = s0.nout;
  P.n1 = s0.nin;
  P.m0 = m[0];
  P.k_out = s0.nout / bS;
  P.k_magic = magic_of((int64_t)P.load_lines * P.k_out);
  std::vector<int> tw_off((size_t)d, 0);
  for (int k = 1; k < d; ++k) tw_off[(size_t)k] = tw_off[(size_t)k - 1] + m[k - 1];
  out.tab.clear();
  out.order.clear();
  std::vector<int> cur((size_t)ns);
  for (int i = 0; i < ns; ++i) cur[(size_t)i] = st[(size_t)i].nin;
  // the offsets of the lines along the stages a and b (b = -1: a alone), at the extents `cur`, and their twiddle steps
  // where `twiddle`; returns the first entry of each (-1: no steps)
  auto put_lines = [&](int a, int b, int64_t lines, bool twiddle) {
    const int at = (int)out.tab.size();
    std::vector<uint16_t> steps;
    for (int64_t line = 0; line < lines; ++line) {
      int64_t r = line, off = 0, j = 0;
      for (int k = ns - 1; k >= 0; --k) {
        if (k == a || k == b) continue;
        const int64_t digit = r % cur[(size_t)k];
        r /= cur[(size_t)k];
        off += digit * bL.stride[(size_t)k];
        if (st[(size_t)k].axis == st[(size_t)a].axis && k > a) j += digit * st[(size_t)k].rem;
      }
      out.tab.push_back((uint16_t)off);
      steps.push_back((uint16_t)(j * st[(size_t)a].done));
    }
    int tj = -1;
    if (twiddle) {
      tj = (int)out.tab.size();
      out.tab.insert(out.tab.end(), steps.begin(), steps.end());
    }
    return std::pair<int, int>(at, tj);
  };
  const auto load = put_lines(0, -1, bL.load_lines, bS > 1 && s0.rem > 1);
  P.load_tab = load.first;
  P.load_tj = load.second;
  if (bS > 1) cur[0] = P.k_out;
  for (size_t p = 0; p < bL.order.size(); ++p) {
    const Unit& u = bL.order[p];
    const Stage& s = st[(size_t)u.a];
    LinePass& q = P.pass[p];
    q.type = unit_type(st, u);
    q.stride = bL.stride[(size_t)u.a];
    if (u.b >= 0) q.stride2 = bL.stride[(size_t)u.b];
    q.lines = (int32_t)bL.lines[p];
    q.magic = magic_of(q.lines);
    q.tw = tw_off[(size_t)s.axis];
    const auto t = put_lines(u.a, u.b, bL.lines[p], s.rem > 1);
    q.tab = t.first;
    q.tj = t.second;
    for (int k : {u.a, u.b})
      if (k >= 0) {
        cur[(size_t)k] = k == 0 ? P.k_out : st[(size_t)k].nout;
        out.order.push_back(st[(size_t)k].axis);
      }
  }
  P.n_tab = (int32_t)out.tab.size();

  // cell (split residue c, output q of the last pass, line) -> natural frequency index
  const Unit lu = bL.order.back();
  std::vector<int64_t> nat((size_t)d, 1);
  for (int k = d - 2; k >= 0; --k) nat[(size_t)k] = nat[(size_t)k + 1] * m[k + 1];
  out.kmap.assign((size_t)(bS * bL.cells), 0);
  const int64_t lines = bL.lines.back();
  for (int c = 0; c < bS; ++c)
    for (int64_t cell = 0; cell < bL.cells; ++cell) {
      int64_t r = cell % lines, at = 0;
      const int64_t o = cell / lines;
      auto put = [&](int k, int64_t digit) {
        const Stage& s = st[(size_t)k];
        if (k == 0) digit = c + digit * bS;
        at += digit * s.done * nat[(size_t)s.axis];
      };
      if (lu.b >= 0) {
        put(lu.a, o / st[(size_t)lu.b].nout);
        put(lu.b, o % st[(size_t)lu.b].nout);
      } else {
        put(lu.a, o);
      }
      for (int k = ns - 1; k >= 0; --k) {
        if (k == lu.a || k == lu.b) continue;
        put(k, r % cur[(size_t)k]);
        r /= cur[(size_t)k];
      }
      out.kmap[(size_t)(c * bL.cells + cell)] = (int32_t)at;
    }
  out.threads = bNT;
  out.per_cu = bfit;
  out.lds = (size_t)(bB * bL.w_size * 8 + (int64_t)P.n_tw * 8 + bG * bL.cells * 4 + (int64_t)P.n_tab * 2);
  return true;
}

// Groups: axes are taken from the outermost on while a group's cells leave room for several columns (at most
// kGroupCells; a whole channel of at most kChannelCells cells is one group).  Columns per work-group: as many as fit
// kTileCells cells, fewer where there would be under two work-groups a CU.
std::vector<InvGroup> plan_inverse(int d, const int* n, const int* m, int64_t channels, int64_t inner,
                                   const int* tw_off) {
  constexpr int64_t kGroupCells = 1024, kChannelCells = 4096, kTileCells = 4096, kLineCells = int64_t(1) << 25;
  std::vector<InvGroup> out;
  std::vector<int> chain;
  int64_t all = inner;
  bool whole = inner == 1;
  for (int k = 0; k < d; ++k) {
    all *= m[k];
    whole = whole && plain_chain(m[k], chain, kInvPlain);
  }
  whole = whole && all <= kChannelCells;
  int64_t outer = channels, rest = all;
  size_t tab_off = 0;
  for (int k = 0; k < d;) {
    InvGroup g;
    g.axis0 = k;
    g.tab_off = tab_off;
    if (!plain_chain(m[k], chain, kInvPlain) || m[k] > kTileCells) {
      g.axes = 1;
      g.direct = true;
      rest /= m[k];
      outer *= 2 * n[k] - 1;
      ++k;
      out.push_back(g);
      continue;
    }
    // An array beyond the last-level cache (256 MB) goes through HBM with every pass: threads that transform a line
    // each in registers run at its rate, a group at half of it, so they win where their reads are whole cache lines.
    if (inner == 1 && !whole && channels * all >= kLineCells && rest / m[k] >= 64 && (m[k] == 8 || m[k] == 16 || m[k] == 32)) {
      g.axes = 1;
      g.line = true;
      rest /= m[k];
      outer *= 2 * n[k] - 1;
      ++k;
      out.push_back(g);
      continue;
    }
    int64_t Mg = 1, Ng = 1;
    std::vector<Stage> st;
    while (k < d && plain_chain(m[k], chain, kInvPlain) && (g.axes == 0 || whole || Mg * m[k] <= kGroupCells)) {
      int done = 1, rem = m[k];
      std::vector<Stage> one;
      for (int f : chain) {
        rem /= f;
        one.push_back({k, f, f, false, done, rem});
        done *= f;
      }
      if ((int)(st.size() + one.size()) > kInvMaxPass - 1) break;
      st.insert(st.end(), one.begin(), one.end());
      Mg *= m[k];
      Ng *= 2 * n[k] - 1;
      rest /= m[k];
      ++g.axes;
      ++k;
    }
    InvP& P = g.P;
    P.Mg = (int32_t)Mg;
    P.Ng = (int32_t)Ng;
    P.col_fast = rest > 1 ? 1 : 0;
    const int64_t columns = outer * rest;
    int cols = 1, lg = 0;
    // (neighbouring columns share 64-byte runs of HBM: at least four where they are interleaved)
    while (cols * 2 * Mg <= kTileCells && cols < 64 && (columns / (2 * cols) >= 512 || (P.col_fast && cols < 4))) {
      cols *= 2;
      ++lg;
    }
    P.cols = cols;
    P.lg_cols = lg;
    if (!P.col_fast && g.axes > 1 && (st.size() < 2 || st[1].axis != st[0].axis) && m[g.axis0] > 2) {
      // whole columns: the last pass' lines must be neighbouring lags of the inner axes, so the first axis gets two
      // stages, one to read with and one to write with
      const int mm = m[g.axis0];
      int f = 2;
      for (int v : kInvPlain)
        if (mm % v == 0 && v * v <= mm && has(kInvPlain, mm / v)) f = v;
      st.insert(st.begin(), st[0]);
      st[0] = {g.axis0, f, f, false, 1, mm / f};
      st[1] = {g.axis0, mm / f, mm / f, false, f, 1};
    }
    const int ns = (int)st.size();
    std::vector<int> stride((size_t)ns);
    // strides in slots of one cell (col_fast: of all columns' values of a cell).  An LDS access serves 16 lanes of
    // 16 bytes at a time: lanes run over the innermost digit, or, in the innermost stage's pass, over the next one,
    // whose stride is made odd.
    const int64_t slot = P.col_fast ? cols : 1;
    int64_t s = 1;
    for (int i = ns - 1; i >= 0; --i) {
      stride[(size_t)i] = (int)(s * slot);
      s *= st[(size_t)i].nout;
      if (i == ns - 1 && slot < 16) s |= 1;
    }
    // (16 neighbouring lanes are in different columns only where a pass has fewer than 16 lines a column)
    if (!P.col_fast && Mg < 16 * 8) s |= 1;
    P.col_stride = P.col_fast ? 1 : (int32_t)s;
    g.lds = (size_t)(P.col_fast ? s * slot : s * cols) * 16;
    P.n_pass = ns;
    // pass order: stage 0 first, the first axis' last stage last
    int own = 1;
    while (own < ns && st[(size_t)own].axis == st[0].axis) ++own;
    std::vector<int> order;
    for (int i = 0; i < own - 1; ++i) order.push_back(i);
    if (own == 1 && ns > 1) {
      // the first axis has one stage, which reads HBM: another axis' last stage writes
      order.push_back(0);
      own = 0;
    }
    for (int i = std::max(own, 1); i < ns; ++i) order.push_back(i);
    if (own > 0) order.push_back(own - 1);
    for (int at = 0; at < ns; ++at) {
      const int i = order[(size_t)at];
      InvPass& p = P.pass[at];
      p.f = st[(size_t)i].nin;
      p.stride = stride[(size_t)i];
      p.lines = (int32_t)(Mg / p.f);
      p.magic = magic_of(p.lines);
      p.tab = (int32_t)g.tab.size();
      p.tj = -1;
      p.tw = tw_off[st[(size_t)i].axis];
      std::vector<uint16_t> steps;
      // whole columns of one axis: the last pass takes its lines in the order of their lags
      const bool by_lag = at + 1 == ns && ns > 1 && g.axes == 1 && !P.col_fast;
      for (int64_t line = 0; line < p.lines; ++line) {
        int64_t r = line, off = 0, j = 0;
        for (int q0 = ns - 1; q0 >= 0; --q0) {
          const int q = by_lag ? ns - 1 - q0 : q0;
          if (q == i) continue;
          const int64_t digit = r % st[(size_t)q].nin;
          r /= st[(size_t)q].nin;
          off += digit * stride[(size_t)q];
          if (st[(size_t)q].axis == st[(size_t)i].axis && q > i) j += digit * st[(size_t)q].rem;
        }
        g.tab.push_back((uint16_t)off);
        steps.push_back((uint16_t)(j * st[(size_t)i].done));
      }
      if (st[(size_t)i].rem > 1) {
        p.tj = (int32_t)g.tab.size();
        g.tab.insert(g.tab.end(), steps.begin(), steps.end());
      }
    }
    // value k of each line of the last pass -> its lag (row-major over the group's axes, Delta_k + n_k - 1)
    P.out_tab = (int32_t)g.tab.size();
    const int li = order.back(), lf = st[(size_t)li].nin;
    std::vector<int> digit((size_t)ns);
    for (int k = 0; k < lf; ++k)
      for (int64_t line = 0; line < Mg / lf; ++line) {
        int64_t r = line;
        for (int q0 = ns - 1; q0 >= 0; --q0) {
          const int q = ns > 1 && g.axes == 1 && !P.col_fast ? ns - 1 - q0 : q0;
          if (q == li) {
            digit[(size_t)q] = k;
            continue;
          }
          digit[(size_t)q] = (int)(r % st[(size_t)q].nin);
          r /= st[(size_t)q].nin;
        }
        int64_t o = 0;
        bool valid = true;
        for (int a = g.axis0; a < g.axis0 + g.axes; ++a) {
          int delta = 0;
          for (int q = 0; q < ns; ++q)
            if (st[(size_t)q].axis == a) delta += digit[(size_t)q] * st[(size_t)q].done;
          if (delta == n[a]) valid = false;
          if (delta >= n[a]) delta -= m[a];
          o = o * (2 * n[a] - 1) + delta + n[a] - 1;
        }
        g.tab.push_back(valid ? (uint16_t)o : (uint16_t)kInvNoLag);
      }
    tab_off += g.tab.size();
    outer *= Ng;
    out.push_back(std::move(g));
  }
  return out;
}

}  // namespace omni
