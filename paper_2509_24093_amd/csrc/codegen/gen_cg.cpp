// Build-time generator of the frequency-domain CG contraction bodies.
//
// For every L_max in [0, LGEN] it emits a specialisation CgBody<L>::run that
// evaluates, fully unrolled with compile-time register indices, the sparse
// complex-basis contraction of cg_table.h (selection rule M = m1 + m2,
// arXiv 2509.24093 §4.3) for one frequency of one channel:
//
//   w[J,M] += coef * (imag ? i : 1) * qa[l1,m1] * ka[l2,m2]
//
// Work is organised in phases mu = |M| so that only the accumulators of one
// phase are live.  Inside a phase the blocks (m1, M - m1) and (M - m1, m1)
// are taken together: by the swap symmetry of the CG coefficients,
// <l2 m2 l1 m1|J M> = (-1)^(l1+l2-J) <l1 m1 l2 m2|J M>, the two terms of an
// unordered pair of components a = (l1,m1), b = (l2,m2) share one
// coefficient, and their sum is
//   coef * (x + sigma y),  x = qa[a] ka[b],  y = qa[b] ka[a],  sigma = (-1)^(l1+l2-J).
// For every row l1 of such a block the generator takes whichever form needs
// fewer operations:
//   pair form:    per l2, s = x + y and/or d = x - y (8 ops for one of them,
//                 12 for both), then 2 FMAs per J;
//   split form:   the x terms and the y terms separately, each as
//     product form: p = qa * ka once per l2 (4 ops), then 2 FMAs per J;
//     key form:     t_J = sum_l2 coef * (the l2 factor) (2 FMAs per term),
//                   then w[J] += (the l1 factor) * t_J (4 FMAs per J).
// At L_max = 6 this is 18.8k operations per point against 21.6k without the
// pairing (23.4k for the plain product form).
// Every output component is handed to st(k, value) as soon as it is final;
// st.end_phase(mu) follows the last component of phase mu.
// Coefficients are emitted as float literals (the double value rounded to
// nearest float).  The one subtraction of every complex product goes through
// fnma() (c - a*b as a single v_fma_f32 with a negated operand, see
// cg_common.h): written as ordinary C++, the compiler turns -(a*b) into
// a*(-b) and keeps a negated copy of every input alive for the whole kernel.
//
// Further bodies per L: CgMirrorBody<L>, the lane-pair form of the same
// contraction (emit_mirror_body); CgPathSplitBody<L>, which keeps the paths
// apart for the channel-mixing kernel, in steps (emit_path_split_body); and
// CgRealBody<L>, the token-wise product of real components of the value tensor
// product (emit_real_body).
//
// Usage: gen_cg <output-dir> <LGEN>   (writes cg_body_L<L>.inc and cg_lgen.h)
#include <algorithm>
#include <array>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "../cg_table.h"

using namespace cgconv;

namespace {

int L_cur = 0;  // L_max of the body being emitted

std::string lit(double c) {
  char buf[64];
  std::snprintf(buf, sizeof buf, "%.9ef", (double)(float)c);
  return buf;
}

std::string acc_name(int M, int J) {
  char buf[32];
  std::snprintf(buf, sizeof buf, "a%c%d", M >= 0 ? 'p' : 'm', J);
  return buf;
}

struct Emitter {
  FILE* f;
  std::set<std::string> inited;
  long ops = 0;

  // acc += coef * (imag ? i : 1) * (pr + i pi)
  void acc_add_scaled(const std::string& a, double c, bool imag, const std::string& pr, const std::string& pi) {
    const bool first = !inited.count(a);
    inited.insert(a);
    std::string re_src = imag ? pi : pr, im_src = imag ? pr : pi;
    double re_c = imag ? -c : c, im_c = c;
    if (first) {
      std::fprintf(f, "      %s.x = %s * %s; %s.y = %s * %s;\n", a.c_str(), lit(re_c).c_str(), re_src.c_str(),
                   a.c_str(), lit(im_c).c_str(), im_src.c_str());
    } else {
      std::fprintf(f, "      %s.x = fmaf(%s, %s, %s.x); %s.y = fmaf(%s, %s, %s.y);\n", a.c_str(),
                   lit(re_c).c_str(), re_src.c_str(), a.c_str(), a.c_str(), lit(im_c).c_str(), im_src.c_str(),
                   a.c_str());
    }
    ops += 2;
  }

  // acc += q * t  (complex multiply-accumulate)
  void acc_cmac(const std::string& a, const std::string& q) {
    const bool first = !inited.count(a);
    inited.insert(a);
    if (first) {
      std::fprintf(f, "      %s.x = fnma(%s.y, ti, %s.x * tr); %s.y = fmaf(%s.y, tr, %s.x * ti);\n", a.c_str(),
                   q.c_str(), q.c_str(), a.c_str(), q.c_str(), q.c_str());
    } else {
      std::fprintf(f,
                   "      %s.x = fmaf(%s.x, tr, %s.x); %s.x = fnma(%s.y, ti, %s.x);"
                   " %s.y = fmaf(%s.x, ti, %s.y); %s.y = fmaf(%s.y, tr, %s.y);\n",
                   a.c_str(), q.c_str(), a.c_str(), a.c_str(), q.c_str(), a.c_str(), a.c_str(), q.c_str(),
                   a.c_str(), a.c_str(), q.c_str(), a.c_str());
    }
    ops += 4;
  }
};

// Terms of one ordered component pair, by J.
using TermMap = std::map<std::array<int, 4>, std::vector<Term>>;  // (l1, m1, l2, m2) -> terms

std::string qname(int l, int m) { return "qa[" + std::to_string(comp(l, m)) + "]"; }
std::string kname(int l, int m) { return "ka[" + std::to_string(comp(l, m)) + "]"; }

// Cheaper of product and key form for one half (fixed factor f1 of the l1
// side, varying factor of the l2 side) with the given (l2 -> terms) lists.
long half_cost(const std::vector<std::pair<int, const std::vector<Term>*>>& rows) {
  long nnz = 0;
  std::set<int> Js;
  for (auto& r : rows) {
    nnz += (long)r.second->size();
    for (const Term& t : *r.second) Js.insert(t.J);
  }
  return std::min(4L * (long)rows.size() + 2 * nnz, 2 * nnz + 4L * (long)Js.size());
}

// Emits one half: sum over l2 of coef * fixed * var(l2), grouped by J.
// fixed/var are the register names of the two factors of every term.
void emit_half(Emitter& e, int M, const std::string& fixed,
               const std::vector<std::pair<std::string, const std::vector<Term>*>>& rows) {
  FILE* f = e.f;
  long nnz = 0;
  std::set<int> Js;
  for (auto& r : rows) {
    nnz += (long)r.second->size();
    for (const Term& t : *r.second) Js.insert(t.J);
  }
  if (4L * (long)rows.size() + 2 * nnz <= 2 * nnz + 4L * (long)Js.size()) {
    for (auto& r : rows) {  // product form
      const std::string& v = r.first;
      std::fprintf(f, "      { const float pr = fnma(%s.y, %s.y, %s.x * %s.x);", fixed.c_str(), v.c_str(),
                   fixed.c_str(), v.c_str());
      std::fprintf(f, " const float pi = fmaf(%s.y, %s.x, %s.x * %s.y);\n", fixed.c_str(), v.c_str(), fixed.c_str(),
                   v.c_str());
      e.ops += 4;
      for (const Term& t : *r.second) e.acc_add_scaled(acc_name(M, t.J), t.coef, t.imag, "pr", "pi");
      std::fprintf(f, "      }\n");
    }
    return;
  }
  for (int J : Js) {  // key form
    std::fprintf(f, "      { float tr, ti;\n");
    bool first = true;
    for (auto& r : rows)
      for (const Term& t : *r.second) {
        if (t.J != J) continue;
        const std::string& v = r.first;
        // t += coef * (imag ? i : 1) * v
        const std::string rs = t.imag ? v + ".y" : v + ".x";
        const std::string is = t.imag ? v + ".x" : v + ".y";
        const double rc = t.imag ? -t.coef : t.coef;
        if (first)
          std::fprintf(f, "      tr = %s * %s; ti = %s * %s;\n", lit(rc).c_str(), rs.c_str(), lit(t.coef).c_str(),
                       is.c_str());
        else
          std::fprintf(f, "      tr = fmaf(%s, %s, tr); ti = fmaf(%s, %s, ti);\n", lit(rc).c_str(), rs.c_str(),
                       lit(t.coef).c_str(), is.c_str());
        first = false;
        e.ops += 2;
      }
    e.acc_cmac(acc_name(M, J), fixed);
    std::fprintf(f, "      }\n");
  }
}

// Register names of a row's operands and the weight of its pairs: the fixed
// component a = (l1, m1) of both inputs, the varying component b = (l2, m2),
// and a factor on the coefficients of pair (l1, l2) (0: the pair is left out).
struct RowOperands {
  std::string qa, ka;
  std::string (*qb)(int l, int m);
  std::string (*kb)(int l, int m);
  double (*weight)(int l1, int l2);
};

std::vector<Term> weighted(const std::vector<Term>& t, double w) {
  std::vector<Term> r = t;
  for (Term& x : r) x.coef *= w;
  return r;
}

// Row l1 of the merged block (m1, m2 = M - m1), m1 <= m2: every pair
// a = (l1, m1), b = (l2, m2) with l2 > l1 if m1 == m2 (the diagonal a == b
// has a single term per J and takes the product form).
void emit_row(Emitter& e, const TermMap& terms_of, int M, int l1, int m1, int m2, const RowOperands& op) {
  FILE* f = e.f;
  static const std::vector<Term> none;
  auto get = [&](int a, int b, int c, int d) -> const std::vector<Term>& {
    auto it = terms_of.find({a, b, c, d});
    return it == terms_of.end() ? none : it->second;
  };
  if (m1 == m2 && op.weight(l1, l1) != 0.0) {
    const std::vector<Term> dg = weighted(get(l1, m1, l1, m1), op.weight(l1, l1));
    if (!dg.empty()) emit_half(e, M, op.qa, {{op.kb(l1, m1), &dg}});
  }
  // off-diagonal pairs of this row
  struct Pair {
    int l2;
    std::vector<Term> x;  // terms of (a, b): qa[a] ka[b]
    std::vector<Term> y;  // terms of (b, a): qa[b] ka[a]
  };
  std::vector<Pair> pairs;
  for (int l2 = std::abs(m2); l2 <= L_cur; ++l2) {
    const double w = op.weight(l1, l2);
    if ((m1 == m2 && l2 <= l1) || w == 0.0) continue;
    const std::vector<Term> x = weighted(get(l1, m1, l2, m2), w);
    const std::vector<Term> y = weighted(get(l2, m2, l1, m1), w);
    if (x.size() != y.size()) {
      std::fprintf(stderr, "gen_cg: swap partner missing (%d %d %d %d)\n", l1, m1, l2, m2);
      std::exit(1);
    }
    if (!x.empty()) pairs.push_back({l2, x, y});
  }
  if (pairs.empty()) return;
  long pair_cost = 0;
  std::vector<std::pair<int, const std::vector<Term>*>> xs, ys;
  for (const Pair& p : pairs) {
    bool ev = false, od = false;
    for (const Term& t : p.x) ((l1 + p.l2 - t.J) % 2 == 0 ? ev : od) = true;
    pair_cost += (ev && od ? 12 : 8) + 2 * (long)p.x.size();
    xs.push_back({p.l2, &p.x});
    ys.push_back({p.l2, &p.y});
  }
  if (half_cost(xs) + half_cost(ys) < pair_cost) {
    std::vector<std::pair<std::string, const std::vector<Term>*>> xr, yr;
    for (const Pair& p : pairs) {
      xr.push_back({op.kb(p.l2, m2), &p.x});
      yr.push_back({op.qb(p.l2, m2), &p.y});
    }
    emit_half(e, M, op.qa, xr);  // qa[a] * ka[b]
    emit_half(e, M, op.ka, yr);  // ka[a] * qa[b]
    return;
  }
  const std::string &qa_ = op.qa, &ka_ = op.ka;
  for (const Pair& p : pairs) {
    const std::string qb = op.qb(p.l2, m2), kb = op.kb(p.l2, m2);
    bool ev = false, od = false;
    for (const Term& t : p.x) {
      // the two terms share the coefficient up to the swap sign
      const Term* u = nullptr;
      for (const Term& w : p.y)
        if (w.J == t.J) u = &w;
      const double sigma = ((l1 + p.l2 - t.J) % 2 == 0) ? 1.0 : -1.0;
      if (!u || u->imag != t.imag || std::fabs(u->coef - sigma * t.coef) > 1e-12 * std::fabs(t.coef) + 1e-15) {
        std::fprintf(stderr, "gen_cg: swap symmetry violated (%d %d %d %d J=%d)\n", l1, m1, p.l2, m2, t.J);
        std::exit(1);
      }
      (sigma > 0 ? ev : od) = true;
    }
    std::fprintf(f, "      {\n");
    if (ev && od) {
      std::fprintf(f, "      const float xr = fnma(%s.y, %s.y, %s.x * %s.x), xi = fmaf(%s.y, %s.x, %s.x * %s.y);\n",
                   qa_.c_str(), kb.c_str(), qa_.c_str(), kb.c_str(), qa_.c_str(), kb.c_str(), qa_.c_str(), kb.c_str());
      std::fprintf(f, "      const float yr = fnma(%s.y, %s.y, %s.x * %s.x), yi = fmaf(%s.y, %s.x, %s.x * %s.y);\n",
                   qb.c_str(), ka_.c_str(), qb.c_str(), ka_.c_str(), qb.c_str(), ka_.c_str(), qb.c_str(), ka_.c_str());
      std::fprintf(f, "      const float sr = xr + yr, si = xi + yi, dr = xr - yr, di = xi - yi;\n");
      e.ops += 12;
    } else if (ev) {  // s = x + y
      std::fprintf(f, "      const float sr = fmaf(%s.x, %s.x, fnma(%s.y, %s.y, fnma(%s.y, %s.y, %s.x * %s.x)));\n",
                   qb.c_str(), ka_.c_str(), qb.c_str(), ka_.c_str(), qa_.c_str(), kb.c_str(), qa_.c_str(), kb.c_str());
      std::fprintf(f, "      const float si = fmaf(%s.x, %s.y, fmaf(%s.y, %s.x, fmaf(%s.y, %s.x, %s.x * %s.y)));\n",
                   qb.c_str(), ka_.c_str(), qb.c_str(), ka_.c_str(), qa_.c_str(), kb.c_str(), qa_.c_str(), kb.c_str());
      e.ops += 8;
    } else {  // d = x - y
      std::fprintf(f, "      const float dr = fnma(%s.x, %s.x, fmaf(%s.y, %s.y, fnma(%s.y, %s.y, %s.x * %s.x)));\n",
                   qb.c_str(), ka_.c_str(), qb.c_str(), ka_.c_str(), qa_.c_str(), kb.c_str(), qa_.c_str(), kb.c_str());
      std::fprintf(f, "      const float di = fnma(%s.x, %s.y, fnma(%s.y, %s.x, fmaf(%s.y, %s.x, %s.x * %s.y)));\n",
                   qb.c_str(), ka_.c_str(), qb.c_str(), ka_.c_str(), qa_.c_str(), kb.c_str(), qa_.c_str(), kb.c_str());
      e.ops += 8;
    }
    for (const Term& t : p.x) {
      const bool even = (l1 + p.l2 - t.J) % 2 == 0;
      e.acc_add_scaled(acc_name(M, t.J), t.coef, t.imag, even ? "sr" : "dr", even ? "si" : "di");
    }
    std::fprintf(f, "      }\n");
  }
}

void emit_body(FILE* f, int L, long* ops_out) {
  const int K = (L + 1) * (L + 1);
  std::vector<Term> terms = contraction_terms(L);
  TermMap terms_of;
  for (const Term& t : terms) terms_of[{t.l1, t.m1, t.l2, t.m2}].push_back(t);
  L_cur = L;

  Emitter e{f, {}, 0};
  std::fprintf(f, "template <>\nstruct CgBody<%d> {\n  static constexpr int K = %d;\n", L, K);
  std::fprintf(f, "  template <class Store>\n");
  std::fprintf(f, "  static __device__ __forceinline__ void run(const float2 (&qa)[%d], const float2 (&ka)[%d], Store& st) {\n", K,
               K);
  for (int mu = 0; mu <= L; ++mu) {
    std::fprintf(f, "    {  // phase |M| = %d\n", mu);
    std::vector<int> Ms = mu == 0 ? std::vector<int>{0} : std::vector<int>{mu, -mu};
    for (int M : Ms)
      for (int J = mu; J <= L; ++J) std::fprintf(f, "      float2 %s;\n", acc_name(M, J).c_str());
    for (int M : Ms) {
      for (int m1 = -L; m1 <= L; ++m1) {
        const int m2 = M - m1;
        if (m2 < -L || m2 > L || m1 > m2) continue;
        std::fprintf(f, "      // blocks m1=%d m2=%d and swapped\n", m1, m2);
        for (int l1 = std::abs(m1); l1 <= L; ++l1)
          emit_row(e, terms_of, M, l1, m1, m2,
                   {qname(l1, m1), kname(l1, m1), qname, kname, [](int, int) { return 1.0; }});
      }
    }
    // output transform and stores
    for (int J = mu; J <= L; ++J) {
      for (int M : Ms)
        if (!e.inited.count(acc_name(M, J))) std::fprintf(f, "      %s = make_float2(0.f, 0.f);\n", acc_name(M, J).c_str());
      if (mu == 0) {
        std::fprintf(f, "      st(%d, %s);\n", comp(J, 0), acc_name(0, J).c_str());
      } else {
        const std::string p = acc_name(mu, J), m = acc_name(-mu, J);
        std::fprintf(f, "      st(%d, make_float2(%s.x + %s.x, %s.y + %s.y));\n", comp(J, mu), m.c_str(),
                     p.c_str(), m.c_str(), p.c_str());
        std::fprintf(f, "      st(%d, make_float2(%s.y - %s.y, %s.x - %s.x));\n", comp(J, -mu), m.c_str(),
                     p.c_str(), p.c_str(), m.c_str());
        e.ops += 4;
      }
    }
    e.inited.clear();
    std::fprintf(f, "      st.end_phase(%d);\n", mu);
    std::fprintf(f, "    }\n");
  }
  std::fprintf(f, "  }\n");
  std::fprintf(f, "  static constexpr long kOps = %ld;  // VALU ops of the contraction per point\n", e.ops);
  std::fprintf(f, "  static constexpr long kNnz = %ld;  // complex-basis non-zeros\n};\n\n", (long)terms.size());
  *ops_out = e.ops;
}

}  // namespace

// Lane-pair per-path body for the channel-mixing kernel
// (CgPathSplitBody<L>): one point per pair of adjacent lanes (even lane
// x = qa, odd lane x[(l,m)] = (-1)^l ka[(l,m)]), the products of every path
// kept apart.  The work is cut into pair steps over
// unordered degree pairs {l1 <= l2}, each with a run Ja..Jb of output
// degrees (at most kPairHalfSlots outputs (J, M) and kPairHalfPaths degrees).
// In a step with l1 < l2 every product x[(l1,m1)] * partner(x[(l2,m2)]),
// taken with the coefficient (-1)^l2 c((l1,m1),(l2,m2),J), is a term of path
// (l1, l2, J) in the even lane and (-1)^J times a term of path (l2, l1, J)
// in the odd lane (swap symmetry c(q,o,J) = (-1)^(l1+l2-J) c(o,q,J), checked
// for every pair): the two lanes evaluate the two ordered paths at once.  In
// a step with l1 == l2 both ordered terms of an unordered pair belong to the
// same path: the lanes take one each (diagonal pairs half
// the coefficient) and combine, w = acc + (-1)^J partner(acc).  Either way
// the odd lane's value is (-1)^J times its path value; st.put<B, S0>(slot,
// value, odd_J) corrects the sign and stages the value at slot (odd lanes
// at slot + S0, the second path's slots, when l1 < l2; the same slot as the
// even lane, with the same value, when l1 == l2).  Slots follow J ascending,
// then M = -J..J, zeros included; st.end_step() follows each step.
// CgPathSplitBody<L>::consume<W> is, for matrix-core wave W, the matching
// sequence of st.step<W, B, JA, JB, S0, TWO, P0aN, P0bN, NPN>() calls (TWO: the step has
// the second path set; P0aN, P0bN, NPN: the first paths of the next step's
// two path sets and their length, NPN = 0 after the last step), preceded by
// st.first<P0a, P0b, NP>() (P0b = -1 without a second set).
constexpr int kPairHalfSlots = 13;
constexpr int kPairHalfPaths = 2;

struct PairStep {
  int l1, l2, Ja, Jb, P0a, P0b;  // P0b = -1 when l1 == l2
};

int path_index(int L, int l1, int l2, int J) {
  int path = 0;
  for (int a = 0; a <= L; ++a)
    for (int b = 0; b <= L; ++b) {
      const int Jmin = std::abs(a - b), Jmax = std::min(a + b, L);
      if (Jmin > Jmax) continue;
      if (a == l1 && b == l2) return path + (J - Jmin);
      path += Jmax - Jmin + 1;
    }
  std::fprintf(stderr, "gen_cg: no path (%d %d %d)\n", l1, l2, J);
  std::exit(1);
}

std::vector<PairStep> pair_steps(int L) {
  std::vector<PairStep> steps;
  for (int l1 = 0; l1 <= L; ++l1)
    for (int l2 = l1; l2 <= L; ++l2) {
      const int Jmin = l2 - l1, Jmax = std::min(l1 + l2, L);
      if (Jmin > Jmax) continue;
      // a step with l1 == l2 stages one path set and may take both halves' room
      const int slot_cap = l1 == l2 ? 2 * kPairHalfSlots : kPairHalfSlots;
      const int path_cap = l1 == l2 ? 2 * kPairHalfPaths : kPairHalfPaths;
      int J = Jmax;
      while (J >= Jmin) {
        const int Jb = J;
        int slots = 2 * J + 1, n = 1;
        --J;
        while (J >= Jmin && n < path_cap && slots + 2 * J + 1 <= slot_cap) {
          slots += 2 * J-- + 1;
          ++n;
        }
        const int Ja = J + 1;
        steps.push_back({l1, l2, Ja, Jb, path_index(L, l1, l2, Ja), l1 == l2 ? -1 : path_index(L, l2, l1, Ja)});
      }
    }
  return steps;
}

void emit_path_split_body(FILE* f, int L, long* ops_out) {
  const int K = (L + 1) * (L + 1);
  std::vector<Term> terms = contraction_terms(L);
  TermMap terms_of;
  for (const Term& t : terms) terms_of[{t.l1, t.m1, t.l2, t.m2}].push_back(t);
  const std::vector<PairStep> steps = pair_steps(L);
  Emitter e{f, {}, 0};
  int max_slots = 0, max_paths = 0;
  auto sname = [](int J, int M) { return "s" + std::to_string(J) + "_" + std::to_string(M + J); };
  std::fprintf(f, "template <>\nstruct CgPathSplitBody<%d> {\n  static constexpr int K = %d;\n", L, K);
  std::fprintf(f, "  template <class Store>\n");
  std::fprintf(f, "  static __device__ __forceinline__ void produce(const float2 (&x)[%d], Store& st) {\n", K);
  for (size_t si = 0; si < steps.size(); ++si) {
    const PairStep& sp = steps[si];
    const int B = (int)(si & 1);
    const bool two = sp.l1 != sp.l2;
    int S0 = 0;
    for (int J = sp.Ja; J <= sp.Jb; ++J) S0 += 2 * J + 1;
    max_slots = std::max(max_slots, two ? 2 * S0 : S0);
    max_paths = std::max(max_paths, (two ? 2 : 1) * (sp.Jb - sp.Ja + 1));
    std::fprintf(f, "    {  // step %zu: degrees %d, %d, J = %d..%d\n", si, sp.l1, sp.l2, sp.Ja, sp.Jb);
    for (int J = sp.Ja; J <= sp.Jb; ++J)
      for (int M = -J; M <= J; ++M) std::fprintf(f, "      float2 %s;\n", sname(J, M).c_str());
    for (int m2 = -sp.l2; m2 <= sp.l2; ++m2) {
      const int q = comp(sp.l2, m2);
      std::vector<std::pair<int, const std::vector<Term>*>> prods;  // (m1, terms)
      for (int m1 = -sp.l1; m1 <= sp.l1; ++m1) {
        if (!two && m1 > m2) continue;  // unordered pairs o <= q
        auto it = terms_of.find({sp.l1, m1, sp.l2, m2});
        if (it == terms_of.end()) continue;
        bool any = false;
        for (const Term& t : it->second) any |= t.J >= sp.Ja && t.J <= sp.Jb;
        if (!any) continue;
        // swap symmetry of the pair, which both lane roles rely on
        auto sw = terms_of.find({sp.l2, m2, sp.l1, m1});
        if (sw == terms_of.end() || sw->second.size() != it->second.size()) {
          std::fprintf(stderr, "gen_cg: swap partner missing (per-path split body)\n");
          std::exit(1);
        }
        for (const Term& t : it->second) {
          const Term* u = nullptr;
          for (const Term& w : sw->second)
            if (w.J == t.J) u = &w;
          const double sigma = ((t.l1 + t.l2 - t.J) % 2 == 0) ? 1.0 : -1.0;
          if (!u || u->imag != t.imag || std::fabs(u->coef - sigma * t.coef) > 1e-12 * std::fabs(t.coef) + 1e-15) {
            std::fprintf(stderr, "gen_cg: swap symmetry violated (per-path split body)\n");
            std::exit(1);
          }
          if (!two && m1 == m2 && t.J % 2 != 0) {
            std::fprintf(stderr, "gen_cg: diagonal term of odd J (per-path split body)\n");
            std::exit(1);
          }
        }
        prods.push_back({m1, &it->second});
      }
      if (prods.empty()) continue;
      std::fprintf(f, "      { const float2 pq = lane_partner2(x[%d]);\n", q);
      e.ops += 2;
      for (auto& pr : prods) {
        const int m1 = pr.first, o = comp(sp.l1, m1);
        std::fprintf(f, "      { const float pr = fnma(x[%d].y, pq.y, x[%d].x * pq.x);", o, o);
        std::fprintf(f, " const float pi = fmaf(x[%d].y, pq.x, x[%d].x * pq.y);\n", o, o);
        e.ops += 4;
        const double scale = ((sp.l2 % 2) ? -1.0 : 1.0) * (!two && m1 == m2 ? 0.5 : 1.0);
        for (const Term& t : *pr.second)
          if (t.J >= sp.Ja && t.J <= sp.Jb) e.acc_add_scaled(sname(t.J, t.M), scale * t.coef, t.imag, "pr", "pi");
        std::fprintf(f, "      }\n");
      }
      std::fprintf(f, "      }\n");
      std::fprintf(f, "      __builtin_amdgcn_sched_barrier(0);\n");
    }
    int base = 0;
    for (int J = sp.Ja; J <= sp.Jb; ++J) {
      for (int M = -J; M <= J; ++M) {
        const std::string a = sname(J, M);
        if (!e.inited.count(a)) {
          std::fprintf(f, "      %s = make_float2(0.f, 0.f);\n", a.c_str());
        } else if (!two) {
          const char* op = J % 2 ? "-" : "+";
          std::fprintf(f, "      %s.x = %s.x %s lane_partner(%s.x); %s.y = %s.y %s lane_partner(%s.y);\n", a.c_str(),
                       a.c_str(), op, a.c_str(), a.c_str(), a.c_str(), op, a.c_str());
          e.ops += 4;
        }
        std::fprintf(f, "      st.template put<%d, %d>(%d, %s, %s);\n", B, two ? S0 : 0, base + M + J, a.c_str(),
                     J % 2 ? "true" : "false");
      }
      base += 2 * J + 1;
    }
    e.inited.clear();
    std::fprintf(f, "      st.end_step();\n    }\n");
  }
  std::fprintf(f, "  }\n");
  std::fprintf(f, "  template <int W, class Store>\n  static __device__ __forceinline__ void consume(Store& st) {\n");
  std::fprintf(f, "    st.template first<%d, %d, %d>();\n", steps[0].P0a, steps[0].P0b, steps[0].Jb - steps[0].Ja + 1);
  for (size_t si = 0; si < steps.size(); ++si) {
    const PairStep& sp = steps[si];
    int S0 = 0;
    for (int J = sp.Ja; J <= sp.Jb; ++J) S0 += 2 * J + 1;
    const bool last = si + 1 == steps.size();
    const PairStep* nx = last ? nullptr : &steps[si + 1];
    std::fprintf(f, "    st.template step<W, %d, %d, %d, %d, %s, %d, %d, %d>();\n", (int)(si & 1), sp.Ja, sp.Jb, S0,
                 sp.l1 != sp.l2 ? "true" : "false", nx ? nx->P0a : 0, nx ? nx->P0b : -1,
                 nx ? nx->Jb - nx->Ja + 1 : 0);
  }
  std::fprintf(f, "  }\n");
  std::fprintf(f, "  static constexpr int kSteps = %d;\n", (int)steps.size());
  std::fprintf(f, "  static constexpr int kMaxStepSlots = %d;  // most staged outputs of one step (both paths)\n",
               max_slots);
  std::fprintf(f, "  static constexpr int kMaxStepPaths = %d;  // most paths of one step\n", max_paths);
  std::fprintf(f, "  static constexpr long kOps = %ld;  // VALU ops of the products per lane (two lanes per point)\n};\n\n",
               e.ops);
  *ops_out = e.ops;
}

// Mirror lane-pair body (CgMirrorBody<L>::run(q, k, st)): one point per pair
// of adjacent lanes, which share the contraction by the sign of M.  The
// coefficients obey c(l1 -m1, l2 -m2, J) = (-1)^(l1+l2-J) c(l1 m1, l2 m2, J)
// (checked here for every term), so the outputs w[J, -M] are the outputs
// w[J, +M] of the mirrored inputs up to signs of the degrees.  The even lane
// holds the components m >= 0 of both inputs, q[l,m] = qa[l,m], the odd lane
// the mirrored ones, q[l,m] = (-1)^l qa[l,-m] (k alike): (L+1)(L+2)/2 instead
// of (L+1)^2 components each.  Both run the same instructions for
// the phases M = mu >= 0: the even lane's sum is w[J,mu], the odd lane's
// (-1)^J w[J,-mu].  A component of m < 0 is the partner lane's value of +m
// times (-1)^l (a lane swap, once per row; the sign goes into the
// coefficients).  Of the phase mu = 0, whose pairs of components mirror into
// each other, each lane takes the pairs {(l1,-a), (l2,a)} with l1 < l2 and
// half the weight of the self-mirrored ones.  st.put(J, mu, acc) receives
// both lanes' sums (mirror_out in cg_common.h turns them into the real-basis
// outputs).  Per lane this is 1.08-1.1 times half the single-lane body's
// operations at L_max 7 and 8 (1.12 at 6, 1.21 at 4), with 2 (L+1)(L+2) input
// floats instead of 4 (L+1)^2.
int hidx(int l, int m) { return l * (l + 1) / 2 + m; }
std::string mqname(int l, int m) { return "q[" + std::to_string(hidx(l, m)) + "]"; }
std::string mkname(int l, int m) { return "k[" + std::to_string(hidx(l, m)) + "]"; }

void emit_mirror_body(FILE* f, int L, long* ops_out) {
  const int H = (L + 1) * (L + 2) / 2;
  std::vector<Term> terms = contraction_terms(L);
  TermMap terms_of;
  for (const Term& t : terms) terms_of[{t.l1, t.m1, t.l2, t.m2}].push_back(t);
  for (const Term& t : terms) {
    const double sg = ((t.l1 + t.l2 - t.J) % 2 == 0) ? 1.0 : -1.0;
    bool ok = false;
    for (const Term& u : terms_of[{t.l1, -t.m1, t.l2, -t.m2}])
      if (u.J == t.J) ok = u.imag == t.imag && std::fabs(u.coef - sg * t.coef) <= 1e-12 * std::fabs(t.coef) + 1e-15;
    if (!ok) {
      std::fprintf(stderr, "gen_cg: mirror symmetry violated (%d %d %d %d J=%d)\n", t.l1, t.m1, t.l2, t.m2, t.J);
      std::exit(1);
    }
  }
  L_cur = L;
  Emitter e{f, {}, 0};
  std::fprintf(f, "template <>\nstruct CgMirrorBody<%d> {\n  static constexpr int H = %d;\n", L, H);
  std::fprintf(f, "  // outputs M = +-MU\n  template <int MU, class Store>\n");
  std::fprintf(f, "  static __device__ __forceinline__ void phase(const float2 (&q)[%d], const float2 (&k)[%d], Store& st) {\n",
               H, H);
  std::vector<long> phase_ops;
  for (int mu = 0; mu <= L; ++mu) {
    const long ops0 = e.ops;
    std::fprintf(f, "    if constexpr (MU == %d) {\n", mu);
    for (int J = mu; J <= L; ++J) std::fprintf(f, "      float2 %s;\n", acc_name(mu, J).c_str());
    for (int m1 = mu - L; 2 * m1 <= mu; ++m1) {
      const int m2 = mu - m1;
      std::fprintf(f, "      // blocks m1=%d m2=%d and swapped\n", m1, m2);
      for (int l1 = std::abs(m1); l1 <= L; ++l1) {
        if (m1 >= 0) {
          if (mu == 0)
            emit_row(e, terms_of, mu, l1, m1, m2,
                     {mqname(l1, m1), mkname(l1, m1), mqname, mkname, [](int, int) { return 0.5; }});
          else
            emit_row(e, terms_of, mu, l1, m1, m2,
                     {mqname(l1, m1), mkname(l1, m1), mqname, mkname, [](int, int) { return 1.0; }});
          continue;
        }
        std::fprintf(f, "      { float2 fq, fk; lane_partner4(%s, %s, fq, fk);\n", mqname(l1, -m1).c_str(),
                     mkname(l1, -m1).c_str());
        e.ops += 4;
        if (mu == 0)
          emit_row(e, terms_of, mu, l1, m1, m2, {"fq", "fk", mqname, mkname, [](int a, int b) {
                                                   const double s = (a % 2) ? -1.0 : 1.0;
                                                   return b < a ? 0.0 : (b == a ? 0.5 * s : s);
                                                 }});
        else
          emit_row(e, terms_of, mu, l1, m1, m2,
                   {"fq", "fk", mqname, mkname, [](int a, int) { return (a % 2) ? -1.0 : 1.0; }});
        std::fprintf(f, "      }\n");
      }
      std::fprintf(f, "      __builtin_amdgcn_sched_barrier(0);\n");
    }
    for (int J = mu; J <= L; ++J) {
      const std::string a = acc_name(mu, J);
      if (!e.inited.count(a)) std::fprintf(f, "      %s = make_float2(0.f, 0.f);\n", a.c_str());
      std::fprintf(f, "      st.put(%d, %d, %s);\n", J, mu, a.c_str());
      e.ops += 6;
    }
    e.inited.clear();
    std::fprintf(f, "      st.end_phase(%d);\n", mu);
    std::fprintf(f, "    }\n");
    phase_ops.push_back(e.ops - ops0);
  }
  std::fprintf(f, "  }\n");
  // the phases of a bit mask (uniform over the wave)
  std::fprintf(f, "  template <class Store>\n");
  std::fprintf(f, "  static __device__ __forceinline__ void run(const float2 (&q)[%d], const float2 (&k)[%d], Store& st, unsigned phases = ~0u) {\n",
               H, H);
  for (int mu = 0; mu <= L; ++mu)
    std::fprintf(f, "    if (phases & %uu) phase<%d>(q, k, st);\n", 1u << mu, mu);
  std::fprintf(f, "  }\n");
  std::fprintf(f, "  static constexpr long kOps = %ld;  // VALU ops per lane (two lanes per point)\n", e.ops);
  std::fprintf(f, "  static constexpr int kPhaseOps[%d] = {", L + 1);
  for (int mu = 0; mu <= L; ++mu) std::fprintf(f, "%s%ld", mu ? ", " : "", phase_ops[mu]);
  std::fprintf(f, "};\n};\n\n");
  *ops_out = e.ops;
}

// Contraction of every channel pair of a head (CgPairsBody<L>::run), one
// point per wave: for 8 query channels c1 and 8 key channels c2,
//   w[J,M](c1, c2) = sum_x t[J,M,x](c2) q[x](c1),  x = (l1, m1),
//   t[J,M,x](c2) = sum_l2 coef k[l2, M - m1](c2).
// t depends on the key channel only, so its coefficients are applied once per
// key channel instead of once per pair, and the second sum is an outer
// product of t (rows) and q (columns): v_mfma_f32_4x4x1 (16 blocks), block b =
// lanes 4b .. 4b+3.  Block 2 c2 + h holds the columns c1 = 4h + (lane & 3);
// its four rows are the real and imaginary parts of t of two output degrees,
// row r = part (r & 1) of degree Ja + (r >> 1), computed by lane 4b + r from
// its own part kp of the key components.  The two blocks of a key channel
// compute t for two different x (l1 and l1 + 1) and broadcast them to each
// other (cbsz = 1).  All coefficients are real: the factor i of the terms with
// l1 + l2 + J odd is i^J i^l1 i^l2 (parities) times a sign, so kp and q carry
// i^l and the outputs i^J.  The lane-dependent coefficients (two degrees, two
// x) come from a table of 4-slot entries [entry][2 h + (r >> 1)][4].
// At L_max = 6: 2424 matrix instructions (four FMAs per lane each) and 2.2k
// FMAs per wave, against 18.9k operations of one pair per lane.
struct PairsTable {
  std::vector<std::array<float, 4>> slots;  // [slot][2 h + row degree]
};
constexpr size_t kPairsSlots = 16;  // slots of one pipeline stage
constexpr int kPairsLmax = 6;       // highest L_max with an inter-channel kernel

void emit_pairs_body(FILE* f, int L, long* ops_out, long* mfma_out) {
  const int K = (L + 1) * (L + 1);
  std::vector<Term> terms = contraction_terms(L);
  std::map<std::array<int, 5>, const Term*> at;  // (l1, m1, l2, m2, J)
  for (const Term& t : terms) at[{t.l1, t.m1, t.l2, t.m2, t.J}] = &t;
  auto coef = [&](int l1, int m1, int l2, int m2, int J) {
    auto it = at.find({l1, m1, l2, m2, J});
    if (it == at.end()) return 0.0;
    const int a = J & 1, p1 = l1 & 1, p2 = l2 & 1, b = p1 ^ p2;
    if (it->second->imag != ((a ^ b) != 0)) {
      std::fprintf(stderr, "gen_cg: parity of a pair term (%d %d %d %d J=%d)\n", l1, m1, l2, m2, J);
      std::exit(1);
    }
    return it->second->coef * ((a & b) ? -1.0 : 1.0) * ((p1 & p2) ? -1.0 : 1.0);
  };
  PairsTable tab;
  long ops = 0, mfmas = 0;
  std::fprintf(f, "template <>\nstruct CgPairsBody<%d> {\n  static constexpr int K = %d;\n", L, K);
  std::fprintf(f, "  template <class Tab, class Store>\n");
  std::fprintf(f, "  static __device__ __forceinline__ void run(const float2 (&q)[%d], const float (&kp)[%d], Tab tab, Store& st) {\n",
               K, K);
  for (int mu = 0; mu <= L; ++mu) {
    std::fprintf(f, "    {  // phase |M| = %d\n", mu);
    const int nj = L + 1 - mu, ng = (nj + 1) / 2;
    const std::vector<int> Ms = mu == 0 ? std::vector<int>{0} : std::vector<int>{mu, -mu};
    for (int M : Ms)
      for (int J = mu; J <= L; ++J) std::fprintf(f, "      float2 %s;\n", acc_name(M, J).c_str());
    for (int M : Ms) {
      std::fprintf(f, "      {\n");
      for (int g = 0; g < ng; ++g) std::fprintf(f, "      v4f dr%d = {0.f, 0.f, 0.f, 0.f}, di%d = {0.f, 0.f, 0.f, 0.f};\n", g, g);
      // one t of every unit (m1, l1, l1 + 1, group): its slots and outer products
      struct Unit {
        int g, m1, l1;
        std::vector<int> k;  // key components of the slots
        std::vector<std::array<float, 4>> c;
        bool any[2] = {false, false};
      };
      std::vector<Unit> units;
      for (int m1 = std::max(-L, M - L); m1 <= std::min(L, M + L); ++m1) {
        const int m2 = M - m1;
        for (int l1 = std::abs(m1); l1 <= L; l1 += 2) {
          for (int g = 0; g < ng; ++g) {
            const int Ja = mu + 2 * g;
            Unit u;
            u.g = g;
            u.m1 = m1;
            u.l1 = l1;
            for (int l2 = std::abs(m2); l2 <= L; ++l2) {
              std::array<float, 4> c;
              bool any = false;
              for (int h = 0; h < 2; ++h)
                for (int d = 0; d < 2; ++d) {
                  const bool in = l1 + h <= L && Ja + d <= L;
                  c[2 * h + d] = in ? (float)coef(l1 + h, m1, l2, m2, Ja + d) : 0.f;
                  if (c[2 * h + d] != 0.f) any = u.any[h] = true;
                }
              if (!any) continue;
              u.k.push_back(comp(l2, m2));
              u.c.push_back(c);
            }
            if (!u.k.empty()) units.push_back(u);
          }
        }
      }
      // stages of consecutive units with at most kPairsSlots slots
      std::vector<std::vector<int>> stages;
      size_t left = 0;
      for (size_t i = 0; i < units.size(); ++i) {
        if (units[i].k.size() > left) {
          stages.push_back({});
          left = kPairsSlots;
        }
        stages.back().push_back((int)i);
        left -= units[i].k.size();
      }
      std::vector<size_t> first;  // first table entry of each stage, and the end
      std::vector<std::vector<std::pair<int, int>>> order;  // (unit, slot of the unit), the chains side by side
      for (auto& st : stages) {
        first.push_back(tab.slots.size() / 4);
        order.push_back({});
        for (size_t i = 0;; ++i) {
          bool more = false;
          for (int u : st)
            if (i < units[u].k.size()) {
              tab.slots.push_back(units[u].c[i]);
              order.back().push_back({u, (int)i});
              more = true;
            }
          if (!more) break;
        }
        while (tab.slots.size() % 4) tab.slots.push_back({0.f, 0.f, 0.f, 0.f});
      }
      first.push_back(tab.slots.size() / 4);
      // Software pipeline, kept by scheduling barriers: step s loads the
      // coefficients of stage s, computes the t of stage s - 1 and runs the
      // outer products of stage s - 2, so that no instruction waits for the
      // one before it.
      for (auto& st : stages)
        for (int u : st) std::fprintf(f, "      float t%d;\n", u);
      for (size_t e = first.front(); e < first.back(); ++e) std::fprintf(f, "      v4f c%zu;\n", e);
      const int ns = (int)stages.size();
      for (int step = 0; step < ns + 2; ++step) {
        if (step < ns) {
          std::fprintf(f, "      { const auto tb = tab.fresh();\n");
          for (size_t e = first[step]; e < first[step + 1]; ++e) std::fprintf(f, "      c%zu = tb.at(%zu);\n", e, e);
          std::fprintf(f, "      }\n");
        }
        if (step >= 1 && step - 1 < ns) {
          const size_t s0 = 4 * first[step - 1];
          for (size_t i = 0; i < order[step - 1].size(); ++i) {
            const int u = order[step - 1][i].first, j = order[step - 1][i].second;
            const size_t slot = s0 + i;
            if (j == 0)
              std::fprintf(f, "      t%d = c%zu[%zu] * kp[%d];\n", u, slot / 4, slot % 4, units[u].k[j]);
            else
              std::fprintf(f, "      t%d = fmaf(c%zu[%zu], kp[%d], t%d);\n", u, slot / 4, slot % 4, units[u].k[j], u);
            ++ops;
          }
        }
        if (step >= 2) {
          for (int h = 0; h < 2; ++h)
            for (int u : stages[step - 2]) {
              if (!units[u].any[h]) continue;
              const int x = comp(units[u].l1 + h, units[u].m1), g = units[u].g;
              std::fprintf(f, "      dr%d = __builtin_amdgcn_mfma_f32_4x4x1f32(t%d, q[%d].x, dr%d, 1, %d, 0);\n", g, u, x, g, h);
              std::fprintf(f, "      di%d = __builtin_amdgcn_mfma_f32_4x4x1f32(t%d, q[%d].y, di%d, 1, %d, 0);\n", g, u, x, g, h);
              mfmas += 2;
            }
        }
        std::fprintf(f, "      __builtin_amdgcn_sched_barrier(0);\n");
      }
      // w = i^J ((dr[re] - di[im]) + i (di[re] + dr[im]))
      for (int J = mu; J <= L; ++J) {
        const int g = (J - mu) / 2, r = 2 * ((J - mu) & 1);
        char re[64], im[64];
        std::snprintf(re, sizeof re, "dr%d[%d] - di%d[%d]", g, r, g, r + 1);
        std::snprintf(im, sizeof im, "di%d[%d] + dr%d[%d]", g, r, g, r + 1);
        if (J & 1)
          std::fprintf(f, "      %s = make_float2(-(%s), %s);\n", acc_name(M, J).c_str(), im, re);
        else
          std::fprintf(f, "      %s = make_float2(%s, %s);\n", acc_name(M, J).c_str(), re, im);
        ops += 2;
      }
      std::fprintf(f, "      }\n");
    }
    for (int J = mu; J <= L; ++J) {
      if (mu == 0) {
        std::fprintf(f, "      st(%d, %s);\n", comp(J, 0), acc_name(0, J).c_str());
      } else {
        const std::string p = acc_name(mu, J), m = acc_name(-mu, J);
        std::fprintf(f, "      st(%d, make_float2(%s.x + %s.x, %s.y + %s.y));\n", comp(J, mu), m.c_str(), p.c_str(),
                     m.c_str(), p.c_str());
        std::fprintf(f, "      st(%d, make_float2(%s.y - %s.y, %s.x - %s.x));\n", comp(J, -mu), m.c_str(), p.c_str(),
                     p.c_str(), m.c_str());
        ops += 4;
      }
    }
    std::fprintf(f, "      st.end_phase(%d);\n    }\n", mu);
  }
  while (tab.slots.size() % 4) tab.slots.push_back({0.f, 0.f, 0.f, 0.f});
  std::fprintf(f, "  }\n  static constexpr int kEntries = %zu;  // table entries of 16 floats\n", tab.slots.size() / 4);
  std::fprintf(f, "  static __device__ const float* table();\n};\n");
  std::fprintf(f, "static __device__ __attribute__((aligned(16))) const float pairs_table_L%d[%zu] = {\n", L, tab.slots.size() * 4);
  for (size_t e = 0; e < tab.slots.size() / 4; ++e) {
    for (int sel = 0; sel < 4; ++sel)
      for (int i = 0; i < 4; ++i) std::fprintf(f, "%.9ef, ", (double)tab.slots[4 * e + i][sel]);
    std::fprintf(f, "\n");
  }
  std::fprintf(f, "};\ninline __device__ const float* CgPairsBody<%d>::table() { return pairs_table_L%d; }\n\n", L, L);
  *ops_out = ops;
  *mfma_out = mfmas;
}

// Token-wise product for the value tensor product (CgRealBody<L>::run):
//   f[J,M] = sum R^{(l1 l2 J)}[M,m1,m2] a[l1,m1] b[l2,m2]   (a, b, f real)
// in the complex-m basis, where the selection rule leaves fewer terms than in
// the real one: A[l,m] = a_c - i a_s for m > 0 (a_c, a_s the components +-m),
// A[l,-m] its conjugate, A[l,0] real; no operation is spent on the change of
// basis, the parts are the inputs themselves up to signs.  For real inputs
// w[J,-M] is the conjugate of w[J,M], so only M >= 0 is evaluated, and
//   f[J,0] = w[J,0],  f[J,M] = 2 Re w[J,M],  f[J,-M] = -2 Im w[J,M].
// Per pair of components the two ordered products x, y share a coefficient up
// to the swap sign, as in CgBody: s = x + y for the real coefficients and/or
// d = x - y for the imaginary ones, then two FMAs per coefficient.  Of M = 0,
// whose result is real, the pairs {(l1,-m), (l2,m)} and {(l1,m), (l2,-m)} are
// conjugates: one of them is taken, and only the real part (one FMA per
// coefficient).  8.9k operations at L_max = 6 against 10.6k in the real basis.
void emit_real_body(FILE* f, int L, long* ops_out) {
  const int K = (L + 1) * (L + 1);
  std::vector<Term> terms = contraction_terms(L);
  TermMap terms_of;
  for (const Term& t : terms) terms_of[{t.l1, t.m1, t.l2, t.m2}].push_back(t);
  long ops = 0;
  std::set<int> inited;
  std::fprintf(f, "template <>\nstruct CgRealBody<%d> {\n  static constexpr int K = %d;\n", L, K);
  std::fprintf(f,
               "  static __device__ __forceinline__ void run(const float (&a)[%d], const float (&b)[%d], "
               "float (&f)[%d]) {\n",
               K, K, K);
  auto acc = [&](int o, double c, const char* src) {
    if (!inited.count(o))
      std::fprintf(f, "      f[%d] = %s * %s;\n", o, lit(c).c_str(), src);
    else
      std::fprintf(f, "      f[%d] = fmaf(%s, %s, f[%d]);\n", o, lit(c).c_str(), src, o);
    inited.insert(o);
    ++ops;
  };
  // a part of a component: sign * array[index], nothing if the component is
  // real and the part imaginary
  struct Part {
    int sign;  // 0: absent
    char arr;
    int idx;
  };
  auto part = [](char arr, int l, int m, bool im) {
    if (!im) return Part{1, arr, comp(l, std::abs(m))};
    return Part{m > 0 ? -1 : (m < 0 ? 1 : 0), arr, comp(l, -std::abs(m))};
  };
  // expr = sum of sign * p * q as nested FMAs; returns false if it is empty
  auto sum_of = [&](const char* name, std::vector<std::array<Part, 2>> products) {
    std::string e;
    for (auto& pq : products) {
      const int sg = pq[0].sign * pq[1].sign;
      if (sg == 0) continue;
      char x[32], y[32];
      std::snprintf(x, sizeof x, "%c[%d]", pq[0].arr, pq[0].idx);
      std::snprintf(y, sizeof y, "%c[%d]", pq[1].arr, pq[1].idx);
      if (e.empty()) {
        if (sg < 0) {
          std::fprintf(stderr, "gen_cg: a product chain starts with a negative term\n");
          std::exit(1);
        }
        e = "mul_here<" + std::to_string(ops) + ">(" + x + ", " + y + ")";
      } else {
        e = std::string(sg > 0 ? "fmaf(" : "fnma(") + x + ", " + y + ", " + e + ")";
      }
      ++ops;
    }
    std::fprintf(f, "      const float %s = %s;\n", name, e.c_str());
  };
  // parts of the product u v (u of the first array's component, v of the
  // second's), as signed products; the imaginary part times `flip`, chosen so
  // that a chain can start with a positive term
  auto re_of = [&](char ua, int ul, int um, char va, int vl, int vm) {
    std::vector<std::array<Part, 2>> r;
    r.push_back({part(ua, ul, um, false), part(va, vl, vm, false)});
    Part i = part(ua, ul, um, true);
    i.sign = -i.sign;
    r.push_back({i, part(va, vl, vm, true)});
    return r;
  };
  auto im_of = [&](char ua, int ul, int um, char va, int vl, int vm) {
    std::vector<std::array<Part, 2>> r;
    r.push_back({part(ua, ul, um, false), part(va, vl, vm, true)});
    r.push_back({part(ua, ul, um, true), part(va, vl, vm, false)});
    return r;
  };
  auto join = [](std::vector<std::array<Part, 2>> p, const std::vector<std::array<Part, 2>>& q, int sq) {
    for (std::array<Part, 2> e : q) {
      e[0].sign *= sq;
      p.push_back(e);
    }
    return p;
  };
  // sign that makes the first present product positive, applied to all
  auto lead = [](std::vector<std::array<Part, 2>>& p) {
    for (auto& e : p)
      if (e[0].sign * e[1].sign != 0) {
        const int sg = e[0].sign * e[1].sign;
        for (auto& x : p) x[0].sign *= sg;
        return sg;
      }
    return 1;
  };
  for (int M = 0; M <= L; ++M)
    for (int m1 = M - L; 2 * m1 <= M; ++m1) {
      const int m2 = M - m1;
      for (int l1 = std::abs(m1); l1 <= L; ++l1)
        for (int l2 = std::abs(m2); l2 <= L; ++l2) {
          if ((m1 == m2 || M == 0) && l2 < l1) continue;
          auto it = terms_of.find({l1, m1, l2, m2});
          if (it == terms_of.end()) continue;
          const bool diag = l1 == l2 && m1 == m2;
          bool ev = false, od = false;
          for (const Term& t : it->second) {
            const double sigma = ((l1 + l2 - t.J) % 2 == 0) ? 1.0 : -1.0;
            const Term* u = nullptr;
            auto sw = terms_of.find({l2, m2, l1, m1});
            if (sw != terms_of.end())
              for (const Term& w : sw->second)
                if (w.J == t.J) u = &w;
            if (!u || u->imag != t.imag || t.imag != (sigma < 0) || (diag && sigma < 0) ||
                std::fabs(u->coef - sigma * t.coef) > 1e-12 * std::fabs(t.coef) + 1e-15) {
              std::fprintf(stderr, "gen_cg: swap symmetry violated (real product, %d %d %d %d J=%d)\n", l1, m1, l2, m2, t.J);
              std::exit(1);
            }
            (sigma > 0 ? ev : od) = true;
          }
          std::fprintf(f, "    {  // (%d,%d) (%d,%d)\n", l1, m1, l2, m2);
          // x = A[l1,m1] B[l2,m2], y = A[l2,m2] B[l1,m1]
          auto xr = re_of('a', l1, m1, 'b', l2, m2), xi = im_of('a', l1, m1, 'b', l2, m2);
          auto yr = re_of('a', l2, m2, 'b', l1, m1), yi = im_of('a', l2, m2, 'b', l1, m1);
          if (M == 0) {
            // half of the conjugate pairs, the real part alone
            // (l1 == l2: y is the conjugate of x, s = 2 Re x, d = 2 i Im x)
            const bool self = l1 == l2 && m1 != 0;
            const double twice = m1 != 0 ? 2.0 : 1.0;
            if (ev) sum_of("sr", diag || self ? xr : join(xr, yr, 1));
            int sd = 1;
            if (od) {  // i d: the real part is -Im d
              auto d = self ? xi : join(xi, yi, -1);
              bool empty = true;
              for (auto& e : d) empty = empty && e[0].sign * e[1].sign == 0;
              if (empty) {
                std::fprintf(stderr, "gen_cg: odd term of two real components\n");
                std::exit(1);
              }
              sd = lead(d);
              sum_of("di", d);
            }
            for (const Term& t : it->second)
              acc(comp(t.J, 0), (t.imag ? -sd : 1) * 4.0 * twice * t.coef, t.imag ? "di" : "sr");
          } else {
            int ss = 1, sd = 1;
            if (diag) {
              sum_of("sr", xr);
              ss = lead(xi);
              sum_of("si", xi);
            } else if (ev && od) {
              const int s1 = lead(xi);
              sum_of("xr", xr);
              sum_of("xi", xi);
              for (auto& e : yi) e[0].sign *= s1;
              const int s2 = lead(yi);
              sum_of("yr", yr);
              sum_of("yi", yi);
              std::fprintf(f, "      const float sr = xr + yr, dr = xr - yr, si = xi %c yi, di = xi %c yi;\n",
                           s2 > 0 ? '+' : '-', s2 > 0 ? '-' : '+');
              ops += 4;
              ss = sd = s1;
            } else if (ev) {
              auto si = join(xi, yi, 1);
              ss = lead(si);
              sum_of("sr", join(xr, yr, 1));
              sum_of("si", si);
            } else {
              auto di = join(xi, yi, -1), dr = join(xr, yr, -1);
              sd = lead(di);
              sum_of("dr", dr);
              sum_of("di", di);
            }
            // real coefficient: w += c s; imaginary: w += i c d
            for (const Term& t : it->second) {
              const double c = 8.0 * t.coef;
              acc(comp(t.J, M), t.imag ? -sd * c : c, t.imag ? "di" : "sr");
              acc(comp(t.J, -M), t.imag ? -c : -ss * c, t.imag ? "dr" : "si");
            }
          }
          std::fprintf(f, "    }\n");
        }
    }
  for (int o = 0; o < K; ++o)
    if (!inited.count(o)) std::fprintf(f, "    f[%d] = 0.f;\n", o);
  std::fprintf(f, "  }\n");
  std::fprintf(f, "  static constexpr long kOps = %ld;  // VALU ops per token and channel\n};\n\n", ops);
  *ops_out = ops;
}

int main(int argc, char** argv) {
  if (argc != 3) {
    std::fprintf(stderr, "usage: %s <output-dir> <LGEN>\n", argv[0]);
    return 2;
  }
  const std::string dir = argv[1];
  const int lgen = std::atoi(argv[2]);
  for (int L = 0; L <= lgen; ++L) {
    const std::string path = dir + "/cg_body_L" + std::to_string(L) + ".inc";
    FILE* f = std::fopen(path.c_str(), "w");
    if (!f) {
      std::perror(path.c_str());
      return 1;
    }
    std::fprintf(f, "// Generated by csrc/codegen/gen_cg.cpp -- do not edit.\n");
    std::fprintf(f, "// Frequency-domain CG contraction body, L_max = %d.\n#pragma once\n\n", L);
    long ops = 0, rops = 0, sops = 0, psops = 0;
    emit_body(f, L, &ops);
    emit_real_body(f, L, &rops);
    emit_mirror_body(f, L, &sops);
    emit_path_split_body(f, L, &psops);
    if (L <= kPairsLmax) {
      long pops = 0, pmfma = 0;
      std::fprintf(f, "#ifdef CGCONV_PAIRS_BODY  // the inter-channel kernel only\n");
      emit_pairs_body(f, L, &pops, &pmfma);
      std::fprintf(f, "#endif\n");
      std::fprintf(stderr, "gen_cg: L=%d channel-pairs body: %ld ops and %ld matrix instructions per wave\n", L, pops,
                   pmfma);
    }
    std::fclose(f);
    std::fprintf(stderr,
                 "gen_cg: L=%d ops/point=%ld real token-wise ops=%ld mirror lane-pair ops/lane=%ld "
                 "per-path lane-pair ops/lane=%ld\n",
                 L, ops, rops, sops, psops);
  }
  const std::string hpath = dir + "/cg_lgen.h";
  FILE* h = std::fopen(hpath.c_str(), "w");
  if (!h) {
    std::perror(hpath.c_str());
    return 1;
  }
  std::fprintf(h, "// Generated by csrc/codegen/gen_cg.cpp -- do not edit.\n#pragma once\n#define CGCONV_LGEN %d\n", lgen);
  std::fclose(h);
  return 0;
}
