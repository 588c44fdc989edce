// Host-side drive of the transforms (ff::Mix) in every shape that a kernel
// gives them: the lanes, the interleaved groups and so the padding of the
// exchange areas are those of the kernels' own shape structs.
//
// The argument names a family of shapes. Each shape transforms the same white
// input of its length; the output must match a double-precision DFT, be the
// same bit for bit for every shape of one plan, write every position once, and
// keep to its exchange area (one float2 more on either side is checked), for
// the first and the last of the interleaved groups. Prints the number of shapes.
#include <cmath>
#include <complex>
#include <cstdio>
#include <cstring>
#include <map>
#include <random>
#include <set>
#include <string>
#include <tuple>
#include <vector>

#include "transform_shapes.hpp"

namespace {

struct TableFetch {
  const float2* tw;
  float2 operator()(int i) const { return tw[i]; }
};
template <int N>
struct Regs {
  float2 a[N];
};

template <class M, bool INV, int P = 0>
void passes(std::vector<Regs<M::REGS>>& x, float2* lds, const float2* tw) {
  if constexpr (P < M::NPASS) {
    for (int t = 0; t < M::G; ++t) {
      float2 w[M::tw_count(P)] = {};
      if constexpr (P > 0) M::template load_twiddles<P>(w, TableFetch{tw}, t);
      M::template butterflies<P, INV, INV>(x[t].a, t, w);
    }
    if constexpr (P + 1 < M::NPASS) {
      for (int t = 0; t < M::G; ++t) M::template put<P>(x[t].a, t, lds);
      for (int t = 0; t < M::G; ++t) M::template get<P + 1>(x[t].a, t, lds);
      passes<M, INV, P + 1>(x, lds, tw);
    }
  }
}

int g_failed = 0;
void fail(const char* what, int n, int g, int t, bool inv) {
  std::printf("%s: length %d, %d lanes, %d groups, %s\n", what, n, g, t, inv ? "inverse" : "forward");
  ++g_failed;
}

// White input of length n (inverse: kept in the first and last `kept` places), and its DFT.
struct Problem {
  std::vector<float2> in;
  std::vector<std::complex<double>> out;
};
const Problem& problem(int n, int kept, bool inv) {
  static std::map<std::tuple<int, int, bool>, Problem> all;
  Problem& p = all[{n, kept, inv}];
  if (!p.in.empty()) return p;
  std::mt19937 rng(n + inv);
  std::normal_distribution<float> gauss;
  p.in.resize(n);
  for (int i = 0; i < n; ++i) {
    p.in[i] = make_float2(gauss(rng), gauss(rng));
    if (inv && i >= kept && i < n - kept) p.in[i] = make_float2(0.f, 0.f);
  }
  std::vector<std::complex<double>> root(n);
  for (int i = 0; i < n; ++i) root[i] = std::polar(1.0, (inv ? 2.0 : -2.0) * M_PI * i / n);
  p.out.resize(n);
  for (int k = 0; k < n; ++k) {
    double re = 0.0, im = 0.0;
    for (int j = 0, e = 0; j < n; ++j) {
      re += p.in[j].x * root[e].real() - p.in[j].y * root[e].imag();
      im += p.in[j].x * root[e].imag() + p.in[j].y * root[e].real();
      e += k;
      if (e >= n) e -= n;
    }
    p.out[k] = {re, im};
  }
  return p;
}

std::set<std::tuple<int, int, int, bool>> g_seen;
std::map<std::pair<std::vector<int>, bool>, std::vector<float2>> g_bits;  // the first output of each plan

// One shape; `tw` is its table and `kept` the modes on each side.
template <class M, bool INV>
void shape(const float2* tw, int kept) {
  std::vector<int> radices;
  for (int p = 0; p < M::NPASS; ++p) radices.push_back(M::radix(p));
  if (!g_seen.insert({M::N * 32 + M::radix(0), M::G, M::T, INV}).second) return;
  const Problem& pr = problem(M::N, kept, INV);
  const float2 guard = make_float2(1e30f, -1e30f);
  for (const int group : {0, M::T - 1}) {
    std::vector<Regs<M::REGS>> x(M::G);
    for (int t = 0; t < M::G; ++t)
      for (int b = 0; b < M::rounds(0); ++b)
        if (M::template active<0>(t, b))
          for (int r = 0; r < M::radix(0); ++r)
            x[t].a[b * M::radix(0) + r] = pr.in[t + M::G * b + r * M::bf(0)];
    std::vector<float2> lds(M::LDS + 2, guard);
    passes<M, INV>(x, lds.data() + 1 + group, tw);
    for (int i = 0; i < M::LDS + 2; ++i)
      if ((i == 0 || i == M::LDS + 1 || (i - 1) % M::T != group) && std::memcmp(&lds[i], &guard, sizeof guard))
        return fail("writes outside its exchange area", M::N, M::G, M::T, INV);
    constexpr int P = M::NPASS - 1;
    std::vector<int> seen(M::N, 0);
    std::vector<float2> out(M::N);
    for (int t = 0; t < M::G; ++t)
      for (int b = 0; b < M::rounds(P); ++b)
        if (M::template active<P>(t, b))
          for (int r = 0; r < M::radix(P); ++r) {
            const int at = t + M::G * b + r * M::bf(P);
            out[at] = x[t].a[b * M::radix(P) + r];
            ++seen[at];
          }
    double err = 0.0, ref = 0.0;
    for (int i = 0; i < M::N; ++i) {
      if (seen[i] != 1) return fail("an output position is not written once", M::N, M::G, M::T, INV);
      err += std::norm(std::complex<double>(out[i].x, out[i].y) - pr.out[i]);
      ref += std::norm(pr.out[i]);
    }
    // a transform of b bits rounds about 2 b times at 2^-24 / sqrt(3) each in the mean square: 2.6e-7 at 2^14
    if (!(std::sqrt(err / ref) < 5e-7)) return fail("differs from the DFT", M::N, M::G, M::T, INV);
    std::vector<float2>& first = g_bits[{radices, INV}];
    if (first.empty()) first = out;
    if (std::memcmp(first.data(), out.data(), sizeof(float2) * M::N))
      return fail("bits differ from another shape's", M::N, M::G, M::T, INV);
  }
}

// The transforms of a length with product grid 3 * 2^LOGN / 4, or (FULL) of 2^LOGN points.
template <int LOGN, bool FULL, class M, bool INV>
void mixed() {
  using Plan = typename std::conditional<FULL, ff::FullPlan<FULL ? LOGN : 4>, ff::MixPlan<FULL ? 6 : LOGN>>::type;
  static std::vector<float2> tab;
  if (tab.empty()) {
    tab.resize(ff::mix_tables_size(LOGN, FULL) + 1);
    ff::build_mix_tables(LOGN, tab.data(), FULL);
  }
  shape<M, INV>(tab.data() + (INV ? 0 : ff::MixTables<Plan>::F_OFF), FULL ? M::N / 4 : M::N / 3);
}

template <int L>
void step() {
  if constexpr (L <= flame::kMaxLog) {
    mixed<L, false, typename flame::RowMix<L>::F, false>();
    mixed<L, false, typename flame::RowMix<L>::I, true>();
    if constexpr (L < 12) {
      mixed<L, false, typename flame::RowSplit<L>::F, false>();
      mixed<L, false, typename flame::RowSplit<L>::I, true>();
    }
    if constexpr (L == 13) {
      mixed<L, false, typename flame::RowMix<L, flame::kFewLanes13>::F, false>();
      mixed<L, false, typename flame::RowMix<L, flame::kFewLanes13>::I, true>();
    }
    if constexpr (L >= flame::kMinLogProduct) {
      mixed<L, false, typename flame::ColMix<L>::F, false>();
      mixed<L, false, typename flame::ColMix<L>::I, true>();
      if constexpr (L < 12) {
        mixed<L, false, typename flame::ColSplit<L>::F, false>();
        mixed<L, false, typename flame::ColSplit<L>::I, true>();
      }
      if constexpr (L == 13) {
        mixed<L, false, typename flame::ColMix<L, flame::kFewLanes13>::F, false>();
        mixed<L, false, typename flame::ColMix<L, flame::kFewLanes13>::I, true>();
      }
    }
    step<L + 1>();
  }
}

template <int L, int NG>
void adjoint_shape() {
  mixed<L, false, typename flame::AdjMix<L, NG>::F, false>();
  mixed<L, false, typename flame::AdjMix<L, NG>::I, true>();
}
template <int L>
void adjoint() {
  if constexpr (L <= flame::kMaxLog) {
    adjoint_shape<L, 1>();
    if constexpr (L <= 11) {
      adjoint_shape<L, 2>();
      adjoint_shape<L, 3>();
    }
    adjoint<L + 1>();
  }
}

template <int L>
void averages() {
  if constexpr (L <= flame::kMaxLogSide) {
    const ff::PassPlan pp = ff::make_pass_plan(L, 16);
    std::vector<float2> tab(pp.tw_size + 1);
    ff::build_twiddles(L, tab.data(), 16);
    using I = typename flame::PhysSplit<L>::I;
    shape<I, true>(tab.data(), I::N / 4);
    averages<L + 1>();
  }
}

template <int L1, int L2>
void resident() {
  if constexpr (L1 + L2 <= flame::kResMaxLogs) {
    using C = flame::Res<L1, L2>;
    if constexpr (C::OK) {
      constexpr bool f1 = L1 < flame::kMinLogProduct, f2 = L2 < flame::kMinLogRowProduct;
      mixed<L1, f1, typename C::CI, true>();
      mixed<L1, f1, typename C::CF, false>();
      mixed<L2, f2, typename C::RI, true>();
      mixed<L2, f2, typename C::RF, false>();
    }
    resident<L1, L2 + 1>();
  } else if constexpr (L1 + 1 + flame::kMinLog <= flame::kResMaxLogs) {
    resident<L1 + 1, flame::kMinLog>();
  }
}

}  // namespace

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  if (what == "step")
    step<flame::kMinLogRowProduct>();
  else if (what == "adjoint")
    adjoint<flame::kMinLogRowProduct>();
  else if (what == "averages")
    averages<flame::kMinLog>();
  else if (what == "resident")
    resident<flame::kMinLog, flame::kMinLog>();
  else
    return 2;
  std::printf("%zu shapes\n", g_seen.size());
  return g_failed ? 1 : 0;
}
