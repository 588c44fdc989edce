// Host-side drive of the mixed-radix product-grid transforms (ff::Mix), lane
// by lane, for CPU tests.
//
// Reads "logn inv lanes full" then the complex64 input (length 3 * 2^logn / 4,
// or 2^logn with full) from stdin, runs every pass with each of the N/16 * lanes
// lanes emulated in turn (lanes: 0 for half of N/16, else 1, 2 or 4 times it),
// for a group interleaved with as many others as fill 256 threads, and writes
// the transform to stdout. The inverse plan takes its input as the kernels
// give it, kept in the first and last third (quarter), and prunes its first
// pass. Every output position must be written exactly once.
#include <cstdio>
#include <type_traits>
#include <vector>

#include "mixed_fft.hpp"

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

template <class PLAN, int LOGN, bool INV, int G>
void run(std::vector<float2>& io, bool full) {
  constexpr int T = G >= 256 ? 1 : 256 / G;
  using M = ff::Mix<typename std::conditional<INV, typename PLAN::I, typename PLAN::F>::type, G, T>;
  std::vector<float2> tab(ff::mix_tables_size(LOGN, full) + 1);
  ff::build_mix_tables(LOGN, tab.data(), full);
  const float2* tw = tab.data() + (INV ? 0 : ff::MixTables<PLAN>::F_OFF);
  std::vector<Regs<M::REGS>> x(G);
  for (int t = 0; t < G; ++t)
    for (int b = 0; b < M::rounds(0); ++b)
      if (M::template active<0>(t, b))
        for (int r = 0; r < M::radix(0); ++r) x[t].a[b * M::radix(0) + r] = io[t + G * b + r * M::bf(0)];
  std::vector<float2> lds(M::LDS, make_float2(1e30f, 1e30f));
  passes<M, INV>(x, lds.data() + (T - 1), tw);
  constexpr int P = M::NPASS - 1;
  std::vector<int> seen(M::N, 0);
  for (int t = 0; t < G; ++t)
    for (int b = 0; b < M::rounds(P); ++b)
      if (M::template active<P>(t, b))
        for (int r = 0; r < M::radix(P); ++r) {
          const int at = t + G * b + r * M::bf(P);
          io[at] = x[t].a[b * M::radix(P) + r];
          ++seen[at];
        }
  for (int i = 0; i < M::N; ++i)
    if (seen[i] != 1) io[i] = make_float2(1e30f, 1e30f);
}

template <class PLAN, int LOGN, int G>
void both(std::vector<float2>& io, int inv, bool full) {
  if constexpr (G > 0) {
    if (inv)
      run<PLAN, LOGN, true, G>(io, full);
    else
      run<PLAN, LOGN, false, G>(io, full);
  }
}

template <class PLAN, int LOGN>
bool lanes_of(std::vector<float2>& io, int inv, int lanes, bool full) {
  constexpr int NB = (1 << LOGN) / 16;
  if (lanes == 0) both<PLAN, LOGN, NB / 2>(io, inv, full);
  if (lanes == 1) both<PLAN, LOGN, NB>(io, inv, full);
  if (lanes == 2) both<PLAN, LOGN, 2 * NB>(io, inv, full);
  if (lanes == 4) both<PLAN, LOGN, 4 * NB>(io, inv, full);
  return true;
}

template <int L>
bool dispatch(int logn, std::vector<float2>& io, int inv, int lanes) {
  if constexpr (L > 14) {
    return false;
  } else {
    return logn == L ? lanes_of<ff::MixPlan<L>, L>(io, inv, lanes, false) : dispatch<L + 1>(logn, io, inv, lanes);
  }
}

}  // namespace

int main() {
  int hdr[4];
  if (fread(hdr, sizeof(int), 4, stdin) != 4) return 2;
  const int logn = hdr[0], inv = hdr[1], lanes = hdr[2], full = hdr[3];
  if (logn < 4 || logn > 14) return 3;
  std::vector<float2> io(full ? size_t(1) << logn : size_t(3) << (logn - 2));
  if (fread(io.data(), sizeof(float2), io.size(), stdin) != io.size()) return 4;
  bool ok = false;
  if (full) {
    if (logn == 4) ok = lanes_of<ff::FullPlan<4>, 4>(io, inv, lanes, true);
    if (logn == 5) ok = lanes_of<ff::FullPlan<5>, 5>(io, inv, lanes, true);
    if (logn == 6) ok = lanes_of<ff::FullPlan<6>, 6>(io, inv, lanes, true);
  } else if (logn >= 6) {
    ok = dispatch<6>(logn, io, inv, lanes);
  }
  if (!ok) return 5;
  fwrite(io.data(), sizeof(float2), io.size(), stdout);
  return 0;
}
