// Mixed-radix transforms of the product grids' lengths, L = 3 N / 4 = 12 * 2^q.
//
// A length-L transform belongs to a group of G threads of a workgroup that
// holds T such groups, interleaved (thread tid: group tid % T, lane tid / T).
// A pass of radix R has L / R butterflies; lane t runs butterflies
// j = t + G b, b < rounds, its inputs x[j + r L / R] and, after the pass, its
// outputs in registers b R + r. Where L / R is no multiple of G the last
// round leaves whole waves idle rather than every wave a part of a
// butterfly: the radices then need not divide the points per thread, so
// that three passes of radix 8 to 16 do what five passes of radix 12, 4, 4,
// 4, 2 did, with two exchanges through LDS instead of four.
//
// The inverse transforms, whose input is a spectrum kept in the first and
// last third of the length, start with the radix-12 pass, pruned to the
// eight inputs that do not vanish; the forward transforms run the radices in
// reverse and end with it. So a lane holds the same modes, t + (L/12) r with
// r = 0..3 (k >= 0) and r = 8..11 (k - L < 0), where a forward transform ends
// and the inverse ones begin, and the same points where an inverse ends and a
// forward one begins.

#pragma once

#include "fft_engine.hpp"

namespace ff {

template <int... RS>
struct Radices {
  static constexpr int count = sizeof...(RS);
  static constexpr int radix[sizeof...(RS)] = {RS...};
};

// The passes of a length 3 * 2^LOGN / 4 transform, inverse (I) and forward (F).
template <int LOGN>
struct MixPlan;
template <>
struct MixPlan<6> {
  using I = Radices<12, 4>;
  using F = Radices<4, 12>;
};
template <>
struct MixPlan<7> {
  using I = Radices<12, 8>;
  using F = Radices<8, 12>;
};
template <>
struct MixPlan<8> {
  using I = Radices<12, 16>;
  using F = Radices<16, 12>;
};
template <>
struct MixPlan<9> {
  using I = Radices<12, 8, 4>;
  using F = Radices<4, 8, 12>;
};
template <>
struct MixPlan<10> {
  using I = Radices<12, 8, 8>;
  using F = Radices<8, 8, 12>;
};
template <>
struct MixPlan<11> {
  using I = Radices<12, 16, 8>;
  using F = Radices<8, 16, 12>;
};
template <>
struct MixPlan<12> {
  using I = Radices<12, 16, 16>;
  using F = Radices<16, 16, 12>;
};
template <>
struct MixPlan<13> {
  using I = Radices<12, 8, 8, 8>;
  using F = Radices<8, 8, 8, 12>;
};
template <>
struct MixPlan<14> {
  using I = Radices<12, 16, 8, 8>;
  using F = Radices<8, 8, 16, 12>;
};

// Spare slots of an exchange area: element i is stored at slot
// i + i / g1 + m (i / g2); a granule of 0 adds nothing.
struct MixPad {
  int g1, g2, m;
};
constexpr int mix_spare(const MixPad& p, int i) { return (p.g1 ? i / p.g1 : 0) + (p.g2 ? p.m * (i / p.g2) : 0); }

// An exchange writes output r of butterfly j at (j / ns) ns R + j % ns + r ns
// and reads j + r L / R2 for the next pass. With a granule that is a multiple
// of ns, divides or is divided by ns R, and divides L / R2, the spare slots
// of r's part are a constant that adds to j's, so that they cost nothing per
// element.
constexpr bool mix_granule_ok(int g, int radix, int ns, int next_bf) {
  return g == 0 || (g % ns == 0 && (g % (ns * radix) == 0 || (ns * radix) % g == 0) && next_bf % g == 0);
}

// Passes over the LDS banks that the first wave's 8-byte accesses take (32
// lanes at a time, conflict-free when they hit 32 distinct slots modulo 32).
constexpr int mix_bank_cost(const MixPad& p, int radix, int ns, int bf, int next_radix, int next_bf, int g, int t) {
  int total = 0;
  for (int side = 0; side < 2; ++side)
    for (int r = 0; r < (side ? next_radix : radix); ++r) {
      int hits[32] = {};
      int most = 0;
      for (int lane = 0; lane < 32; ++lane) {
        const int j = lane / t;
        if (j >= g || j >= (side ? next_bf : bf)) break;
        const int i = side ? j + r * next_bf : (j / ns) * ns * radix + j % ns + r * ns;
        const int h = ++hits[((i + mix_spare(p, i)) * t + lane % t) % 32];
        most = h > most ? h : most;
      }
      total += most;
    }
  return total;
}

constexpr MixPad mix_best_pad(int radix, int ns, int bf, int next_radix, int next_bf, int g, int t) {
  constexpr MixPad cand[] = {{0, 0, 0},  {4, 0, 0},  {8, 0, 0},  {16, 0, 0},  {32, 0, 0},  {12, 0, 0},
                             {24, 0, 0}, {48, 0, 0}, {96, 0, 0}, {192, 0, 0}, {0, 32, 4},  {0, 64, 4},
                             {0, 96, 4}, {8, 64, 4}, {16, 64, 4}, {0, 48, 2}, {0, 192, 2}, {0, 192, 4}};
  MixPad best{0, 0, 0};
  int cost = mix_bank_cost(best, radix, ns, bf, next_radix, next_bf, g, t);
  for (const MixPad& p : cand) {
    if (!mix_granule_ok(p.g1, radix, ns, next_bf) || !mix_granule_ok(p.g2, radix, ns, next_bf)) continue;
    const int c = mix_bank_cost(p, radix, ns, bf, next_radix, next_bf, g, t);
    if (c < cost) {
      cost = c;
      best = p;
    }
  }
  return best;
}

// The same for the whole length 2^LOGN of a short axis, LOGN = 4 .. 6, kept in
// the first and last quarter: the spectral end is a radix-16 pass, so that a
// lane holds the modes t + (N/16) r, r = 0..3 and 12..15.
template <int LOGN>
struct FullPlan;
template <>
struct FullPlan<4> {
  using I = Radices<16>;
  using F = Radices<16>;
};
template <>
struct FullPlan<5> {
  using I = Radices<16, 2>;
  using F = Radices<2, 16>;
};
template <>
struct FullPlan<6> {
  using I = Radices<16, 4>;
  using F = Radices<4, 16>;
};

// The transform with radices RX on G lanes, T groups interleaved.
template <class RX, int G_, int T_>
struct Mix {
  static constexpr int G = G_, T = T_, NPASS = RX::count;
  static constexpr int radix(int p) { return RX::radix[p]; }
  static constexpr int ns(int p) { return p == 0 ? 1 : ns(p - 1) * radix(p - 1); }
  static constexpr int N = ns(NPASS);
  static constexpr int bf(int p) { return N / radix(p); }
  static constexpr int rounds(int p) { return (bf(p) + G - 1) / G; }
  static constexpr bool whole(int p) { return bf(p) % G == 0; }  // no idle lanes in the last round
  static constexpr int regs_up_to(int p) {
    return p < 0 ? 0 : (rounds(p) * radix(p) > regs_up_to(p - 1) ? rounds(p) * radix(p) : regs_up_to(p - 1));
  }
  static constexpr int REGS = regs_up_to(NPASS - 1);
  // twiddle table: entry r of butterfly k at tw_off(p) + (r - 1) ns(p) + k, p >= 1 (tw_butterfly)
  static constexpr int tw_off(int p) { return p <= 1 ? 0 : tw_off(p - 1) + ns(p - 1) * (radix(p - 1) - 1); }
  static constexpr int TW = tw_off(NPASS);
  // exchange area after pass P
  template <int P>
  static constexpr MixPad pad = mix_best_pad(radix(P), ns(P), bf(P), radix(P + 1), bf(P + 1), G, T);
  template <int P = 0>
  static constexpr int slots() {
    if constexpr (P + 1 < NPASS) {
      const int here = N + mix_spare(pad<P>, N - 1), rest = slots<P + 1>();
      return here > rest ? here : rest;
    } else {
      return N;
    }
  }
  static constexpr int SLOTS = slots();
  static constexpr int LDS = SLOTS * T;  // float2 of one exchange area

  template <int P>
  static __host__ __device__ __forceinline__ bool active(int t, int b) {
    return whole(P) || b + 1 < rounds(P) || t + G * b < bf(P);
  }

  // Twiddles of lane t in pass P >= 1: those of round b from b (R - 1) on.
  static constexpr int tw_count(int p) { return p < 1 || p >= NPASS ? 1 : rounds(p) * (radix(p) - 1); }
  template <int P, class F>
  static __host__ __device__ __forceinline__ void load_twiddles(float2 (&w)[tw_count(P)], const F& fetch, int t) {
#pragma unroll
    for (int b = 0; b < rounds(P); ++b) {
      const int k = mod_ns<ns(P)>(t + G * b);
#pragma unroll
      for (int r = 1; r < radix(P); ++r) w[b * (radix(P) - 1) + r - 1] = fetch(tw_off(P) + (r - 1) * ns(P) + k);
    }
  }

  // Pass P on the registers. ZMID: in pass 0, the inputs between the first
  // and the last four are zero (radix 12 or 16).
  template <int P, bool INV, bool ZMID>
  static __host__ __device__ __forceinline__ void butterflies(float2 (&x)[REGS], int t, const float2 (&w)[tw_count(P)]) {
    constexpr int R = radix(P);
#pragma unroll
    for (int b = 0; b < rounds(P); ++b) {
      if (!active<P>(t, b)) continue;
      float2 y[R];
#pragma unroll
      for (int r = 0; r < R; ++r) y[r] = x[b * R + r];
      if constexpr (P > 0) {
#pragma unroll
        for (int r = 1; r < R; ++r) y[r] = twmul<INV>(y[r], w[b * (R - 1) + r - 1]);
      }
      if constexpr (P == 0 && R == 12 && ZMID)
        dft12<INV, true>(y);
      else if constexpr (P == 0 && R == 16 && ZMID)
        dft16_outer<INV>(y);
      else
        dft<R, INV>(y);
#pragma unroll
      for (int r = 0; r < R; ++r) x[b * R + r] = y[r];
    }
  }

  // The outputs of pass P into the exchange area (the group's element i at
  // lds[slot T]), and from there the inputs of pass P + 1.
  template <int P>
  static __host__ __device__ __forceinline__ void put(const float2 (&x)[REGS], int t, float2* lds) {
    constexpr int R = radix(P), NS = ns(P);
    constexpr MixPad pd = pad<P>;
#pragma unroll
    for (int b = 0; b < rounds(P); ++b) {
      if (!active<P>(t, b)) continue;
      const unsigned j = t + G * b;
      const unsigned q = j / NS;  // block of NS R elements
      unsigned at = q * (NS * R) + (j - q * NS);
      if constexpr (pd.g1 > 0) at += NS * R >= pd.g1 ? q * (NS * R / pd.g1) : q / (pd.g1 / (NS * R) > 0 ? pd.g1 / (NS * R) : 1);
      if constexpr (pd.g2 > 0)
        at += pd.m * (NS * R >= pd.g2 ? q * (NS * R / pd.g2) : q / (pd.g2 / (NS * R) > 0 ? pd.g2 / (NS * R) : 1));
      float2* const p = lds + at * T;
#pragma unroll
      for (int r = 0; r < R; ++r) p[(r * NS + mix_spare(pd, r * NS)) * T] = x[b * R + r];
    }
  }
  template <int P>
  static __host__ __device__ __forceinline__ void get(float2 (&x)[REGS], int t, const float2* lds) {
    constexpr int R = radix(P), BF = bf(P);
    constexpr MixPad pd = pad<P - 1>;
#pragma unroll
    for (int b = 0; b < rounds(P); ++b) {
      if (!active<P>(t, b)) continue;
      const unsigned j = t + G * b;
      unsigned at = j;
      if constexpr (pd.g1 > 0) at += j / (pd.g1 > 0 ? pd.g1 : 1);
      if constexpr (pd.g2 > 0) at += pd.m * (j / (pd.g2 > 0 ? pd.g2 : 1));
      const float2* const p = lds + at * T;
#pragma unroll
      for (int r = 0; r < R; ++r) x[b * R + r] = p[(r * BF + mix_spare(pd, r * BF)) * T];
    }
  }
};

// The table of one axis: the inverse plan's twiddles, then the forward plan's.
template <class PLAN>
struct MixTables {
  using I = Mix<typename PLAN::I, 1, 1>;
  using F = Mix<typename PLAN::F, 1, 1>;
  static constexpr int F_OFF = I::TW, SIZE = I::TW + F::TW;
};

// Passes of one of an axis's two plans, for building its table (ns, radix and
// offset per pass; the first pass has no twiddles).
struct MixPassList {
  int npass, ns[5], radix[5], off[5], size;
};
template <class PLAN>
constexpr MixPassList mix_pass_list(bool forward) {
  using I = typename MixTables<PLAN>::I;
  using F = typename MixTables<PLAN>::F;
  MixPassList l{};
  l.npass = I::NPASS;
  for (int p = 0; p < I::NPASS; ++p) {
    l.ns[p] = forward ? F::ns(p) : I::ns(p);
    l.radix[p] = forward ? F::radix(p) : I::radix(p);
    l.off[p] = forward ? F::tw_off(p) : I::tw_off(p);
  }
  l.size = forward ? F::TW : I::TW;
  return l;
}
// full: the whole length (FullPlan) instead of 3/4 of it (MixPlan)
inline MixPassList mix_passes(int logn, bool forward, bool full = false) {
  if (full) {
    switch (logn) {
      case 4: return mix_pass_list<FullPlan<4>>(forward);
      case 5: return mix_pass_list<FullPlan<5>>(forward);
      case 6: return mix_pass_list<FullPlan<6>>(forward);
      default: return MixPassList{};
    }
  }
  switch (logn) {
    case 6: return mix_pass_list<MixPlan<6>>(forward);
    case 7: return mix_pass_list<MixPlan<7>>(forward);
    case 8: return mix_pass_list<MixPlan<8>>(forward);
    case 9: return mix_pass_list<MixPlan<9>>(forward);
    case 10: return mix_pass_list<MixPlan<10>>(forward);
    case 11: return mix_pass_list<MixPlan<11>>(forward);
    case 12: return mix_pass_list<MixPlan<12>>(forward);
    case 13: return mix_pass_list<MixPlan<13>>(forward);
    case 14: return mix_pass_list<MixPlan<14>>(forward);
    default: return MixPassList{};
  }
}
inline int mix_tables_size(int logn, bool full = false) {
  return mix_passes(logn, false, full).size + mix_passes(logn, true, full).size;
}
inline void build_mix_tables(int logn, float2* out, bool full = false) {
  for (int dir = 0; dir < 2; ++dir) {
    const MixPassList l = mix_passes(logn, dir == 1, full);
    for (int p = 1; p < l.npass; ++p) build_twiddle_pass(l.ns[p], l.radix[p], out + l.off[p]);
    out += l.size;
  }
}

}  // namespace ff
