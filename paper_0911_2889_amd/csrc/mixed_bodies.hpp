// Bodies of the step's kernels on the product grids (3 N1/4 theta rows, 3 N2/4
// phi points), with the mixed-radix transforms of mixed_fft.hpp: one
// workgroup's work on one column tile or one group of row pairs of a flame.
// The kernels of mixed_kernels.hip run one body per workgroup; the persistent
// ensemble kernel (ensemble_kernel.hip) runs many, one after another.

#pragma once

#include <hip/hip_runtime.h>

#include "flame_dev.hpp"
#include "kernel_common.hpp"
#include "mixed_fft.hpp"

namespace flame {

// Lanes per transform: L/12 of them, so that the radix-12 pass is one
// butterfly per lane; half as many at 8192 points, where every pass of
// 12 * 8 * 8 * 8 then fills its lanes (2 and 3 butterflies each) and two
// workgroups of 256 threads share a compute unit instead of one of 512.
constexpr int mix_lanes(int logn) { return (1 << logn) / (logn == 13 ? 32 : 16); }

// Lanes per transform of 8192 points where there are few: one butterfly each
// in the radix-8 passes (the radix-12 pass leaves 4 of the 12 waves idle). A
// compute unit has one transform at a time, of 768 lanes rather than 512: 8192x16
// column kernel 16.0 -> 15.6 us (15.2 with its inverse's twiddles loaded late),
// 16x8192 row kernel 13.3 -> 12.6. (Plans of 16, 16, 4 and 6 points took 15.0
// and 12.6. Both inverse transforms of a column pass by pass, in the same waits:
// 16.0.)
constexpr int kFewLanes13 = 768;

// Whether a transform's exchanges alternate between two areas, so that each
// needs one workgroup barrier instead of two: for that workgroup, whose
// barriers are idle time. Measured: 8192x16 column kernel 17.0 -> 15.6 us,
// 16x8192 row kernel 13.9 -> 12.8.
constexpr bool mix_two_areas(int logn, int g) { return logn == 13 && g == kFewLanes13; }

// Column kernel: G lanes and T columns as the N1-row kernels (ColCfg).
template <int LOGN1, int G_ = mix_lanes(LOGN1)>
struct ColMix {
  static constexpr int N1 = 1 << LOGN1, NB = N1 / 16;
  static constexpr int G = G_, RB = G > NB ? 1 : NB / G;  // RB: radix-12 butterflies per lane (lanes t >= NB: none)
  static constexpr int T = col_tile_for(NB), TQ = q_tile_for(NB), QS = ff::ilog2c(TQ);
  using F = ff::Mix<typename ff::MixPlan<LOGN1>::F, G, T>;
  using I = ff::Mix<typename ff::MixPlan<LOGN1>::I, G, T>;
  static constexpr int L = F::N;
  static constexpr int THREADS = G * T;
  static constexpr bool TWO = mix_two_areas(LOGN1, G);
  static constexpr int AREA = F::LDS > I::LDS ? F::LDS : I::LDS;
  static constexpr int LDS_BYTES = 8 * (TWO ? 2 : 1) * AREA;
  static constexpr int WPE = COL_WAVES_PER_EU;
};

// Row kernel: G lanes per row pair, B pairs interleaved.
template <int LOGN2, int G_ = mix_lanes(LOGN2)>
struct RowMix {
  static constexpr int N2 = 1 << LOGN2, NB = N2 / 16;
  static constexpr int G = G_, RB = G > NB ? 1 : NB / G;
  static constexpr int B = NB >= 256 ? 1 : 256 / NB;
  using F = ff::Mix<typename ff::MixPlan<LOGN2>::F, G, B>;
  using I = ff::Mix<typename ff::MixPlan<LOGN2>::I, G, B>;
  static constexpr int L = F::N;
  static constexpr int THREADS = G * B;
  static constexpr bool TWO = mix_two_areas(LOGN2, G);
  static constexpr int AREA = F::LDS > I::LDS ? F::LDS : I::LDS;
  static constexpr int LDS_BYTES = 8 * (TWO ? 2 : 1) * AREA;
  static constexpr int WPE = LOGN2 >= 13 ? 2 : ROW_WAVES_PER_EU;
};

// Twiddles of one transform of a kernel: held in registers from the kernel's
// start (its inverse transforms run twice), or read from the table by each
// pass while it waits for the exchange before it. At 16384 a workgroup is
// 1024 threads of at most 128 registers, which cannot hold them.
template <class M, bool HELD>
struct MixTw {
  static constexpr int first(int p) { return p <= 1 ? 0 : first(p - 1) + M::tw_count(p - 1); }
  GlobalFetch fetch;
  int t;
  float2 w[HELD && M::NPASS > 1 ? first(M::NPASS) : 1];
  __device__ __forceinline__ MixTw() {}
  __device__ __forceinline__ MixTw(const float2* table, int t_) { init(table, t_); }
  __device__ __forceinline__ void init(const float2* table, int t_) {
    fetch = GlobalFetch{(const gf2*)table};
    t = t_;
    if constexpr (HELD) load<1>();
  }
  template <int P>
  __device__ __forceinline__ void load() {
    if constexpr (P < M::NPASS) {
      float2 v[M::tw_count(P)];
      M::template load_twiddles<P>(v, fetch, t);
#pragma unroll
      for (int i = 0; i < M::tw_count(P); ++i) w[first(P) + i] = v[i];
      load<P + 1>();
    }
  }
  template <int P>
  __device__ __forceinline__ void pass(float2 (&v)[M::tw_count(P)]) const {
    if constexpr (P > 0 && HELD) {
#pragma unroll
      for (int i = 0; i < M::tw_count(P); ++i) v[i] = w[first(P) + i];
    } else if constexpr (P > 0) {
      // a pointer the compiler cannot follow, so that it does not keep one
      // transform's twiddles in registers for the next
      const gf2* tab = fetch.tw;
      asm volatile("" : "+s"(tab));
      M::template load_twiddles<P>(v, GlobalFetch{tab}, t);
    }
  }
};
// Rows (logn, g: the transform's 2^logn and its lanes): reading them late costs
// 3 % of the row kernel at 2048x4096.
constexpr bool mix_held(int logn, int g) { return logn < 13 || (logn == 13 && g == kFewLanes13); }
// Columns: up to 1024 points the registers are worth more as further waves
// (32 flames of 512x1024: column kernel 25.6 -> 24.0 us).
constexpr bool mix_held_col(int logn, int g) { return logn > 10 && mix_held(logn, g); }

// Run passes P.. of a transform whose pass-P inputs are in x (every thread of
// the workgroup calls it: it contains workgroup barriers; the last one is
// before the last pass, after every read of the exchange area).
template <class M, bool INV, bool ZMID, int P = 0, class TW>
__device__ __forceinline__ void mix_fft(float2 (&x)[M::REGS], float2* lds, const TW& tw,
                                        const float2 (&w)[M::tw_count(P)]) {
  M::template butterflies<P, INV, ZMID>(x, tw.t, w);
  if constexpr (P + 1 < M::NPASS) {
    M::template put<P>(x, tw.t, lds);
    float2 next[M::tw_count(P + 1)];
    tw.template pass<P + 1>(next);
    __syncthreads();
    M::template get<P + 1>(x, tw.t, lds);
    __syncthreads();
    mix_fft<M, INV, ZMID, P + 1>(x, lds, tw, next);
  }
}
template <class M, bool INV, bool ZMID, class TW>
__device__ __forceinline__ void mix_fft(float2 (&x)[M::REGS], float2* lds, const TW& tw) {
  const float2 none[1] = {make_float2(0.f, 0.f)};
  mix_fft<M, INV, ZMID, 0>(x, lds, tw, none);
}

// The same with exchange P in area a (P even) or b (P odd). A thread's reads
// of one area are over before the barrier of the next exchange, so that area
// may be written after it; the next transform starts with the area that this
// one's last exchange did not use.
template <class M, bool INV, bool ZMID, int P = 0, class TW>
__device__ __forceinline__ void mix_fft2(float2 (&x)[M::REGS], float2* a, float2* b, const TW& tw,
                                         const float2 (&w)[M::tw_count(P)]) {
  static_assert(M::NPASS % 2 == 0, "the first and the last exchange use the same area");
  M::template butterflies<P, INV, ZMID>(x, tw.t, w);
  if constexpr (P + 1 < M::NPASS) {
    M::template put<P>(x, tw.t, a);
    float2 next[M::tw_count(P + 1)];
    tw.template pass<P + 1>(next);
    __syncthreads();
    M::template get<P + 1>(x, tw.t, a);
    mix_fft2<M, INV, ZMID, P + 1>(x, b, a, tw, next);
  }
}
// One area (b unused, every exchange in a) or two.
template <class M, bool INV, bool ZMID, bool TWO, class TW>
__device__ __forceinline__ void mix_fft_in(float2 (&x)[M::REGS], float2* a, float2* b, const TW& tw) {
  const float2 none[1] = {make_float2(0.f, 0.f)};
  if constexpr (TWO)
    mix_fft2<M, INV, ZMID, 0>(x, a, b, tw, none);
  else
    mix_fft<M, INV, ZMID, 0>(x, a, tw, none);
}

// One column tile of the step (COL_STEP), or the column transforms of a
// spectrum (COL_FIRST: src, or the state).
template <int LOGN1, int MODE, int SV, int G_ = mix_lanes(LOGN1)>
__device__ __forceinline__ void colm_body(const FlameDev& f, long long n, const float2* src, int tile, int tid) {
  constexpr int VAR = SV & ~VAR_NT;
  constexpr bool NT = MODE == COL_STEP && (SV & VAR_NT) != 0;
  static_assert(MODE == COL_STEP || MODE == COL_FIRST, "step modes only");
  using C = ColMix<LOGN1, G_>;
  using F = typename C::F;
  using I = typename C::I;
  constexpr int T = C::T, G = C::G, NB = C::NB, RB = C::RB, L = C::L, N1 = C::N1, TQ = C::TQ, QS = C::QS;
  extern __shared__ float2 lds[];
  const int c = tid % T, t = tid / T;
  const bool act = G <= NB || t < NB;  // lanes of the radix-12 pass; the others read lane 0's modes (unused)
  const int jt = act ? t : 0;
  const int m = tile * T + c;
  const bool live = m < f.m;
  float2* const my = lds + c;
  float2* const my2 = my + (C::TWO ? C::AREA : 0);
  gf2* const Sc = glob(MODE == COL_FIRST && src ? const_cast<float2*>(src) : f.S) + (size_t)m * f.h1 + N1 / 4;
  // kept mode i = 8 b + kk of this lane, in butterfly t + G b of the radix-12
  // pass: k1 = t + G b + NB kk >= 0 for kk < 4, then t + G b - NB (8 - kk) < 0;
  // it is input or output kk, or kk + 4, of that butterfly
  auto k1_of = [&](int i) { return jt + G * (i >> 3) + NB * ((i & 7) < 4 ? (i & 7) : (i & 7) - 8); };
  auto reg_of = [](int i) { return 12 * (i >> 3) + ((i & 7) < 4 ? (i & 7) : (i & 7) + 4); };
  constexpr int KEEP = 8 * RB;

  float2 sv[KEEP];
  MixTw<I, mix_held_col(LOGN1, G_)> wi;
  if constexpr (MODE == COL_STEP) {
    gf2* const Qc = glob(f.Q) + ((((size_t)m >> QS) * L) << QS) + (m & (TQ - 1));  // column m: Qc[j1 * TQ]
    gf2* const Pc = glob(VAR >= VAR_HEUN_P ? f.S2 : f.S) + (size_t)m * f.h1 + N1 / 4;  // Heun's predictor
    // The loads carry no condition that depends on the column, so that no
    // branch between them makes one wait for another: a column past the grid
    // reads its padded slots of Q and column 0 of the state (its results are
    // never stored). Waves that a partly idle round leaves out skip theirs.
    const int ms = live ? m : 0;
    gf2* const Sl = glob(f.S) + (size_t)ms * f.h1 + N1 / 4;
    gf2* const Pl = glob(VAR >= VAR_HEUN_P ? f.S2 : f.S) + (size_t)ms * f.h1 + N1 / 4;
    float2 v[F::REGS];
#pragma unroll
    for (int b = 0; b < F::rounds(0); ++b)
      if (F::template active<0>(t, b)) {
#pragma unroll
        for (int r = 0; r < F::radix(0); ++r) v[b * F::radix(0) + r] = ld(Qc + (t + G * b + r * F::bf(0)) * TQ);
      }
    constexpr bool FORCED = VAR != VAR_EULER;
    float2 old[KEEP], frc[KEEP], prd[KEEP];
#pragma unroll
    for (int kk = 0; kk < KEEP; ++kk) {
      old[kk] = ld(Sl + k1_of(kk));
      frc[kk] = FORCED ? forcing_at(f, ms, k1_of(kk)) : make_float2(0.f, 0.f);
      prd[kk] = VAR == VAR_HEUN_C ? ld(Pl + k1_of(kk)) : make_float2(0.f, 0.f);
    }
    const MixTw<F, mix_held_col(LOGN1, G_)> wf(f.twma + ff::MixTables<ff::MixPlan<LOGN1>>::F_OFF, t);
    mix_fft_in<F, false, false, C::TWO>(v, my, my2, wf);
    // The inverse's twiddles are loaded here, not beside the forward's: a
    // workgroup's loads of both tables before its first transform are as long as
    // those of its column (2048x4096 column kernel 17.4 -> 17.0 us, 4096x2048
    // 18.4 -> 17.9, 8192x16 15.6 -> 15.2).
    wi.init(f.twma, t);
    const StepScalars sc = step_scalars(f, n, L, f.cols);
    const float ac = VAR == VAR_HEUN_C ? step_scalars(f, n + 1, L, f.cols).a : 0.f;  // the corrector's dt c_{n+1} / P
    const float kap2c = f.s2 * (float)m;
    const float dtf = (float)f.dt;
#pragma unroll
    for (int kk = 0; kk < KEEP; ++kk) {
      const int k1 = k1_of(kk);
      const float2 q = v[reg_of(kk)];
      const float kap1 = f.s1 * (float)k1;
      const float e = growth_factor(norm2(kap1, kap2c), sc, f.gamma);
      float2 val = update_mode<VAR>(e, old[kk], q, frc[kk], prd[kk], sc.a, ac, dtf);
      if (kk == 4 && jt == 0) val = make_float2(0.f, 0.f);  // k1 = -N1/4 lies outside the box
      sv[kk] = val;
    }
    if (tile == 0) {
      // symmetrise column k2 = 0 (group c == 0): copy k1 > 0 conjugated onto -k1
      if (c == 0 && act) {
#pragma unroll
        for (int kk = 0; kk < KEEP; ++kk)
          if ((kk & 7) < 4) my2[k1_of(kk)] = sv[kk];
      }
      __syncthreads();
      if (c == 0 && act) {
#pragma unroll
        for (int kk = 0; kk < KEEP; ++kk)
          if ((kk & 7) >= 4 && k1_of(kk) > -N1 / 4) sv[kk] = ff::cconj(my2[-k1_of(kk)]);
        if (t == 0) sv[0].y = 0.f;
      }
      __syncthreads();
    }
    if (live && act) {
      gf2* const Dc = VAR == VAR_HEUN_P ? Pc : Sc;  // the predictor goes to S2
#pragma unroll
      for (int kk = 0; kk < KEEP; ++kk) st(Dc + k1_of(kk), sv[kk]);
    }
  } else {
#pragma unroll
    for (int kk = 0; kk < KEEP; ++kk) sv[kk] = live ? ld(Sc + k1_of(kk)) : make_float2(0.f, 0.f);
  }

  if (MODE == COL_FIRST) wi.init(f.twma, t);
  const float kap2 = f.s2 * (float)m;
  gf2* const Wpc = glob(f.Wp);
  gf2* const Wmc = glob(f.Wm);
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    // pass 0: Z+ = IFFT_k1((i kappa1 - kappa2) Phi~) -> Wp; pass 1: conj(IFFT_k1((i kappa1 + kappa2) Phi~)) -> Wm
    const float kp = pass == 0 ? -kap2 : kap2;
    float2 v[I::REGS];
#pragma unroll
    for (int kk = 0; kk < KEEP; ++kk) {
      const float kap1 = f.s1 * (float)k1_of(kk);
      v[reg_of(kk)] = slope(kap1, kp, sv[kk]);
    }
    mix_fft_in<I, true, true, C::TWO>(v, pass == 0 ? my2 : my, pass == 0 ? my : my2, wi);
    if (live) {
      constexpr int P = I::NPASS - 1, R = I::radix(P);
#pragma unroll
      for (int b = 0; b < I::rounds(P); ++b)
        if (I::template active<P>(t, b)) {
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const int j1 = t + G * b + r * I::bf(P);
            if (pass == 0)
              st_nt<NT>(Wpc + w_index(j1, m, f.m), v[b * R + r]);
            else
              st_nt<NT>(Wmc + w_index(j1, m, f.m), ff::cconj(v[b * R + r]));
          }
        }
    }
  }
}

// One group of row pairs of the step: the quadratic term on 3 N2/4 phi points.
template <int LOGN2, bool NT, int G_ = mix_lanes(LOGN2)>
__device__ __forceinline__ void rowm_body(const FlameDev& f, int group, int tid) {
  using C = RowMix<LOGN2, G_>;
  using F = typename C::F;
  using I = typename C::I;
  constexpr int B = C::B, G = C::G, NB = C::NB, RB = C::RB;
  extern __shared__ float2 lds[];
  const int p = tid % B, t = tid / B;
  const bool act = G <= NB || t < NB;  // as colm_body
  const int jt = act ? t : 0;
  const int pair = group * B + p;
  const int n1 = f.rows, ts = f.tshift, mcols = f.m;
  const bool live = pair < n1 / 2;
  const int ja = 2 * pair, jb = 2 * pair + 1;
  float2* const my = lds + p;
  float2* const my2 = my + (C::TWO ? C::AREA : 0);
  gf2* const Wp = glob(f.Wp);
  gf2* const Wm = glob(f.Wm);
  gf2* const Q = glob(f.Q);
  // both rows' inputs come in one 16-byte load per register (w_index layout),
  // without conditions: a pair past the grid reads pair 0 (its results are
  // never stored), and the one position past the box (k2 = -N2/4, at t = 0)
  // is read in bounds and zeroed once every load is issued
  float2 v[2][I::REGS];
  const int pl = live ? pair : 0;
  const int pbase4 = (pl >> 1) * mcols, poff = (pl & 1) << 1;
#pragma unroll
  for (int b = 0; b < RB; ++b) {
    const int j = jt + G * b;
#pragma unroll
    for (int r = 0; r < 4; ++r) ld_pair(Wp + (((pbase4 + j + NB * r) << 2) + poff), v[0][12 * b + r], v[1][12 * b + r]);
#pragma unroll
    for (int r = 8; r < 12; ++r) {
      const int mm = NB * (12 - r) - j;  // k2 = -mm; mm = mcols at r = 8, j = 0
      ld_pair(Wm + (((pbase4 + (r > 8 || b > 0 || jt > 0 ? mm : 0)) << 2) + poff), v[0][12 * b + r], v[1][12 * b + r]);
    }
  }
  const MixTw<I, mix_held(LOGN2, G_)> wi(f.twmb, t);
  v[0][8] = jt > 0 ? v[0][8] : make_float2(0.f, 0.f);  // b = 0, r = 8
  v[1][8] = jt > 0 ? v[1][8] : make_float2(0.f, 0.f);
  constexpr int PL = I::NPASS - 1;  // an inverse's last pass and the forward's first share their register map
  static_assert(I::radix(PL) == F::radix(0) && I::rounds(PL) == F::rounds(0), "forward plan = inverse plan reversed");
  constexpr int NV = I::rounds(PL) * I::radix(PL);
  float qa[NV];
  float2 y[F::REGS];
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    mix_fft_in<I, true, true, C::TWO>(v[half], half == 0 ? my : my2, half == 0 ? my2 : my, wi);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const float2 z = v[half][i];
      const float q = norm2(z.x, z.y);
      if (half == 0)
        qa[i] = q;
      else
        y[i] = make_float2(qa[i], q);
    }
  }
  mix_fft_in<F, false, false, C::TWO>(
      y, my, my2, MixTw<F, mix_held(LOGN2, G_)>(f.twmb + ff::MixTables<ff::MixPlan<LOGN2>>::F_OFF, t));
  // The forward transform of the two packed real rows, split by
  // Q_a(k) = (Y(k) + conj(Y(-k)))/2, Q_b(k) = (Y(k) - conj(Y(-k)))/(2i),
  // k = j + NB r in [0, K2] (r < 4): Y(-k) is output 11 - r of butterfly NB - j
  // (of this one, output 12 - r, for j = 0). Only those four go through LDS.
  static_assert(F::bf(F::NPASS - 1) == NB, "radix-12 last pass");
  if (act) {
#pragma unroll
    for (int b = 0; b < RB; ++b)
#pragma unroll
      for (int r = 8; r < 12; ++r) my2[(t + G * b + NB * (r - 8)) * B] = y[12 * b + r];
  }
  __syncthreads();
  if (live && act) {
#pragma unroll
    for (int b = 0; b < RB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int j = t + G * b, k = j + NB * r;
        const float2 yk = y[12 * b + r];
        // L - k = NB (12 - r) - j; k = 0 pairs with itself
        const float2 yo = my2[(NB * (4 - r) - j - (k == 0 ? 1 : 0)) * B];
        const float2 ym = k == 0 ? yk : yo;
        float2 qa2, qb2;
        split_pair(yk, ym, qa2, qb2);
        st_nt<NT>(Q + tiled(ja, k, n1, ts), qa2);
        st_nt<NT>(Q + tiled(jb, k, n1, ts), qb2);
      }
  }
}

// ------------------------------------------------------- few transforms
// Bodies for launches that leave most of the chip idle (split_pays): there a
// step's time is the length of the chain of loads, passes and exchanges, not
// the work. The two inverse transforms of a column (or of a row pair) run side
// by side on two groups of lanes, each in its own exchange area, and the
// forward transform on the lanes of both; up to 1024 points there are lanes
// enough for one butterfly per lane in every pass. A workgroup holds few
// transforms, so that more compute units take part. Every transform has the
// radices and the arithmetic of the bodies above, so the results are the same
// bit for bit. Measured against those bodies (one flame, us per row and column
// kernel): 256x512 7.5 + 7.5 -> 5.0 + 5.4, 512x1024 8.0 + 8.9 -> 5.8 + 5.4,
// 1024x2048 9.4 + 11.6 -> 9.0 + 9.4.
constexpr int kSplitThreads = 128;  // per workgroup; 64 and 256 were 0-2 % and 5-15 % slower
constexpr int split_lanes(int logn) { return (1 << logn) / (logn <= 10 ? 8 : 16); }

template <int LOGN1>
struct ColSplit {
  static constexpr int N1 = 1 << LOGN1, NB = N1 / 16;
  static constexpr int G = split_lanes(LOGN1), GF = 2 * G;  // lanes per inverse and per forward transform
  static constexpr int T = GF >= kSplitThreads ? 1 : kSplitThreads / GF;  // columns per workgroup
  static constexpr int TQ = q_tile_for(NB), QS = ff::ilog2c(TQ);
  using F = ff::Mix<typename ff::MixPlan<LOGN1>::F, GF, T>;
  using I = ff::Mix<typename ff::MixPlan<LOGN1>::I, G, T>;
  static constexpr int L = F::N;
  static constexpr int THREADS = GF * T;
  static constexpr int AREA = I::LDS;  // of one inverse transform's exchange
  static constexpr int LDS_BYTES = 8 * (F::LDS > 2 * AREA ? F::LDS : 2 * AREA);
};

template <int LOGN2>
struct RowSplit {
  static constexpr int N2 = 1 << LOGN2, NB = N2 / 16;
  static constexpr int G = split_lanes(LOGN2), GF = 2 * G;
  static constexpr int B = GF >= kSplitThreads ? 1 : kSplitThreads / GF;
  using F = ff::Mix<typename ff::MixPlan<LOGN2>::F, GF, B>;
  using I = ff::Mix<typename ff::MixPlan<LOGN2>::I, G, B>;
  static constexpr int L = F::N;
  static constexpr int THREADS = GF * B;
  static constexpr int AREA = I::LDS;
  static constexpr int LDS_BYTES = 8 * (F::LDS > 2 * AREA ? F::LDS : 2 * AREA);
};

template <int LOGN1, int MODE, int VAR>
__device__ __forceinline__ void cols_body(const FlameDev& f, long long n, const float2* src, int tile, int tid) {
  static_assert(MODE == COL_STEP || MODE == COL_FIRST, "step modes only");
  using C = ColSplit<LOGN1>;
  using F = typename C::F;
  using I = typename C::I;
  constexpr int T = C::T, G = C::G, GF = C::GF, NB = C::NB, L = C::L, N1 = C::N1, TQ = C::TQ, QS = C::QS;
  extern __shared__ float2 lds[];
  const int c = tid % T, u = tid / T;  // forward lane u; inverse transform h, lane t
  const int h = u / G, t = u % G;
  const int m = tile * T + c;
  const bool live = m < f.m;
  float2* const my = lds + c;
  gf2* const Sc = glob(MODE == COL_FIRST && src ? const_cast<float2*>(src) : f.S) + (size_t)m * f.h1 + N1 / 4;
  // kept mode kk = 0..7 of butterfly j of a radix-12 pass (j < NB)
  auto k1_of = [](int j, int kk) { return kk < 4 ? j + NB * kk : j - NB * (8 - kk); };
  const bool inv_act = G == NB || t < NB;  // lanes of an inverse transform's radix-12 pass
  MixTw<I, true> wi;
  float2 sv[8];
  if constexpr (MODE == COL_STEP) {
    gf2* const Qc = glob(f.Q) + ((((size_t)m >> QS) * L) << QS) + (m & (TQ - 1));
    gf2* const Pc = glob(VAR >= VAR_HEUN_P ? f.S2 : f.S) + (size_t)m * f.h1 + N1 / 4;
    const int ms = live ? m : 0;
    gf2* const Sl = glob(f.S) + (size_t)ms * f.h1 + N1 / 4;
    gf2* const Pl = glob(VAR >= VAR_HEUN_P ? f.S2 : f.S) + (size_t)ms * f.h1 + N1 / 4;
    float2 v[F::REGS];
#pragma unroll
    for (int b = 0; b < F::rounds(0); ++b)
      if (F::template active<0>(u, b)) {
#pragma unroll
        for (int r = 0; r < F::radix(0); ++r) v[b * F::radix(0) + r] = ld(Qc + (u + GF * b + r * F::bf(0)) * TQ);
      }
    constexpr bool FORCED = VAR != VAR_EULER;
    const int ju = u < NB ? u : 0;  // lanes past the radix-12 pass read lane 0's modes (unused)
    float2 old[8], frc[8], prd[8];
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      old[kk] = ld(Sl + k1_of(ju, kk));
      frc[kk] = FORCED ? forcing_at(f, ms, k1_of(ju, kk)) : make_float2(0.f, 0.f);
      prd[kk] = VAR == VAR_HEUN_C ? ld(Pl + k1_of(ju, kk)) : make_float2(0.f, 0.f);
    }
    mix_fft<F, false, false>(v, my, MixTw<F, true>(f.twma + ff::MixTables<ff::MixPlan<LOGN1>>::F_OFF, u));
    wi.init(f.twma, t);  // not before the forward transform (colm_body): 1024x2048 11.1 -> 9.8 us
    const StepScalars sc = step_scalars(f, n, L, f.cols);
    const float ac = VAR == VAR_HEUN_C ? step_scalars(f, n + 1, L, f.cols).a : 0.f;
    const float kap2c = f.s2 * (float)m;
    const float dtf = (float)f.dt;
    // the updated modes in order of kk, to both groups
    if (u < NB) {
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) {
        const int k1 = k1_of(u, kk);
        const float2 q = v[kk < 4 ? kk : kk + 4];
        const float kap1 = f.s1 * (float)k1;
        const float e = growth_factor(norm2(kap1, kap2c), sc, f.gamma);
        float2 val = update_mode<VAR>(e, old[kk], q, frc[kk], prd[kk], sc.a, ac, dtf);
        if (kk == 4 && u == 0) val = make_float2(0.f, 0.f);  // k1 = -N1/4 lies outside the box
        if (m == 0 && kk == 0 && u == 0) val.y = 0.f;
        my[(u + NB * kk) * T] = val;
      }
    }
    __syncthreads();
    if (inv_act) {
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) {
        sv[kk] = my[(t + NB * kk) * T];
        // column k2 = 0: the k1 > 0 half conjugated onto k1 < 0 (symmetrisation)
        if (kk >= 4 && m == 0 && k1_of(t, kk) > -N1 / 4) sv[kk] = ff::cconj(my[-k1_of(t, kk) * T]);
      }
    }
    __syncthreads();
    if (live && inv_act && h == 0) {
      gf2* const Dc = VAR == VAR_HEUN_P ? Pc : Sc;
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) st(Dc + k1_of(t, kk), sv[kk]);
    }
  } else {
    wi.init(f.twma, t);
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) sv[kk] = live && inv_act ? ld(Sc + k1_of(t, kk)) : make_float2(0.f, 0.f);
  }
  // group 0: Z+ = IFFT_k1((i kappa1 - kappa2) Phi~) -> Wp; group 1: conj(IFFT_k1((i kappa1 + kappa2) Phi~)) -> Wm
  const float kp = h == 0 ? -(f.s2 * (float)m) : f.s2 * (float)m;
  float2 v[I::REGS];
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) {
    const float kap1 = f.s1 * (float)k1_of(t, kk);
    v[kk < 4 ? kk : kk + 4] = slope(kap1, kp, sv[kk]);
  }
  mix_fft<I, true, true>(v, my + h * C::AREA, wi);
  if (live) {
    gf2* const dst = glob(h == 0 ? f.Wp : f.Wm);
    const float cs = h == 0 ? 1.f : -1.f;  // Wm holds the conjugate
    constexpr int P = I::NPASS - 1, R = I::radix(P);
#pragma unroll
    for (int b = 0; b < I::rounds(P); ++b)
      if (I::template active<P>(t, b)) {
#pragma unroll
        for (int r = 0; r < R; ++r)
          st(dst + w_index(t + G * b + r * I::bf(P), m, f.m), make_float2(v[b * R + r].x, cs * v[b * R + r].y));
      }
  }
}

template <int LOGN2>
__device__ __forceinline__ void rows_body(const FlameDev& f, int group, int tid) {
  using C = RowSplit<LOGN2>;
  using F = typename C::F;
  using I = typename C::I;
  constexpr int B = C::B, G = C::G, GF = C::GF, NB = C::NB;
  extern __shared__ float2 lds[];
  const int p = tid % B, u = tid / B;  // forward lane u; inverse transform of row h, lane t
  const int h = u / G, t = u % G;
  const int pair = group * B + p;
  const int n1 = f.rows, ts = f.tshift, mcols = f.m;
  const bool live = pair < n1 / 2;
  float2* const my = lds + p;
  gf2* const Q = glob(f.Q);
  float2 v[I::REGS];
  {
    const int row = live ? 2 * pair + h : h;  // a pair past the grid reads pair 0 (never stored)
    const int jt = G == NB || t < NB ? t : 0;  // lanes past the radix-12 pass read lane 0's inputs (unused)
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = ld(glob(f.Wp) + w_index(row, jt + NB * r, mcols));
#pragma unroll
    for (int r = 8; r < 12; ++r) {
      const int mm = NB * (12 - r) - jt;  // k2 = -mm; mm = mcols at r = 8, t = 0
      v[r] = ld(glob(f.Wm) + w_index(row, r > 8 || jt > 0 ? mm : 0, mcols));
    }
    const MixTw<I, true> wi(f.twmb, t);
    v[8] = jt > 0 ? v[8] : make_float2(0.f, 0.f);
    mix_fft<I, true, true>(v, my + h * C::AREA, wi);
  }
  const MixTw<F, true> wf(f.twmb + ff::MixTables<ff::MixPlan<LOGN2>>::F_OFF, u);
  {
    // |z|^2 of the two rows side by side, as the real and the imaginary part of the forward transform's input
    constexpr int P = I::NPASS - 1, R = I::radix(P);
    float* const qf = reinterpret_cast<float*>(my) + h;
#pragma unroll
    for (int b = 0; b < I::rounds(P); ++b)
      if (I::template active<P>(t, b)) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const float2 z = v[b * R + r];
          qf[2 * (t + G * b + r * I::bf(P)) * B] = norm2(z.x, z.y);
        }
      }
  }
  __syncthreads();
  float2 y[F::REGS];
#pragma unroll
  for (int b = 0; b < F::rounds(0); ++b)
    if (F::template active<0>(u, b)) {
#pragma unroll
      for (int r = 0; r < F::radix(0); ++r) y[b * F::radix(0) + r] = my[(u + GF * b + r * F::bf(0)) * B];
    }
  __syncthreads();
  mix_fft<F, false, false>(y, my, wf);
  // split by Hermitian symmetry, as rowm_body
  if (u < NB) {
#pragma unroll
    for (int r = 8; r < 12; ++r) my[(u + NB * (r - 8)) * B] = y[r];
  }
  __syncthreads();
  if (live && u < NB) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int k = u + NB * r;
      const float2 yk = y[r];
      const float2 yo = my[(NB * (4 - r) - u - (k == 0 ? 1 : 0)) * B];
      const float2 ym = k == 0 ? yk : yo;
      float2 qa2, qb2;
      split_pair(yk, ym, qa2, qb2);
      st(Q + tiled(2 * pair, k, n1, ts), qa2);
      st(Q + tiled(2 * pair + 1, k, n1, ts), qb2);
    }
  }
}

}  // namespace flame
