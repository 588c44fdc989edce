// Adjoint of the flame step and of the area functional (gfx950).
//
// Cotangents hold the Fourier coefficients of a real band-limited grid field
// (the gradient with respect to the grid values of Phi), in the state layout.
// For the step n -> n+1 (integrating-factor Euler)
//     Phi^{n+1} = E^n (Phi^n + dt c_n Pi |grad Phi^n|^2),
// the transpose of its Jacobian is
//     lambda^n = mu - 2 dt c_n Pi div(m grad Phi^n),   mu = E^n lambda^{n+1},
// with m the grid field of mu; E^n is a real even multiplier (self-adjoint),
// the projection Pi is self-adjoint, and the adjoint of the spectral gradient
// restricted to the box is -Pi div with div taken by the grid transform.
// The area excess J = (1/P) sum sqrt(1 + |grad Phi|^2/r0^2) - 1 has
//     dJ/dPhi = -Pi div( grad Phi / (P r0^2 sqrt(1 + |grad Phi|^2/r0^2)) ).
//
// One adjoint step is three kernels on the step's grid: adjm_col (3 N1/4 rows)
// or adj_col (N1 rows), and adjm_row (3 N2/4 phi points) or adj_row (N2):
//  * adj_col<ADJ_A>: mu = E lambda per column; column inverse transforms of mu
//    (-> Q) and of (i kappa1 -+ kappa2) Phi~^n (-> Wp, Wm, as the forward step);
//  * adj_row<ROW_ADJ>: per row pair, m (one packed real synthesis for two
//    rows), z = g1 + i g2, zeta = m z = w1 + i w2, forward row transform of
//    zeta split by Hermitian symmetry into the row transforms of w1 (-> A1)
//    and i kappa2 w2 (-> A2);
//  * adj_col<ADJ_C>: column forward transforms of A1 and A2, divergence
//    i kappa1 A1 + A2 on the box, lambda^n = mu - 2 dt c_n div / P.
// The seed uses adj_row<ROW_SEED> (zeta = z / (r0^2 sqrt(1 + x))) and
// adj_col<SEED_C> (lambda = -div / P^2) after the column transforms of the
// state.

#include <hip/hip_runtime.h>

#include "fft_engine.hpp"
#include "flame_dev.hpp"
#include "flame_kernels.hpp"
#include "kernel_common.hpp"
#include "mixed_bodies.hpp"
#include "transform_shapes.hpp"

namespace flame {

namespace {

__device__ __forceinline__ float efactor(const FlameDev& f, const StepScalars& sc, int k1, float kap2) {
  const float kap1 = f.s1 * (float)k1;
  const float kk2 = kap1 * kap1 + kap2 * kap2;
  return growth_factor(kk2, sc, f.gamma);
}

}  // namespace

template <int LOGN1, int MODE>
__global__ void __launch_bounds__(ColCfg<LOGN1>::THREADS) __attribute__((amdgpu_waves_per_eu(COL_WAVES_PER_EU)))
    adj_col_kernel(const FlameDev* __restrict__ fls, long long n, const float2* state, const float2* lam_in,
                   float2* lam_out) {
  using S = ff::Shape<LOGN1>;
  constexpr int G = S::G, T = ColCfg<LOGN1>::T, N1 = S::N;
  extern __shared__ float2 lds[];
  const FlameDev f = fls[blockIdx.y];
  const int tid = threadIdx.x;
  const int c = tid % T, t = tid / T;
  const int tile = xcd_swizzle(blockIdx.x, gridDim.x);
  const int m = tile * T + c;
  const bool live = m < f.m;
  float2* my = lds + c;
  constexpr int TQ = ColCfg<LOGN1>::TQ, QS = ColCfg<LOGN1>::QS;
  const size_t tile_base = ((((size_t)m >> QS) * N1) << QS) + (m & (TQ - 1));  // column m of Q, A1, A2
  const size_t col = (size_t)m * f.h1 + N1 / 4;  // element k1 of column m at col + k1
  // loads carry no condition (a branch around a load makes the compiler wait
  // for every load issued before it): a column past the grid reads column 0
  // of the spectra and its padded slots of A1 and A2, and is never stored
  const size_t coll = (size_t)(live ? m : 0) * f.h1 + N1 / 4;
  const auto tw1 = KernelTw<LOGN1>::make(f.tw1, t);
  const float kap2 = f.s2 * (float)m;

  float2 v[ff::kPts];
  float2 lam[8];
  if constexpr (MODE != SEED_C) {
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      const int i = kept_reg<LOGN1, ff::kPts>(kk);
      const int k1 = t + G * i - (i >= 12 ? N1 : 0);
      lam[kk] = ld(glob(const_cast<float2*>(lam_in)) + coll + k1);
    }
  }

  if constexpr (MODE == ADJ_A) {
    const StepScalars sc = step_scalars(f, n, f.n1, f.n2);
    float2 sv[8];
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      const int i = kept_reg<LOGN1, ff::kPts>(kk);
      const int k1 = t + G * i - (i >= 12 ? N1 : 0);
      sv[kk] = ld(glob(const_cast<float2*>(state)) + coll + k1);
    }
    // M = column synthesis of mu = E lambda  -> Q
#pragma unroll
    for (int i = 0; i < ff::kPts; ++i) v[i] = make_float2(0.f, 0.f);
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      const int i = kept_reg<LOGN1, ff::kPts>(kk);
      const int k1 = t + G * i - (i >= 12 ? N1 : 0);
      v[i] = ff::cscale(lam[kk], efactor(f, sc, k1, kap2));
    }
    fft<LOGN1, true, kPrune>(v, t, my, T, tw1);
    if (live) {
#pragma unroll
      for (int i = 0; i < ff::kPts; ++i) st(glob(f.Q) + tile_base + (t + G * i) * TQ, v[i]);
    }
    // Z+ and Z- of the state, exactly as the forward column kernel
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
      const float sgn = pass == 0 ? -1.f : 1.f;
#pragma unroll
      for (int i = 0; i < ff::kPts; ++i) v[i] = make_float2(0.f, 0.f);
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) {
        const int i = kept_reg<LOGN1, ff::kPts>(kk);
        const float kap1 = f.s1 * (float)(t + G * i - (i >= 12 ? N1 : 0));
        v[i] = make_float2(-kap1 * sv[kk].y + sgn * kap2 * sv[kk].x, kap1 * sv[kk].x + sgn * kap2 * sv[kk].y);
      }
      fft<LOGN1, true, kPrune>(v, t, my, T, tw1);
      if (live) {
        gf2* dst = glob(pass == 0 ? f.Wp : f.Wm);
#pragma unroll
        for (int i = 0; i < ff::kPts; ++i)
          st(dst + w_index(t + G * i, m, f.m), pass == 0 ? v[i] : ff::cconj(v[i]));
      }
    }
  } else {
    // forward column transforms of the row transforms of w1 and i kappa2 w2
    float2 u[8], w[8];
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
      gf2* srcp = glob(pass == 0 ? f.A1 : f.A2) + tile_base;
#pragma unroll
      for (int i = 0; i < ff::kPts; ++i) v[i] = ld(srcp + (t + G * i) * TQ);
      fft<LOGN1, false>(v, t, my, T, tw1);
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) (pass == 0 ? u : w)[kk] = v[kept_reg<LOGN1, ff::kPts>(kk)];
    }
    float2 out[8];
    const float inv_p = 1.0f / ((float)f.n1 * (float)f.n2);
    StepScalars sc{};
    if constexpr (MODE == ADJ_C) sc = step_scalars(f, n, f.n1, f.cols);
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      const int i = kept_reg<LOGN1, ff::kPts>(kk);
      const int k1 = t + G * i - (i >= 12 ? N1 : 0);
      const float kap1 = f.s1 * (float)k1;
      // raw divergence i kappa1 U1 + V2 (sums without the 1/P factors)
      const float2 div = make_float2(-kap1 * u[kk].y + w[kk].x, kap1 * u[kk].x + w[kk].y);
      float2 val;
      if constexpr (MODE == ADJ_C) {
        const float e = efactor(f, sc, k1, kap2);
        val = make_float2(e * lam[kk].x - 2.f * sc.a * div.x, e * lam[kk].y - 2.f * sc.a * div.y);
      } else {
        val = ff::cscale(div, -inv_p * inv_p);
      }
      if (k1 == -N1 / 4) val = make_float2(0.f, 0.f);
      out[kk] = val;
    }
    if (tile == 0) {  // symmetrise column k2 = 0: copy k1 > 0 conjugated onto -k1
      if (c == 0) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) lds[t + G * kk] = out[kk];
      }
      __syncthreads();
      if (c == 0) {
#pragma unroll
        for (int kk = 4; kk < 8; ++kk) {
          const int k1 = t + G * kept_reg<LOGN1, ff::kPts>(kk) - N1;
          if (k1 > -N1 / 4) out[kk] = ff::cconj(lds[-k1]);
        }
        if (t == 0) out[0].y = 0.f;
      }
      __syncthreads();
    }
    if (live) {
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) {
        const int i = kept_reg<LOGN1, ff::kPts>(kk);
        const int k1 = t + G * i - (i >= 12 ? N1 : 0);
        st(glob(lam_out) + col + k1, out[kk]);
      }
    }
  }
}

template <int LOGN1, int MODE, int NG>
__global__ void __launch_bounds__((AdjMix<LOGN1, NG>::THREADS))
    __attribute__((amdgpu_waves_per_eu(ADJ_ROW_WAVES_PER_EU)))
    adjm_col_kernel(const FlameDev* __restrict__ fls, long long n, const float2* state, const float2* lam_in,
                    float2* lam_out) {
  static_assert(MODE == ADJ_A || MODE == ADJ_C, "product-grid adjoint modes");
  using C = AdjMix<LOGN1, NG>;
  using F = typename C::F;
  using I = typename C::I;
  constexpr int G = C::G, T = C::T, NB = C::NB, L = C::L, N1 = C::N;
  constexpr int TQ = q_tile_for(NB), QS = ff::ilog2c(TQ);
  extern __shared__ float2 lds[];
  const FlameDev f = fls[blockIdx.y];
  const int tid = threadIdx.x;
  const int c = tid % T, u = tid / T;
  const int h = u / G, t = u % G;
  const int tile = xcd_swizzle(blockIdx.x, gridDim.x);
  const int m = tile * T + c;
  const bool live = m < f.m;
  const bool act = G == NB || t < NB;  // lanes of the radix-12 pass
  float2* const my = lds + c + h * C::AREA;
  float2* const my2 = my + (C::TWO ? C::AREA : 0);
  const size_t tile_base = ((((size_t)m >> QS) * L) << QS) + (m & (TQ - 1));  // column m of Q, A1, A2
  const size_t col = (size_t)m * f.h1 + N1 / 4;  // element k1 of column m at col + k1
  // loads carry no condition (a branch around a load makes the compiler wait
  // for every load issued before it): a column past the grid reads column 0
  // of the spectra and its padded slots of A1 and A2, and is never stored
  const size_t coll = (size_t)(live ? m : 0) * f.h1 + N1 / 4;
  const float kap2 = f.s2 * (float)m;
  const StepScalars sc = step_scalars(f, n, L, f.cols);
  // 1024 threads of 128 registers: what a transform does not need is loaded after it
  constexpr bool LATE = LOGN1 == 14;
  const int jt = act ? t : 0;
  auto k1_of = [&](int kk) { return kk < 4 ? jt + NB * kk : jt - NB * (8 - kk); };
  gf2* const lin = glob(const_cast<float2*>(lam_in));

  if constexpr (MODE == ADJ_A) {
    // job 0: the column synthesis of mu = E lambda -> Q; jobs 1 and 2: Z+ and
    // Z- of the state, as the forward column kernel -> Wp, Wm
    float2 lm[8], sv[8];
    gf2* const one = NG == 1 || h == 0 ? lin : glob(const_cast<float2*>(state));
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) lm[kk] = ld(one + coll + k1_of(kk));
    auto load_state = [&] {
#pragma unroll
      for (int kk = 0; kk < 8; ++kk)
        sv[kk] = NG == 1 ? ld(glob(const_cast<float2*>(state)) + coll + k1_of(kk)) : lm[kk];
    };
    if (!LATE) load_state();
    const MixTw<I, C::HELD> tw(f.twma, t);
#pragma unroll
    for (int q = 0; q < (NG == 1 ? 3 : 1); ++q) {
      const int job = NG == 1 ? q : h;
      if (LATE && q == 1) load_state();
      const float kp = job == 1 ? -kap2 : kap2;
      float2 v[I::REGS];
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) {
        const int k1 = k1_of(kk);
        const float kap1 = f.s1 * (float)k1;
        const int i = kk < 4 ? kk : kk + 4;
        if (NG > 1 || q == 0) v[i] = ff::cscale(lm[kk], efactor(f, sc, k1, kap2));
        if (NG > 1 || q > 0) v[i] = NG > 1 && job == 0 ? v[i] : slope(kap1, kp, sv[kk]);
      }
      mix_fft_in<I, true, true, C::TWO>(v, q & 1 ? my2 : my, q & 1 ? my : my2, tw);
      if (live) {
        constexpr int P = I::NPASS - 1, R = I::radix(P);
        gf2* const wd = glob(job == 1 ? f.Wp : f.Wm);
        const float cs = job == 1 ? 1.f : -1.f;  // Wm holds the conjugate
#pragma unroll
        for (int b = 0; b < I::rounds(P); ++b)
          if (I::template active<P>(t, b)) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
              const int j1 = t + G * b + r * I::bf(P);
              const float2 x = v[b * R + r];
              if (job == 0)
                st(glob(f.Q) + tile_base + (size_t)j1 * TQ, x);
              else
                st(wd + w_index(j1, m, f.m), make_float2(x.x, cs * x.y));
            }
          }
      }
    }
  } else {
    // forward column transforms of the row transforms of w1 (job 0) and i kappa2 w2 (job 1)
    float2 lam[8], u1[8], w2[8];
#pragma unroll
    for (int kk = 0; kk < 8; ++kk)
      if (!LATE) lam[kk] = ld(lin + coll + k1_of(kk));
    const MixTw<F, C::HELD> tw(f.twma + ff::MixTables<ff::MixPlan<LOGN1>>::F_OFF, t);
#pragma unroll
    for (int q = 0; q < (NG == 1 ? 2 : 1); ++q) {
      const int job = NG == 1 ? q : h;
      gf2* const srcp = glob(job == 0 ? f.A1 : f.A2) + tile_base;
      float2 v[F::REGS];
#pragma unroll
      for (int b = 0; b < F::rounds(0); ++b)
        if (F::template active<0>(t, b)) {
#pragma unroll
          for (int r = 0; r < F::radix(0); ++r)
            v[b * F::radix(0) + r] = ld(srcp + (size_t)(t + G * b + r * F::bf(0)) * TQ);
        }
      mix_fft_in<F, false, false, C::TWO>(v, q & 1 ? my2 : my, q & 1 ? my : my2, tw);
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) (q == 0 ? u1 : w2)[kk] = v[kk < 4 ? kk : kk + 4];
    }
    if constexpr (NG == 2) {  // the second transform's modes to the first group
      if (h == 1 && act) {
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) my[(t + NB * kk) * T] = u1[kk];
      }
      __syncthreads();
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) w2[kk] = lds[c + C::AREA + (jt + NB * kk) * T];
    }
    if (LATE) {
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) lam[kk] = ld(lin + coll + k1_of(kk));
    }
    float2 out[8];
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      const int k1 = k1_of(kk);
      const float kap1 = f.s1 * (float)k1;
      // raw divergence i kappa1 U1 + V2 (sums without the 1/P factors)
      const float2 div = make_float2(-kap1 * u1[kk].y + w2[kk].x, kap1 * u1[kk].x + w2[kk].y);
      const float e = efactor(f, sc, k1, kap2);
      out[kk] = make_float2(e * lam[kk].x - 2.f * sc.a * div.x, e * lam[kk].y - 2.f * sc.a * div.y);
      if (kk == 4 && t == 0) out[kk] = make_float2(0.f, 0.f);  // k1 = -N1/4 lies outside the box
    }
    if (tile == 0) {  // symmetrise column k2 = 0: copy k1 > 0 conjugated onto -k1
      float2* const sym = lds;  // the first group's area; every read of it is behind a barrier
      if (m == 0 && h == 0 && act) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) sym[k1_of(kk)] = out[kk];
      }
      __syncthreads();
      if (m == 0 && h == 0 && act) {
#pragma unroll
        for (int kk = 4; kk < 8; ++kk)
          if (k1_of(kk) > -N1 / 4) out[kk] = ff::cconj(sym[-k1_of(kk)]);
        if (t == 0) out[0].y = 0.f;
      }
    }
    if (live && act && h == 0) {
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) st(glob(lam_out) + col + k1_of(kk), out[kk]);
    }
  }
}

// ROW_ADJ on 3 N2/4 phi points: per row pair m (both rows in one packed real
// synthesis, job 0), z = g1 + i g2 of each row (jobs 1 and 2), zeta = m z, and
// the forward transforms of the two zetas.
template <int LOGN2, int NG>
__global__ void __launch_bounds__((AdjMix<LOGN2, NG>::THREADS))
    __attribute__((amdgpu_waves_per_eu(ADJ_ROW_WAVES_PER_EU)))
    adjm_row_kernel(const FlameDev* __restrict__ fls) {
  using C = AdjMix<LOGN2, NG>;
  using F = typename C::F;
  using I = typename C::I;
  constexpr int G = C::G, B = C::T, NB = C::NB;
  static_assert(I::radix(I::NPASS - 1) == F::radix(0) && I::rounds(I::NPASS - 1) == F::rounds(0),
                "an inverse's last pass and the forward's first share their register map");
  extern __shared__ float2 lds[];
  const FlameDev f = fls[blockIdx.y];
  const int tid = threadIdx.x;
  const int p = tid % B, u = tid / B;
  const int h = u / G, t = u % G;
  const int pair = xcd_swizzle(blockIdx.x, gridDim.x) * B + p;
  const int n1 = f.rows, ts = f.tshift, mcols = f.m;
  const bool live = pair < n1 / 2;
  const int ja = live ? 2 * pair : 0;  // a pair past the grid reads pair 0 (never stored)
  float2* const my = lds + p + h * C::AREA;
  float2* const my2 = my + (C::TWO ? C::AREA : 0);
  const bool act = G == NB || t < NB;
  const int jt = act ? t : 0;
  gf2* const Wp = glob(f.Wp);
  gf2* const Wm = glob(f.Wm);
  gf2* const Q = glob(f.Q);
  auto load_z = [&](float2(&v)[I::REGS], int row) {
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = ld(Wp + w_index(row, jt + NB * r, mcols));
#pragma unroll
    for (int r = 8; r < 12; ++r) {
      const int mm = NB * (12 - r) - jt;  // k2 = -mm; mm = mcols at r = 8, t = 0
      v[r] = ld(Wm + w_index(row, r > 8 || jt > 0 ? mm : 0, mcols));
    }
  };
  auto load_m = [&](float2(&v)[I::REGS]) {
    // Y = X_a + i X_b, X(k2) = M(k2), X(-k2) = conj(M(k2))
#pragma unroll
    for (int r = 0; r < 12; ++r) {
      if (r >= 4 && r < 8) continue;
      const int mm = NB * (12 - r) - jt;
      const int k = r < 4 ? jt + NB * r : (r > 8 || jt > 0 ? mm : 0);
      const float2 a = ld(Q + tiled(ja, k, n1, ts)), b = ld(Q + tiled(ja + 1, k, n1, ts));
      v[r] = r < 4 ? make_float2(a.x - b.y, a.y + b.x) : make_float2(a.x + b.y, -a.y + b.x);
    }
  };
  // forward transform of zeta and its split by Hermitian symmetry: the row
  // transform of w1, (Xi(k) + conj(Xi(-k)))/2 -> A1, and of i kappa2 w2,
  // kappa2 (Xi(k) - conj(Xi(-k)))/2 -> A2 (outputs as in rowm_body)
  auto forward = [&](float2(&y)[F::REGS], const MixTw<F, C::HELD_ROW>& wf, bool store, int row, float2* a,
                     float2* b) {
    mix_fft_in<F, false, false, C::TWO>(y, a, b, wf);
    float2* const ex = C::TWO ? b : a;  // free once every lane has passed the last exchange's barrier
    if (act) {
#pragma unroll
      for (int r = 8; r < 12; ++r) ex[(t + NB * (r - 8)) * B] = y[r];
    }
    __syncthreads();
    if (store && act) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int k = t + NB * r;
        const float2 xk = y[r];
        const float2 xo = ex[(NB * (4 - r) - t - (k == 0 ? 1 : 0)) * B];
        const float2 xm = k == 0 ? xk : xo;
        const float hk = 0.5f * f.s2 * (float)k;
        st(glob(f.A1) + tiled(row, k, n1, ts), make_float2(0.5f * (xk.x + xm.x), 0.5f * (xk.y - xm.y)));
        st(glob(f.A2) + tiled(row, k, n1, ts), make_float2(hk * (xk.x - xm.x), hk * (xk.y + xm.y)));
      }
    }
  };
  constexpr int P = I::NPASS - 1, R = I::radix(P), NV = I::rounds(P) * R;
  const MixTw<I, C::HELD_ROW> wi(f.twmb, t);
  const float2* const ftab = f.twmb + ff::MixTables<ff::MixPlan<LOGN2>>::F_OFF;
  if constexpr (NG == 3) {
    float2 v[I::REGS];
    if (h == 0)
      load_m(v);
    else
      load_z(v, ja + h - 1);
    v[8] = jt > 0 ? v[8] : make_float2(0.f, 0.f);  // the position past the box
    mix_fft<I, true, true>(v, my, wi);
    const MixTw<F, C::HELD_ROW> wf(ftab, t);
    // m to the groups of the two rows, in the first group's area
    float2* const ms = lds + p;
    if (h == 0) {
#pragma unroll
      for (int b = 0; b < I::rounds(P); ++b)
        if (I::template active<P>(t, b)) {
#pragma unroll
          for (int r = 0; r < R; ++r) ms[(t + G * b + r * I::bf(P)) * B] = v[b * R + r];
        }
    }
    __syncthreads();
    float2 y[F::REGS];
#pragma unroll
    for (int b = 0; b < I::rounds(P); ++b)
      if (I::template active<P>(t, b)) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const float2 mm = ms[(t + G * b + r * I::bf(P)) * B];
          y[b * R + r] = ff::cscale(v[b * R + r], h == 1 ? mm.x : mm.y);
        }
      }
    __syncthreads();  // the first group's forward pass, which nobody reads, writes its area
    forward(y, wf, live && h > 0, ja + h - 1, my, my2);
  } else {
    float2 v[I::REGS], z[2][I::REGS];
    // both rows' values in one 16-byte load (8192x8192 adjoint step 640 -> 627 us)
#pragma unroll
    for (int r = 0; r < 4; ++r) ld_pair(Wp + w_index(ja, jt + NB * r, mcols), z[0][r], z[1][r]);
#pragma unroll
    for (int r = 8; r < 12; ++r) {
      const int mm = NB * (12 - r) - jt;  // as load_z
      ld_pair(Wm + w_index(ja, r > 8 || jt > 0 ? mm : 0, mcols), z[0][r], z[1][r]);
    }
    load_m(v);
    v[8] = jt > 0 ? v[8] : make_float2(0.f, 0.f);
    mix_fft_in<I, true, true, C::TWO>(v, my, my2, wi);
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      z[half][8] = jt > 0 ? z[half][8] : make_float2(0.f, 0.f);
      // the areas alternate over the transforms; a forward one's split takes the one its last exchange left
      float2 *const a = half == 0 ? my : my2, *const b = half == 0 ? my2 : my;
      mix_fft_in<I, true, true, C::TWO>(z[half], b, a, wi);
      float2 y[F::REGS];
#pragma unroll
      for (int i = 0; i < NV; ++i) y[i] = ff::cscale(z[half][i], half == 0 ? v[i].x : v[i].y);
      forward(y, MixTw<F, C::HELD_ROW>(ftab, t), live, ja + half, a, b);
      if (!C::TWO) __syncthreads();  // the next transform writes the exchange area
    }
  }
}

template <int LOGN2, int MODE>
__global__ void __launch_bounds__(RowCfg<LOGN2>::THREADS) __attribute__((amdgpu_waves_per_eu(ADJ_ROW_WAVES_PER_EU)))
    adj_row_kernel(const FlameDev* __restrict__ fls, long long n) {
  using S = ff::Shape<LOGN2>;
  constexpr int G = S::G, B = RowCfg<LOGN2>::B, N2 = S::N;
  extern __shared__ float2 lds[];
  const FlameDev f = fls[blockIdx.y];
  const int tid = threadIdx.x;
  const int p = tid % B, t = tid / B;
  const int pair = xcd_swizzle(blockIdx.x, gridDim.x) * B + p;
  // the adjoint step runs on the step's product grid; the seed on the grid's rows
  const int n1 = MODE == ROW_ADJ ? f.rows : f.n1, ts = f.tshift, mcols = f.m;
  const bool live = pair < n1 / 2;
  const int ja = 2 * pair, jb = 2 * pair + 1;
  // rows the loads read: a pair past the grid reads pair 0 (never stored), so
  // that no load sits behind a branch
  const int jal = live ? ja : 0, jbl = live ? jb : 1;
  float2* my = lds + p;
  const auto tw2 = KernelTw<LOGN2>::make(f.tw2, t);
  gf2* const Wp = glob(f.Wp);
  gf2* const Wm = glob(f.Wm);
  gf2* const Q = glob(f.Q);
  gf2* const A1 = glob(f.A1);
  gf2* const A2 = glob(f.A2);
  const float inv_r2 = [&] {
    const double r = r0_at(f, n);
    return (float)(1.0 / (r * r));
  }();

  // both rows' packed-gradient spectra, loaded before m's transform so that
  // their latency is hidden behind it
  float2 wv[2][ff::kPts];
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const int row = half ? jbl : jal;
#pragma unroll
    for (int i = 0; i < ff::kPts; ++i) {
      const int idx = t + G * i;
      float2 val = make_float2(0.f, 0.f);
      if (i < 4) {
        val = ld(Wp + w_index(row, idx, mcols));
      } else if (i >= 12) {
        const int mm = N2 - idx;  // < mcols except at i = 12, t = 0
        val = ld(Wm + w_index(row, i > 12 || t > 0 ? mm : 0, mcols));
      }
      wv[half][i] = val;
    }
  }

  float ma[ff::kPts], mb[ff::kPts];
  if constexpr (MODE == ROW_ADJ) {
    // m for both rows: Y = X_a + i X_b, X(k2) = M(k2), X(-k2) = conj(M(k2))
    float2 y[ff::kPts];
#pragma unroll
    for (int i = 0; i < ff::kPts; ++i) {
      const int idx = t + G * i;
      float2 val = make_float2(0.f, 0.f);
      if (i < 4) {
        const float2 a = ld(Q + tiled(jal, idx, n1, ts)), b = ld(Q + tiled(jbl, idx, n1, ts));
        val = make_float2(a.x - b.y, a.y + b.x);
      } else if (i >= 12) {
        const int mm = N2 - idx;  // < mcols except at i = 12, t = 0
        const int mc = i > 12 || t > 0 ? mm : 0;
        const float2 a = ld(Q + tiled(jal, mc, n1, ts)), b = ld(Q + tiled(jbl, mc, n1, ts));
        val = make_float2(a.x + b.y, -a.y + b.x);
      }
      y[i] = val;
    }
    y[12] = t > 0 ? y[12] : make_float2(0.f, 0.f);  // a select once every load is issued
    fft<LOGN2, true, kPrune>(y, t, my, B, tw2);
#pragma unroll
    for (int i = 0; i < ff::kPts; ++i) {
      ma[i] = y[i].x;
      mb[i] = y[i].y;
    }
  }

#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const int row = half ? jb : ja;  // the row this half stores (live pairs only)
    float2 v[ff::kPts];
#pragma unroll
    for (int i = 0; i < ff::kPts; ++i) v[i] = wv[half][i];
    v[12] = t > 0 ? v[12] : make_float2(0.f, 0.f);  // the position past the box
    fft<LOGN2, true, kPrune>(v, t, my, B, tw2);  // z = g1 + i g2 on the row
#pragma unroll
    for (int i = 0; i < ff::kPts; ++i) {
      float s;
      if constexpr (MODE == ROW_ADJ) {
        s = half ? mb[i] : ma[i];
      } else {
        const float x = (v[i].x * v[i].x + v[i].y * v[i].y) * inv_r2;
        s = inv_r2 / sqrtf(1.f + x);
      }
      v[i] = ff::cscale(v[i], s);  // zeta = w1 + i w2
    }
    fft<LOGN2, false>(v, t, my, B, tw2);
    __syncthreads();
    ff::Fft<LOGN2, false>::scatter(v, t, my, B);
    __syncthreads();
    if (live) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int k = t + G * i;
        const float2 xk = my[ff::Shape<LOGN2>::nat(k) * B];
        const float2 xm = my[ff::Shape<LOGN2>::nat((N2 - k) & (N2 - 1)) * B];
        // row transform of w1: (Xi(k) + conj(Xi(-k)))/2; of i kappa2 w2: kappa2 (Xi(k) - conj(Xi(-k)))/2
        const float2 u1 = make_float2(0.5f * (xk.x + xm.x), 0.5f * (xk.y - xm.y));
        const float h = 0.5f * f.s2 * (float)k;
        const float2 v2 = make_float2(h * (xk.x - xm.x), h * (xk.y + xm.y));
        st(A1 + tiled(row, k, n1, ts), u1);
        st(A2 + tiled(row, k, n1, ts), v2);
      }
    }
    __syncthreads();
  }
}

namespace {

template <int LOGN>
struct AdjColTable {
  static void launch(int mode, dim3 grid, hipStream_t st, const FlameDev* fl, long long n, const float2* s,
                     const float2* li, float2* lo) {
    constexpr int th = ColCfg<LOGN>::THREADS, lds = ColCfg<LOGN>::LDS_BYTES;
    switch (mode) {
      case ADJ_A: hipLaunchKernelGGL((adj_col_kernel<LOGN, ADJ_A>), grid, dim3(th), lds, st, fl, n, s, li, lo); break;
      case ADJ_C: hipLaunchKernelGGL((adj_col_kernel<LOGN, ADJ_C>), grid, dim3(th), lds, st, fl, n, s, li, lo); break;
      default: hipLaunchKernelGGL((adj_col_kernel<LOGN, SEED_C>), grid, dim3(th), lds, st, fl, n, s, li, lo); break;
    }
  }
};

template <int LOGN>
struct AdjRowTable {
  static void launch(int mode, dim3 grid, hipStream_t st, const FlameDev* fl, long long n) {
    constexpr int th = RowCfg<LOGN>::THREADS, lds = RowCfg<LOGN>::LDS_BYTES;
    if (mode == ROW_SEED)
      hipLaunchKernelGGL((adj_row_kernel<LOGN, ROW_SEED>), grid, dim3(th), lds, st, fl, n);
    else
      hipLaunchKernelGGL((adj_row_kernel<LOGN, ROW_ADJ>), grid, dim3(th), lds, st, fl, n);
  }
};

template <template <int> class Tab, int L, class... A>
void dispatch_adj(int logn, A... args) {
  if constexpr (L <= kMaxLog) {
    if (logn == L)
      Tab<L>::launch(args...);
    else
      dispatch_adj<Tab, L + 1>(logn, args...);
  }
}

}  // namespace

namespace {

template <int L, int NG>
void adjm_col_launch(int mode, int columns, hipStream_t st, const FlameDev* fl, long long n, const float2* s,
                     const float2* li, float2* lo) {
  using C = AdjMix<L, NG>;
  const dim3 grid((columns + C::T - 1) / C::T, 1);
  if (mode == ADJ_A)
    hipLaunchKernelGGL((adjm_col_kernel<L, ADJ_A, NG>), grid, dim3(C::THREADS), C::LDS_BYTES, st, fl, n, s, li, lo);
  else
    hipLaunchKernelGGL((adjm_col_kernel<L, ADJ_C, NG>), grid, dim3(C::THREADS), C::LDS_BYTES, st, fl, n, s, li, lo);
}

template <int L>
void dispatch_adjm_col(int logn, int mode, int columns, hipStream_t st, const FlameDev* fl, long long n,
                       const float2* s, const float2* li, float2* lo) {
  if constexpr (L <= kMaxLog) {
    if (logn != L) return dispatch_adjm_col<L + 1>(logn, mode, columns, st, fl, n, s, li, lo);
    if constexpr (L <= 11) {
      if (split_pays(L, columns, true)) {
        if (mode == ADJ_A) {
          using C = AdjMix<L, 3>;
          hipLaunchKernelGGL((adjm_col_kernel<L, ADJ_A, 3>), dim3((columns + C::T - 1) / C::T, 1), dim3(C::THREADS),
                             C::LDS_BYTES, st, fl, n, s, li, lo);
        } else {
          using C = AdjMix<L, 2>;
          hipLaunchKernelGGL((adjm_col_kernel<L, ADJ_C, 2>), dim3((columns + C::T - 1) / C::T, 1), dim3(C::THREADS),
                             C::LDS_BYTES, st, fl, n, s, li, lo);
        }
        return;
      }
    }
    adjm_col_launch<L, 1>(mode, columns, st, fl, n, s, li, lo);
  }
}

template <int L>
void dispatch_adjm_row(int logn, int pairs, hipStream_t st, const FlameDev* fl) {
  if constexpr (L <= kMaxLog) {
    if (logn != L) return dispatch_adjm_row<L + 1>(logn, pairs, st, fl);
    if constexpr (L <= 11) {
      if (split_pays(L, pairs, false)) {
        using C = AdjMix<L, 3>;
        hipLaunchKernelGGL((adjm_row_kernel<L, 3>), dim3((pairs + C::T - 1) / C::T, 1), dim3(C::THREADS), C::LDS_BYTES,
                           st, fl);
        return;
      }
    }
    using C = AdjMix<L, 1>;
    hipLaunchKernelGGL((adjm_row_kernel<L, 1>), dim3((pairs + C::T - 1) / C::T, 1), dim3(C::THREADS), C::LDS_BYTES, st,
                       fl);
  }
}

template <int L>
int adj_mixed_lds(int logn) {
  if constexpr (L <= kMaxLog) {
    if (logn != L) return adj_mixed_lds<L + 1>(logn);
    if constexpr (L <= 11) return AdjMix<L, 3>::LDS_BYTES > AdjMix<L, 1>::LDS_BYTES ? AdjMix<L, 3>::LDS_BYTES : AdjMix<L, 1>::LDS_BYTES;
    return AdjMix<L, 1>::LDS_BYTES;
  }
  return 0;
}

}  // namespace

int adj_mixed_lds_bytes(int logn) { return logn < kMinLogRowProduct ? 0 : adj_mixed_lds<kMinLogRowProduct>(logn); }

void launch_adjp_col(int logn1, int mode, int tiles, hipStream_t st, const FlameDev* fl, long long n,
                     const void* state, const void* lam_in, void* lam_out) {
  if (logn1 < kMinLogProduct || (mode != ADJ_A && mode != ADJ_C)) return;
  dispatch_adjm_col<kMinLogProduct>(logn1, mode, tiles * col_tile(logn1), st, fl, n, static_cast<const float2*>(state),
                                    static_cast<const float2*>(lam_in), static_cast<float2*>(lam_out));
}

void launch_adj_col(int logn1, int mode, int tiles, hipStream_t st, const FlameDev* fl, long long n,
                    const void* state, const void* lam_in, void* lam_out) {
  dispatch_adj<AdjColTable, kMinLog>(logn1, mode, dim3(tiles, 1), st, fl, n, static_cast<const float2*>(state),
                                     static_cast<const float2*>(lam_in), static_cast<float2*>(lam_out));
}

void launch_adj_row(int logn2, int mode, int groups, hipStream_t st, const FlameDev* fl, long long n) {
  if (mode == ROW_ADJ && logn2 >= kMinLogRowProduct) {  // as the step's row kernel, on 3 N2/4 points
    dispatch_adjm_row<kMinLogRowProduct>(logn2, groups * row_pairs(logn2), st, fl);
    return;
  }
  dispatch_adj<AdjRowTable, kMinLog>(logn2, mode, dim3(groups, 1), st, fl, n);
}

}  // namespace flame
