// Steps of small flames, one workgroup per flame (gfx950): every step of a
// call in one launch, with the state in registers and the intermediates W
// and Q of the two-kernel step (flame_kernels.hip) in LDS.
//
// What bounds a small flame's step otherwise is not work but two launches and
// their chains: at 64x128 each of the two kernels took 5 to 6 us for some 2 us
// of one compute unit's arithmetic (12.3 us a step, here 6.4). Many flames take
// their turns at the compute units and still gain where the last turn has one
// flame: 257 of 64x128 12.6 us for 18.4, of 128x128 17.7 for 25.7, of 32x256, the
// closest, 16.6 for 17.1. Here a step is the four phases below with
// nine to seventeen workgroup barriers between them.
//
//  column inverse: 2 M jobs (column m; Wp and Wm), lanes as the split bodies
//  row inverse:    R jobs (row j1), then |z|^2 of a row pair as one complex field
//  row forward:    R/2 jobs, split by Hermitian symmetry into Q
//  column forward: M jobs, the update on the lanes that hold the modes
//
// Lane tid works on job tid % jobs, so that the lanes of a wave touch
// neighbouring jobs: the exchange areas are interleaved over the jobs, and W
// and Q, [m][j1] with an odd stride R + 1, are free of bank conflicts from
// both sides. The transforms are those of the two-kernel step on a product
// grid (ff::MixPlan); an axis without one (N1 < 128, N2 < 64) takes
// ff::FullPlan.

#include <hip/hip_runtime.h>

#include <type_traits>

#include "flame_dev.hpp"
#include "flame_kernels.hpp"
#include "kernel_common.hpp"
#include "mixed_bodies.hpp"
#include "transform_shapes.hpp"

namespace flame {

namespace {

// Resident: every grid of N1 N2 <= 2^kResMaxLogs but three, which need 162 to 189 KB.
template <int L1, int L2>
constexpr bool resident_as_documented() {
  if constexpr (L1 + L2 <= kResMaxLogs) {
    constexpr bool out = (L1 == 4 && L2 == 10) || (L1 == 5 && L2 == 9) || (L1 == 6 && L2 == 8);
    return Res<L1, L2>::OK != out && resident_as_documented<L1, L2 + 1>();
  } else if constexpr (L1 + 1 + kMinLog <= kResMaxLogs) {
    return resident_as_documented<L1 + 1, kMinLog>();
  } else {
    return true;
  }
}
static_assert(resident_as_documented<kMinLog, kMinLog>(), "the grids that flame_step's description names");

// A value the compiler cannot see through: what a phase derives from the
// thread index (addresses, wavenumbers) is then formed in that phase, instead
// of being kept, and spilled, across all the phases of all the steps.
__device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// A transform of the lanes t < M::G (`on`); every thread of the workgroup
// calls it. The exchange area must be free on entry; on return other lanes
// may still read it.
template <class M, bool INV, bool ZMID, int P = 0>
__device__ __forceinline__ void res_fft(float2 (&x)[M::REGS], float2* lds, const MixTw<M, false>& tw, bool on,
                                        const float2 (&w)[M::tw_count(P)]) {
  if (on) M::template butterflies<P, INV, ZMID>(x, tw.t, w);
  if constexpr (P + 1 < M::NPASS) {
    if constexpr (P > 0) __syncthreads();  // the last exchange has been read
    float2 next[M::tw_count(P + 1)];
    if (on) {
      M::template put<P>(x, tw.t, lds);
      tw.template pass<P + 1>(next);
    }
    __syncthreads();
    if (on) M::template get<P + 1>(x, tw.t, lds);
    res_fft<M, INV, ZMID, P + 1>(x, lds, tw, on, next);
  }
}
template <class M, bool INV, bool ZMID>
__device__ __forceinline__ void res_fft(float2 (&x)[M::REGS], float2* lds, const MixTw<M, false>& tw, bool on) {
  const float2 none[1] = {make_float2(0.f, 0.f)};
  res_fft<M, INV, ZMID, 0>(x, lds, tw, on, none);
}

}  // namespace

// `steps` steps of flame blockIdx.x from step index n (+ *nbase); the index of
// step s is n + s dn (dn = 0 for timing without moving on). VAR: VAR_EULER,
// VAR_EULER_F (a forcing may be bound) or VAR_HEUN_P (both stages of Heun).
template <int L1, int L2, int VAR>
__global__ void __launch_bounds__((Res<L1, L2>::THREADS))
    res_kernel(const FlameDev* __restrict__ fls, long long n, const long long* nbase, int steps, int dn) {
  using C = Res<L1, L2>;
  using A1 = typename C::A1;
  using A2 = typename C::A2;
  using CI = typename C::CI;
  using CF = typename C::CF;
  using RI = typename C::RI;
  using RF = typename C::RF;
  constexpr int M = C::M, R = C::R, NP = C::NP, S = C::S, N1 = C::N1, NB1 = A1::NB, NB2 = A2::NB;
  constexpr bool HEUN = VAR == VAR_HEUN_P, FORCED = VAR != VAR_EULER;
  extern __shared__ float2 lds[];
  float2* const la = lds;
  float2* const lb = lds + C::AREA_A;
  if (nbase) n += *nbase;
  const FlameDev f = fls[blockIdx.x];
  const int tid = threadIdx.x;
  const float2* const tab1 = L1 >= kMinLogProduct ? f.twma : f.twfa;
  const float2* const tab2 = L2 >= kMinLogRowProduct ? f.twmb : f.twfb;
  // column forward and update: column cf, lane uf; the lanes uf < NB1 hold the state
  const int cf = tid % M, uf = tid / M;
  const bool hold = uf < NB1;
  auto k1_of = [](int j, int kk) { return kk < 4 ? j + NB1 * kk : j - NB1 * (8 - kk); };
  gf2* const Sc = glob(f.S) + (size_t)cf * f.h1 + N1 / 4;
  float2 sv[8], frc[8], prd[8];
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) {
    const int k1 = k1_of(hold ? uf : 0, kk);
    sv[kk] = ld(Sc + k1);
    frc[kk] = FORCED ? forcing_at(f, cf, k1) : make_float2(0.f, 0.f);
    prd[kk] = make_float2(0.f, 0.f);
  }
  // the modes to the column inverse's lanes
  if (hold) {
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) lb[(uf + NB1 * kk) * M + cf] = sv[kk];
  }
  StepScalars* const scal = reinterpret_cast<StepScalars*>(lb + C::AREA_B);
  for (int step = 0; step < steps; ++step) {
    if (step % kResChunk == 0) {
      for (int i = tid; i < kResChunk1; i += C::THREADS)
        scal[i] = step_scalars(f, n + (long long)(step + i) * dn + (dn == 0 && i == kResChunk ? 1 : 0), R, A2::L);
      __syncthreads();  // also: the modes are in place
    }
#pragma unroll 1
    for (int stage = 0; stage < (HEUN ? 2 : 1); ++stage) {
      // ---- column inverse transforms of (i kappa1 -+ kappa2) Phi~ -> W
      {
        const int id = opaque(tid), c = id % M, h = (id / M) & 1, t = id / (2 * M);
        const bool on = t < C::GCI, act = t < NB1;
        const float kap2 = f.s2 * (float)c, kp = h == 0 ? -kap2 : kap2;
        float2 v[CI::REGS];
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
          const int jt = act ? t : 0;
          v[A1::reg(kk)] = slope(f.s1 * (float)k1_of(jt, kk), kp, lb[(jt + NB1 * kk) * M + c]);
        }
        res_fft<CI, true, true>(v, la + h * M + c, MixTw<CI, false>(tab1, t), on);
        if constexpr (CI::NPASS == 1) __syncthreads();  // every lane has read its modes before W takes their place
        constexpr int P = CI::NPASS - 1, RX = CI::radix(P);
        const float cs = h == 0 ? 1.f : -1.f;  // Wm holds the conjugate
        if (on) {
#pragma unroll
          for (int b = 0; b < CI::rounds(P); ++b)
            if (CI::template active<P>(t, b)) {
#pragma unroll
              for (int r = 0; r < RX; ++r)
                lb[(h * M + c) * S + t + CI::G * b + r * CI::bf(P)] = make_float2(v[b * RX + r].x, cs * v[b * RX + r].y);
            }
        }
      }
      __syncthreads();
      // ---- row inverse transforms, |z|^2
      {
        const int id = opaque(tid), j1 = id % R, t = id / R;
        const bool on = t < C::GRI, act = t < NB2;
        const int jt = act ? t : 0;
        float2 v[RI::REGS];
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
          const int k2 = kk < 4 ? jt + NB2 * kk : NB2 * (8 - kk) - jt;  // |k2|; M (past the box) at kk = 4, jt = 0
          const int at = kk < 4 ? k2 : M + (kk > 4 || jt > 0 ? k2 : 0);
          v[A2::reg(kk)] = lb[at * S + j1];
        }
        v[A2::reg(4)] = jt > 0 ? v[A2::reg(4)] : make_float2(0.f, 0.f);
        res_fft<RI, true, true>(v, la + j1, MixTw<RI, false>(tab2, t), on);
        if constexpr (RI::NPASS == 1) __syncthreads();  // W has been read
        constexpr int P = RI::NPASS - 1, RX = RI::radix(P);
        float* const q = reinterpret_cast<float*>(lb) + j1;  // pair j1 / 2, real or imaginary part
        if (on) {
#pragma unroll
          for (int b = 0; b < RI::rounds(P); ++b)
            if (RI::template active<P>(t, b)) {
#pragma unroll
              for (int r = 0; r < RX; ++r)
                q[(t + RI::G * b + r * RI::bf(P)) * R] = norm2(v[b * RX + r].x, v[b * RX + r].y);
            }
        }
      }
      __syncthreads();
      // ---- row forward transforms, split into Q
      {
        const int id = opaque(tid), pj = id % NP, t = id / NP;
        const bool on = t < C::GRF, act = t < NB2;
        float2 y[RF::REGS];
        if (on) {
#pragma unroll
          for (int b = 0; b < RF::rounds(0); ++b)
            if (RF::template active<0>(t, b)) {
#pragma unroll
              for (int r = 0; r < RF::radix(0); ++r)
                y[b * RF::radix(0) + r] = lb[(t + RF::G * b + r * RF::bf(0)) * NP + pj];
            }
        }
        res_fft<RF, false, false>(y, la + pj, MixTw<RF, false>(tab2 + ff::MixTables<typename A2::Plan>::F_OFF, t), on);
        if constexpr (RF::NPASS == 1) __syncthreads();  // |z|^2 has been read
        float2* const ex = lb + M * S + pj;
        if (act) {
#pragma unroll
          for (int kk = 4; kk < 8; ++kk) ex[(t + NB2 * (kk - 4)) * NP] = y[A2::reg(kk)];
        }
        __syncthreads();
        if (act) {
#pragma unroll
          for (int kk = 0; kk < 4; ++kk) {
            const int k = t + NB2 * kk;
            const float2 yk = y[A2::reg(kk)];
            const float2 yo = ex[(NB2 * (4 - kk) - t - (k == 0 ? 1 : 0)) * NP];
            float2 qa, qb;
            split_pair(yk, k == 0 ? yk : yo, qa, qb);
            lb[k * S + 2 * pj] = qa;
            lb[k * S + 2 * pj + 1] = qb;
          }
        }
      }
      __syncthreads();
      // ---- column forward transforms, update
      {
        const int id = opaque(tid), cf = id % M, uf = id / M;
        const bool on_cf = uf < C::GCF, hold = uf < NB1;
        float2 v[CF::REGS];
        if (on_cf) {
#pragma unroll
          for (int b = 0; b < CF::rounds(0); ++b)
            if (CF::template active<0>(uf, b)) {
#pragma unroll
              for (int r = 0; r < CF::radix(0); ++r)
                v[b * CF::radix(0) + r] = lb[cf * S + uf + CF::G * b + r * CF::bf(0)];
            }
        }
        res_fft<CF, false, false>(v, la + cf, MixTw<CF, false>(tab1 + ff::MixTables<typename A1::Plan>::F_OFF, uf), on_cf);
        if constexpr (CF::NPASS == 1) __syncthreads();  // Q has been read
        const StepScalars sc = scal[step % kResChunk];
        const float kap2c = f.s2 * (float)cf, dtf = (float)f.dt;
        const bool corrector = HEUN && stage == 1;
        const float ac = corrector ? scal[dn == 0 ? kResChunk : step % kResChunk + 1].a : 0.f;
        float2 now[8];
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
          const int k1 = k1_of(uf, kk);
          const float e = growth_factor(norm2(f.s1 * (float)k1, kap2c), sc, f.gamma);
          const float2 q = v[A1::reg(kk)];
          if (corrector)
            now[kk] = update_mode<VAR_HEUN_C>(e, sv[kk], q, frc[kk], prd[kk], sc.a, ac, dtf);
          else
            now[kk] = update_mode<VAR>(e, sv[kk], q, frc[kk], prd[kk], sc.a, ac, dtf);
          if (kk == 4 && uf == 0) now[kk] = make_float2(0.f, 0.f);  // k1 = -N1/4 lies outside the box
          if (kk == 0 && uf == 0 && cf == 0) now[kk].y = 0.f;
        }
        if (hold) {
#pragma unroll
          for (int kk = 0; kk < 8; ++kk) lb[(uf + NB1 * kk) * M + cf] = now[kk];
        }
        __syncthreads();
        if (cf == 0 && hold) {
          // column k2 = 0: the k1 > 0 half conjugated onto k1 < 0 (symmetrisation)
#pragma unroll
          for (int kk = 4; kk < 8; ++kk)
            if (k1_of(uf, kk) > -N1 / 4) {
              now[kk] = ff::cconj(lb[-k1_of(uf, kk) * M]);
              lb[(uf + NB1 * kk) * M] = now[kk];
            }
        }
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
          if (HEUN && stage == 0)
            prd[kk] = now[kk];
          else
            sv[kk] = now[kk];
        }
        __syncthreads();
      }
    }
  }
  if (hold) {
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) st(Sc + k1_of(uf, kk), sv[kk]);
  }
}

namespace {

template <int L1, int L2>
KernelLaunch res_info(int var) {
  if constexpr (Res<L1, L2>::OK) {
    using C = Res<L1, L2>;
    const void* fn = var == VAR_EULER     ? reinterpret_cast<const void*>(&res_kernel<L1, L2, VAR_EULER>)
                     : var == VAR_EULER_F ? reinterpret_cast<const void*>(&res_kernel<L1, L2, VAR_EULER_F>)
                                          : reinterpret_cast<const void*>(&res_kernel<L1, L2, VAR_HEUN_P>);
    return KernelLaunch{fn, C::THREADS, C::LDS_BYTES};
  } else {
    return KernelLaunch{nullptr, 0, 0};
  }
}

template <int L1, int L2>
KernelLaunch res_pick(int logn1, int logn2, int var) {
  if constexpr (L1 + L2 > kResMaxLogs) {
    if constexpr (L1 + 1 + kMinLog > kResMaxLogs)
      return KernelLaunch{nullptr, 0, 0};
    else
      return logn1 > L1 ? res_pick<L1 + 1, kMinLog>(logn1, logn2, var) : KernelLaunch{nullptr, 0, 0};
  } else {
    if (logn1 == L1 && logn2 == L2) return res_info<L1, L2>(var);
    if (logn1 == L1) return res_pick<L1, L2 + 1>(logn1, logn2, var);
    if constexpr (L1 + 1 + kMinLog <= kResMaxLogs) return res_pick<L1 + 1, kMinLog>(logn1, logn2, var);
    return KernelLaunch{nullptr, 0, 0};
  }
}

KernelLaunch resident_info(int logn1, int logn2, int var) { return res_pick<kMinLog, kMinLog>(logn1, logn2, var); }

void launch_resident(const KernelLaunch& kl, int flames, hipStream_t st, const FlameDev* fl, long long n, int steps,
                     int dn) {
  const long long* nb = nullptr;
  void* args[] = {&fl, &n, &nb, &steps, &dn};
  (void)hipLaunchKernel(kl.func, dim3(flames), dim3(kl.threads), args, kl.lds, st);
}

// the runtime asks through these pointers (flame_kernels.hpp)
const bool registered = (resident_kernel = &resident_info, resident_launch = &launch_resident, true);

}  // namespace

}  // namespace flame
