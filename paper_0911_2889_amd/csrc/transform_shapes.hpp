// Shapes of the kernels that run the product grids' transforms (mixed_fft.hpp)
// otherwise than the step's two: lanes, interleaved groups and exchange areas of
// the adjoint, of the averages on the physical grid, and of the resident step.
// No device code here: the host can drive every one of them lane by lane.

#pragma once

#include <type_traits>

#include "flame_dev.hpp"
#include "kernel_common.hpp"
#include "mixed_bodies.hpp"
#include "mixed_fft.hpp"

namespace flame {

// ------------------------------------------------ averages (physical_kernels.hip)

// The power-of-two plans' inverse transforms (ff::make_pass_plan, 16 points
// per thread: radix 16, the remainder last) as ff::Mix passes, so that they
// run on any number of lanes with the tables of those plans.
template <int LOGN>
struct PowPlan;
#define FLAME_POW_PLAN(L, ...)     \
  template <>                      \
  struct PowPlan<L> {              \
    using I = ff::Radices<__VA_ARGS__>; \
  }
FLAME_POW_PLAN(4, 16);
FLAME_POW_PLAN(5, 16, 2);
FLAME_POW_PLAN(6, 16, 4);
FLAME_POW_PLAN(7, 16, 8);
FLAME_POW_PLAN(8, 16, 16);
FLAME_POW_PLAN(9, 16, 16, 2);
FLAME_POW_PLAN(10, 16, 16, 4);
FLAME_POW_PLAN(11, 16, 16, 8);
#undef FLAME_POW_PLAN
constexpr int kMaxLogSide = 11;  // longer transforms run one after another (split_pays)

// Two inverse transforms side by side on two groups of G lanes (ColSplit, RowSplit).
template <int LOGN>
struct PhysSplit {
  static constexpr int N = 1 << LOGN, NB = N / 16;
  static constexpr int G = LOGN <= 10 ? 2 * NB : NB;
  static constexpr int T = 2 * G >= kSplitThreads ? 1 : kSplitThreads / (2 * G);
  using I = ff::Mix<typename PowPlan<LOGN>::I, G, T>;
  static constexpr int THREADS = 2 * G * T;
  static constexpr int LDS_BYTES = 8 * (2 * I::LDS > THREADS ? 2 * I::LDS : THREADS);  // and the sums of a workgroup
};

// ------------------------------------------------ adjoint (adjoint_kernels.hip)

// The product-grid kernels hold NG transforms side by side, on NG groups of G
// lanes and in NG exchange areas (NG = 3: the three inverse transforms of a
// column or row pair; NG = 2: the two forward ones of a column), or run them
// one after another on N/16 lanes (NG = 1). As for the step's kernels
// (split_pays), side by side is for launches that leave most of the chip idle.
// At 8192 points one after another means 768 lanes and two exchange areas, for
// the reasons at kFewLanes13 and mix_two_areas; here for many transforms too,
// since three transforms' data leave no registers for a second workgroup
// (adjoint steps: 16x8192 33.1 -> 30.3 us, 8192x64 31.8 -> 29.0, 8192x8192 682
// -> 641; 512 lanes with two areas 31.6, 30.7 and 659, 768 with one 32.1, 31.1
// and 675).
template <int LOGN, int NG>
struct AdjMix {
  static constexpr int N = 1 << LOGN, NB = N / 16;
  static constexpr int G = NG > 1 ? split_lanes(LOGN) : (LOGN == 13 ? kFewLanes13 : NB);
  static constexpr int T = NG > 1 ? (G >= 64 ? 1 : 64 / G) : (G >= 256 ? 1 : 256 / G);
  // twiddles in registers (MixTw); one after another, a row kernel holds both
  // rows' inputs and m beside its transform, and at 2048 points, and from 8192
  // on, has no registers for them (4096 points: 64x4096 28.1 -> 27.6 us)
  static constexpr bool HELD = LOGN < 14, HELD_ROW = NG > 1 || LOGN < 11 || LOGN == 12;
  using F = ff::Mix<typename ff::MixPlan<LOGN>::F, G, T>;
  using I = ff::Mix<typename ff::MixPlan<LOGN>::I, G, T>;
  static constexpr int L = F::N, AREA = F::LDS > I::LDS ? F::LDS : I::LDS;
  static constexpr int THREADS = NG * G * T;
  static constexpr bool TWO = NG == 1 && LOGN == 13;  // two exchange areas (mix_two_areas)
  static constexpr int LDS_BYTES = 8 * NG * (TWO ? 2 : 1) * AREA;
};

// ------------------------------------------------ resident step (resident_kernel.hip)

constexpr int imin(int a, int b) { return a < b ? a : b; }
constexpr int imax(int a, int b) { return a > b ? a : b; }

template <int LOGN, bool PRODUCT>
struct ResAxis {
  using Plan = typename std::conditional<PRODUCT, ff::MixPlan<PRODUCT ? LOGN : 6>, ff::FullPlan<PRODUCT ? 4 : LOGN>>::type;
  static constexpr int N = 1 << LOGN, NB = N / 16;
  static constexpr int RS = PRODUCT ? 12 : 16;  // radix at the spectral end
  static constexpr int L = RS * NB;
  // register of kept mode kk = 0..7 (k = j + NB kk >= 0 for kk < 4, else j - NB (8 - kk))
  static constexpr int reg(int kk) { return kk < 4 ? kk : kk + RS - 8; }
  static constexpr int min_radix() {
    int r = 16;
    for (int x : Plan::I::radix) r = imin(r, x);
    return r;
  }
  // lanes per job: at least NB, doubled while a pass has more butterflies than
  // that and `jobs` jobs still fit `threads`
  static constexpr int lanes(int jobs, int threads) {
    int g = NB;
    while (jobs * g * 2 <= threads && g < L / min_radix()) g *= 2;
    return g;
  }
};

constexpr int kResMaxThreads = 1024;
// Steps whose scalars (logarithm, divisions in double) are formed at once, a
// step per lane, and read from LDS step by step; one more for Heun's corrector.
constexpr int kResChunk = 64, kResChunk1 = kResChunk + 1;
constexpr int kResMaxLds = 160 * 1024;

template <int L1, int L2>
struct Res {
  using A1 = ResAxis<L1, (L1 >= kMinLogProduct)>;
  using A2 = ResAxis<L2, (L2 >= kMinLogRowProduct)>;
  static constexpr int N1 = A1::N, N2 = A2::N, M = N2 / 4, R = A1::L, NP = R / 2;
  static constexpr int GCI = A1::lanes(2 * M, kResMaxThreads), GCF = A1::lanes(M, kResMaxThreads);
  static constexpr int GRI = A2::lanes(R, kResMaxThreads), GRF = A2::lanes(NP, kResMaxThreads);
  using CI = ff::Mix<typename A1::Plan::I, GCI, 2 * M>;
  using CF = ff::Mix<typename A1::Plan::F, GCF, M>;
  using RI = ff::Mix<typename A2::Plan::I, GRI, R>;
  using RF = ff::Mix<typename A2::Plan::F, GRF, NP>;
  static constexpr int S = R + 1;  // stride of a column of W and Q
  // area A: the exchanges; area B: W, then |z|^2, then Q and the split's
  // exchange, then the updated modes
  static constexpr int AREA_A = imax(imax(CI::LDS, CF::LDS), imax(RI::LDS, RF::LDS));
  static constexpr int AREA_B = imax(imax(2 * M * S, A2::L * NP), imax(M * S + M * NP, 8 * A1::NB * M));
  static constexpr int LDS_BYTES = 8 * (AREA_A + AREA_B) + kResChunk1 * (int)sizeof(StepScalars);
  static constexpr int JOBS = imax(imax(2 * M * GCI, M * GCF), imax(R * GRI, NP * GRF));
  static constexpr int THREADS = (JOBS + 63) / 64 * 64;
  static constexpr bool OK = THREADS <= kResMaxThreads && LDS_BYTES <= kResMaxLds;
};

}  // namespace flame
