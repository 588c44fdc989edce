// HIP kernels of the spectral flame step on N1 rows and on N2 phi points, and
// of the physical grid's transforms (gfx950); on the product grids the step
// runs the kernels of mixed_kernels.hip, in the same two parts.
//
// One step of Eq. (1) is two kernels:
//  * row_kernel<ROW_STEP>: for each pair of grid rows j1, load the column-
//    transformed gradient spectrum Z(j1, k2) (k2 in [-K2, K2]), inverse
//    transform along phi to z = g1 + i g2 (the two gradient components packed
//    into one complex field), form q = |z|^2 = |grad Phi|^2, and transform the
//    two real rows back with one complex forward transform, keeping
//    k2 in [0, K2] -> Q. (Section 3: row transform, pointwise product, row
//    inverse transform.)
//  * col_kernel<COL_STEP>: for each stored column k2 = m, forward transform Q
//    along theta, keep |k1| <= K1, apply the integrating-factor Euler update
//    with the exact linear propagator, symmetrise the k2 = 0 column (Section 3),
//    store the state, then immediately form the next step's column transforms
//    of (i kappa1 -+ kappa2) Phi~ -> Wp, Wm. (Section 3: column transforms of
//    k1 Psi and k2 Psi; the inverse column transform of the product.)
// The global transposes of Section 3 are the layouts of Wp/Wm and Q in HBM:
// each kernel reads long contiguous runs and writes pieces of at least 64
// bytes (2 rows x 4 columns of Q; 4 rows x 2 columns of Wp, and of Wm).

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <initializer_list>
#include <type_traits>

#include "fft_engine.hpp"
#include "flame_dev.hpp"
#include "flame_kernels.hpp"
#include "kernel_common.hpp"
#include "step_bodies.hpp"

namespace flame {

template <int LOGN1, int MODE, int PTS = ff::kPts, int SV = VAR_EULER>
__global__ void __launch_bounds__((ColCfg<LOGN1, PTS>::THREADS)) __attribute__((amdgpu_waves_per_eu(COL_WAVES_PER_EU)))
    col_kernel(const FlameDev* __restrict__ fls, long long n, const long long* nbase, const float2* src) {
  if (nbase) n += *nbase;  // graph replays read the step index from device memory
  col_body<LOGN1, MODE, PTS, SV>(fls[blockIdx.y], n, src, xcd_swizzle(blockIdx.x, gridDim.x), threadIdx.x);
}

template <int LOGN2, int MODE, int PTS = ff::kPts, bool NT = false>
__global__ void __launch_bounds__((RowCfg<LOGN2, PTS>::THREADS)) __attribute__((amdgpu_waves_per_eu(RowCfg<LOGN2, PTS>::WPE)))
    row_kernel(const FlameDev* __restrict__ fls, long long n, const long long* nbase,
               const float* __restrict__ phys_in, float* __restrict__ phys_out) {
  if (nbase) n += *nbase;
  row_body<LOGN2, MODE, PTS, NT>(fls[blockIdx.y], n, phys_in, phys_out, xcd_swizzle(blockIdx.x, gridDim.x),
                                 threadIdx.x);
}

// ------------------------------------------------------------------ dispatch

namespace {

template <int LOGN>
struct ColTable {
  static void launch(int mode, dim3 grid, hipStream_t st, const FlameDev* fl, long long n, const float2* src) {
    constexpr int th = ColCfg<LOGN>::THREADS, lds = ColCfg<LOGN>::LDS_BYTES;
    const long long* nb = nullptr;
    switch (mode) {
      case COL_STEP: hipLaunchKernelGGL((col_kernel<LOGN, COL_STEP>), grid, dim3(th), lds, st, fl, n, nb, src); break;
      case COL_FIRST:
        hipLaunchKernelGGL((col_kernel<LOGN, COL_FIRST>), grid, dim3(th), lds, st, fl, n, nb, src);
        break;
      case COL_PROJECT:
        hipLaunchKernelGGL((col_kernel<LOGN, COL_PROJECT>), grid, dim3(th), lds, st, fl, n, nb, src);
        break;
      default: hipLaunchKernelGGL((col_kernel<LOGN, COL_SYNTH>), grid, dim3(th), lds, st, fl, n, nb, src); break;
    }
  }
  template <int VAR>
  static KernelLaunch step_kernel_v(int pts) {
    if (pts == 12) return KernelLaunch{nullptr, 0, 0};  // product grid only (colp_kernel_info)
    if (pts == 8) {
      if constexpr (LOGN <= kMaxLog8)
        return KernelLaunch{reinterpret_cast<const void*>(&col_kernel<LOGN, COL_STEP, 8, VAR>),
                            ColCfg<LOGN, 8>::THREADS, ColCfg<LOGN, 8>::LDS_BYTES};
      else
        return KernelLaunch{nullptr, 0, 0};
    }
    return KernelLaunch{reinterpret_cast<const void*>(&col_kernel<LOGN, COL_STEP, ff::kPts, VAR>),
                        ColCfg<LOGN>::THREADS, ColCfg<LOGN>::LDS_BYTES};
  }
  static KernelLaunch step_kernel(int pts, int var) {
    switch (var) {
      case VAR_EULER_F: return step_kernel_v<VAR_EULER_F>(pts);
      case VAR_HEUN_P: return step_kernel_v<VAR_HEUN_P>(pts);
      case VAR_HEUN_C: return step_kernel_v<VAR_HEUN_C>(pts);
      case VAR_NT | VAR_EULER: return step_kernel_v<VAR_NT | VAR_EULER>(pts);
      case VAR_NT | VAR_EULER_F: return step_kernel_v<VAR_NT | VAR_EULER_F>(pts);
      case VAR_NT | VAR_HEUN_P: return step_kernel_v<VAR_NT | VAR_HEUN_P>(pts);
      case VAR_NT | VAR_HEUN_C: return step_kernel_v<VAR_NT | VAR_HEUN_C>(pts);
      default: return step_kernel_v<VAR_EULER>(pts);
    }
  }
};

template <int LOGN>
struct RowTable {
  static void launch(int mode, dim3 grid, hipStream_t st, const FlameDev* fl, long long n, const float* in,
                     float* out) {
    constexpr int th = RowCfg<LOGN>::THREADS, lds = RowCfg<LOGN>::LDS_BYTES;
    const long long* nb = nullptr;
    switch (mode) {
      case ROW_FORWARD:
        hipLaunchKernelGGL((row_kernel<LOGN, ROW_FORWARD>), grid, dim3(th), lds, st, fl, n, nb, in, out);
        break;
      default: hipLaunchKernelGGL((row_kernel<LOGN, ROW_SYNTH>), grid, dim3(th), lds, st, fl, n, nb, in, out); break;
    }
  }
  template <bool NT>
  static KernelLaunch step_kernel_nt(int pts) {
    if (pts == 8) {
      if constexpr (LOGN <= kMaxLog8)
        return KernelLaunch{reinterpret_cast<const void*>(&row_kernel<LOGN, ROW_STEP, 8, NT>),
                            RowCfg<LOGN, 8>::THREADS, RowCfg<LOGN, 8>::LDS_BYTES};
      else
        return KernelLaunch{nullptr, 0, 0};
    }
    return KernelLaunch{reinterpret_cast<const void*>(&row_kernel<LOGN, ROW_STEP, ff::kPts, NT>),
                        RowCfg<LOGN>::THREADS, RowCfg<LOGN>::LDS_BYTES};
  }
  static KernelLaunch step_kernel(int pts, bool nt) { return nt ? step_kernel_nt<true>(pts) : step_kernel_nt<false>(pts); }
};

template <template <int> class Tab, int L, class... A>
void dispatch_log(int logn, A... args) {
  if constexpr (L <= kMaxLog) {
    if (logn == L)
      Tab<L>::launch(args...);
    else
      dispatch_log<Tab, L + 1>(logn, args...);
  }
}

template <template <int> class Tab, int L, class... A>
void dispatch_info(int logn, KernelLaunch* out, A... args) {
  if constexpr (L <= kMaxLog) {
    if (logn == L)
      *out = Tab<L>::step_kernel(args...);
    else
      dispatch_info<Tab, L + 1>(logn, out, args...);
  }
}

}  // namespace

// Step-mode launches go through the kernel tables; with timing events they
// use hipExtLaunchKernel, which records the events in the kernel's own
// dispatch (kernel start and end, no extra queue packets).
void launch_col(int logn1, int mode, int tiles, int nfl, hipStream_t st, const FlameDev* fl, long long n,
                const void* src, int pts, hipEvent_t ev_start, hipEvent_t ev_stop, int var) {
  if (mode == COL_STEP && (var != VAR_EULER || pts != ff::kPts || ev_start || ev_stop)) {
    const KernelLaunch kl = col_step_kernel(logn1, pts, var);
    if (!kl.func) return;
    const long long* nb = nullptr;
    const float2* s = static_cast<const float2*>(src);
    void* args[] = {&fl, &n, &nb, &s};
    if (ev_start || ev_stop)
      (void)hipExtLaunchKernel(kl.func, dim3(tiles * kl.mult, nfl), dim3(kl.threads), args, kl.lds, st, ev_start, ev_stop, 0);
    else
      (void)hipLaunchKernel(kl.func, dim3(tiles * kl.mult, nfl), dim3(kl.threads), args, kl.lds, st);
    return;
  }
  if (mode == COL_FIRST && nfl == 1 &&
      launch_first_side(logn1, tiles * col_tile(logn1), st, fl, static_cast<const float2*>(src)))
    return;
  dispatch_log<ColTable, kMinLog>(logn1, mode, dim3(tiles, nfl), st, fl, n, static_cast<const float2*>(src));
}

void launch_row(int logn2, int mode, int groups, int nfl, hipStream_t st, const FlameDev* fl, long long n,
                const float* in, float* out, int pts, hipEvent_t ev_start, hipEvent_t ev_stop, bool nt) {
  if (mode == ROW_STEP) {
    const KernelLaunch kl = row_step_kernel(logn2, pts, nt);
    if (!kl.func) return;
    const long long* nb = nullptr;
    void* args[] = {&fl, &n, &nb, &in, &out};
    if (ev_start || ev_stop)
      (void)hipExtLaunchKernel(kl.func, dim3(groups * kl.mult, nfl), dim3(kl.threads), args, kl.lds, st, ev_start, ev_stop, 0);
    else
      (void)hipLaunchKernel(kl.func, dim3(groups * kl.mult, nfl), dim3(kl.threads), args, kl.lds, st);
    return;
  }
  if (mode == ROW_DIAG) {
    launch_diag(logn2, groups, pts, st, fl, n, reinterpret_cast<double*>(out));
    return;
  }
  dispatch_log<RowTable, kMinLog>(logn2, mode, dim3(groups, nfl), st, fl, n, in, out);
}

namespace {

template <int L>
int col_lds(int logn1) {
  if constexpr (L <= kMaxLog) {
    if (logn1 != L) return col_lds<L + 1>(logn1);
    int b = ColCfg<L, 16>::LDS_BYTES > ColCfg<L, 8>::LDS_BYTES ? ColCfg<L, 16>::LDS_BYTES : ColCfg<L, 8>::LDS_BYTES;
    return b;
  }
  return 0;
}

template <int L>
int row_lds(int logn2) {
  if constexpr (L <= kMaxLog) {
    if (logn2 != L) return row_lds<L + 1>(logn2);
    int b = RowCfg<L, 16>::LDS_BYTES > RowCfg<L, 8>::LDS_BYTES ? RowCfg<L, 16>::LDS_BYTES : RowCfg<L, 8>::LDS_BYTES;
    return b;
  }
  return 0;
}

}  // namespace

int lds_bytes_needed(int logn1, int logn2) {
  const int c = col_lds<kMinLog>(logn1), r = row_lds<kMinLog>(logn2);
  const int m1 = mixed_lds_bytes(logn1), m2 = mixed_lds_bytes(logn2);
  const int a1 = adj_mixed_lds_bytes(logn1), a2 = adj_mixed_lds_bytes(logn2);
  const int p1 = phys_lds_bytes(logn1), p2 = phys_lds_bytes(logn2);
  int most = c;
  for (const int b : {r, m1, m2, a1, a2, p1, p2}) most = b > most ? b : most;
  return most;
}

KernelLaunch col_step_kernel(int logn1, int pts, int var) {
  KernelLaunch out{nullptr, 0, 0};
  dispatch_info<ColTable, kMinLog>(logn1, &out, pts, var);
  return out;
}

// The row kernel forms the quadratic term on 3 N2/4 phi points where it has a
// transform of that length (N2 >= 64) and the caller did not ask for all N2
// (kRowFull): three quarters of the butterflies of N2 points in as many passes
// or fewer.
KernelLaunch row_step_kernel(int logn2, int pts, bool nt) {
  if (logn2 >= kMinLogRowProduct && !(pts & kRowFull)) return rowp_kernel_info(logn2, pts, nt);
  KernelLaunch out{nullptr, 0, 0};
  dispatch_info<RowTable, kMinLog>(logn2, &out, pts & ~kRowFull, nt);
  return out;
}

// One thread stores the step index that graph replays read (a vector store).
__global__ void set_step_kernel(long long* __restrict__ counter, long long value) {
  if (threadIdx.x == 0) {
    volatile long long* p = counter;
    *p = value;
  }
}

void launch_set_step(hipStream_t st, long long* counter, long long value) {
  hipLaunchKernelGGL(set_step_kernel, dim3(1), dim3(64), 0, st, counter, value);
}

}  // namespace flame
