// Step kernels on the product grids (gfx950): the column kernel on 3 N1/4
// theta rows and the row kernel on 3 N2/4 phi points (mixed_bodies.hpp). The
// split of a step into the two kernels and the arrays between them are those
// of flame_kernels.hip.

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include "flame_dev.hpp"
#include "flame_kernels.hpp"
#include "mixed_bodies.hpp"

namespace flame {

template <int LOGN1, int MODE, int SV, int G = mix_lanes(LOGN1)>
__global__ void __launch_bounds__((ColMix<LOGN1, G>::THREADS)) __attribute__((amdgpu_waves_per_eu(COL_WAVES_PER_EU)))
    colm_kernel(const FlameDev* __restrict__ fls, long long n, const long long* nbase, const float2* src) {
  if (nbase) n += *nbase;  // graph replays read the step index from device memory
  colm_body<LOGN1, MODE, SV, G>(fls[blockIdx.y], n, src, xcd_swizzle(blockIdx.x, gridDim.x), threadIdx.x);
}

template <int LOGN2, bool NT, int G = mix_lanes(LOGN2)>
__global__ void __launch_bounds__((RowMix<LOGN2, G>::THREADS))
    __attribute__((amdgpu_waves_per_eu(RowMix<LOGN2, G>::WPE)))
    rowm_kernel(const FlameDev* __restrict__ fls, long long, const long long*, const float*, float*) {
  rowm_body<LOGN2, NT, G>(fls[blockIdx.y], xcd_swizzle(blockIdx.x, gridDim.x), threadIdx.x);
}

template <int LOGN1, int MODE, int VAR>
__global__ void __launch_bounds__(ColSplit<LOGN1>::THREADS)
    cols_kernel(const FlameDev* __restrict__ fls, long long n, const long long* nbase, const float2* src) {
  if (nbase) n += *nbase;
  cols_body<LOGN1, MODE, VAR>(fls[blockIdx.y], n, src, xcd_swizzle(blockIdx.x, gridDim.x), threadIdx.x);
}

template <int LOGN2>
__global__ void __launch_bounds__(RowSplit<LOGN2>::THREADS)
    rows_kernel(const FlameDev* __restrict__ fls, long long, const long long*, const float*, float*) {
  rows_body<LOGN2>(fls[blockIdx.y], xcd_swizzle(blockIdx.x, gridDim.x), threadIdx.x);
}

namespace {

template <int L, int VAR>
KernelLaunch colm_info(int mode) {
  using C = ColMix<L>;
  if (mode == COL_FIRST)
    return KernelLaunch{reinterpret_cast<const void*>(&colm_kernel<L, COL_FIRST, VAR_EULER>), C::THREADS, C::LDS_BYTES};
  return KernelLaunch{reinterpret_cast<const void*>(&colm_kernel<L, COL_STEP, VAR>), C::THREADS, C::LDS_BYTES};
}

template <int L>
KernelLaunch colm_dispatch(int logn1, int mode, int var) {
  if constexpr (L > kMaxLog) {
    return KernelLaunch{nullptr, 0, 0};
  } else {
    if (logn1 != L) return colm_dispatch<L + 1>(logn1, mode, var);
    switch (var) {
      case VAR_EULER_F: return colm_info<L, VAR_EULER_F>(mode);
      case VAR_HEUN_P: return colm_info<L, VAR_HEUN_P>(mode);
      case VAR_HEUN_C: return colm_info<L, VAR_HEUN_C>(mode);
      case VAR_NT | VAR_EULER: return colm_info<L, VAR_NT | VAR_EULER>(mode);
      case VAR_NT | VAR_EULER_F: return colm_info<L, VAR_NT | VAR_EULER_F>(mode);
      case VAR_NT | VAR_HEUN_P: return colm_info<L, VAR_NT | VAR_HEUN_P>(mode);
      case VAR_NT | VAR_HEUN_C: return colm_info<L, VAR_NT | VAR_HEUN_C>(mode);
      default: return colm_info<L, VAR_EULER>(mode);
    }
  }
}

template <int L>
KernelLaunch rowm_dispatch(int logn2, bool nt) {
  if constexpr (L > kMaxLog) {
    return KernelLaunch{nullptr, 0, 0};
  } else {
    if (logn2 != L) return rowm_dispatch<L + 1>(logn2, nt);
    using C = RowMix<L>;
    return KernelLaunch{nt ? reinterpret_cast<const void*>(&rowm_kernel<L, true>)
                           : reinterpret_cast<const void*>(&rowm_kernel<L, false>),
                        C::THREADS, C::LDS_BYTES};
  }
}

template <int L, int VAR>
KernelLaunch cols_info(int mode) {
  if constexpr (L > 12) {  // side by side would take 1024 threads of 128 registers: one after the other (kFewLanes13)
    using C = ColMix<L, kFewLanes13>;
    const void* fn = mode == COL_FIRST ? reinterpret_cast<const void*>(&colm_kernel<L, COL_FIRST, VAR_EULER, kFewLanes13>)
                                       : reinterpret_cast<const void*>(&colm_kernel<L, COL_STEP, VAR, kFewLanes13>);
    return KernelLaunch{fn, C::THREADS, C::LDS_BYTES};
  } else {
    using C = ColSplit<L>;
    const void* fn = mode == COL_FIRST ? reinterpret_cast<const void*>(&cols_kernel<L, COL_FIRST, VAR_EULER>)
                                       : reinterpret_cast<const void*>(&cols_kernel<L, COL_STEP, VAR>);
    return KernelLaunch{fn, C::THREADS, C::LDS_BYTES, ColMix<L>::T > C::T ? ColMix<L>::T / C::T : 1};
  }
}

// The bodies with side-by-side transforms; they have plain stores only, which
// the store kind of a grid allows (the results are the same).
template <int L>
KernelLaunch cols_dispatch(int logn1, int mode, int var) {
  if constexpr (L == 12) {  // never the faster one (split_pays)
    return logn1 == L ? colm_dispatch<L>(logn1, mode, var) : cols_dispatch<L + 1>(logn1, mode, var);
  } else if constexpr (L > kMaxLog8) {
    return KernelLaunch{nullptr, 0, 0};
  } else {
    if (logn1 != L) return cols_dispatch<L + 1>(logn1, mode, var);
    switch (var & ~VAR_NT) {
      case VAR_EULER_F: return cols_info<L, VAR_EULER_F>(mode);
      case VAR_HEUN_P: return cols_info<L, VAR_HEUN_P>(mode);
      case VAR_HEUN_C: return cols_info<L, VAR_HEUN_C>(mode);
      default: return cols_info<L, VAR_EULER>(mode);
    }
  }
}

template <int L>
KernelLaunch rows_dispatch(int logn2) {
  if constexpr (L == 12) {
    return rows_dispatch<L + 1>(logn2);  // never the faster one (split_pays)
  } else if constexpr (L > kMaxLog8) {
    return KernelLaunch{nullptr, 0, 0};
  } else {
    if (logn2 != L) return rows_dispatch<L + 1>(logn2);
    if constexpr (L > 12) {
      using C = RowMix<L, kFewLanes13>;
      return KernelLaunch{reinterpret_cast<const void*>(&rowm_kernel<L, false, kFewLanes13>), C::THREADS, C::LDS_BYTES};
    } else {
      using C = RowSplit<L>;
      return KernelLaunch{reinterpret_cast<const void*>(&rows_kernel<L>), C::THREADS, C::LDS_BYTES,
                          RowMix<L>::B > C::B ? RowMix<L>::B / C::B : 1};
    }
  }
}

}  // namespace

KernelLaunch colp_kernel_info(int logn1, int mode, int pts, int var) {
  if (logn1 < kMinLogProduct) return KernelLaunch{nullptr, 0, 0};
  if (pts == 8) return cols_dispatch<kMinLogProduct>(logn1, mode, var);
  return colm_dispatch<kMinLogProduct>(logn1, mode, var);
}

KernelLaunch rowp_kernel_info(int logn2, int pts, bool nt) {
  if (logn2 < kMinLogRowProduct) return KernelLaunch{nullptr, 0, 0};
  if (pts == 8) return logn2 == 12 ? rowm_dispatch<12>(logn2, nt) : rows_dispatch<kMinLogRowProduct>(logn2);
  return rowm_dispatch<kMinLogRowProduct>(logn2, nt);
}

void launch_colp(int logn1, int mode, int tiles, int nfl, hipStream_t st, const FlameDev* fl, long long n,
                 const void* src, int pts, hipEvent_t ev_start, hipEvent_t ev_stop, int var) {
  const KernelLaunch kl = colp_kernel_info(logn1, mode, pts, var);
  if (!kl.func) return;
  const long long* nb = nullptr;
  const float2* s = static_cast<const float2*>(src);
  void* args[] = {&fl, &n, &nb, &s};
  if (ev_start || ev_stop)
    (void)hipExtLaunchKernel(kl.func, dim3(tiles * kl.mult, nfl), dim3(kl.threads), args, kl.lds, st, ev_start, ev_stop, 0);
  else
    (void)hipLaunchKernel(kl.func, dim3(tiles * kl.mult, nfl), dim3(kl.threads), args, kl.lds, st);
}

namespace {
template <int L>
int mixed_lds(int logn) {
  if constexpr (L <= kMaxLog) {
    if (logn != L) return mixed_lds<L + 1>(logn);
    int b = RowMix<L>::LDS_BYTES;
    if constexpr (L < 12) b = RowSplit<L>::LDS_BYTES > b ? RowSplit<L>::LDS_BYTES : b;
    if constexpr (L == 13) b = RowMix<L, kFewLanes13>::LDS_BYTES > b ? RowMix<L, kFewLanes13>::LDS_BYTES : b;
    if constexpr (L >= kMinLogProduct) {
      b = ColMix<L>::LDS_BYTES > b ? ColMix<L>::LDS_BYTES : b;
      if constexpr (L < 12) b = ColSplit<L>::LDS_BYTES > b ? ColSplit<L>::LDS_BYTES : b;
      if constexpr (L == 13) b = ColMix<L, kFewLanes13>::LDS_BYTES > b ? ColMix<L, kFewLanes13>::LDS_BYTES : b;
    }
    return b;
  }
  return 0;
}
}  // namespace

int mixed_lds_bytes(int logn) { return logn < kMinLogRowProduct ? 0 : mixed_lds<kMinLogRowProduct>(logn); }

}  // namespace flame
