// Kernels on the physical N1 x N2 grid and of the state's layouts (gfx950):
// the averages of a state (Section 3), the column transforms they need, and
// the canonical half spectrum to and from the state layout.

#include <hip/hip_runtime.h>

#include "flame_dev.hpp"
#include "flame_kernels.hpp"
#include "kernel_common.hpp"
#include "mixed_bodies.hpp"
#include "step_bodies.hpp"
#include "transform_shapes.hpp"

namespace flame {

namespace {

// Whether a row pair's two transforms of the averages run side by side: as the
// step's (split_pays), but short rows less long, because the spectral sums
// fill part of the chip beside them. Averages one after the other and side by
// side, us: rows of at most 512 points, at 1024 waves 8192x256 25.4 and 31.4,
// 4096x512 23.6 and 27.8, at 512 waves 4096x256 19.2 and 20.8; 1024 points, at
// 1024 waves 23.7 and 24.0, at 512 17.6 and 16.5; 2048 points, at 1024 21.7 and 20.8.
constexpr bool diag_split_pays(int logn, long long pairs) {
  const long long waves = pairs * ((1 << logn) / 16) / 64;
  return split_pays(logn, pairs, false) && waves <= (logn <= 9 ? 256 : logn == 10 ? 512 : 1024);
}

// Partial sums that other workgroups read in the same launch: stores and loads
// at agent scope, which do not stay in one XCD's L2.
__device__ __forceinline__ void put_part(double* p, double x) {
  __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double get_part(const double* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sum over the workgroup in a fixed order (THREADS a power of two), valid in thread 0.
template <int THREADS>
__device__ __forceinline__ double group_sum(double x, double* red) {
  const int tid = threadIdx.x;
  red[tid] = x;
  __syncthreads();
  for (int w = THREADS / 2; w > 0; w >>= 1) {
    if (tid < w) red[tid] += red[tid + w];
    __syncthreads();
  }
  return red[0];
}

// Spectral sums of block b of n: sum_k w_k |kappa|^2 |Phi~_k|^2 (w = 1 on
// k2 = 0, 2 elsewhere) and a count of non-finite entries.
template <int THREADS>
__device__ __forceinline__ void spectral_part(const FlameDev& f, int b, int n, double* part, double* red) {
  const int total = f.m * f.h1, lh = __builtin_ctz((unsigned)f.h1);
  double acc = 0.0, nb = 0.0;
  for (int e = b * THREADS + (int)threadIdx.x; e < total; e += n * THREADS) {
    const int m = e >> lh, s = e & (f.h1 - 1);
    const float2 v = f.S[e];
    if (!isfinite(v.x) || !isfinite(v.y)) {
      nb += 1.0;
      continue;
    }
    const double k1 = (double)f.s1 * (double)(s - f.n1 / 4), k2 = (double)f.s2 * (double)m;
    const double w = m == 0 ? 1.0 : 2.0;
    acc += w * (k1 * k1 + k2 * k2) * ((double)v.x * v.x + (double)v.y * v.y);
  }
  const double a = group_sum<THREADS>(acc, red);
  __syncthreads();
  const double c = group_sum<THREADS>(nb, red);
  if (threadIdx.x == 0) {
    put_part(part + 2 * b, a);
    put_part(part + 2 * b + 1, c);
  }
}

// The workgroup that finishes last adds up the partial sums and writes the
// averages. Each counts in after its partial sums are stored (waited for), at
// one of kTickets counters, and the last of each of those at a master counter:
// at one counter the workgroups queue up (2300 of them, 4096x512: 23 us). Every
// counter is left at zero for the next launch.
template <int THREADS>
__device__ __forceinline__ void finish(const FlameDev& f, long long n, int n_area, int n_spec, double* out,
                                       double* red) {
  __shared__ unsigned last;
  if (threadIdx.x == 0) {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt 0: this thread's partial sums are in memory
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    const unsigned blocks = (unsigned)(n_area + n_spec), g = blockIdx.x % kTickets;
    unsigned* const mine = f.ticket + (g + 1) * kTicketStride;
    bool all = __hip_atomic_fetch_add(mine, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 ==
               (blocks - g + kTickets - 1) / kTickets;
    if (all) {
      __hip_atomic_store(mine, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      all = __hip_atomic_fetch_add(f.ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 ==
            (blocks < kTickets ? blocks : kTickets);
    }
    last = all;
  }
  __syncthreads();
  if (!last) return;
  double a = 0.0, s = 0.0, b = 0.0;
  for (int i = threadIdx.x; i < n_area; i += THREADS) a += get_part(f.part + i);
  const double* sp = f.part + n_area;
  for (int i = threadIdx.x; i < n_spec; i += THREADS) {
    s += get_part(sp + 2 * i);
    b += get_part(sp + 2 * i + 1);
  }
  a = group_sum<THREADS>(a, red);
  __syncthreads();
  s = group_sum<THREADS>(s, red);
  __syncthreads();
  b = group_sum<THREADS>(b, red);
  if (threadIdx.x == 0) {
    const double r = r0_at(f, n);
    const float2 s00 = f.S[f.n1 / 4];
    out[0] = r + (double)s00.x;
    out[1] = s / (2.0 * r * r);
    out[2] = a / ((double)f.n1 * (double)f.n2);
    out[3] = (b == 0.0 && isfinite(out[2])) ? 1.0 : 0.0;
    __hip_atomic_store(f.ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

}  // namespace

// Averages of the state from its column transforms W on N1 rows: blocks
// [0, n_area) take a group of row pairs each (the area sums), blocks [n_area,
// n_area + n_spec) a part of the spectral sums, and the last one to finish the
// rest: one launch for what were three, the spectral sums beside the row
// transforms. (The spectral blocks first: 2048 x 4096 51 us for 44.) One after
// another: row_body's transforms.
template <int LOGN2>
__global__ void __launch_bounds__(RowCfg<LOGN2>::THREADS) __attribute__((amdgpu_waves_per_eu(2)))
    diag_kernel(const FlameDev* __restrict__ fls, long long n, int n_area, int n_spec, double* __restrict__ out) {
  constexpr int THREADS = RowCfg<LOGN2>::THREADS;
  extern __shared__ float2 lds[];
  const FlameDev f = fls[0];
  double* const red = reinterpret_cast<double*>(lds);
  const int group = blockIdx.x;
  if (group < n_area) {
    const double area = row_body<LOGN2, ROW_DIAG>(f, n, nullptr, nullptr, xcd_swizzle(group, n_area), threadIdx.x);
    __syncthreads();
    const double a = group_sum<THREADS>(area, red);
    if (threadIdx.x == 0) put_part(f.part + group, a);
  } else {
    spectral_part<THREADS>(f, group - n_area, n_spec, f.part + n_area, red);
  }
  __syncthreads();
  finish<THREADS>(f, n, n_area, n_spec, out, red);
}

// The same with a row pair's two transforms side by side.
template <int LOGN2>
__global__ void __launch_bounds__(PhysSplit<LOGN2>::THREADS)
    diag_side_kernel(const FlameDev* __restrict__ fls, long long n, int n_area, int n_spec, double* __restrict__ out) {
  using C = PhysSplit<LOGN2>;
  using I = typename C::I;
  constexpr int G = C::G, T = C::T, NB = C::NB;
  extern __shared__ float2 lds[];
  const FlameDev f = fls[0];
  double* const red = reinterpret_cast<double*>(lds);
  const int group = blockIdx.x;
  if (group < n_area) {
    const int p = threadIdx.x % T, u = threadIdx.x / T, h = u / G, t = u % G;
    const int pair = xcd_swizzle(group, n_area) * T + p;
    const bool live = pair < f.n1 / 2;
    const int row = live ? 2 * pair + h : h;  // a pair past the grid reads pair 0 (not counted)
    const int jt = G == NB || t < NB ? t : 0;
    float2 v[I::REGS];
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = ld(glob(f.Wp) + w_index(row, jt + NB * r, f.m));
#pragma unroll
    for (int r = 12; r < 16; ++r) {
      const int mm = NB * (16 - r) - jt;  // k2 = -mm; mm = M at r = 12, t = 0
      v[r] = ld(glob(f.Wm) + w_index(row, r > 12 || jt > 0 ? mm : 0, f.m));
    }
    const MixTw<I, true> tw(f.tw2, t);
    v[12] = jt > 0 ? v[12] : make_float2(0.f, 0.f);
    mix_fft<I, true, true>(v, lds + p + h * I::LDS, tw);
    const double r0 = r0_at(f, n);
    const float inv_r2 = (float)(1.0 / (r0 * r0));
    constexpr int P = I::NPASS - 1, R = I::radix(P), NV = I::rounds(P) * R;
    float q[NV];
#pragma unroll
    for (int b = 0; b < I::rounds(P); ++b)
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const float2 z = v[b * R + r];
        q[b * R + r] = I::template active<P>(t, b) ? z.x * z.x + z.y * z.y : 0.f;
      }
    const double area = excess_sum(q, inv_r2);
    __syncthreads();
    const double a = group_sum<C::THREADS>(live ? area : 0.0, red);
    if (threadIdx.x == 0) put_part(f.part + group, a);
  } else {
    spectral_part<C::THREADS>(f, group - n_area, n_spec, f.part + n_area, red);
  }
  __syncthreads();
  finish<C::THREADS>(f, n, n_area, n_spec, out, red);
}

// Column transforms of a spectrum on N1 rows (COL_FIRST), Wp and Wm side by side.
template <int LOGN1>
__global__ void __launch_bounds__(PhysSplit<LOGN1>::THREADS)
    first_side_kernel(const FlameDev* __restrict__ fls, const float2* src) {
  using C = PhysSplit<LOGN1>;
  using I = typename C::I;
  constexpr int G = C::G, T = C::T, NB = C::NB, N1 = C::N;
  extern __shared__ float2 lds[];
  const FlameDev f = fls[0];
  const int c = threadIdx.x % T, u = threadIdx.x / T, h = u / G, t = u % G;
  const int m = xcd_swizzle(blockIdx.x, gridDim.x) * T + c;
  const bool live = m < f.m;
  const int jt = G == NB || t < NB ? t : 0;
  gf2* const Sc = glob(src ? const_cast<float2*>(src) : f.S) + (size_t)(live ? m : 0) * f.h1 + N1 / 4;
  float2 v[I::REGS];
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) v[kk < 4 ? kk : kk + 8] = ld(Sc + (kk < 4 ? jt + NB * kk : jt - NB * (8 - kk)));
  const MixTw<I, true> tw(f.tw1, t);
  const float kp = h == 0 ? -(f.s2 * (float)m) : f.s2 * (float)m;
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) {
    const int k1 = kk < 4 ? jt + NB * kk : jt - NB * (8 - kk);
    v[kk < 4 ? kk : kk + 8] = slope(f.s1 * (float)k1, kp, v[kk < 4 ? kk : kk + 8]);
  }
  mix_fft<I, true, true>(v, lds + c + h * I::LDS, tw);
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

// Canonical half spectrum half[k1 + K1][k2] to and from the state S[k2][k1 +
// N1/4] in tiles through LDS, so that both sides are read and written in runs
// of 256 bytes (element by element, one of them went 8 bytes at a time: 8 us
// instead of 4 at 2048x4096). The k2 = 0 column is symmetrised on the way in.
constexpr int kTile = 32, kTileThreads = 256;
template <bool SET>
__global__ void __launch_bounds__(kTileThreads)
    spectrum_kernel(const FlameDev* __restrict__ fls, int flame, float2* __restrict__ half) {
  __shared__ float2 tile[kTile][kTile + 1];
  const FlameDev f = fls[flame];
  const int k1max = f.n1 / 4 - 1;
  const int tm = (f.m + kTile - 1) / kTile, tiles = tm * ((f.h1 + kTile - 1) / kTile);
  const int x = threadIdx.x % kTile, y0 = threadIdx.x / kTile;
  for (int b = blockIdx.x; b < tiles; b += gridDim.x) {
    const int m0 = b % tm * kTile, s0 = b / tm * kTile;  // slot s holds k1 = s - N1/4, row s - 1 of half
#pragma unroll
    for (int i = 0; i < kTile; i += kTileThreads / kTile) {
      const int y = y0 + i;
      if (SET) {
        const int m = m0 + x, s = s0 + y;
        tile[x][y] = m < f.m && s > 0 && s < f.h1 ? half[(size_t)(s - 1) * f.m + m] : make_float2(0.f, 0.f);
      } else {
        const int m = m0 + y, s = s0 + x;
        tile[y][x] = m < f.m && s < f.h1 ? f.S[(size_t)m * f.h1 + s] : make_float2(0.f, 0.f);
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kTile; i += kTileThreads / kTile) {
      const int y = y0 + i;
      if (SET) {
        const int m = m0 + y, s = s0 + x, k1 = s - f.n1 / 4;
        if (m < f.m && s < f.h1) {
          float2 v = tile[y][x];
          if (m == 0 && s > 0 && k1 < 0) v = ff::cconj(half[(size_t)(k1max - k1) * f.m]);
          if (m == 0 && k1 == 0) v.y = 0.f;
          f.S[(size_t)m * f.h1 + s] = v;
        }
      } else {
        const int m = m0 + x, s = s0 + y;
        if (m < f.m && s > 0 && s < f.h1) half[(size_t)(s - 1) * f.m + m] = tile[x][y];
      }
    }
    __syncthreads();
  }
}

namespace {

template <int L>
void diag_dispatch(int logn2, int groups, int n_spec, hipStream_t st, const FlameDev* fl, long long n, double* out) {
  if constexpr (L <= kMaxLog) {
    if (logn2 != L) return diag_dispatch<L + 1>(logn2, groups, n_spec, st, fl, n, out);
    if constexpr (L <= kMaxLogSide) {
      using C = PhysSplit<L>;
      const int pairs = groups * RowCfg<L>::B;
      if (diag_split_pays(L, pairs)) {
        const int n_area = (pairs + C::T - 1) / C::T;
        hipLaunchKernelGGL(diag_side_kernel<L>, dim3(n_area + n_spec), dim3(C::THREADS), C::LDS_BYTES, st, fl, n,
                           n_area, n_spec, out);
        return;
      }
    }
    hipLaunchKernelGGL(diag_kernel<L>, dim3(groups + n_spec), dim3(RowCfg<L>::THREADS), RowCfg<L>::LDS_BYTES, st, fl, n,
                       groups, n_spec, out);
  }
}

template <int L>
bool first_dispatch(int logn1, int columns, hipStream_t st, const FlameDev* fl, const float2* src) {
  if constexpr (L <= kMaxLogSide) {
    if (logn1 != L) return first_dispatch<L + 1>(logn1, columns, st, fl, src);
    if (!split_pays(L, columns, true)) return false;
    using C = PhysSplit<L>;
    hipLaunchKernelGGL(first_side_kernel<L>, dim3((columns + C::T - 1) / C::T), dim3(C::THREADS), C::LDS_BYTES, st, fl,
                       src);
    return true;
  }
  return false;
}

template <int L>
int phys_lds(int logn) {
  if constexpr (L <= kMaxLogSide)
    return logn == L ? PhysSplit<L>::LDS_BYTES : phys_lds<L + 1>(logn);
  return 0;
}

}  // namespace

int phys_lds_bytes(int logn) { return phys_lds<kMinLog>(logn); }

void launch_diag(int logn2, int groups, int n_spec, hipStream_t st, const FlameDev* fl, long long n, double* out) {
  diag_dispatch<kMinLog>(logn2, groups, n_spec, st, fl, n, out);
}

bool launch_first_side(int logn1, int columns, hipStream_t st, const FlameDev* fl, const float2* src) {
  return first_dispatch<kMinLog>(logn1, columns, st, fl, src);
}

// Workgroups for a box of `total` modes: one per tile. A box of few columns k2
// fills its tiles only in part: there are at most 256 of those (k1 <= 8192),
// and a workgroup past them ends at once (4096x16 in and out 17.2 us with one
// per 1024 modes, 10.2 with these).
static int spectrum_blocks(int total) {
  const int full = total / (kTile * kTile), thin = total / (4 * kTile);
  const int blocks = full > 256 ? full : (thin < 256 ? thin : 256);
  return blocks < 1 ? 1 : (blocks < 4096 ? blocks : 4096);
}

void launch_set_spectrum(hipStream_t st, const FlameDev* fl, int flame, int total, const void* half) {
  const int blocks = spectrum_blocks(total);
  hipLaunchKernelGGL(spectrum_kernel<true>, dim3(blocks), dim3(kTileThreads), 0, st, fl, flame,
                     static_cast<float2*>(const_cast<void*>(half)));
}

void launch_get_spectrum(hipStream_t st, const FlameDev* fl, int flame, int total, void* half) {
  const int blocks = spectrum_blocks(total);
  hipLaunchKernelGGL(spectrum_kernel<false>, dim3(blocks), dim3(kTileThreads), 0, st, fl, flame,
                     static_cast<float2*>(half));
}

}  // namespace flame
