// Device-side description of one flame and the kernel configuration shared
// by the kernels and the host runtime.

#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "fft_engine.hpp"

namespace flame {

// Minimum waves per SIMD the row and column kernels are compiled for (a
// register budget of 512 / waves VGPRs).
#ifndef ROW_WAVES_PER_EU
#define ROW_WAVES_PER_EU 3
#endif
#ifndef COL_WAVES_PER_EU
#define COL_WAVES_PER_EU 2
#endif
#ifndef ADJ_ROW_WAVES_PER_EU
#define ADJ_ROW_WAVES_PER_EU 2
#endif

// Per-flame pointers and constants read by every kernel (one entry per flame
// in a device array; blockIdx.y selects the flame inside a launch).
struct FlameDev {
  float2* S;           // state, [M][H1]
  float2* Wp;          // column transforms of (i kappa1 - kappa2) Phi~ and ...
  float2* Wm;          // ... the conj of those of (i kappa1 + kappa2) Phi~, interleaved
                       // [j1/4][m][j1%4], Wp and Wm in the two halves of W (index with w_index)
  float2* Q;           // row transforms of |grad Phi|^2 (and scratch), tiled [m/TQ][j1][m%TQ]
  float2* A1;          // adjoint scratch, same layout: row transform of w1 = m g1
  float2* A2;          // adjoint scratch, same layout: i kappa2 x row transform of w2 = m g2
  const float2* tw1;   // twiddles of the length-N1 transform, 16 points per thread
  const float2* tw2;   // twiddles of the length-N2 transform, 16 points per thread
  const float2* tw1_8; // the same for 8 points per thread
  const float2* tw2_8;
  const float2* twma;  // twiddles of the length-3N1/4 transforms (ff::MixTables), or null
  const float2* twmb;  // the same for length 3N2/4
  const float2* twfa;  // twiddles of the length-N1 transforms of ff::FullPlan (N1 <= 64), or null
  const float2* twfb;  // the same for length N2
  double* part;        // per-workgroup partial sums of the diagnostics
  unsigned* ticket;    // counters of the workgroups of a diagnostics launch that have finished: a
                       // master and kTickets others, kTicketStride apart, zero between launches
  const double* r0tab; // reference-radius table {r0(t_n), I1_n, I2_n} (r0_law = 1), or null for r0 = t
  long long r0n;       // its entries
  const float2* F;     // forcing f~ of Eq. (1) in the state layout [M][H1], or null (f~ = 0)
  float2* S2;          // Heun's predictor Phi* in the state layout (workspace; the A2 scratch)
  int n1, n2;
  int m;               // stored k2 columns, N2/4
  int h1;              // stored k1 slots, N1/2
  int tshift;          // log2 of the tile width TQ of Q, A1, A2
  int rows;            // theta rows of the step's product grid: 3 N1/4, or N1
  float s1, s2;        // axis scales of kappa
  float gamma;
  int cols;            // phi points of the step's product grid: 3 N2/4, or N2
  double t0, dt;
};

// A batch of circular flames (the one-dimensional form of Eq. (1)) of one
// grid: spectra S[c][k], k = 0 .. N/4 - 1, complex64, caller-owned.
struct CircleDev {
  float2* S;
  int n_circles;
  float seg;     // segment integer: kappa_k = seg k
  float gamma;
  int pad_;
  double t0, dt;
};

// Register shape of a length-N transform with PTS (8 or 16) points per
// thread. LOW, HIGH: registers i < LOW hold the spectral positions
// k = t + G i >= 0 of the retained box, i >= HIGH the negative ones (k - N);
// the registers between hold padding.
template <int LOGN, int PTS>
struct TfShape {
  using S = ff::Shape<LOGN, PTS>;
  static constexpr int LOW = PTS / 4, HIGH = 3 * PTS / 4;
};
template <int LOGN, int PTS>
using TShape = typename TfShape<LOGN, PTS>::S;

// Column kernel: T = max(1, 16*256/N1) columns per workgroup, interleaved
// (thread tid works on column tid % T, FFT lane tid / T); the transform of
// each column uses G = N1/PTS threads. T does not depend on PTS.
//
// Q is tiled [m/TQ][j1][m%TQ] with TQ = 2T for N1 >= 2048 (else TQ = T): a
// row-kernel workgroup at N2 = 4096 holds one row pair, so with TQ = T its
// pieces of Q (2 rows x TQ columns of 8 bytes) would be 32 or 16 bytes, and
// HBM writes in pieces under 64 bytes run at about half the bandwidth of
// longer ones. The column kernel then reads half of each 2-row piece and the
// neighbouring workgroup (same XCD) the other half.
constexpr int col_tile_for(int g16) { return g16 >= 256 ? 1 : 256 / g16; }
constexpr int q_tile_for(int g16) { return g16 >= 128 ? 2 * col_tile_for(g16) : col_tile_for(g16); }

template <int LOGN1, int PTS = ff::kPts>
struct ColCfg {
  static constexpr int G16 = ff::Shape<LOGN1>::G;
  static constexpr int G = TShape<LOGN1, PTS>::G;
  static constexpr int T = col_tile_for(G16);
  static constexpr int TQ = q_tile_for(G16);
  static constexpr int QS = ff::ilog2c(TQ);
  static constexpr int THREADS = T * G;
  static constexpr int LDS_BYTES = TShape<LOGN1, PTS>::LDS * T * 8;
};

// Product grid of the step: |grad Phi|^2 is formed on M1 = 3 N1/4 theta rows
// instead of N1. The product of two fields with |k1| <= K1 = N1/4 - 1 has
// |k1| <= 2 K1, and on M1 >= 3 K1 + 1 rows no alias of it lands in
// |k1| <= K1, so the truncated quadratic term is the same as on N1 rows up to
// rounding. Used for N1 >= 128. The same holds along phi: the step's row
// kernel forms the term on 3 N2/4 points for N2 >= 64 (mixed_bodies.hpp).
constexpr int kMinLogProduct = 7;
constexpr int kMinLogRowProduct = 6;
// Added to the row kernel's points per thread: on all N2 phi points.
constexpr int kRowFull = 64;

// One set of counters per flame, as of partial sums: the averages of two flames
// of a plan, captured apart, may be replayed at the same time.
constexpr unsigned kTickets = 32, kTicketStride = 32, kTicketWords = (kTickets + 1) * kTicketStride;

// Resident kernels (resident_kernel.hip) exist for N1 N2 <= 2^kResMaxLogs and
// where a flame's intermediates fit one workgroup's LDS.
constexpr int kResMaxLogs = 14;
// Steps per resident launch at most.
constexpr int kResMaxSteps = 2000;
// FullPlan twiddles exist for lengths up to 2^kMaxLogFull.
constexpr int kMaxLogFull = 6;

// Whether a step kernel on a product grid runs the bodies for few transforms
// (mixed_bodies.hpp, "few transforms"): `transforms` columns or row pairs of
// length 2^logn in the launch, which the other bodies run on N/16 lanes each.
// Measured: up to 2048 points they win while those lanes make at most half a
// wave per SIMD of the chip for the columns (512 waves: 1024x2048 9.4 against
// 11.6 us; at 1024 waves, 1024x4096, 15.2 against 14.9) and one wave per SIMD
// for the rows (768 waves: 9.0 against 9.4 us). At 4096 points a workgroup of
// either kind is one transform and fills its compute unit's issue slots, and
// side by side is slower (9.5 against 8.5 us for 96 row pairs). At 8192 points
// the variant is 768 lanes instead of 256: faster while every compute unit
// has at most one transform (128x8192 12.8 against 16.9 us), slower where two
// workgroups of 256 threads can share one (8192x8192: 198 against 162 us).
constexpr bool split_pays(int logn, long long transforms, bool columns) {
  const long long waves = transforms * ((1 << logn) / 16) / 64;
  return logn <= 11 ? waves <= (columns ? 512 : 1024) : logn == 13 && transforms <= 256;
}
// The step's row kernel. Rows of at most 256 points have two passes and one
// exchange, little to wait for, and half as many waves are enough for them: at
// 768 waves 8192x256 takes 7.5 us side by side and 6.6 one after the other,
// 16384x128 6.6 and 6.1 (4096x512 7.8 and 8.0); at 384, 4096x256, 5.3 and 5.7.
constexpr bool split_pays_rows(int logn, long long pairs) {
  return split_pays(logn, pairs, false) && (logn > 8 || pairs * ((1 << logn) / 16) / 64 <= 512);
}

// Row kernel: B = max(1, 16*256/N2) row pairs per workgroup, interleaved.
// WPE: the minimum waves per SIMD it is compiled for; at N2 = 8192 with 16
// points per thread a workgroup is 8 waves (2 per SIMD), which may then use
// the whole register budget instead of spilling.
template <int LOGN2, int PTS = ff::kPts>
struct RowCfg {
  static constexpr int G16 = ff::Shape<LOGN2>::G;
  static constexpr int G = TShape<LOGN2, PTS>::G;
  static constexpr int B = G16 >= 256 ? 1 : 256 / G16;
  static constexpr int THREADS = B * G;
  static constexpr int LDS_BYTES = TShape<LOGN2, PTS>::LDS * B * 8;
  static constexpr int WPE = THREADS >= 512 && PTS == 16 ? 2 : ROW_WAVES_PER_EU;
};

constexpr int col_tile(int logn1) { return col_tile_for((1 << logn1) / ff::kPts); }
constexpr int q_tile(int logn1) { return q_tile_for((1 << logn1) / ff::kPts); }
constexpr int row_pairs(int logn2) { return (1 << logn2) / ff::kPts >= 256 ? 1 : 256 / ((1 << logn2) / ff::kPts); }

enum ColMode : int { COL_STEP = 0, COL_FIRST = 1, COL_PROJECT = 2, COL_SYNTH = 3 };
// Variants of the step's column kernel (COL_STEP): integrating-factor Euler
// without the forcing term (compiled out) or with it, and the two stages of
// integrating-factor Heun, which read the forcing when one is bound:
//   VAR_HEUN_P: predictor Phi* = E (Phi~^n + dt (f~ - c_n N(Phi~^n))) -> S2;
//   VAR_HEUN_C: corrector Phi~^{n+1} = (Phi* + E Phi~^n + dt (f~ - c_{n+1} N(Phi*))) / 2 -> S.
enum StepVar : int { VAR_EULER = 0, VAR_EULER_F = 1, VAR_HEUN_P = 2, VAR_HEUN_C = 3 };
// Or-ed into a StepVar: the column kernel writes W with non-temporal stores
// (the row kernel's Q stores take the same choice through its NT argument).
constexpr int VAR_NT = 4;
enum RowMode : int { ROW_STEP = 0, ROW_FORWARD = 1, ROW_SYNTH = 2, ROW_DIAG = 3 };
// Adjoint column kernel: ADJ_A forms mu = E lambda and the column transforms
// of mu and of the state's packed gradient; ADJ_C / SEED_C form the
// divergence from the row transforms in A1, A2 and write the cotangent.
enum AdjColMode : int { ADJ_A = 0, ADJ_C = 1, SEED_C = 2 };
// Adjoint row kernel: ROW_ADJ forms w = m grad Phi (on 3 N2/4 phi points where
// there is a transform of that length; ROW_ADJ_FULL: on N2), ROW_SEED forms
// w = grad Phi / (r0^2 sqrt(1 + |grad Phi|^2 / r0^2)); all write the row
// transforms of w1 and i kappa2 w2 to A1, A2.
enum AdjRowMode : int { ROW_ADJ = 0, ROW_SEED = 1, ROW_ADJ_FULL = 2 };

// Keep each thread's twiddles in registers for a kernel's lifetime (the
// alternative reads the table in every pass).
#ifndef FLAME_CACHE_TWIDDLES
#define FLAME_CACHE_TWIDDLES 1
#endif
constexpr bool kCacheTwiddles = FLAME_CACHE_TWIDDLES != 0;
// Passes with Ns >= this keep their twiddles in registers (2: every pass).
#ifndef FLAME_TW_CACHE_MIN_NS
#define FLAME_TW_CACHE_MIN_NS 2
#endif
constexpr int kTwCacheMinNs = FLAME_TW_CACHE_MIN_NS;
// Prune the first butterfly of inverse transforms whose input is zero in the
// middle half of the padded spectrum.
#ifndef FLAME_PRUNE
#define FLAME_PRUNE 1
#endif
constexpr bool kPrune = FLAME_PRUNE != 0;


constexpr int kMinLog = 4;
constexpr int kMaxLog = 14;
// Lengths up to 2^kMaxLog8 have the 8-points-per-thread kernels (beyond it
// they would need more than 1024 threads per workgroup).
constexpr int kMaxLog8 = 13;

// Persistent ensemble kernel: one co-resident grid of workgroups steps every
// flame of a plan for all steps of a launch. A workgroup's share is either
// `nfl` whole flames from `flame` on, which it steps alone (parts == 1), or
// part `part` of the `parts` workgroups that share flame `flame`: it takes
// the row-pair groups and column tiles part, part + parts, ... of each step
// and meets the others at that flame's arrival counter after each phase.
struct EnsembleItem {
  int flame, nfl, part, parts;
  int logn1, logn2;    // the grid of its flames
  int rtiles, ctiles;  // row-pair groups and column tiles of one flame
};
// Its step kernels' bodies: the product-grid columns (N1 = 2^7 .. 2^10) and
// rows (N2 = 2^7 .. 2^11), all of them 256 threads per workgroup.
constexpr int kEnsThreads = 256;
constexpr int kEnsMinLog1 = 7, kEnsMaxLog1 = 10;
constexpr int kEnsMinLog2 = 7, kEnsMaxLog2 = 11;
constexpr int kEnsArriveStride = 32;  // 128 bytes between two flames' arrival counters

}  // namespace flame
