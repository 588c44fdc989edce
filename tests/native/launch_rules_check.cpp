// Host-sanitizer drive of the rules by which flame_api.hip picks its launches,
// on devices that the checked model of the HIP calls (hipstub) does not have:
// built like plan_bookkeeping_check.cpp, with the model's device queries
// replaced by the ones below. The argument names the check; each prints "OK".
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include <hip/hip_runtime.h>

#include "flame_kernels.hpp"

#define launch_row stub_launch_row
#define col_step_kernel stub_col_step_kernel
#define row_step_kernel stub_row_step_kernel
#define colp_kernel_info stub_colp_kernel_info
#define ensemble_blocks_per_cu stub_blocks_per_cu
#define hipDeviceGetAttribute stub_device_attribute
#include "hipstub/hip_stub.cpp"
#undef hipDeviceGetAttribute
#undef ensemble_blocks_per_cu
#undef launch_row
#undef col_step_kernel
#undef row_step_kernel
#undef colp_kernel_info

#include "flame.h"

namespace {
int g_blocks_per_cu = 2;
int g_max_lds = 160 * 1024;
}  // namespace

hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int dev) {
  if (a != hipDeviceAttributeMaxSharedMemoryPerBlock) return stub_device_attribute(v, a, dev);
  *v = g_max_lds;
  return hipSuccess;
}

namespace {
flame::FlameDev g_diag;  // the flame of the last launch of averages
flame::FlameDev g_step;  // and of the last row kernel of a step, with its points per thread
int g_step_pts = 0;
long g_row_steps = 0;

// A kernel for each choice, as the library has them: on a product grid 8
// points are the bodies for few transforms, which have plain stores only.
const char g_kernels[4][128] = {};
flame::KernelLaunch a_kernel(int kind, int pts, int var) {
  return flame::KernelLaunch{&g_kernels[kind][(pts & 31) * 4 + (var & 3)], 256, 0};
}
}

namespace flame {
int ensemble_blocks_per_cu() { return g_blocks_per_cu; }
KernelLaunch col_step_kernel(int, int pts, int var) {
  return pts == 12 ? KernelLaunch{nullptr, 0, 0} : a_kernel(0, pts, (var & VAR_NT) != 0);
}
KernelLaunch colp_kernel_info(int logn1, int, int pts, int var) {
  if (logn1 < kMinLogProduct) return KernelLaunch{nullptr, 0, 0};
  return a_kernel(1, pts == 8 ? 8 : 12, pts != 8 && (var & VAR_NT) != 0);
}
KernelLaunch row_step_kernel(int logn2, int pts, bool nt) {
  if (logn2 < kMinLogRowProduct || (pts & kRowFull)) return a_kernel(2, pts, nt);
  return a_kernel(3, pts == 8 ? 8 : 12, pts != 8 && nt);
}
void launch_row(int logn2, int mode, int groups, int nfl, hipStream_t st, const FlameDev* fl, long long n,
                const float* in, float* out, int pts, hipEvent_t e0, hipEvent_t e1, bool nt) {
  if (mode == ROW_DIAG) g_diag = *fl;
  if (mode == ROW_STEP) {
    g_step = *fl;
    g_step_pts = pts;
    ++g_row_steps;
  }
  stub_launch_row(logn2, mode, groups, nfl, st, fl, n, in, out, pts, e0, e1, nt);
}
}  // namespace flame

// Resident kernels of 100 KB for n1 n2 <= 2^14, as resident_kernel.hip
// registers its own; the launches are counted.
namespace {
constexpr int kResidentLds = 100 * 1024;
long g_resident_launches = 0, g_resident_steps = 0;

flame::KernelLaunch resident_info(int logn1, int logn2, int) {
  if (logn1 + logn2 > flame::kResMaxLogs) return flame::KernelLaunch{nullptr, 0, 0};
  return flame::KernelLaunch{flame::kDummyKernel, 256, kResidentLds};
}
void resident_run(const flame::KernelLaunch& kl, int flames, hipStream_t st, const flame::FlameDev* fl, long long,
                  int steps, int) {
  if (kl.func != flame::kDummyKernel || kl.lds > g_max_lds) violation("resident launch past the device's LDS");
  if (flames < 1 || steps < 1 || steps > flame::kResMaxSteps) violation("resident launch out of range");
  flame::touch(fl, flames);
  ++g_resident_launches;
  g_resident_steps += steps;
  hip_stub_launch(kl.func, st);
}
const bool g_registered =
    (flame::resident_kernel = &resident_info, flame::resident_launch = &resident_run, true);
}  // namespace

namespace {

#define CHECK(x)                                                                             \
  do {                                                                                       \
    const int rc_ = (x);                                                                     \
    if (rc_ != FLAME_OK) {                                                                   \
      std::fprintf(stderr, "%s:%d: %s returned %d: %s\n", __FILE__, __LINE__, #x, rc_,      \
                   flame_last_error());                                                      \
      std::exit(3);                                                                          \
    }                                                                                        \
  } while (0)
#define EXPECT(x)                                                             \
  do {                                                                        \
    if (!(x)) {                                                               \
      std::fprintf(stderr, "%s:%d: not so: %s\n", __FILE__, __LINE__, #x);    \
      std::exit(4);                                                           \
    }                                                                         \
  } while (0)

flame_desc desc(int n1, int n2, int integrator = 0) {
  flame_desc d;
  std::memset(&d, 0, sizeof d);
  d.n1 = n1;
  d.n2 = n2;
  d.gamma = 0.8;
  d.theta_pi = 1.0;
  d.t0 = 200.0;
  d.dt = 0.25;
  d.integrator = integrator;
  return d;
}

void* aligned(size_t bytes) {
  void* p = std::aligned_alloc(256, (bytes + 255) / 256 * 256);
  if (!p) std::exit(5);
  std::memset(p, 0, bytes);
  return p;
}

struct Plan {
  std::vector<flame_desc> d;
  std::vector<void*> states;
  void* ws = nullptr;
  flame_plan p = nullptr;
  explicit Plan(std::vector<flame_desc> descs) : d(std::move(descs)) {
    size_t b = 0;
    for (const flame_desc& x : d) {
      CHECK(flame_state_bytes(&x, &b));
      states.push_back(aligned(b));
    }
    CHECK(flame_workspace_bytes(d.data(), (int)d.size(), &b));
    ws = aligned(b);
    CHECK(flame_init(d.data(), (int)d.size(), states.data(), ws, b, nullptr, &p));
  }
  ~Plan() {
    if (p) CHECK(flame_destroy(p));
    for (void* s : states) std::free(s);
    std::free(ws);
  }
};

// The persistent grid takes two workgroups of each compute unit unless the
// caller asks for another count, also where more would fit.
void persistent_default() {
  for (int per_cu : {1, 2, 3}) {
    g_blocks_per_cu = per_cu;
    std::vector<flame_desc> ds(256, desc(128, 256));
    for (int i = 0; i < 64; ++i) ds.push_back(desc(512, 1024));
    Plan pl(ds);
    CHECK(flame_set_points_per_thread(pl.p, 128, 256, 12, 16));
    CHECK(flame_set_points_per_thread(pl.p, 512, 1024, 12, 16));
    CHECK(flame_set_persistent(pl.p, 1, 0, 0));
    CHECK(flame_step(pl.p, 1));
    int32_t on = 0, wgs = 0;
    CHECK(flame_get_persistent(pl.p, &on, &wgs));
    EXPECT(on == 1 && wgs > 256 * (per_cu > 1 ? 1 : 0) && wgs <= 256 * (per_cu < 2 ? per_cu : 2));
  }
}

// Where a device has less LDS than a resident kernel asks for, the small
// flames take the two launches a step, here and in the allocation-free call.
void resident_lds() {
  for (int lds : {160 * 1024, 64 * 1024}) {
    g_max_lds = lds;
    g_resident_launches = g_resident_steps = 0;
    Plan pl({desc(64, 128), desc(32, 64, 1)});
    CHECK(flame_step(pl.p, 3));
    CHECK(flame_set_graph_steps(pl.p, 2));
    CHECK(flame_step(pl.p, 4));
    flame_desc d = desc(64, 128);
    std::vector<float> s(64 * 128 / 4, 0.f);
    CHECK(flame_step_noalloc(&d, s.data(), 0, 5, nullptr));
    EXPECT(lds >= kResidentLds ? g_resident_steps == 3 + 3 + 5 : g_resident_launches == 0);
  }
}

// The resident paths of flame_step, its graphs, timing, autotuning and the
// settings that enter and leave them, in a plan that has other groups too.
void resident_paths() {
  for (int graph : {0, 1, 7, 2001}) {
    Plan pl({desc(64, 128), desc(64, 128), desc(32, 64, 1), desc(128, 128), desc(256, 512)});
    flame_plan p = pl.p;
    std::vector<float> spec(256 * 512 / 4, 0.f);
    for (int f = 0; f < 5; ++f) CHECK(flame_set_spectrum(p, f, spec.data(), 0));
    g_resident_steps = 0;
    CHECK(flame_set_graph_steps(p, graph));
    int64_t n = 0;
    CHECK(flame_step(p, 2003));
    CHECK(flame_step_index(p, &n));
    EXPECT(n == 2003);
    EXPECT(g_resident_steps == 3 * (graph ? 2003 % graph : 2003));  // three groups; the others are in the graphs
    for (int it = 0; it < 24; ++it) {
      CHECK(flame_set_points_per_thread(p, 64, 128, it % 3 == 1 ? 8 : 16, 16));
      CHECK(flame_set_product_grid(p, 128, 128, it % 2));
      CHECK(flame_set_forcing(p, 0, it % 4 == 1 ? spec.data() : nullptr));
      if (it % 5 == 0) CHECK(flame_set_graph_steps(p, it % 10 ? 0 : graph));
      CHECK(flame_timing_begin(p));
      CHECK(flame_step(p, it % 3));
      double ms[4];
      int64_t cnt[4];
      CHECK(flame_timing_end(p, ms, cnt));
    }
    CHECK(flame_autotune(p, 1, nullptr));
    CHECK(flame_step(p, 9));
    CHECK(flame_step_index(p, &n));
    EXPECT(n == 2003 + 8 * 3 + 9);
  }
}

// Two flames' averages share nothing that a launch writes.
void averages_apart() {
  Plan pl({desc(64, 128), desc(64, 128), desc(256, 512)});
  std::vector<flame::FlameDev> seen;
  for (int f = 0; f < 3; ++f) {
    double out[4];
    CHECK(flame_diagnostics(pl.p, f, out, nullptr));
    for (unsigned i = 0; i < (flame::kTickets + 1) * flame::kTicketStride; ++i) EXPECT(g_diag.ticket[i] == 0);
    for (const flame::FlameDev& d : seen) {
      const long long apart = g_diag.ticket - d.ticket;
      EXPECT(std::llabs(apart) >= (long long)((flame::kTickets + 1) * flame::kTicketStride));
      EXPECT(d.part != g_diag.part && d.Wp != g_diag.Wp);
    }
    seen.push_back(g_diag);
  }
}

// The step's grid: the product grid by default, the paper's N1 x N2 where the
// product grid is disabled, with 3 N2/4 of its phi points at 12 row points.
void step_grids() {
  for (const auto& g : {std::pair<int, int>{256, 512}, {64, 512}, {128, 32}}) {
    const int n1 = g.first, n2 = g.second;
    const int m1 = n1 >= 128 ? 3 * n1 / 4 : n1, m2 = n2 >= 64 ? 3 * n2 / 4 : n2;
    Plan pl({desc(n1, n2), desc(n1, n2, 1)});
    auto grid = [&](int rows, int cols) {
      CHECK(flame_step(pl.p, 1));
      EXPECT(g_step.rows == rows && g_step.cols == cols);
      EXPECT(((g_step_pts & flame::kRowFull) != 0) == (cols == n2));
      EXPECT((g_step_pts & ~flame::kRowFull) != 12 || cols == m2);
    };
    CHECK(flame_set_points_per_thread(pl.p, n1, n2, 8, 16));  // no resident kernel
    grid(m1, m2);
    CHECK(flame_set_product_grid(pl.p, n1, n2, 0));
    for (int pts : {8, 16, 12}) {
      if (pts == 12 && n2 < 64) continue;
      CHECK(flame_set_points_per_thread(pl.p, n1, n2, 16, pts));
      grid(n1, pts == 12 ? m2 : n2);
    }
    CHECK(flame_set_points_per_thread(pl.p, n1, n2, 8, 8));
    grid(n1, n2);
    if (n1 >= 128) {
      CHECK(flame_set_product_grid(pl.p, n1, n2, 1));
      grid(m1, m2);
    }
  }
}

// Configurations of the same kernels are timed once, and equal times leave the default.
void autotune_equals() {
  for (int joint : {0, 1}) {
    std::vector<flame_desc> ds{desc(256, 512)};
    if (joint) ds.push_back(desc(512, 512));
    Plan pl(ds);
    CHECK(flame_set_points_per_thread(pl.p, 256, 512, 8, 8));
    if (joint) CHECK(flame_set_graph_steps(pl.p, 2));
    g_row_steps = 0;
    int32_t tried = 0, cp = 0, rp = 0, product = 0, nt = -1;
    CHECK(flame_autotune(pl.p, 1, &tried));
    EXPECT(tried == 30 * (int)ds.size());
    // 12 kernel pairs on N1 rows; on the product grid three column and three
    // row kernels (few; many; many, non-temporal), without the two pairs that
    // mix the bodies for many transforms with different store kinds. Each
    // pair takes two launches in each of three rounds; jointly, three
    // repetitions of one step for the other 18 pairs of each group (and the
    // first trial), with the other group beside it.
    const long alone = 6 * (12 + 7);
    EXPECT(g_row_steps == (joint ? 2 * alone + 2 * 3 * (1 + 2 * 18) : alone));
    CHECK(flame_get_points_per_thread(pl.p, 256, 512, &cp, &rp));
    CHECK(flame_get_product_grid(pl.p, 256, 512, &product));
    CHECK(flame_get_streaming_stores(pl.p, 256, 512, &nt));
    EXPECT(cp == 16 && rp == 16 && product == 1 && nt == 0);
  }
}

}  // namespace

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  if (what == "persistent_default")
    persistent_default();
  else if (what == "resident_lds")
    resident_lds();
  else if (what == "resident_paths")
    resident_paths();
  else if (what == "averages_apart")
    averages_apart();
  else if (what == "step_grids")
    step_grids();
  else if (what == "autotune_equals")
    autotune_equals();
  else
    return 2;
  std::printf("OK\n");
  return 0;
}
