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

#define ensemble_blocks_per_cu stub_blocks_per_cu
#include "hipstub/hip_stub.cpp"
#undef ensemble_blocks_per_cu

#include "flame.h"

namespace {
int g_blocks_per_cu = 2;
}

namespace flame {
int ensemble_blocks_per_cu() { return g_blocks_per_cu; }
}  // namespace flame

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

}  // namespace

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  if (what == "persistent_default")
    persistent_default();
  else
    return 2;
  std::printf("OK\n");
  return 0;
}
