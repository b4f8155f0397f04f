// Host side of the lattice steps on the CPU: the queueing of steps with the
// launches replaced by recorders (no device is touched).
#include <hip/hip_runtime.h>

#include "no_device.h"

#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(...) ((void)0)
#include "../../paper_1806_10251_amd/csrc/lbm_api.hip"

namespace lbmk {

static StepArgs g_single;
static int g_multi_calls;

template <int ST, int FL>
void launch_step(int, int, int, const void*, void*, const StepArgs& a, const void*, hipStream_t) {
  g_single = a;
}
template <int ST>
bool launch_multi(int, const void*, void*, const StepArgs&, const uint8_t*, const void*,
                  hipStream_t) {
  ++g_multi_calls;
  return false;   // as where the device refuses the LDS
}

}  // namespace lbmk

// A two-step launch that is refused: the single step that takes its place
// covers the lattice with its own tiles.
static int refused() {
  static lbm_ctx c;
  c.grid = lbm_grid{};
  c.grid.nx = 200;
  c.grid.ny = 100;
  for (int i = 0; i < 4; ++i) c.grid.side[i] = LBM_SIDE_WALL;
  c.p.check_every = 100;
  c.p.storage = LBM_STORE_F32;
  c.tiles_x = 4;
  c.tiles_y = 25;
  c.ntiles = 100;
  c.out_rows = 4;
  c.multi = 0;
  const int taken = enqueue_steps(&c, 10, nullptr);
  std::printf("%d %d %d %d %d %lld\n", taken, lbmk::g_multi_calls, lbmk::g_single.tiles_x,
              lbmk::g_single.ntiles, c.cur, (long long)c.t);
  return 0;
}

// shape of the two-step kernel and allowed share of rows near solid nodes:
// nx ny W E S N storage mask
static int shape(char** v) {
  static lbm_ctx c;
  static uint8_t solid;
  c.grid.nx = std::atoi(v[0]);
  c.grid.ny = std::atoi(v[1]);
  for (int i = 0; i < 4; ++i) c.grid.side[i] = std::atoi(v[2 + i]);
  c.p.storage = std::atoi(v[6]);
  c.esize = storage_bytes(c.p.storage);
  c.d_solid = std::atoi(v[7]) ? &solid : nullptr;
  const int s = multi_shape(&c);
  std::printf("%d %g\n", s, s < 0 ? 0.0 : multi_near_share(&c, s));
  return 0;
}

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  if (what == "refused") return refused();
  if (what == "shape" && argc == 10) return shape(argv + 2);
  return 2;
}
