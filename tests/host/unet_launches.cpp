// Which kernels a convolution of the network's layers launches, on the CPU:
// launches replaced by recorders.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include <hip/hip_runtime.h>

#include "no_device.h"

static void record(const char* fn, dim3 g, dim3 b) {
  // (the tiled forms are launched through a pointer)
  const std::string name(fn, std::strcspn(fn, "<"));
  std::printf("%s %u %u %u\n", name == "fn" ? "tile" : name.c_str(), g.x, g.y, b.x);
}

#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(fn, grid, block, ...) record(NAME_OF(fn), grid, block)
#define hipFuncSetAttribute(...) hipSuccess
#define hipGetLastError() hipSuccess
template <class F>
static const char* name_of(F, const char* text) {
  return text;
}
#define NAME_OF(fn) name_of(fn, #fn)
#include "../../paper_1806_10251_amd/csrc/unet.hip"

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  static char mem[4096];
  int v[8] = {};
  for (int i = 2; i < argc && i < 10; ++i) v[i - 2] = std::atoi(argv[i]);
  const int n = v[0], h = v[1], w = v[2], ci = v[3], co = v[4];
  if (what == "fwd")
    return unet_conv3x3_fwd(mem, ci, mem, nullptr, mem, co, n, h, w, ci, co, 0, 0, nullptr);
  if (what == "bwdw")
    return unet_conv3x3_bwd_weight(mem, co, mem, ci, (float*)mem, (float*)mem, n, h, w, ci, co,
                                   (float*)mem, nullptr);
  if (what == "work") {
    std::printf("%lld\n", (long long)unet_wgrad_work_floats(n, h, w, ci, co));
    return 0;
  }
  return 2;
}
