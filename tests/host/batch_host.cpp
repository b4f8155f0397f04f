// Host side of a batch on the CPU: device memory from malloc, launches and
// copies replaced by recorders.
#include <algorithm>
#include <chrono>
#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <set>
#include <string>
#include <thread>
#include <tuple>
#include <vector>

#include <hip/hip_runtime.h>

#include "no_device.h"

namespace rec {

std::mutex mu;
std::condition_variable cv;
std::set<char*> live;         // allocations
int allocs = 0, uploads = 0, waiting = 0, meet = 0;
bool stale = false;           // a copy from memory that was given back
thread_local char* exported;  // destination of this thread's last export
std::vector<char*> exports;

hipError_t alloc(void** p, size_t n) {
  std::lock_guard<std::mutex> l(mu);
  *p = std::malloc(n + 64);
  live.insert((char*)*p);
  ++allocs;
  return hipSuccess;
}
hipError_t give_back(void* p) {
  std::lock_guard<std::mutex> l(mu);
  live.erase((char*)p);       // (kept by malloc: addresses stay distinct)
  return hipSuccess;
}
hipError_t copy(void* dst, const void* src, size_t n, hipMemcpyKind kind) {
  std::lock_guard<std::mutex> l(mu);
  if (kind == hipMemcpyHostToDevice) {
    ++uploads;
    std::memcpy(dst, src, n);
  } else if (exported && src >= exported && !live.count(exported)) {
    stale = true;
  }
  return hipSuccess;
}
// Waits until `meet` threads are here, two seconds at most.
hipError_t sync() {
  std::unique_lock<std::mutex> l(mu);
  ++waiting;
  cv.notify_all();
  cv.wait_for(l, std::chrono::seconds(2), [] { return waiting >= meet; });
  return hipSuccess;
}
template <class... A>
void launch(A... a) {
  if constexpr (sizeof...(A) == 14) {   // export_kernel: the last three are the outputs
    std::lock_guard<std::mutex> l(mu);
    exported = (char*)std::get<11>(std::tuple<A...>(a...));
    exports.push_back(exported);
  }
}

}  // namespace rec

#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(fn, grid, block, lds, st, ...) rec::launch(__VA_ARGS__)
#define hipMalloc(p, n) rec::alloc((void**)(p), n)
#define hipFree(p) rec::give_back(p)
#define hipMemcpy(d, s, n, k) rec::copy(d, s, n, k)
#define hipStreamSynchronize(s) rec::sync()
#include "../../paper_1806_10251_amd/csrc/lbm_batch.hip"

namespace lbmh {
int fail(int code, const std::string& msg) {
  std::fprintf(stderr, "%s\n", msg.c_str());
  return code;
}
}  // namespace lbmh
extern "C" const char* lbm_last_error(void) { return ""; }

// Cases "nx ny W E S N solid" (solid: every solid-th node, 0 none).
static void add_case(lbm_batch& b, char** v) {
  HostCase c;
  c.grid = lbm_grid{};
  c.grid.nx = std::atoi(v[0]);
  c.grid.ny = std::atoi(v[1]);
  for (int i = 0; i < 4; ++i) c.grid.side[i] = std::atoi(v[2 + i]);
  c.g = make_geom_for(c.grid.nx, c.grid.ny, c.grid.side, b.storage == LBM_STORE_F64 ? 8 : 4);
  c.h_mask.assign((size_t)c.grid.nx * c.grid.ny, 0);
  if (const int every = std::atoi(v[6]))
    for (size_t i = 0; i < c.h_mask.size(); i += every) c.h_mask[i] = 1;
  b.cs.push_back(c);
  ++b.n;
  b.enabled.push_back(1);
  b.h_active.push_back(1);
}

// Two threads read the fields of two cases at the same time.
static int fields() {
  static lbm_batch b;
  b.storage = LBM_STORE_F32;
  char* v[] = {(char*)"400", (char*)"300", (char*)"1", (char*)"1", (char*)"1", (char*)"2", (char*)"0"};
  add_case(b, v);
  v[0] = (char*)"800";
  add_case(b, v);
  rec::meet = 2;
  std::vector<double> out[2];
  std::thread t[2];
  for (int i = 0; i < 2; ++i)
    t[i] = std::thread([&, i] {
      out[i].resize(800 * 300);
      lbm_batch_fields(&b, i, out[i].data(), nullptr, nullptr);
    });
  for (auto& x : t) x.join();
  std::printf("%d %d %d\n", (int)rec::exports.size(), rec::exports[0] != rec::exports[1],
              (int)rec::stale);
  return 0;
}

// Item lists over runs of the given lengths (a negative length drops case 0):
// shape, items and uploads so far after each.  Then the launch order of the
// last list: every item once, ranges of equal cost, dearest first.
static int items(int argc, char** argv) {
  static lbm_batch b;
  b.storage = LBM_STORE_F64;
  b.K = std::atoi(argv[0]);
  char* cavity[] = {(char*)"190", (char*)"200", (char*)"1", (char*)"1", (char*)"1", (char*)"2",
                    (char*)"977"};
  char* channel[] = {(char*)"400", (char*)"260", (char*)"3", (char*)"4", (char*)"1", (char*)"1",
                     (char*)"0"};
  for (int i = 0; i < 4; ++i) {
    add_case(b, cavity);
    add_case(b, channel);
  }
  if (configure(&b)) return 1;
  for (int i = 1; i < argc; ++i) {
    int left = std::atoi(argv[i]);
    if (left < 0) {
      b.h_active[0] = 0;
      left = -left;
    }
    rec::uploads = 0;
    if (rebuild_items(&b, left)) return 1;
    std::printf("%d %d %d\n", b.multi, b.n_mitems, rec::uploads);
  }
  std::set<std::pair<int, int>> seen;
  long long cost[8] = {}, dear = 0;
  for (int k = 0; k < 8; ++k) {
    int last = 3;
    for (int i = k; i < b.n_mitems; i += 8) {
      const int2 it = b.d_mitems[i];
      if (it.x < 0) continue;
      seen.insert({it.x, it.y & kTileMask});
      const HostCase& c = b.cs[it.x];
      const int tx = multi_tiles_x(c), x = (it.y & kTileMask) % tx;
      const int w = it.y >> kInteriorBit & 1 ? 1 : it.x % 2 && x == tx - 1 ? 3 : 2;
      if (w > last) ++dear;
      last = w;
      cost[k] += w;
    }
  }
  long long want = 0;
  for (int i = 0; i < b.n; ++i)
    if (b.h_active[i]) want += (long long)multi_tiles_x(b.cs[i]) * multi_tiles_y(b.cs[i], b.multi);
  std::printf("%d %lld %d\n", seen.size() == (size_t)want, dear,
              *std::max_element(cost, cost + 8) - *std::min_element(cost, cost + 8) <= 6);
  return 0;
}

// Allocations after reading a case of nx x 300 nodes three times.
static int staging(char* nx) {
  static lbm_batch b;
  b.storage = LBM_STORE_F32;
  char* v[] = {nx, (char*)"300", (char*)"1", (char*)"1", (char*)"1", (char*)"2", (char*)"0"};
  add_case(b, v);
  std::vector<double> out((size_t)b.cs[0].grid.nx * 300);
  for (int i = 0; i < 3; ++i) lbm_batch_fields(&b, 0, out.data(), nullptr, nullptr);
  std::printf("%d %d\n", rec::allocs, (int)rec::live.size());
  return 0;
}

// Shape of the two-step kernel: storage, then per kind of case its number and
// the case.
static int shape(int argc, char** argv) {
  static lbm_batch b;
  b.storage = std::atoi(argv[0]);
  for (int i = 1; i + 8 <= argc; i += 8)
    for (int k = 0; k < std::atoi(argv[i]); ++k) add_case(b, argv + i + 1);
  std::printf("%d\n", batch_multi_shape(&b));
  return 0;
}

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  if (what == "fields") return fields();
  if (what == "shape" && argc > 3) return shape(argc - 2, argv + 2);
  if (what == "staging" && argc == 3) return staging(argv[2]);
  if (what == "items" && argc > 3) return items(argc - 2, argv + 2);
  return 2;
}
