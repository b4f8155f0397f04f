// Batched steady solver: many independent lattices (cases of different size,
// Re, gamma and geometry) advanced together in windows of check_every steps.
//
// Graph schedules: a window is one captured sequence of launches over the
// tiles of all active cases, plain steps two per launch where that pays
// (batch_multi_shape).  Launches, not steps, swap the two lattices, so the
// batch keeps the index of its current one.
//
// Dataflow schedule: one persistent kernel per window.  Work is a stream of
// tickets (step, case, tile) taken in order from one atomic counter; the order
// is step-major, so while the last tiles of one step run, the first tiles of
// the next are already handed out.  A tile of case c at step s may start once
// all tiles of case c at step s-1 are done (a per-case completion counter):
// cases advance independently, with no grid-wide barrier.  A block only ever
// waits for tickets that running blocks already hold, so progress does not
// depend on co-residency; the wait is bounded anyway (an error flag ends the
// launch).  The block that completes a case's last tile of the window reduces,
// in a fixed order, that case's residual partials and retires it when
// converged, stalled or diverged; the host drops retired cases from the next
// window's ticket list.
//
// All cases share one step counter and one storage type: FP32 or FP64
// deviations.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "../../include/lbm.h"
#include "lbm_aux.h"
#include "lbm_host.h"
#include "lbm_multi.h"

using namespace lbmk;
using namespace lbmh;

namespace {


// Per-case descriptor (device).
struct CaseDev {
  StepArgs a[2];       // per lattice parity: geometry, tiling, mask, ubuf,
                       // partials (case base), outlet history in/out
  Consts<float> kf;
  Consts<double> kd;
  void* lat[2];
  int outlet;
  int ntiles;
  int mtiles_x;        // tiles per row of the two-step kernel
};

template <class C>
__device__ __forceinline__ const Consts<C>& case_consts(const CaseDev& cd);
template <>
__device__ __forceinline__ const Consts<float>& case_consts<float>(const CaseDev& cd) {
  return cd.kf;
}
template <>
__device__ __forceinline__ const Consts<double>& case_consts<double>(const CaseDev& cd) {
  return cd.kd;
}


__device__ __forceinline__ int load_flag(const int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Work items carry the tile index and, in bit kInteriorBit, whether the
// tile's region (the tile with its one-node ring) is all fluid and keeps away
// from every side: such tiles take the path without boundary, mask and outlet
// logic.
constexpr int kInteriorBit = 30;
constexpr int kTileMask = (1 << kInteriorBit) - 1;

// Below this many active items the graph schedule launches one kernel per
// step for all classes (kClsAny).
constexpr long long kSplitMinItems = 2048;

// Item classes of the graph schedule: each class is one launch per step, so
// that each gets the registers of its own path (the interior path and the
// closed-lattice boundary path fit eight blocks per compute unit; the outlet
// path needs more).  kClsAny decides per item (the dataflow kernel).
enum ItemClass : int { kClsInt = 0, kClsClosed = 1, kClsOutlet = 2, kClsOther = 3, kClsAny = 4 };
constexpr int kNumClasses = 4;

template <class S, int BY, int R, int FL, int VAR = 0, int CLS = kClsAny>
__device__ __forceinline__ void run_item(const CaseDev& cd, int par, int item_tile,
                                         typename S::C (*s_rho)[kLanes + 2], double (*s_red)[4]) {
  using T = typename S::T;
  using C = typename S::C;
  const T* fa = static_cast<const T*>(cd.lat[par]);
  T* fb = static_cast<T*>(cd.lat[par ^ 1]);
  const int tile = item_tile & kTileMask;
  // the case's step arguments and constants as local (scalar) copies, read
  // before the first population load: read where used, a field needed for
  // an address after the population loads are issued costs a second round
  // trip (its load waits for every load before it)
  const StepArgs args = cd.a[par];
  const Consts<C> k = case_consts<C>(cd);
  if constexpr (CLS == kClsInt) {
    step_tile<S, BY, R, FL, false, false, VAR, true>(fa, fb, args, k, tile, s_rho, s_red);
    return;
  } else if constexpr (CLS == kClsClosed) {
    step_tile<S, BY, R, FL, true, false, VAR, false, true>(fa, fb, args, k, tile, s_rho, s_red);
    return;
  } else if constexpr (CLS == kClsOutlet) {
    step_tile<S, BY, R, FL, true, true, VAR>(fa, fb, args, k, tile, s_rho, s_red);
    return;
  } else if constexpr (CLS == kClsOther) {
    step_tile<S, BY, R, FL, true, false, VAR>(fa, fb, args, k, tile, s_rho, s_red);
    return;
  }
  if (item_tile >> kInteriorBit)
    step_tile<S, BY, R, FL, false, false, VAR, true>(fa, fb, cd.a[par], case_consts<C>(cd), tile,
                                                     s_rho, s_red);
  else if (cd.outlet)
    step_tile<S, BY, R, FL, true, true, VAR>(fa, fb, cd.a[par], case_consts<C>(cd), tile, s_rho,
                                             s_red);
  else
    step_tile<S, BY, R, FL, true, false, VAR>(fa, fb, cd.a[par], case_consts<C>(cd), tile, s_rho,
                                              s_red);
}

// Retirement state shared by both batch schedules.
struct RetireArgs {
  const CaseDev* cases;
  double tol;
  long long min_steps;
  int* active;
  long long* done_step;
  int* status;
  double* best;
  int* stall;
  double* case_res;
  int plateau_checks;
  double plateau_factor;
};

// Residual of case c from its per-tile partials (fixed order: lane-strided
// sums, then lane 0 adds the 64 lane sums in order) and the retirement rule.
// t: steps done before the check step.  Uses threads (lane, 0) of the block.
__device__ void retire_check(const RetireArgs& b, int c, long long t, double (*s_sum)[kLanes]) {
  const CaseDev& cd = b.cases[c];
  const int lane = threadIdx.x, w = threadIdx.y;
  if (w == 0) {
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int i = lane; i < cd.ntiles; i += kLanes)
      for (int q = 0; q < 4; ++q) acc[q] += cd.a[0].partials[(long long)i * 4 + q];
    for (int q = 0; q < 4; ++q) s_sum[q][lane] = acc[q];
  }
  __syncthreads();
  if (w == 0 && lane == 0) {
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    for (int i = 0; i < kLanes; ++i)
      for (int q = 0; q < 4; ++q) v[q] += s_sum[q][i];
    for (int q = 0; q < 4; ++q) b.case_res[(long long)c * 4 + q] = v[q];
    const bool finite = isfinite(v[0]) && isfinite(v[1]) && isfinite(v[2]);
    const double r = v[1] > 0.0 ? sqrt(v[0] / v[1]) : (v[0] > 0.0 ? INFINITY : 0.0);
    int st = 0;
    if (!finite) {
      st = 3;
    } else if (t + 1 >= b.min_steps) {
      if (r < b.tol) {
        st = 1;
      } else if (b.plateau_checks > 0) {
        // plateau: no improvement by plateau_factor for plateau_checks checks
        if (r < b.best[c] * b.plateau_factor) {
          b.best[c] = r;
          b.stall[c] = 0;
        } else if (++b.stall[c] >= b.plateau_checks) {
          st = 2;
        }
      }
    }
    if (st) {
      b.status[c] = st;
      b.done_step[c] = st == 3 ? -(t + 1) : t + 1;
      __hip_atomic_store(&b.active[c], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  __syncthreads();
}

// Arguments of the persistent dataflow kernel (one launch per window).
struct BatchArgs {
  const CaseDev* cases;
  int ncases;
  const int* item_case;   // work items of the window: (case, tile)
  const int* item_tile;
  int n_items;
  long long t0;           // steps done before this window
  int par0;               // lattice that holds the state at t0
  int nsteps;             // steps in this window
  int K;                  // check cadence
  unsigned* ticket;       // ticket counter (zero at launch)
  unsigned* done;         // [ncases] tiles finished in this window (zero at launch)
  RetireArgs ret;
  int* err;               // set when a wait timed out
  long long spin_limit;
};

// ---- schedule "graph": one multi-case step kernel per time step (one block
// per active tile of any case, tiles handed out XCD by XCD), then a per-case
// reduction kernel on check steps; a window of check_every steps is captured
// once into a graph and replayed while the set of active cases is unchanged.
struct StepLaunch {
  const CaseDev* cases;
  const int* item_case;
  const int* item_tile;
  int n_items;
  const int* active;
  int par;
};

// NTS: non-temporal population stores (the active lattices together exceed
// the last-level cache).
template <class S, int BY, int R, int FL, bool NTS, int CLS>
__global__ __launch_bounds__(kLanes* BY) void batch_step_kernel(StepLaunch L) {
  __shared__ typename S::C s_rho[BY * R + 2][kLanes + 2];
  __shared__ double s_red[BY][4];
  const int it = xcd_tile(blockIdx.x, L.n_items);
  const int c = L.item_case[it];
  if (!L.active[c]) return;
  run_item<S, BY, R, FL, NTS ? kVarNts : 0, CLS>(L.cases[c], L.par, L.item_tile[it], s_rho,
                                                 s_red);
}

// Two plain steps of every active case in one launch (see lbm_multi.h): one
// block per tile of the two-step kernel, the path per item.  Cases retire at
// check steps only, and the host then drops their items, so no item needs a
// look at the active flags (one dependent load less before the populations).
// Bound: small FP64 batches by the latency of a block (item, descriptor and
// population loads in a row, one or two blocks per compute unit by registers),
// large FP32 ones by vector instructions.  Per step, one step | two steps per
// launch: 12 FP64 cases with sides of 64 to 128 26.4 | 13.9 us, 20 FP32 cases
// with sides of 64 to 512 115 | 71 us.
template <class S, int NW, int RPW>
__global__ __launch_bounds__(kLanes* NW, (multi_waves<S, NW, RPW>()))
void batch_multi_kernel(const CaseDev* __restrict__ cases, const int2* __restrict__ items,
                        int par) {
  using T = typename S::T;
  using C = typename S::C;
  extern __shared__ __align__(16) char smem[];
  using F = T[NW * RPW - 2][kLanes];
  using R = C[kLanes + 2];
  F* s_f = reinterpret_cast<F*>(smem);
  R* s_rho = reinterpret_cast<R*>(smem + 9 * sizeof(F));
  const int2 it = items[blockIdx.x];
  const int c = __builtin_amdgcn_readfirstlane(it.x);
  if (c < 0) return;
  const int code = __builtin_amdgcn_readfirstlane(it.y);
  const CaseDev& cd = cases[c];
  const T* fa = static_cast<const T*>(cd.lat[par]);
  T* fb = static_cast<T*>(cd.lat[par ^ 1]);
  StepArgs args = cd.a[par];
  args.tiles_x = cd.mtiles_x;
  const Consts<C> k = case_consts<C>(cd);
  const int tile = code & kTileMask;
  if (code >> kInteriorBit)
    multi_tile<S, NW, RPW, kMultiSteps, false, false, false, true>(fa, fb, args, k, tile, s_f,
                                                                   s_rho);
  else if (cd.outlet)
    multi_tile<S, NW, RPW, kMultiSteps, true, true, false, false>(fa, fb, args, k, tile, s_f,
                                                                  s_rho);
  else
    multi_tile<S, NW, RPW, kMultiSteps, true, false, false, false>(fa, fb, args, k, tile, s_f,
                                                                   s_rho);
}

// one block per case: residual of the check step that ends the window
__global__ __launch_bounds__(kLanes) void batch_reduce_kernel(RetireArgs r, int ncases,
                                                              const long long* tnow, int nsteps) {
  __shared__ double s_sum[4][kLanes];
  const int c = blockIdx.x;
  if (c >= ncases || !r.active[c]) return;
  retire_check(r, c, *tnow + nsteps - 1, s_sum);
}

__global__ void batch_tick_kernel(long long* tnow, int nsteps) {
  if (threadIdx.x == 0) *tnow += nsteps;
}

// ---- schedule "dataflow": one persistent kernel per window.
template <class S, int BY, int R>
__global__ __launch_bounds__(kLanes* BY) void batch_kernel(BatchArgs b) {
  __shared__ typename S::C s_rho[BY * R + 2][kLanes + 2];
  __shared__ double s_red[BY][4];
  __shared__ double s_sum[4][kLanes];
  __shared__ unsigned s_ticket;
  __shared__ int s_last;
  const bool lead = threadIdx.x == 0 && threadIdx.y == 0;
  const unsigned total = unsigned(b.nsteps) * unsigned(b.n_items);
  for (;;) {
    if (lead) s_ticket = atomicAdd(b.ticket, 1u);
    __syncthreads();
    // uniform across the block: scalar registers (buffer resources and
    // offsets derived from the case must be wave-uniform)
    const unsigned tk = __builtin_amdgcn_readfirstlane(s_ticket);
    if (tk >= total) break;
    const int s = int(tk / unsigned(b.n_items));
    const int it = int(tk % unsigned(b.n_items));
    const int c = b.item_case[it];
    const int tile = b.item_tile[it];   // tile index and interior bit
    const CaseDev& cd = b.cases[c];
    // wait until case c has finished step s - 1 of this window
    if (lead) {
      const unsigned need = unsigned(s) * unsigned(cd.ntiles);
      long long spins = 0;
      while (__hip_atomic_load(&b.done[c], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) < need) {
        __builtin_amdgcn_s_sleep(1);
        if (++spins > b.spin_limit) {
          __hip_atomic_store(b.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          break;
        }
      }
      __atomic_thread_fence(__ATOMIC_ACQUIRE);
    }
    __syncthreads();
    if (__hip_atomic_load(b.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) break;
    const long long t = b.t0 + s;   // steps done before this one
    const int par = (b.par0 + s) & 1;
    const long long idx = (t + 1) % b.K;
    const int flavor = idx == 0 ? kCheck : ((b.K >= 2 && idx == b.K - 1) ? kStore : kPlain);
    if (flavor == kCheck) run_item<S, BY, R, kCheck>(cd, par, tile, s_rho, s_red);
    else if (flavor == kStore) run_item<S, BY, R, kStore>(cd, par, tile, s_rho, s_red);
    else run_item<S, BY, R, kPlain>(cd, par, tile, s_rho, s_red);
    __syncthreads();
    if (lead) {
      __atomic_thread_fence(__ATOMIC_RELEASE);
      const unsigned prev =
          __hip_atomic_fetch_add(&b.done[c], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
      s_last = (prev + 1 == unsigned(b.nsteps) * unsigned(cd.ntiles)) && flavor == kCheck;
      if (s_last) __atomic_thread_fence(__ATOMIC_ACQUIRE);
    }
    __syncthreads();
    if (s_last) retire_check(b.ret, c, t, s_sum);
  }
}

struct Shape {
  int by, rows;
};
constexpr Shape kBatchShapes[] = {{4, 1}, {8, 1}, {16, 1}};

template <class S, int BY, int R>
const void* kernel_ptr() {
  return reinterpret_cast<const void*>(&batch_kernel<S, BY, R>);
}

template <class S>
const void* kernel_for_storage(int by) {
  switch (by) {
    case 8: return kernel_ptr<S, 8, 1>();
    case 16: return kernel_ptr<S, 16, 1>();
    default: return kernel_ptr<S, 4, 1>();
  }
}

const void* batch_kernel_for(int storage, int by) {
  return storage == LBM_STORE_F64 ? kernel_for_storage<StoreF64>(by)
                                  : kernel_for_storage<StoreF32>(by);
}

struct HostCase {
  lbm_grid grid;
  lbm_params p;
  Geom g;
  Consts<float> kf;
  Consts<double> kd;
  void* lat[2] = {nullptr, nullptr};
  void* hist[2] = {nullptr, nullptr};
  float* ubuf = nullptr;
  uint8_t* solid = nullptr;
  int tiles_x = 0, ntiles = 0, tile_base = 0;
  size_t fluid = 0;
  std::vector<uint8_t> h_mask;      // [ny][nx], 1 = solid
  std::vector<uint8_t> tile_int;    // per tile: region all fluid, away from the sides
  std::vector<uint8_t> multi_int[kNumMultiShapes];   // the same per two-step shape (on demand)
  int state_par = 0;  // which lattice holds the case's current state
};

}  // namespace

constexpr size_t kKeptStageMin = 1ull << 20, kKeptStage = 64ull << 20;

struct lbm_batch {
  std::vector<HostCase> cs;
  int n = 0;
  int K = 100;
  int by = 4, rows = 1;
  int blocks = 0;    // 0 = all co-resident blocks
  int schedule = 0;
  int storage = LBM_STORE_F32;
  int plateau_checks = 0;
  double plateau_factor = 0.9;
  int device = 0;
  hipStream_t own_stream = nullptr, stream = nullptr;
  CaseDev* d_cases = nullptr;
  int* d_item_case = nullptr;
  int* d_item_tile = nullptr;
  int n_items = 0, item_cap = 0;
  int cls_off[kNumClasses + 1] = {0, 0, 0, 0, 0};  // graph schedule: items of class k
                                                   // are [cls_off[k], cls_off[k + 1])
  bool merged = false;  // graph schedule with few items: one launch per step
  int multi = -1;       // shape of the two-step kernel, -1: step by step
  int2* d_mitems = nullptr;   // its items (case, tile and interior bit)
  int n_mitems = 0, mitem_cap = 0;
  int mitems_shape = -1;             // shape and active cases the device's items are
  std::vector<int> mitems_active;    // for (built again when either changes)
  double* d_stage = nullptr;   // staging of lbm_batch_fields (see there)
  size_t stage_bytes = 0;
  std::mutex stage_mutex;
  int par = 0;          // lattice that holds the state of the advancing cases
  int window_flips = 0; // lattice swaps of a captured window, modulo 2
  double* d_partials = nullptr;
  double* d_case_res = nullptr;
  int* d_active = nullptr;
  long long* d_done = nullptr;
  int* d_status = nullptr;
  double* d_best = nullptr;
  int* d_stall = nullptr;
  unsigned* d_sync = nullptr;  // [1 + n]: ticket counter, per-case completion counters
  int* d_err = nullptr;
  long long* d_tnow = nullptr; // step counter read by the reduction kernel
  hipGraphExec_t graph[2] = {nullptr, nullptr};  // window graphs by start parity
  int64_t t = 0;
  std::vector<int> h_active;
  std::vector<int> enabled;     // cases a run advances
  std::vector<int> h_status;    // status of the last run
};

namespace {

void free_batch(lbm_batch* b) {
  if (!b) return;
  for (auto& c : b->cs) {
    for (int i = 0; i < 2; ++i) {
      if (c.lat[i]) hipFree(c.lat[i]);
      if (c.hist[i]) hipFree(c.hist[i]);
    }
    if (c.ubuf) hipFree(c.ubuf);
    if (c.solid) hipFree(c.solid);
  }
  hipFree(b->d_cases);
  hipFree(b->d_item_case);
  hipFree(b->d_item_tile);
  hipFree(b->d_mitems);
  hipFree(b->d_stage);
  hipFree(b->d_partials);
  hipFree(b->d_case_res);
  hipFree(b->d_active);
  hipFree(b->d_done);
  hipFree(b->d_status);
  hipFree(b->d_best);
  hipFree(b->d_stall);
  hipFree(b->d_sync);
  hipFree(b->d_tnow);
  for (int i = 0; i < 2; ++i)
    if (b->graph[i]) hipGraphExecDestroy(b->graph[i]);
  hipFree(b->d_err);
  if (b->own_stream) hipStreamDestroy(b->own_stream);
  delete b;
}

// Bytes of the two lattices of every active case.  Beyond the 256 MiB
// Infinity Cache a written lattice is evicted before the next step reads it,
// so the step stores it non-temporally (as the single-lattice path does).
constexpr size_t kLastLevelCacheBytes = size_t(256) << 20;
size_t active_lattice_bytes(const lbm_batch* b) {
  const size_t es = b->storage == LBM_STORE_F64 ? 8 : 4;
  size_t bytes = 0;
  for (int i = 0; i < b->n; ++i)
    if (b->h_active[i]) bytes += 2 * 9 * (size_t)b->cs[i].g.plane * es;
  return bytes;
}

constexpr int kMultiRing = 2 * kMultiSteps - 1, kMultiCols = kLanes - 2 * kMultiRing;
int multi_tiles_x(const HostCase& c) { return (c.grid.nx + kMultiCols - 1) / kMultiCols; }
int multi_tiles_y(const HostCase& c, int shape) {
  const int tyo = kMultiShapes[shape].nw * kMultiShapes[shape].rpw - 2 * kMultiRing;
  return (c.grid.ny + tyo - 1) / tyo;
}

// Per tile of a two-step shape: region all fluid and one node away from every
// side.
const std::vector<uint8_t>& multi_interior(HostCase& c, int shape) {
  std::vector<uint8_t>& f = c.multi_int[shape];
  if (!f.empty()) return f;
  const int nx = c.grid.nx, ny = c.grid.ny, tx = multi_tiles_x(c), ty = multi_tiles_y(c, shape);
  const int nr = kMultiShapes[shape].nw * kMultiShapes[shape].rpw, tyo = nr - 2 * kMultiRing;
  f.assign((size_t)tx * ty, 0);
  for (int j = 0; j < ty; ++j)
    for (int i = 0; i < tx; ++i) {
      const int x0 = i * kMultiCols - kMultiRing, y0 = j * tyo - kMultiRing;
      if (x0 < 1 || x0 + kLanes > nx - 1 || y0 < 1 || y0 + nr > ny - 1) continue;
      bool fluid = true;
      for (int y = y0; fluid && y < y0 + nr; ++y)
        fluid = std::memchr(&c.h_mask[(size_t)y * nx + x0], 1, kLanes) == nullptr;
      f[(size_t)j * tx + i] = fluid ? 1 : 0;
    }
  return f;
}

// Tiles of region length len along a side of length n whose region keeps one
// node away from both ends.
int multi_inner(int n, int tiles, int len) {
  int inner = 0;
  for (int i = 0; i < tiles; ++i) {
    const int lo = i * (len - 2 * kMultiRing) - kMultiRing;
    inner += lo >= 1 && lo + len <= n - 1;
  }
  return inner;
}

// Shape of the two-step kernel for the active cases, or -1: as for a single
// lattice, from the sum of their tiles, whatever the block height of the
// single steps (256 FP32 cases with sides of 64 to 512, height 8: 1066 | 676
// us).  Times per step, one step | two steps per launch:
// - Up to one block per compute unit (or 512 of the 6-row blocks) the launch
//   is what counts: 4 cavities 64^2 FP64 9.3 | 4.5 us, 20 of them 11.0 | 8.9,
//   FP32 9.3 | 5.3.
// - More tiles: as long as a quarter of them keep away from the sides (20 cavities
//   128^2 FP64 21.3 | 14.9 us, FP32 11.8 | 8.9; 20 channels 400 x 100 FP64 38.1 |
//   25.6; 20 cavities 512^2 FP64 157 | 128, FP32 96.3 | 60.7).  Many small
//   lattices have none, and the boundary work is done on the ring as well (200
//   cavities 64^2 FP64 25.7 | 40.3 us, FP32 16.6 | 23.2).
// - Beyond 2048 tiles (eight per compute unit) the work counts, as for a single
//   lattice: the rows a pair collides over those of two single steps, up to 1.7
//   (1.6: 39 cavities 190^2 FP64 53.8 | 46.2 us; 1.8: 76 cavities 128^2 FP64 43.3 |
//   45.9, 512 of them 264 | 301, 76 FP32 21.3 | 22.5).
// Solid nodes do not decide it (60 FP64 cavities 400^2 with solids in every tile
// 650 | 315 us; of all batches measured only 20 of 200^2 lost, 30.0 | 33.0).
int batch_multi_shape(lbm_batch* b) {
  if (b->schedule != 0) return -1;
  long long tiles[kNumMultiShapes] = {};
  double rows = 0;   // of 64 nodes, two single steps
  bool any = false;
  for (int i = 0; i < b->n; ++i) {
    if (!b->h_active[i]) continue;
    const HostCase& c = b->cs[i];
    if (c.grid.nx < 16 || c.grid.ny < 16) return -1;
    any = true;
    rows += 2.0 * ((c.grid.nx + kLanes - 1) / kLanes) * c.grid.ny;
    for (int s = 0; s < kNumMultiShapes; ++s)
      tiles[s] += (long long)multi_tiles_x(c) * multi_tiles_y(c, s);
  }
  if (!any) return -1;
  for (int s = 0; s < 3; ++s)
    if (tiles[s] <= 256) return s;
  if (tiles[1] <= 512) return 1;
  const bool cached = active_lattice_bytes(b) <= kLastLevelCacheBytes;
  const int shape = cached || b->storage == LBM_STORE_F64 ? 3 : 4;
  const int nr = kMultiShapes[shape].nw * kMultiShapes[shape].rpw;
  if (tiles[shape] > 2048 && tiles[shape] * (2.0 * nr - 8.0) > 1.7 * rows) return -1;
  long long inner = 0;
  for (int i = 0; i < b->n; ++i) {
    if (!b->h_active[i]) continue;
    const HostCase& c = b->cs[i];
    inner += (long long)multi_inner(c.grid.nx, multi_tiles_x(c), kLanes) *
             multi_inner(c.grid.ny, multi_tiles_y(c, shape), nr);
  }
  return 4 * inner >= tiles[shape] ? shape : -1;
}

// Items of the two-step kernel in launch order.  Block i runs on XCD i mod 8:
// every XCD gets a contiguous range of about the same cost, so that neighbouring
// tiles share its L2, the dearest items first, so that the last blocks are
// short ones.  Ranges that end earlier are padded with empty items (case -1).
// Cost relative to the others: interior 1, boundary 2, with the outlet column 3
// (us per step in the order of the tiles | ordered with ranges of equal weights |
// with these, mixes of cavities and channels: 12 FP64 cases with sides of 64 to
// 128 18.1 | 16.1 | 14.8, 16 FP64 of 64 to 256 41.0 | 35.6 | 35.6, 32 FP32 of
// 64 to 256 29.2 | 26.9 | 27.2, 20 FP32 of 64 to 512 78.3 | 74.6 | 75.7: the
// order pays everywhere, the weights in few, dear tiles).  Linear in the items,
// as it is host time of a run.
std::vector<int2> multi_items(lbm_batch* b) {
  std::vector<int2> items;
  std::vector<uint8_t> cost;
  long long total = 0;
  for (int i = 0; i < b->n; ++i) {
    if (!b->h_active[i]) continue;
    const std::vector<uint8_t>& f = multi_interior(b->cs[i], b->multi);
    const int tx = multi_tiles_x(b->cs[i]);
    const bool outlet = b->cs[i].grid.side[1] == LBM_SIDE_OUTLET;
    for (int t = 0, x = 0; t < (int)f.size(); ++t, x = x + 1 == tx ? 0 : x + 1) {
      items.push_back(int2{i, t | (int(f[t]) << kInteriorBit)});
      cost.push_back(f[t] ? 1 : outlet && x == tx - 1 ? 3 : 2);
      total += cost.back();
    }
  }
  // count per range and cost, then place in the order of the list
  std::vector<uint8_t> range(items.size());
  size_t count[8][4] = {}, at[8][4], longest = 0;
  long long sum = 0;
  for (size_t i = 0; i < items.size(); ++i) {
    range[i] = uint8_t(std::min<long long>(7, sum * 8 / total));
    ++count[range[i]][cost[i]];
    sum += cost[i];
  }
  for (int k = 0; k < 8; ++k) {
    at[k][3] = 0;
    at[k][2] = count[k][3];
    at[k][1] = at[k][2] + count[k][2];
    longest = std::max(longest, at[k][1] + count[k][1]);
  }
  std::vector<int2> out(8 * longest, int2{-1, 0});
  for (size_t i = 0; i < items.size(); ++i)
    out[8 * at[range[i]][cost[i]]++ + range[i]] = items[i];
  return out;
}

// (Re)build the tiling of every case for the current launch shape, the
// descriptors and the active item list.
int configure(lbm_batch* b) {
  const int ro = b->by * b->rows;
  int total = 0;
  for (auto& c : b->cs) {
    c.tiles_x = (c.grid.nx + kLanes - 1) / kLanes;
    c.ntiles = c.tiles_x * ((c.grid.ny + ro - 1) / ro);
    c.tile_base = total;
    total += c.ntiles;
    // interior tiles: the same margins as the single-lattice kernel, and no
    // solid node in the tile or its ring
    c.tile_int.assign(c.ntiles, 0);
    const int nx = c.grid.nx, ny = c.grid.ny;
    for (int t = 0; t < c.ntiles; ++t) {
      const int x0 = (t % c.tiles_x) * kLanes, y0 = (t / c.tiles_x) * ro;
      if (!(x0 >= 2 && x0 + kLanes + 1 <= nx - 2 && y0 >= 2 && y0 + ro + 1 <= ny - 2)) continue;
      bool fluid = true;
      for (int y = y0 - 1; fluid && y <= y0 + ro; ++y)
        for (int x = x0 - 1; x <= x0 + kLanes; ++x)
          if (c.h_mask[(size_t)y * nx + x]) {
            fluid = false;
            break;
          }
      c.tile_int[t] = fluid ? 1 : 0;
    }
  }
  hipFree(b->d_partials);
  b->d_partials = nullptr;
  HIPCHECK(hipMalloc(&b->d_partials, (size_t)std::max(total, 1) * 4 * sizeof(double)));
  std::vector<CaseDev> desc(b->n);
  for (int i = 0; i < b->n; ++i) {
    const HostCase& c = b->cs[i];
    CaseDev d{};
    for (int par = 0; par < 2; ++par) {
      StepArgs& a = d.a[par];
      a.g = c.g;
      a.tiles_x = c.tiles_x;
      a.ntiles = c.ntiles;
      a.out_rows = ro;
      a.solid = c.solid;
      a.ubuf = c.ubuf;
      a.force = c.ubuf;  // batch cases take the uniform force; any readable buffer
      a.has_force = 0;
      a.partials = b->d_partials + (long long)c.tile_base * 4;
      a.hist_in = c.hist[par];
      a.hist_out = c.hist[par ^ 1];
    }
    d.kf = c.kf;
    d.kd = c.kd;
    d.lat[0] = c.lat[0];
    d.lat[1] = c.lat[1];
    d.outlet = c.grid.side[1] == LBM_SIDE_OUTLET;
    d.ntiles = c.ntiles;
    d.mtiles_x = multi_tiles_x(c);
    desc[i] = d;
  }
  if (!b->d_cases) HIPCHECK(hipMalloc(&b->d_cases, sizeof(CaseDev) * b->n));
  HIPCHECK(hipMemcpy(b->d_cases, desc.data(), sizeof(CaseDev) * b->n, hipMemcpyHostToDevice));
  b->item_cap = 0;  // force the item list to be rebuilt
  return LBM_OK;
}

void drop_graphs(lbm_batch* b) {
  for (int i = 0; i < 2; ++i)
    if (b->graph[i]) {
      hipGraphExecDestroy(b->graph[i]);
      b->graph[i] = nullptr;
    }
}

// left: steps still to take.
int rebuild_items(lbm_batch* b, int64_t left) {
  drop_graphs(b);
  // ticket order within a step: schedule 0 = case by case (a case's tiles
  // contiguous), 1 = tiles interleaved across cases
  // the graph schedules group the items by class (one launch per class and
  // step); the dataflow schedule keeps one list
  std::vector<int> ic, itl;
  auto item_class = [&](int i, int t) {
    if (b->cs[i].tile_int[t]) return int(kClsInt);
    const int32_t* sd = b->cs[i].grid.side;
    if (sd[1] == LBM_SIDE_OUTLET) return int(kClsOutlet);
    bool closed = true;
    for (int q = 0; q < 4; ++q)
      closed = closed && (sd[q] == LBM_SIDE_WALL || sd[q] == LBM_SIDE_LID);
    return int(closed ? kClsClosed : kClsOther);
  };
  // Few items (less than about two rounds of resident blocks): one launch
  // per step that decides the path per item.  Each launch then runs for
  // little more than its start-up latency, and one launch instead of up to
  // four per step is what counts (the tail of a steady run, where a few
  // cases remain).
  long long active_items = 0;
  for (int i = 0; i < b->n; ++i)
    if (b->h_active[i]) active_items += b->cs[i].ntiles;
  b->merged = b->schedule != 2 && active_items < kSplitMinItems;
  const int ncls = (b->schedule == 2 || b->merged) ? 1 : kNumClasses;
  for (int k = 0; k < ncls; ++k) {
    b->cls_off[k] = (int)ic.size();
    auto take = [&](int i, int t) {
      if (ncls > 1 && item_class(i, t) != k) return;
      ic.push_back(i);
      itl.push_back(t | (int(b->cs[i].tile_int[t]) << kInteriorBit));
    };
    if (b->schedule != 1) {
      for (int i = 0; i < b->n; ++i) {
        if (!b->h_active[i]) continue;
        for (int t = 0; t < b->cs[i].ntiles; ++t) take(i, t);
      }
    } else {
      int maxt = 0;
      for (int i = 0; i < b->n; ++i)
        if (b->h_active[i]) maxt = std::max(maxt, b->cs[i].ntiles);
      for (int t = 0; t < maxt; ++t)
        for (int i = 0; i < b->n; ++i)
          if (b->h_active[i] && t < b->cs[i].ntiles) take(i, t);
    }
  }
  for (int k = ncls; k <= kNumClasses; ++k) b->cls_off[k] = (int)ic.size();
  b->n_items = (int)ic.size();
  if (b->n_items > b->item_cap) {
    hipFree(b->d_item_case);
    hipFree(b->d_item_tile);
    b->d_item_case = b->d_item_tile = nullptr;
    b->item_cap = 0;
    HIPCHECK(hipMalloc(&b->d_item_case, sizeof(int) * b->n_items));
    HIPCHECK(hipMalloc(&b->d_item_tile, sizeof(int) * b->n_items));
    b->item_cap = b->n_items;
  }
  // (a run or window without two plain steps in a row before its last one has no
  // pairs: its items would be built for nothing)
  b->multi = left > kMultiSteps && b->K >= kMultiSteps + 2 ? batch_multi_shape(b) : -1;
  if (b->multi >= 0 && (b->multi != b->mitems_shape || b->h_active != b->mitems_active)) {
    b->mitems_shape = -1;
    const std::vector<int2> mi = multi_items(b);
    b->n_mitems = (int)mi.size();
    if (b->n_mitems > b->mitem_cap) {
      hipFree(b->d_mitems);
      b->d_mitems = nullptr;
      b->mitem_cap = 0;
      HIPCHECK(hipMalloc(&b->d_mitems, sizeof(int2) * b->n_mitems));
      b->mitem_cap = b->n_mitems;
    }
    HIPCHECK(hipMemcpy(b->d_mitems, mi.data(), sizeof(int2) * b->n_mitems, hipMemcpyHostToDevice));
    b->mitems_shape = b->multi;
    b->mitems_active = b->h_active;
  }
  if (b->n_items) {
    HIPCHECK(hipMemcpy(b->d_item_case, ic.data(), sizeof(int) * b->n_items, hipMemcpyHostToDevice));
    HIPCHECK(hipMemcpy(b->d_item_tile, itl.data(), sizeof(int) * b->n_items, hipMemcpyHostToDevice));
  }
  return LBM_OK;
}

template <class S, class FT>
void launch_case_init(lbm_batch* b, HostCase& c, const FT* rho, const FT* ux, const FT* uy) {
  using T = typename S::T;
  using C = typename S::C;
  const Consts<C>& k = *reinterpret_cast<const Consts<C>*>(
      sizeof(C) == 8 ? static_cast<const void*>(&c.kd) : static_cast<const void*>(&c.kf));
  const int blocks = int(((long long)c.grid.nx * c.grid.ny + 255) / 256);
  hipLaunchKernelGGL((init_kernel<S, FT>), dim3(blocks), dim3(256), 0, b->stream, (T*)c.lat[0],
                     (T*)c.lat[1], c.g, k, c.solid, rho, ux, uy, (C*)c.ubuf, (C*)c.hist[0],
                     (C*)c.hist[1]);
  hipLaunchKernelGGL((ghost_fill_kernel<S>), dim3(blocks), dim3(256), 0, b->stream, (T*)c.lat[0],
                     c.g, k, c.solid);
}

template <class FT>
int init_case(lbm_batch* b, int ci, const FT* rho, const FT* ux, const FT* uy) {
  HostCase& c = b->cs[ci];
  if (b->storage == LBM_STORE_F64) launch_case_init<StoreF64, FT>(b, c, rho, ux, uy);
  else launch_case_init<StoreF32, FT>(b, c, rho, ux, uy);
  HIPCHECK(hipGetLastError());
  // the batch's current lattice: copy when it is the second one
  if (b->par) {
    const size_t es = b->storage == LBM_STORE_F64 ? 8 : 4;
    const size_t bytes = 9 * (size_t)c.g.plane * es;
    HIPCHECK(hipMemcpyAsync(c.lat[1], c.lat[0], bytes, hipMemcpyDeviceToDevice, b->stream));
    HIPCHECK(hipMemcpyAsync(c.hist[1], c.hist[0], 2 * es * c.grid.ny, hipMemcpyDeviceToDevice,
                            b->stream));
  }
  c.state_par = b->par;
  return LBM_OK;
}

// Before a run: every enabled case must hold its state in lat[par].
int align_parity(lbm_batch* b) {
  const int par = b->par;
  const size_t es = b->storage == LBM_STORE_F64 ? 8 : 4;
  for (int i = 0; i < b->n; ++i) {
    HostCase& c = b->cs[i];
    if (!b->enabled[i] || c.state_par == par) continue;
    HIPCHECK(hipMemcpyAsync(c.lat[par], c.lat[c.state_par], 9 * (size_t)c.g.plane * es,
                            hipMemcpyDeviceToDevice, b->stream));
    HIPCHECK(hipMemcpyAsync(c.hist[par], c.hist[c.state_par], 2 * es * c.grid.ny,
                            hipMemcpyDeviceToDevice, b->stream));
    c.state_par = par;
  }
  return LBM_OK;
}


template <class S, int BY, bool NTS, int CLS>
void launch_step_cls(int flavor, const StepLaunch& L, hipStream_t st) {
  dim3 grid(L.n_items), block(kLanes, BY);
  if (flavor == kCheck)
    hipLaunchKernelGGL((batch_step_kernel<S, BY, 1, kCheck, NTS, CLS>), grid, block, 0, st, L);
  else if (flavor == kStore)
    hipLaunchKernelGGL((batch_step_kernel<S, BY, 1, kStore, NTS, CLS>), grid, block, 0, st, L);
  else
    hipLaunchKernelGGL((batch_step_kernel<S, BY, 1, kPlain, NTS, CLS>), grid, block, 0, st, L);
}

template <class S, int BY, bool NTS>
void launch_step_nts(int flavor, int cls, const StepLaunch& L, hipStream_t st) {
  switch (cls) {
    case kClsInt: launch_step_cls<S, BY, NTS, kClsInt>(flavor, L, st); break;
    case kClsClosed: launch_step_cls<S, BY, NTS, kClsClosed>(flavor, L, st); break;
    case kClsOutlet: launch_step_cls<S, BY, NTS, kClsOutlet>(flavor, L, st); break;
    case kClsOther: launch_step_cls<S, BY, NTS, kClsOther>(flavor, L, st); break;
    default: launch_step_cls<S, BY, NTS, kClsAny>(flavor, L, st); break;
  }
}

template <class S, int BY>
void launch_step_by(int flavor, int cls, bool nts, const StepLaunch& L, hipStream_t st) {
  if (nts) launch_step_nts<S, BY, true>(flavor, cls, L, st);
  else launch_step_nts<S, BY, false>(flavor, cls, L, st);
}

template <class S>
void launch_step_storage(int by, int flavor, int cls, bool nts, const StepLaunch& L,
                         hipStream_t st) {
  if (by == 8) launch_step_by<S, 8>(flavor, cls, nts, L, st);
  else if (by == 16) launch_step_by<S, 16>(flavor, cls, nts, L, st);
  else launch_step_by<S, 4>(flavor, cls, nts, L, st);
}

RetireArgs retire_args(lbm_batch* b, double tol, long long min_steps) {
  RetireArgs r{};
  r.cases = b->d_cases;
  r.tol = tol;
  r.min_steps = min_steps;
  r.active = b->d_active;
  r.done_step = b->d_done;
  r.status = b->d_status;
  r.best = b->d_best;
  r.stall = b->d_stall;
  r.case_res = b->d_case_res;
  r.plateau_checks = b->plateau_checks;
  r.plateau_factor = b->plateau_factor;
  return r;
}

template <class S, int NW, int RPW>
bool launch_batch_multi(const lbm_batch* b, int par, hipStream_t st) {
  constexpr size_t lds = multi_lds<S, NW, RPW>();
  auto* fn = batch_multi_kernel<S, NW, RPW>;
  if (lds > 64 * 1024 &&
      hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) {
    (void)hipGetLastError();   // (handled: single steps instead)
    return false;
  }
  hipLaunchKernelGGL(fn, dim3(b->n_mitems), dim3(kLanes, NW), lds, st, b->d_cases, b->d_mitems,
                     par);
  return true;
}

template <class S>
bool launch_batch_multi_shape(const lbm_batch* b, int par, hipStream_t st) {
  switch (b->multi) {
    case 0: return launch_batch_multi<S, 8, 1>(b, par, st);
    case 1: return launch_batch_multi<S, 12, 1>(b, par, st);
    case 2: return launch_batch_multi<S, 16, 1>(b, par, st);
    case 3: return launch_batch_multi<S, 8, 2>(b, par, st);
    default:
      if constexpr (sizeof(typename S::C) == 4) return launch_batch_multi<S, 8, 4>(b, par, st);
      return false;
  }
}

// Enqueue nsteps steps starting at step counter t in lattice par (graph
// schedule): the step kernels, pairs of plain steps in one launch (never the
// last step of the window, so that the two lattices hold the last two states),
// and when the last one is a check step, the per-case reduction and the
// step-counter tick.  Returns the lattice swaps.
int enqueue_window(lbm_batch* b, long long t, int nsteps, int par, const RetireArgs& r,
                   hipStream_t st) {
  int launches = 0;
  StepLaunch L{};
  L.cases = b->d_cases;
  L.item_case = b->d_item_case;
  L.item_tile = b->d_item_tile;
  L.n_items = b->n_items;
  L.active = b->d_active;
  int last_flavor = kPlain;
  const bool nts = active_lattice_bytes(b) > kLastLevelCacheBytes;
  auto flavor_at = [&](long long tt) {
    const long long idx = (tt + 1) % b->K;
    return idx == 0 ? kCheck : ((b->K >= 2 && idx == b->K - 1) ? kStore : kPlain);
  };
  for (int i = 0; i < nsteps; ++i, ++launches, par ^= 1) {
    const int flavor = flavor_at(t + i);
    if (b->multi >= 0 && nsteps - i > kMultiSteps && flavor == kPlain &&
        flavor_at(t + i + 1) == kPlain &&
        (b->storage == LBM_STORE_F64 ? launch_batch_multi_shape<StoreF64>(b, par, st)
                                     : launch_batch_multi_shape<StoreF32>(b, par, st))) {
      i += kMultiSteps - 1;
      last_flavor = kPlain;
      continue;
    }
    L.par = par;
    if (b->merged) {
      if (b->n_items > 0) {
        if (b->storage == LBM_STORE_F64)
          launch_step_storage<StoreF64>(b->by, flavor, kClsAny, nts, L, st);
        else
          launch_step_storage<StoreF32>(b->by, flavor, kClsAny, nts, L, st);
      }
      last_flavor = flavor;
      continue;
    }
    for (int k = 0; k < kNumClasses; ++k) {
      StepLaunch Lk = L;
      Lk.item_case = b->d_item_case + b->cls_off[k];
      Lk.item_tile = b->d_item_tile + b->cls_off[k];
      Lk.n_items = b->cls_off[k + 1] - b->cls_off[k];
      if (Lk.n_items <= 0) continue;
      if (b->storage == LBM_STORE_F64)
        launch_step_storage<StoreF64>(b->by, flavor, k, nts, Lk, st);
      else
        launch_step_storage<StoreF32>(b->by, flavor, k, nts, Lk, st);
    }
    last_flavor = flavor;
  }
  if (last_flavor == kCheck)
    hipLaunchKernelGGL(batch_reduce_kernel, dim3(b->n), dim3(kLanes), 0, st, r, b->n,
                       (const long long*)b->d_tnow, nsteps);
  hipLaunchKernelGGL(batch_tick_kernel, dim3(1), dim3(64), 0, st, b->d_tnow, nsteps);
  return launches;
}

}  // namespace

extern "C" {

int lbm_batch_create(int32_t n, const lbm_grid* grids, const uint8_t* const* masks,
                     const lbm_params* params, lbm_batch** out) {
  if (!out) return fail(LBM_EINVAL, "null output pointer");
  *out = nullptr;
  if (n < 1 || !grids || !params) return fail(LBM_EINVAL, "need n >= 1 cases");
  const int K = params[0].check_every;
  for (int i = 0; i < n; ++i) {
    int rc = validate(&grids[i], masks ? masks[i] : nullptr, &params[i]);
    if (!rc && (params[i].strain_fd || params[i].mrt))
      rc = fail(LBM_EINVAL, "batch cases use the default kernel (strain_fd 0, mrt 0)");
    if (rc) return fail(rc, "case " + std::to_string(i) + ": " + lbm_last_error());
    if (params[i].storage != params[0].storage ||
        (params[i].storage != LBM_STORE_F32 && params[i].storage != LBM_STORE_F64))
      return fail(LBM_EINVAL, "batch cases must all use LBM_STORE_F32 or all LBM_STORE_F64");
    if (params[i].check_every != K) return fail(LBM_EINVAL, "batch cases must share check_every");
  }
  lbm_batch* b = new (std::nothrow) lbm_batch();
  if (!b) return fail(LBM_ENOMEM, "host allocation failed");
  b->n = n;
  b->K = K;
  b->storage = params[0].storage;
  b->cs.resize(n);
  b->enabled.assign(n, 1);
  b->h_status.assign(n, 0);
  auto dev = [&](hipError_t e, const char* what) {
    if (e != hipSuccess) {
      fail(LBM_EDEVICE, std::string(what) + ": " + hipGetErrorString(e));
      return false;
    }
    return true;
  };
  bool ok = dev(hipGetDevice(&b->device), "hipGetDevice") &&
            dev(hipStreamCreateWithFlags(&b->own_stream, hipStreamNonBlocking), "hipStreamCreate");
  b->stream = b->own_stream;
  for (int i = 0; ok && i < n; ++i) {
    HostCase& c = b->cs[i];
    c.grid = grids[i];
    c.p = params[i];
    if (c.p.omega3 == 0) c.p.omega3 = 1.0;
    if (c.p.omega6 == 0) c.p.omega6 = 1.0;
    if (c.p.omega7 == 0) c.p.omega7 = 1.0;
    if (c.p.omega8 == 0) c.p.omega8 = 1.0;
    if (c.p.rho0 == 0) c.p.rho0 = 1.0;
    c.kf = make_consts<float>(c.p, 1.0);
    c.kd = make_consts<double>(c.p, 1.0);
    const size_t es = b->storage == LBM_STORE_F64 ? 8 : 4;
    c.g = make_geom_for(c.grid.nx, c.grid.ny, c.grid.side, es);
    const size_t np = (size_t)c.grid.nx * c.grid.ny;
    for (int j = 0; ok && j < 2; ++j)
      ok = dev(hipMalloc(&c.lat[j], 9 * (size_t)c.g.plane * es), "hipMalloc lattice") &&
           dev(hipMemset(c.lat[j], 0, 9 * (size_t)c.g.plane * es), "hipMemset") &&
           dev(hipMalloc(&c.hist[j], 2 * es * c.grid.ny), "hipMalloc history");
    ok = ok && dev(hipMalloc(&c.ubuf, 2 * np * es), "hipMalloc velocity");
    // the batch kernel always runs the obstacle path: every case has a mask
    // (all fluid when none was given)
    const uint8_t* m = masks ? masks[i] : nullptr;
    std::vector<uint8_t> hm(np, 0);
    size_t solid = 0;
    if (m)
      for (size_t q = 0; q < np; ++q) {
        hm[q] = m[q] ? 1 : 0;
        solid += hm[q];
      }
    c.fluid = np - solid;
    c.h_mask = hm;
    ok = ok && dev(hipMalloc(&c.solid, np), "hipMalloc mask") &&
         dev(hipMemcpy(c.solid, hm.data(), np, hipMemcpyHostToDevice), "copy mask");
  }
  ok = ok && dev(hipMalloc(&b->d_case_res, sizeof(double) * 4 * n), "hipMalloc") &&
       dev(hipMemset(b->d_case_res, 0, sizeof(double) * 4 * n), "hipMemset") &&
       dev(hipMalloc(&b->d_active, sizeof(int) * n), "hipMalloc") &&
       dev(hipMalloc(&b->d_done, sizeof(long long) * n), "hipMalloc") &&
       dev(hipMalloc(&b->d_status, sizeof(int) * n), "hipMalloc") &&
       dev(hipMalloc(&b->d_best, sizeof(double) * n), "hipMalloc") &&
       dev(hipMalloc(&b->d_stall, sizeof(int) * n), "hipMalloc") &&
       dev(hipMalloc(&b->d_sync, sizeof(unsigned) * (1 + n)), "hipMalloc") &&
       dev(hipMalloc(&b->d_tnow, sizeof(long long)), "hipMalloc") &&
       dev(hipMalloc(&b->d_err, sizeof(int)), "hipMalloc") &&
       dev(hipMemset(b->d_err, 0, sizeof(int)), "hipMemset");
  if (!ok) {
    free_batch(b);
    return LBM_EDEVICE;
  }
  int rc = configure(b);
  for (int i = 0; rc == LBM_OK && i < n; ++i) rc = init_case<double>(b, i, nullptr, nullptr, nullptr);
  if (rc == LBM_OK && hipStreamSynchronize(b->stream) != hipSuccess)
    rc = fail(LBM_EDEVICE, "initialisation failed");
  if (rc) {
    free_batch(b);
    return rc;
  }
  *out = b;
  return LBM_OK;
}

void lbm_batch_destroy(lbm_batch* b) {
  if (!b) return;
  if (b->stream) hipStreamSynchronize(b->stream);
  free_batch(b);
}

int lbm_batch_set_stream(lbm_batch* b, void* s) {
  if (!b) return fail(LBM_EINVAL, "null batch");
  HIPCHECK(hipStreamSynchronize(b->stream));
  b->stream = s ? (hipStream_t)s : b->own_stream;
  return LBM_OK;
}

int lbm_batch_set_launch(lbm_batch* b, int32_t rows_per_item, int32_t schedule) {
  if (!b) return fail(LBM_EINVAL, "null batch");
  // rows_per_item: block height of 4, 8 or 16 wavefronts of one row (0 = 4).
  // schedule: 0 graph of per-step kernels, work case by case; 1 the same
  // with tiles interleaved across cases; 2 persistent dataflow kernel.
  int by = rows_per_item == 0 ? 4 : rows_per_item;
  bool known = false;
  for (auto& s : kBatchShapes) known |= s.by == by;
  if (!known) return fail(LBM_EINVAL, "rows_per_item must be 4, 8 or 16");
  if (schedule < 0 || schedule > 2) return fail(LBM_EINVAL, "schedule must be 0, 1 or 2");
  HIPCHECK(hipStreamSynchronize(b->stream));
  b->by = by;
  b->rows = 1;
  b->schedule = schedule;
  b->blocks = 0;
  drop_graphs(b);
  return configure(b);
}

int lbm_batch_init_fields(lbm_batch* b, int32_t ci, const double* rho, const double* ux,
                          const double* uy) {
  if (!b || ci < 0 || ci >= b->n) return fail(LBM_EINVAL, "bad batch or case index");
  const size_t np = (size_t)b->cs[ci].grid.nx * b->cs[ci].grid.ny;
  double* tmp[3] = {nullptr, nullptr, nullptr};
  const double* src[3] = {rho, ux, uy};
  int rc = LBM_OK;
  for (int i = 0; i < 3 && rc == LBM_OK; ++i) {
    if (!src[i]) continue;
    if (hipMalloc(&tmp[i], np * sizeof(double)) != hipSuccess ||
        hipMemcpy(tmp[i], src[i], np * sizeof(double), hipMemcpyHostToDevice) != hipSuccess)
      rc = fail(LBM_EDEVICE, "upload of initial fields failed");
  }
  if (rc == LBM_OK) rc = init_case<double>(b, ci, tmp[0], tmp[1], tmp[2]);
  if (hipStreamSynchronize(b->stream) != hipSuccess && rc == LBM_OK)
    rc = fail(LBM_EDEVICE, "initialisation failed");
  for (auto p : tmp)
    if (p) hipFree(p);
  return rc;
}

int lbm_batch_init_fields_device(lbm_batch* b, int32_t ci, const float* rho, const float* ux,
                                 const float* uy) {  // NOLINT
  if (!b || ci < 0 || ci >= b->n) return fail(LBM_EINVAL, "bad batch or case index");
  const int rc = init_case<float>(b, ci, rho, ux, uy);
  if (rc) return rc;
  // the caller may release the arrays as soon as this returns
  HIPCHECK(hipStreamSynchronize(b->stream));
  return LBM_OK;
}

int lbm_batch_run(lbm_batch* b, double tol, int64_t max_steps, int64_t* steps_per_case) {
  if (!b) return fail(LBM_EINVAL, "null batch");
  if (max_steps < 0 || !(tol >= 0)) return fail(LBM_EINVAL, "bad tol or max_steps");
  const int n = b->n;
  // enabled cases start active; steps count from the batch's current step
  {
    int rc0 = align_parity(b);
    if (rc0) return rc0;
  }
  b->h_active = b->enabled;
  std::vector<long long> done(n, 0);
  std::vector<int> zeros(n, 0);
  std::vector<double> inf(n, INFINITY);
  HIPCHECK(hipMemcpyAsync(b->d_status, zeros.data(), sizeof(int) * n, hipMemcpyHostToDevice,
                          b->stream));
  HIPCHECK(hipMemcpyAsync(b->d_stall, zeros.data(), sizeof(int) * n, hipMemcpyHostToDevice,
                          b->stream));
  HIPCHECK(hipMemcpyAsync(b->d_best, inf.data(), sizeof(double) * n, hipMemcpyHostToDevice,
                          b->stream));
  HIPCHECK(hipMemcpyAsync(b->d_active, b->h_active.data(), sizeof(int) * n,
                          hipMemcpyHostToDevice, b->stream));
  HIPCHECK(hipMemcpyAsync(b->d_done, done.data(), sizeof(long long) * n, hipMemcpyHostToDevice,
                          b->stream));
  HIPCHECK(hipMemsetAsync(b->d_err, 0, sizeof(int), b->stream));
  const int64_t t_start = b->t;
  int rc = rebuild_items(b, max_steps);
  if (rc) return rc;
  const RetireArgs ret = retire_args(b, tol, t_start + 2LL * b->K);
  {
    long long tn = b->t;
    HIPCHECK(hipMemcpyAsync(b->d_tnow, &tn, sizeof tn, hipMemcpyHostToDevice, b->stream));
    HIPCHECK(hipStreamSynchronize(b->stream));
  }
  // dataflow schedule: resident grid size
  const void* kfn = batch_kernel_for(b->storage, b->by);
  int G = 1;
  if (b->schedule == 2) {
    int per_cu = 0;
    HIPCHECK(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kfn, kLanes * b->by, 0));
    hipDeviceProp_t prop;
    HIPCHECK(hipGetDeviceProperties(&prop, b->device));
    G = std::max(1, per_cu) * prop.multiProcessorCount;
    if (b->blocks > 0) G = std::min(G, b->blocks);
  }
  int64_t left = max_steps;
  int active_n = 0;
  for (int v : b->h_active) active_n += v;
  while (left > 0 && active_n > 0) {
    // one window per launch sequence, ending at the next check step
    const int64_t to_check = b->K - (b->t % b->K);
    const int64_t ns = std::min(left, to_check);
    if (b->schedule == 2) {
      BatchArgs a{};
      a.cases = b->d_cases;
      a.ncases = n;
      a.item_case = b->d_item_case;
      a.item_tile = b->d_item_tile;
      a.n_items = b->n_items;
      a.t0 = b->t;
      a.par0 = b->par;
      a.nsteps = (int)ns;
      a.K = b->K;
      a.ticket = b->d_sync;
      a.done = b->d_sync + 1;
      a.ret = ret;
      a.err = b->d_err;
      a.spin_limit = 1LL << 26;
      HIPCHECK(hipMemsetAsync(b->d_sync, 0, sizeof(unsigned) * (1 + n), b->stream));
      void* kargs[] = {&a};
      HIPCHECK(hipLaunchKernel(kfn, dim3(G), dim3(kLanes, b->by), kargs, 0, b->stream));
      hipLaunchKernelGGL(batch_tick_kernel, dim3(1), dim3(64), 0, b->stream, b->d_tnow, (int)ns);
      b->par ^= int(ns & 1);
    } else if (ns == b->K && b->K >= 4) {
      // full window: captured once per start parity, replayed
      const int par = b->par;
      if (!b->graph[par]) {
        hipGraph_t gr = nullptr;
        HIPCHECK(hipStreamBeginCapture(b->stream, hipStreamCaptureModeThreadLocal));
        b->window_flips = enqueue_window(b, b->t, (int)ns, par, ret, b->stream) & 1;
        hipError_t e = hipStreamEndCapture(b->stream, &gr);
        if (e != hipSuccess) return fail(LBM_EDEVICE, hipGetErrorString(e));
        e = hipGraphInstantiate(&b->graph[par], gr, nullptr, nullptr, 0);
        hipGraphDestroy(gr);
        if (e != hipSuccess) {
          b->graph[par] = nullptr;
          return fail(LBM_EDEVICE, hipGetErrorString(e));
        }
      }
      HIPCHECK(hipGraphLaunch(b->graph[par], b->stream));
      b->par ^= b->window_flips;
    } else {
      b->par ^= enqueue_window(b, b->t, (int)ns, b->par, ret, b->stream) & 1;
    }
    HIPCHECK(hipGetLastError());
    b->t += ns;
    left -= ns;
    if (b->t % b->K == 0) {
      HIPCHECK(hipStreamSynchronize(b->stream));
      int err = 0;
      HIPCHECK(hipMemcpy(&err, b->d_err, sizeof(int), hipMemcpyDeviceToHost));
      if (err) return fail(LBM_EDEVICE, "batch dependency wait timed out");
      std::vector<int> act(n);
      HIPCHECK(hipMemcpy(act.data(), b->d_active, sizeof(int) * n, hipMemcpyDeviceToHost));
      int now = 0;
      for (int v : act) now += v;
      if (now < active_n) {  // drop retired cases from the work list
        for (int i = 0; i < n; ++i)
          if (b->h_active[i] && !act[i]) b->cs[i].state_par = b->par;
        b->h_active = act;
        rc = rebuild_items(b, left);
        if (rc) return rc;
      }
      active_n = now;
    }
  }
  HIPCHECK(hipStreamSynchronize(b->stream));
  HIPCHECK(hipMemcpy(done.data(), b->d_done, sizeof(long long) * n, hipMemcpyDeviceToHost));
  HIPCHECK(hipMemcpy(b->h_status.data(), b->d_status, sizeof(int) * n, hipMemcpyDeviceToHost));
  // (cases that retired hold their state where the batch was then)
  for (int i = 0; i < n; ++i)
    if (b->enabled[i] && b->h_active[i]) b->cs[i].state_par = b->par;
  bool diverged = false;
  for (int i = 0; i < n; ++i) {
    long long v = done[i];
    if (!b->enabled[i]) v = 0;              // not advanced by this run
    else if (v == 0) v = b->t - t_start;    // not converged within max_steps
    else if (v < 0) {
      diverged = true;
      v = -(-v - t_start);
    } else {
      v -= t_start;
    }
    if (steps_per_case) steps_per_case[i] = v;
  }
  if (diverged) return fail(LBM_EUNSTABLE, "some cases diverged (negative step counts)");
  return LBM_OK;
}


int lbm_batch_set_plateau(lbm_batch* b, int32_t checks, double factor) {
  if (!b || checks < 0 || !(factor > 0 && factor <= 1))
    return fail(LBM_EINVAL, "checks >= 0 and 0 < factor <= 1");
  b->plateau_checks = checks;
  b->plateau_factor = factor;
  return LBM_OK;
}

int lbm_batch_status(lbm_batch* b, int32_t* status) {
  if (!b || !status) return fail(LBM_EINVAL, "null argument");
  for (int i = 0; i < b->n; ++i) status[i] = b->h_status[i];
  return LBM_OK;
}

int lbm_batch_set_enabled(lbm_batch* b, const int32_t* enabled) {
  if (!b) return fail(LBM_EINVAL, "null batch");
  for (int i = 0; i < b->n; ++i) b->enabled[i] = enabled ? (enabled[i] != 0) : 1;
  return LBM_OK;
}

int lbm_batch_set_storage(lbm_batch* b, int32_t storage) {
  if (!b) return fail(LBM_EINVAL, "null batch");
  if (storage != LBM_STORE_F32 && storage != LBM_STORE_F64)
    return fail(LBM_EINVAL, "batch storage must be LBM_STORE_F32 or LBM_STORE_F64");
  if (storage == b->storage) return LBM_OK;
  HIPCHECK(hipStreamSynchronize(b->stream));
  const size_t es2 = storage == LBM_STORE_F64 ? 8 : 4, es1 = b->storage == LBM_STORE_F64 ? 8 : 4;
  for (auto& c : b->cs) {
    const int rc = check_lattice_bytes(c.grid.nx, c.grid.ny, es2);
    if (rc) return rc;
  }
  for (auto& c : b->cs) {
    const Geom g2 = make_geom_for(c.grid.nx, c.grid.ny, c.grid.side, es2);
    const size_t np = (size_t)c.grid.nx * c.grid.ny;
    void* lat2[2] = {nullptr, nullptr};
    void* hist2[2] = {nullptr, nullptr};
    void* ub2 = nullptr;
    bool ok = true;
    for (int i = 0; ok && i < 2; ++i)
      ok = hipMalloc(&lat2[i], 9 * (size_t)g2.plane * es2) == hipSuccess &&
           hipMemset(lat2[i], 0, 9 * (size_t)g2.plane * es2) == hipSuccess &&
           hipMalloc(&hist2[i], 2 * es2 * c.grid.ny) == hipSuccess;
    ok = ok && hipMalloc(&ub2, 2 * np * es2) == hipSuccess;
    if (!ok) {
      for (int i = 0; i < 2; ++i) {
        hipFree(lat2[i]);
        hipFree(hist2[i]);
      }
      hipFree(ub2);
      return fail(LBM_ENOMEM, "allocation for the new storage failed");
    }
    const long long nf = (long long)(c.grid.nx + 2) * (c.grid.ny + 2);
    for (int i = 0; i < 2; ++i) {
      hipLaunchKernelGGL(convert_lattice_kernel, dim3(int((nf + 255) / 256)), dim3(256), 0,
                         b->stream, c.lat[i], b->storage, c.g, 1.0, lat2[i], (int)storage, g2, 1.0);
      const long long nh = 2LL * c.grid.ny;
      hipLaunchKernelGGL(convert_values_kernel, dim3(int((nh + 255) / 256)), dim3(256), 0,
                         b->stream, c.hist[i], int(es1 == 8), hist2[i], int(es2 == 8), nh);
    }
    hipLaunchKernelGGL(convert_values_kernel, dim3(int((2 * np + 255) / 256)), dim3(256), 0,
                       b->stream, (const void*)c.ubuf, int(es1 == 8), ub2, int(es2 == 8),
                       (long long)(2 * np));
    HIPCHECK(hipGetLastError());
    HIPCHECK(hipStreamSynchronize(b->stream));
    for (int i = 0; i < 2; ++i) {
      hipFree(c.lat[i]);
      hipFree(c.hist[i]);
      c.lat[i] = lat2[i];
      c.hist[i] = hist2[i];
    }
    hipFree(c.ubuf);
    c.ubuf = static_cast<float*>(ub2);
    c.g = g2;
    c.p.storage = storage;
  }
  b->storage = storage;
  drop_graphs(b);
  return configure(b);
}

int lbm_batch_average_last_two(lbm_batch* b) {
  if (!b) return fail(LBM_EINVAL, "null batch");
  for (int i = 0; i < b->n; ++i) {
    if (!b->enabled[i]) continue;
    HostCase& h = b->cs[i];
    const int cur = h.state_par;
    const long long n = 9LL * h.g.plane;
    HIPCHECK(launch_average(b->storage, h.lat[cur], h.lat[cur ^ 1], n, (double)h.kf.scale,
                            h.hist[cur], h.hist[cur ^ 1], h.hist[0] ? 2LL * h.grid.ny : 0,
                            b->stream));
  }
  HIPCHECK(hipStreamSynchronize(b->stream));
  return LBM_OK;
}

int lbm_batch_residual(lbm_batch* b, int32_t ci, double* r) {
  if (!b || !r || ci < 0 || ci >= b->n) return fail(LBM_EINVAL, "bad argument");
  double v[4];
  HIPCHECK(hipStreamSynchronize(b->stream));
  HIPCHECK(hipMemcpy(v, b->d_case_res + 4 * ci, sizeof v, hipMemcpyDeviceToHost));
  if (!std::isfinite(v[0]) || !std::isfinite(v[1])) {
    *r = NAN;
    return fail(LBM_EUNSTABLE, "residual is not finite");
  }
  *r = v[1] > 0 ? std::sqrt(v[0] / v[1]) : (v[0] > 0 ? INFINITY : 0.0);
  return LBM_OK;
}

int lbm_batch_fields(lbm_batch* b, int32_t ci, double* rho, double* ux, double* uy) {
  if (!b || ci < 0 || ci >= b->n) return fail(LBM_EINVAL, "bad batch or case index");
  HostCase& c = b->cs[ci];
  const size_t np = (size_t)c.grid.nx * c.grid.ny;
  // Staging of kKeptStageMin to kKeptStage bytes stays with the batch (512 x 512
  // nodes: 610 us per call with an allocation of its own, 535 without; 256 x 256
  // 121 either way, 64 x 64 46.2 and 48.6).  Others last for the call, and so do
  // those of a call that finds the kept staging in use by another thread.
  const size_t bytes = 3 * np * sizeof(double);
  std::unique_lock<std::mutex> lock(b->stage_mutex, std::defer_lock);
  const bool kept = bytes >= kKeptStageMin && bytes <= kKeptStage && lock.try_lock();
  if (kept && bytes > b->stage_bytes) {
    hipFree(b->d_stage);
    b->d_stage = nullptr;
    b->stage_bytes = 0;
    HIPCHECK(hipMalloc(&b->d_stage, bytes));
    b->stage_bytes = bytes;
  }
  double* d = kept ? b->d_stage : nullptr;
  if (!kept) HIPCHECK(hipMalloc(&d, bytes));
  const int blocks = int((np + 255) / 256);
  if (b->storage == LBM_STORE_F64)
    hipLaunchKernelGGL((export_kernel<StoreF64>), dim3(blocks), dim3(256), 0, b->stream,
                       (const double*)c.lat[c.state_par], c.g, c.kd, c.solid,
                       (const double*)nullptr, 0LL, (long long)np, (double*)nullptr, (float*)nullptr,
                       (float*)nullptr,
                       (float*)nullptr, d, d + np, d + 2 * np);
  else
    hipLaunchKernelGGL((export_kernel<StoreF32>), dim3(blocks), dim3(256), 0, b->stream,
                       (const float*)c.lat[c.state_par], c.g, c.kf, c.solid,
                       (const float*)nullptr, 0LL, (long long)np, (double*)nullptr, (float*)nullptr,
                       (float*)nullptr,
                       (float*)nullptr, d, d + np, d + 2 * np);
  hipError_t e = hipStreamSynchronize(b->stream);
  double* h[3] = {rho, ux, uy};
  for (int i = 0; i < 3 && e == hipSuccess; ++i)
    if (h[i]) e = hipMemcpy(h[i], d + i * np, np * sizeof(double), hipMemcpyDeviceToHost);
  if (!kept) hipFree(d);
  if (e != hipSuccess) return fail(LBM_EDEVICE, hipGetErrorString(e));
  return LBM_OK;
}

}  // extern "C"
