// Host side of the single-lattice C ABI declared in include/lbm.h, plus the
// small auxiliary kernels (partial-sum finalisation, equilibrium
// initialisation, export).  The fused step kernels live in lbm_kernels.h and
// are instantiated per storage type and flavour in lbm_step.hip.

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "../../include/lbm.h"
#include "lbm_aux.h"
#include "lbm_ctx.h"
#include "lbm_host.h"
#include "lbm_multi.h"

using namespace lbmk;
using namespace lbmh;

namespace lbmh {
namespace {
thread_local std::string g_err;
}
int fail(int code, const std::string& msg) {
  g_err = msg;
  return code;
}

int export_range(lbm_ctx* c, long long first, long long count, double* pops, float* ro,
                 float* uxo, float* uyo, double* rd, double* uxd, double* uyd) {
  const Geom g = make_geom_for(c->grid.nx, c->grid.ny, c->grid.side, c->esize);
  if (count <= 0) return LBM_OK;
  const int blocks = int((count + 255) / 256);
  const void* src = c->lat[c->cur];
  switch (c->p.storage) {
    case LBM_STORE_F64:
      hipLaunchKernelGGL(export_kernel<StoreF64>, dim3(blocks), dim3(256), 0, c->stream,
                         (const double*)src, g, c->kd, c->d_solid, (const double*)c->d_force,
                         first, count, pops, ro, uxo, uyo, rd, uxd, uyd);
      break;
    case LBM_STORE_F32:
      hipLaunchKernelGGL(export_kernel<StoreF32>, dim3(blocks), dim3(256), 0, c->stream,
                         (const float*)src, g, c->kf, c->d_solid, (const float*)c->d_force,
                         first, count, pops, ro, uxo, uyo, rd, uxd, uyd);
      break;
    case LBM_STORE_BF16:
      hipLaunchKernelGGL(export_kernel<StoreBF16>, dim3(blocks), dim3(256), 0, c->stream,
                         (const uint16_t*)src, g, c->kf, c->d_solid, (const float*)c->d_force,
                         first, count, pops, ro, uxo, uyo, rd, uxd, uyd);
      break;
    default:
      hipLaunchKernelGGL(export_kernel<StoreF16>, dim3(blocks), dim3(256), 0, c->stream,
                         (const _Float16*)src, g, c->kf, c->d_solid, (const float*)c->d_force,
                         first, count, pops, ro, uxo, uyo, rd, uxd, uyd);
      break;
  }
  HIPCHECK(hipGetLastError());
  return LBM_OK;
}
}  // namespace lbmh

namespace {

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

struct Shape {
  int by, rows;
};
constexpr Shape kShapes[] = {{16, 1}, {8, 1}, {4, 1}, {4, 2}, {8, 2}, {4, 4}, {8, 4}};
constexpr int kNumShapes = sizeof(kShapes) / sizeof(kShapes[0]);


}  // namespace


namespace {

template <class C>
const Consts<C>& consts_for(const lbm_ctx* c);
template <>
const Consts<double>& consts_for<double>(const lbm_ctx* c) { return c->kd; }
template <>
const Consts<float>& consts_for<float>(const lbm_ctx* c) { return c->kf; }



Geom make_geom(const lbm_ctx* c) { return make_geom_for(c->grid.nx, c->grid.ny, c->grid.side, c->esize); }


int configure_tiles(lbm_ctx* c) {
  c->out_rows = c->by * c->rows;
  c->tiles_x = (c->grid.nx + kLanes - 1) / kLanes;
  c->tiles_y = (c->grid.ny + c->out_rows - 1) / c->out_rows;
  c->ntiles = c->tiles_x * c->tiles_y;
  if ((size_t)c->ntiles > c->partial_cap) {
    if (c->partials) HIPCHECK(hipFree(c->partials));
    c->partials = nullptr;
    HIPCHECK(hipMalloc(&c->partials, (size_t)c->ntiles * 4 * sizeof(double)));
    c->partial_cap = c->ntiles;
  }
  for (int i = 0; i < 2; ++i)
    if (c->graph[i]) {
      hipGraphExecDestroy(c->graph[i]);
      c->graph[i] = nullptr;
    }
  return LBM_OK;
}

constexpr size_t kLastLevelCacheBytes = size_t(256) << 20;

int flavor_of(const lbm_ctx* c, int64_t idx) {
  const int K = c->p.check_every;
  if (idx % K == 0) return kCheck;
  return K >= 2 && idx % K == K - 1 ? kStore : kPlain;
}

constexpr int kMultiRing = 2 * kMultiSteps - 1;
int multi_rows(int shape) { return kMultiShapes[shape].nw * kMultiShapes[shape].rpw; }
int multi_tiles_x(const lbm_ctx* c) {
  const int txo = kLanes - 2 * kMultiRing;
  return (c->grid.nx + txo - 1) / txo;
}
int multi_tiles_y(const lbm_ctx* c, int shape) {
  const int tyo = multi_rows(shape) - 2 * kMultiRing;
  return (c->grid.ny + tyo - 1) / tyo;
}
long long multi_tiles(const lbm_ctx* c, int shape) {
  return (long long)multi_tiles_x(c) * multi_tiles_y(c, shape);
}

// Shape of the two-step kernel for this lattice, or -1 (step by step: the
// variants, a launch shape other than the default, and where two steps at
// once do not pay).  Times are per step, cavities unless named otherwise, one
// step | two steps.
// - Up to one block per compute unit a launch costs its latency, whatever
//   the size: the lowest blocks that still fit (2, 6, 10 output rows, one row
//   per wavefront): 128^2 FP64 3.6 | 2.7 us, 256^2 FP32 3.4 | 2.6 us, 320^2
//   FP32 3.9 | 3.1 us; two rounds of the 6-row blocks up to 512 tiles: 384^2
//   FP32 4.4 | 3.5 us.
// - Larger lattices: two rows per wavefront (10 output rows: 1024^2 FP32
//   13.3 | 10.9, FP64 24.0 | 19.0 us, 2048^2 FP64 117 | 73.5 us); beyond the
//   last-level cache, except in FP64 (registers), four rows (26 output rows:
//   4096^2 FP32 264 | 158 us, channel 4096 x 1024 FP16 52.5 | 47.1 us).
// - The ring costs instructions: the rows a pair collides over those of two
//   single steps (work) are 1.1 to 1.4 where the tiles fit.  At 1.6 (59 to 64
//   columns of 58 over 64, 175 to 192 of 3 x 58 over 3 x 64) every storage
//   loses: 180 x 2000 FP16 6.6 | 8.4 us, FP32 6.8 | 7.3, FP64 11.1 | 13.0.
//   FP64 has the least to spare: in small lattices up to 2 (64 x 1500 at 2.7:
//   5.3 | 7.0 us), and tiles that are partly empty do not pay in strips of one
//   or two tiles (80 x 4000 12.7 | 13.5 us with sides periodic in y) or where
//   few compute units get a second block (129 x 1025 periodic 7.0 | 7.4 us);
//   channels gain there all the same, their outlet being a serial chain
//   (129 x 1025 13.7 | 10.0 us).
// - 16-bit storages in cache are bound by instructions: beyond about 1.1 M
//   nodes one step at a time is up to 3 % faster without an outlet (1280^2
//   FP16 17.4 | 18.1 us, 2048^2 38.1 | 38.8 us), and up to 2.2 M nodes also
//   with one in every 14th tile or fewer (1600 x 750 18.0 | 19.2 us; 2400 x
//   1041 29.5 | 28.6), except with a mask, whose tests the two-step kernel
//   leaves out where a tile has none (1600 x 750 20.5 | 20.2 us).
struct MultiFit {
  long long tiles;
  double work, fill;   // fill: lattice nodes over output nodes of the tiles
};
MultiFit multi_fit(const lbm_ctx* c, int shape) {
  const int nx = c->grid.nx, ny = c->grid.ny, nr = multi_rows(shape);
  MultiFit f{multi_tiles(c, shape), 0, 0};
  f.work = f.tiles * (2.0 * nr - 8.0) / (2.0 * ((nx + kLanes - 1) / kLanes) * ny);
  f.fill = (double)nx * ny /
           ((double)f.tiles * (kLanes - 2 * kMultiRing) * (nr - 2 * kMultiRing));
  return f;
}

// 16-bit lattices in cache beyond 1.1 M nodes
bool multi_big16(const lbm_ctx* c) {
  const Geom g = make_geom(c);
  return c->esize == 2 && 2 * 9 * (size_t)g.plane * c->esize <= kLastLevelCacheBytes &&
         (long long)c->grid.nx * c->grid.ny > 1100000;
}

int multi_shape(const lbm_ctx* c) {
  if (c->by != 4 || c->rows != 1 || c->p.strain_fd || c->p.mrt) return -1;
  const int nx = c->grid.nx, ny = c->grid.ny;
  if (nx < 16 || ny < 16) return -1;
  // 16-bit storages: the copies across a periodic side are rounded to nearest,
  // the node's own values stochastically; a region that continues across the
  // side has only the latter
  if (c->esize == 2 && (c->grid.side[0] == LBM_SIDE_PERIODIC ||
                        c->grid.side[2] == LBM_SIDE_PERIODIC))
    return -1;
  const bool outlet = c->grid.side[1] == LBM_SIDE_OUTLET;
  const bool tight = c->esize == 8 && !outlet;
  int small = -1;
  for (int s = 0; s < 3 && small < 0; ++s)
    if (multi_tiles(c, s) <= 256) small = s;
  if (small < 0 && multi_tiles(c, 1) <= 512) small = 1;
  if (small >= 0) return tight && small > 0 && multi_fit(c, small).work > 2.0 ? -1 : small;
  const Geom g = make_geom(c);
  const bool cached = 2 * 9 * (size_t)g.plane * c->esize <= kLastLevelCacheBytes;
  const bool big16 = multi_big16(c);
  if (big16 && !outlet) return -1;
  const int shape = (cached && !big16) || c->esize == 8 ? 3 : 4;
  const MultiFit f = multi_fit(c, shape);
  if (f.work > 1.55) return -1;
  if (big16 && (f.work > 1.25 || (!c->d_solid && f.work > 1.15 && multi_tiles_x(c) >= 14 &&
                                  (long long)nx * ny < 2200000)))
    return -1;
  if (tight && f.fill < 0.85 && (multi_tiles_x(c) <= 2 || f.tiles <= 384)) return -1;
  return shape;
}

// The share of the regions' rows that may be near a solid node (a row with one
// or next to one takes the tests of every neighbour, in the single step as
// well, but the ring's rows too).  Dots on a share of the lattice, per step,
// one step | two steps, at these shares:
// - channels always gain (1024^2 FP64 with all rows 38.6 | 35.5 us), 16-bit ones
//   in cache beyond 1.1 M nodes up to a quarter (2048^2 FP16 at 0.16 57.1 | 52.1,
//   at 0.40 57.9 | 59.0);
// - FP64 beyond one block per compute unit: 0.15 (512^2 at 0.14 9.5 | 9.3,
//   0.18 9.6 | 9.9; 1024^2 periodic at 0.15 25.3 | 25.1, 0.17 25.1 | 25.5),
//   closed lattices of more tiles 0.5 (1024^2 at 0.41 27.1 | 25.7, at 0.89 28.4 |
//   29.4), and 0.4 where a lattice one tile wide takes two of the two-step tiles
//   (64^2 at 0.29 4.3 | 3.3, 0.46 4.3 | 4.5);
// - FP32: any (1024^2, all rows 17.5 | 15.7), except 0.2 with periodic sides in
//   cache beyond 1.1 M nodes (1500^2 at 0.15 25.1 | 24.5, 0.41 25.9 | 27.1) and
//   0.05 where few compute units get a second, partly empty block (129 x 1025
//   at 0.02 5.1 | 4.9, 0.16 5.2 | 5.7);
// - 16 bits: 0.05 beyond two rounds of small blocks (1024^2 FP16 at 0.03 14.0 |
//   13.7, 0.17 14.2 | 14.9).
double multi_near_share(const lbm_ctx* c, int shape) {
  const MultiFit f = multi_fit(c, shape);
  const int32_t* sd = c->grid.side;
  if (sd[1] == LBM_SIDE_OUTLET) return multi_big16(c) ? 0.25 : 1.0;
  bool closed = true;
  for (int q = 0; q < 4; ++q)
    closed = closed && (sd[q] == LBM_SIDE_WALL || sd[q] == LBM_SIDE_LID);
  if (c->esize == 8) {
    if (f.tiles > 256) return closed && f.tiles > 512 ? 0.5 : 0.15;
    return closed && f.work > 3.0 ? 0.4 : 1.0;
  }
  if (shape < 3) return 1.0;
  if (c->esize == 2 || (f.fill < 0.85 && f.tiles <= 512)) return 0.05;
  return shape == 3 && !closed && (long long)c->grid.nx * c->grid.ny > 1100000 ? 0.2 : 1.0;
}

// fluid[tile] = 1 where the region of the tile (64 x nr nodes from (x0, y0),
// inside the lattice) holds no solid node, and near[tile]: its rows with a solid
// node in them or in the row above or below; one wavefront per tile, nr <= 32.
__global__ __launch_bounds__(kLanes) void multi_fluid_kernel(const uint8_t* __restrict__ solid,
                                                             int nx, int ny, int tiles_x, int txo,
                                                             int tyo, int h, int nr,
                                                             uint8_t* __restrict__ fluid,
                                                             uint8_t* __restrict__ near) {
  const int tile = blockIdx.x, x = tile % tiles_x * txo - h + int(threadIdx.x);
  const int y0 = tile / tiles_x * tyo - h;
  unsigned rows = 0;
  for (int r = 0; r < nr; ++r) {
    const int y = y0 + r;
    const bool s = x >= 0 && x < nx && y >= 0 && y < ny && solid[y * nx + x];
    rows |= __builtin_amdgcn_ballot_w64(s) != 0 ? 1u << r : 0u;
  }
  if (threadIdx.x != 0) return;
  fluid[tile] = rows ? 0 : 1;
  rows |= rows << 1 | rows >> 1;
  if (nr < 32) rows &= (1u << nr) - 1;
  near[tile] = uint8_t(__builtin_popcount(rows));
}

// Choose the two-step shape of the current configuration and mark its tiles
// without solid nodes.  Called where the configuration changes, on the
// context's stream.
int configure_multi(lbm_ctx* c) {
  c->multi = multi_shape(c);
  if (c->multi < 0 || !c->d_solid) return LBM_OK;
  const int tx = multi_tiles_x(c), n = tx * multi_tiles_y(c, c->multi), nr = multi_rows(c->multi);
  uint8_t* d_near = c->d_fluid + n;
  hipLaunchKernelGGL(multi_fluid_kernel, dim3(n), dim3(kLanes), 0, c->stream, c->d_solid,
                     c->grid.nx, c->grid.ny, tx, kLanes - 2 * kMultiRing, nr - 2 * kMultiRing,
                     kMultiRing, nr, c->d_fluid, d_near);
  HIPCHECK(hipGetLastError());
  const double allowed = multi_near_share(c, c->multi);
  if (allowed >= 1.0) return LBM_OK;
  std::vector<uint8_t> near(n);
  HIPCHECK(hipMemcpyAsync(near.data(), d_near, n, hipMemcpyDeviceToHost, c->stream));
  HIPCHECK(hipStreamSynchronize(c->stream));
  long long rows = 0;
  for (uint8_t v : near) rows += v;
  if (rows > allowed * n * nr) c->multi = -1;
  return LBM_OK;
}

StepArgs step_args(const lbm_ctx* c) {
  StepArgs a{};
  a.g = make_geom(c);
  a.tiles_x = c->tiles_x;
  a.ntiles = c->ntiles;
  a.out_rows = c->out_rows;
  a.solid = c->d_solid;
  a.hist_in = c->hist[c->cur];
  a.hist_out = c->hist[c->cur ^ 1];
  a.ubuf = c->ubuf;
  a.partials = c->partials;
  a.force = c->d_force ? c->d_force : c->ubuf;
  a.has_force = c->d_force != nullptr;
  a.rng = c->rng;
  a.rng_slot = c->cur;
  return a;
}

const void* consts_of(const lbm_ctx* c) {
  return c->p.storage == LBM_STORE_F64 ? static_cast<const void*>(&c->kd)
                                       : static_cast<const void*>(&c->kf);
}

// Queue the next step, or kMultiSteps plain steps in one launch, then swap
// lattices; returns the steps taken.  left: steps still to take.  The last
// step of a call is always a step of its own, so that the two lattices then
// hold the states of the last two steps.
int enqueue_steps(lbm_ctx* c, int64_t left, hipStream_t st) {
  const int64_t idx = c->t + 1;
  const int flavor = flavor_of(c, idx);
  const StepArgs a = step_args(c);
  const void* src = c->lat[c->cur];
  void* dst = c->lat[c->cur ^ 1];
  const void* k = consts_of(c);
  const int shape = c->multi;
  if (shape >= 0 && left > kMultiSteps && flavor == kPlain && flavor_of(c, idx + 1) == kPlain) {
    StepArgs m = a;   // (a refused launch leaves the single step its own tiles)
    m.tiles_x = multi_tiles_x(c);
    m.ntiles = m.tiles_x * multi_tiles_y(c, shape);
    bool ok;
    switch (c->p.storage) {
      case 0: ok = launch_multi<0>(shape, src, dst, m, c->d_fluid, k, st); break;
      case 1: ok = launch_multi<1>(shape, src, dst, m, c->d_fluid, k, st); break;
      case 2: ok = launch_multi<2>(shape, src, dst, m, c->d_fluid, k, st); break;
      default: ok = launch_multi<3>(shape, src, dst, m, c->d_fluid, k, st); break;
    }
    if (ok) {
      c->cur ^= 1;
      c->t += kMultiSteps;
      return kMultiSteps;
    }
  }
  int var = (c->p.strain_fd ? kVarFds : 0) | (c->p.mrt ? kVarMrt : 0);
  // When the two lattices together outgrow MI355X's 256 MiB Infinity Cache
  // the default kernel stores non-temporally: measured 6 % faster at 4096^2
  // (F32), while at 1024^2 (75 MB, cache resident) ordinary stores are 24 %
  // faster.
  const size_t elem = c->p.storage == LBM_STORE_F64 ? 8 : c->p.storage == LBM_STORE_F32 ? 4 : 2;
  if (var == 0 && 2 * 9 * (size_t)a.g.plane * elem > kLastLevelCacheBytes) var = kVarNts;
  switch (c->p.storage * 3 + flavor) {
    case 0: launch_step<0, kPlain>(c->by, c->rows, var, src, dst, a, k, st); break;
    case 1: launch_step<0, kStore>(c->by, c->rows, var, src, dst, a, k, st); break;
    case 2: launch_step<0, kCheck>(c->by, c->rows, var, src, dst, a, k, st); break;
    case 3: launch_step<1, kPlain>(c->by, c->rows, var, src, dst, a, k, st); break;
    case 4: launch_step<1, kStore>(c->by, c->rows, var, src, dst, a, k, st); break;
    case 5: launch_step<1, kCheck>(c->by, c->rows, var, src, dst, a, k, st); break;
    case 6: launch_step<2, kPlain>(c->by, c->rows, var, src, dst, a, k, st); break;
    case 7: launch_step<2, kStore>(c->by, c->rows, var, src, dst, a, k, st); break;
    case 8: launch_step<2, kCheck>(c->by, c->rows, var, src, dst, a, k, st); break;
    case 9: launch_step<3, kPlain>(c->by, c->rows, var, src, dst, a, k, st); break;
    case 10: launch_step<3, kStore>(c->by, c->rows, var, src, dst, a, k, st); break;
    default: launch_step<3, kCheck>(c->by, c->rows, var, src, dst, a, k, st); break;
  }
  if (flavor == kCheck) {
    hipLaunchKernelGGL(finalize_kernel<256>, dim3(1), dim3(256), 0, st, c->partials, c->ntiles,
                       c->result);
    c->checked = true;
  }
  c->cur ^= 1;
  c->t = idx;
  return 1;
}

template <class S, class FT>
void launch_init(lbm_ctx* c, const FT* rho, const FT* ux, const FT* uy) {
  using C = typename S::C;
  using T = typename S::T;
  Geom g = make_geom(c);
  const int blocks = int(((long long)g.nx * g.ny + 255) / 256);
  hipLaunchKernelGGL((init_kernel<S, FT>), dim3(blocks), dim3(256), 0, c->stream, (T*)c->lat[0],
                     (T*)c->lat[1], g, consts_for<C>(c), c->d_solid, rho, ux, uy, (C*)c->ubuf,
                     (C*)c->hist[0], (C*)c->hist[1]);
  hipLaunchKernelGGL((ghost_fill_kernel<S>), dim3(blocks), dim3(256), 0, c->stream, (T*)c->lat[0],
                     g, consts_for<C>(c), c->d_solid);
}

template <class S>
void launch_ghost_fill(lbm_ctx* c, int which) {
  using C = typename S::C;
  using T = typename S::T;
  Geom g = make_geom(c);
  const int blocks = int(((long long)g.nx * g.ny + 255) / 256);
  hipLaunchKernelGGL((ghost_fill_kernel<S>), dim3(blocks), dim3(256), 0, c->stream,
                     (T*)c->lat[which], g, consts_for<C>(c), c->d_solid);
}

// The step counter of the stochastic rounding equals the step index: set it
// wherever the state's step index is set (initialisation, checkpoint load),
// in the slot the next step reads.
int set_rng_counter(lbm_ctx* c) {
  c->rng_host[c->cur] = unsigned(c->t);
  HIPCHECK(hipMemcpyAsync(c->rng + c->cur, &c->rng_host[c->cur], sizeof(unsigned),
                          hipMemcpyHostToDevice, c->stream));
  return LBM_OK;
}

template <class FT>
int init_common(lbm_ctx* c, const FT* rho, const FT* ux, const FT* uy) {
  switch (c->p.storage) {
    case LBM_STORE_F64: launch_init<StoreF64, FT>(c, rho, ux, uy); break;
    case LBM_STORE_F32: launch_init<StoreF32, FT>(c, rho, ux, uy); break;
    case LBM_STORE_BF16: launch_init<StoreBF16, FT>(c, rho, ux, uy); break;
    default: launch_init<StoreF16, FT>(c, rho, ux, uy); break;
  }
  HIPCHECK(hipGetLastError());
  c->cur = 0;
  c->t = 0;
  c->checked = false;
  for (int i = 0; i < 2; ++i)
    if (c->graph[i]) {
      hipGraphExecDestroy(c->graph[i]);
      c->graph[i] = nullptr;
    }
  return set_rng_counter(c);
}

int export_common(lbm_ctx* c, double* pops, float* ro, float* uxo, float* uyo, double* rd,
                  double* uxd, double* uyd) {
  return lbmh::export_range(c, 0, (long long)c->grid.nx * c->grid.ny, pops, ro, uxo, uyo, rd,
                            uxd, uyd);
}

// Device copy of the per-node force field in the current compute type and the
// force flag of the constants (a field replaces the uniform force).
int apply_force(lbm_ctx* c) {
  if (c->d_force) HIPCHECK(hipFree(c->d_force));
  c->d_force = nullptr;
  const bool uniform = c->p.fx != 0.0 || c->p.fy != 0.0;
  c->kd.force = c->kf.force = uniform ? 1 : 0;
  if (c->h_force.empty()) return LBM_OK;
  const size_t m = c->h_force.size();
  std::vector<char> buf(m * c->csize);
  if (c->csize == 8) {
    std::memcpy(buf.data(), c->h_force.data(), m * sizeof(double));
  } else {
    float* f = reinterpret_cast<float*>(buf.data());
    for (size_t i = 0; i < m; ++i) f[i] = float(c->h_force[i]);
  }
  HIPCHECK(hipMalloc(&c->d_force, buf.size()));
  HIPCHECK(hipMemcpy(c->d_force, buf.data(), buf.size(), hipMemcpyHostToDevice));
  c->kd.force = c->kf.force = 1;
  return LBM_OK;
}

void free_ctx(lbm_ctx* c) {
  if (!c) return;
  for (int i = 0; i < 2; ++i) {
    if (c->graph[i]) hipGraphExecDestroy(c->graph[i]);
    if (c->lat[i]) hipFree(c->lat[i]);
    if (c->hist[i]) hipFree(c->hist[i]);
  }
  if (c->d_solid) hipFree(c->d_solid);
  if (c->d_force) hipFree(c->d_force);
  if (c->ubuf) hipFree(c->ubuf);
  if (c->partials) hipFree(c->partials);
  if (c->result) hipFree(c->result);
  if (c->rng) hipFree(c->rng);
  if (c->ev0) hipEventDestroy(c->ev0);
  if (c->ev1) hipEventDestroy(c->ev1);
  if (c->own_stream) hipStreamDestroy(c->own_stream);
  delete c;
}

}  // namespace

extern "C" {

const char* lbm_last_error(void) { return lbmh::g_err.c_str(); }

int lbm_launch_shapes(int32_t* shapes, int32_t cap) {
  for (int i = 0; i < kNumShapes && i < cap; ++i) {
    shapes[2 * i] = kShapes[i].by;
    shapes[2 * i + 1] = kShapes[i].rows;
  }
  return kNumShapes;
}

int lbm_create(const lbm_grid* grid, const uint8_t* solid_mask, const lbm_params* params,
               lbm_ctx** out) {
  if (!out) return fail(LBM_EINVAL, "null output pointer");
  *out = nullptr;
  int rc = validate(grid, solid_mask, params);
  if (rc) return rc;
  lbm_ctx* c = new (std::nothrow) lbm_ctx();
  if (!c) return fail(LBM_ENOMEM, "host allocation failed");
  c->grid = *grid;
  c->p = *params;
  if (c->p.omega3 == 0) c->p.omega3 = 1.0;
  if (c->p.omega6 == 0) c->p.omega6 = 1.0;
  if (c->p.omega7 == 0) c->p.omega7 = 1.0;
  if (c->p.omega8 == 0) c->p.omega8 = 1.0;
  if (c->p.rho0 == 0) c->p.rho0 = 1.0;
  double scale = 1.0;
  if (c->p.storage == LBM_STORE_BF16 || c->p.storage == LBM_STORE_F16) {
    scale = c->p.storage_scale > 0 ? c->p.storage_scale
                                   : (c->p.storage == LBM_STORE_F16 ? 4096.0 : 1.0);
    int e;
    if (std::frexp(scale, &e) != 0.5) {
      free_ctx(c);
      return fail(LBM_EINVAL, "storage_scale must be a power of two");
    }
  }
  c->kd = make_consts<double>(c->p, scale);
  c->kf = make_consts<float>(c->p, scale);
  c->esize = storage_bytes(c->p.storage);
  c->csize = c->p.storage == LBM_STORE_F64 ? 8 : 4;
  c->by = 4;
  c->rows = 1;
  auto dev = [&](hipError_t e, const char* what) {
    if (e != hipSuccess) {
      g_err = std::string(what) + ": " + hipGetErrorString(e);
      return false;
    }
    return true;
  };
  const size_t n = (size_t)grid->nx * grid->ny;
  bool ok = dev(hipGetDevice(&c->device), "hipGetDevice") &&
            dev(hipStreamCreateWithFlags(&c->own_stream, hipStreamNonBlocking), "hipStreamCreate");
  c->stream = c->own_stream;
  const Geom g0 = make_geom(c);
  for (int i = 0; ok && i < 2; ++i) {
    ok = dev(hipMalloc(&c->lat[i], 9 * (size_t)g0.plane * c->esize), "hipMalloc lattice") &&
         dev(hipMemset(c->lat[i], 0, 9 * (size_t)g0.plane * c->esize), "hipMemset lattice") &&
         dev(hipMalloc(&c->hist[i], 2 * (size_t)grid->ny * c->csize), "hipMalloc history");
  }
  ok = ok && dev(hipMalloc(&c->ubuf, 2 * n * c->csize), "hipMalloc velocity") &&
       dev(hipMalloc(&c->result, 4 * sizeof(double)), "hipMalloc result") &&
       dev(hipMalloc(&c->rng, 2 * sizeof(unsigned)), "hipMalloc step counter") &&
       dev(hipMemset(c->rng, 0, 2 * sizeof(unsigned)), "hipMemset step counter") &&
       dev(hipEventCreate(&c->ev0), "hipEventCreate") &&
       dev(hipEventCreate(&c->ev1), "hipEventCreate");
  if (ok && solid_mask) {
    bool any = false;
    for (size_t i = 0; i < n; ++i) any |= solid_mask[i] != 0;
    if (any) {
      c->h_solid.assign(solid_mask, solid_mask + n);
      for (auto& v : c->h_solid) v = v ? 1 : 0;
      // followed by two bytes per tile of the two-step kernel (two output rows
      // or more each)
      ok = dev(hipMalloc(&c->d_solid, n + 2 * (size_t)multi_tiles(c, 0)), "hipMalloc mask") &&
           dev(hipMemcpy(c->d_solid, c->h_solid.data(), n, hipMemcpyHostToDevice), "copy mask");
      c->d_fluid = c->d_solid + n;
    }
  }
  if (!ok) {
    free_ctx(c);
    return LBM_EDEVICE;
  }
  rc = configure_tiles(c);
  if (!rc) rc = configure_multi(c);
  if (!rc) rc = init_common<double>(c, nullptr, nullptr, nullptr);
  if (!rc) {
    hipError_t e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) rc = fail(LBM_EDEVICE, hipGetErrorString(e));
  }
  if (rc) {
    free_ctx(c);
    return rc;
  }
  *out = c;
  return LBM_OK;
}

void lbm_destroy(lbm_ctx* c) {
  if (!c) return;
  if (c->stream) hipStreamSynchronize(c->stream);
  free_ctx(c);
}

int lbm_set_stream(lbm_ctx* c, void* s) {
  if (!c) return fail(LBM_EINVAL, "null context");
  HIPCHECK(hipStreamSynchronize(c->stream));
  c->stream = s ? (hipStream_t)s : c->own_stream;
  return LBM_OK;
}

int lbm_init_fields(lbm_ctx* c, const double* rho, const double* ux, const double* uy) {
  if (!c) return fail(LBM_EINVAL, "null context");
  const size_t n = (size_t)c->grid.nx * c->grid.ny;
  double* tmp[3] = {nullptr, nullptr, nullptr};
  const double* src[3] = {rho, ux, uy};
  int rc = LBM_OK;
  for (int i = 0; i < 3 && rc == LBM_OK; ++i) {
    if (!src[i]) continue;
    if (hipMalloc(&tmp[i], n * sizeof(double)) != hipSuccess ||
        hipMemcpy(tmp[i], src[i], n * sizeof(double), hipMemcpyHostToDevice) != hipSuccess)
      rc = fail(LBM_EDEVICE, "upload of initial fields failed");
  }
  if (rc == LBM_OK) rc = init_common<double>(c, tmp[0], tmp[1], tmp[2]);
  hipError_t e = hipStreamSynchronize(c->stream);
  if (rc == LBM_OK && e != hipSuccess) rc = fail(LBM_EDEVICE, hipGetErrorString(e));
  for (int i = 0; i < 3; ++i)
    if (tmp[i]) hipFree(tmp[i]);
  return rc;
}

int lbm_init_fields_device(lbm_ctx* c, const float* rho, const float* ux, const float* uy) {
  if (!c) return fail(LBM_EINVAL, "null context");
  const int rc = init_common<float>(c, rho, ux, uy);
  if (rc) return rc;
  // the caller may release the arrays as soon as this returns
  HIPCHECK(hipStreamSynchronize(c->stream));
  return LBM_OK;
}

int lbm_step(lbm_ctx* c, int64_t n) {
  if (!c) return fail(LBM_EINVAL, "null context");
  if (n < 0) return fail(LBM_EINVAL, "n must be >= 0");
  if (n == 0) return LBM_OK;
  const int K = c->p.check_every;
  hipStream_t st = c->stream;
  if (c->timing) HIPCHECK(hipEventRecord(c->ev0, st));
  int64_t left = n;
  // replay a captured graph of K steps for every aligned block of K steps
  while (left > 0) {
    if (c->t % K == 0 && left >= K && K >= 4) {
      const int par = c->cur;
      if (!c->graph[par]) {
        hipGraph_t gr = nullptr;
        const int64_t t0 = c->t;
        const int cur0 = c->cur;
        const bool chk0 = c->checked;
        HIPCHECK(hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal));
        int launches = 0;
        for (int i = 0; i < K; ++launches) i += enqueue_steps(c, K - i, st);
        c->graph_flips = launches & 1;
        hipError_t e = hipStreamEndCapture(st, &gr);
        c->t = t0;
        c->cur = cur0;
        c->checked = chk0;
        if (e != hipSuccess) return fail(LBM_EDEVICE, hipGetErrorString(e));
        e = hipGraphInstantiate(&c->graph[par], gr, nullptr, nullptr, 0);
        hipGraphDestroy(gr);
        if (e != hipSuccess) {
          c->graph[par] = nullptr;
          return fail(LBM_EDEVICE, hipGetErrorString(e));
        }
      }
      HIPCHECK(hipGraphLaunch(c->graph[par], st));
      c->t += K;
      c->cur ^= c->graph_flips;
      c->checked = true;
      left -= K;
    } else {
      left -= enqueue_steps(c, left, st);
    }
  }
  HIPCHECK(hipGetLastError());
  if (c->timing) {
    HIPCHECK(hipEventRecord(c->ev1, st));
    HIPCHECK(hipEventSynchronize(c->ev1));
    float ms = 0.f;
    HIPCHECK(hipEventElapsedTime(&ms, c->ev0, c->ev1));
    c->last_ms = double(ms) / double(n);
  }
  return LBM_OK;
}

int lbm_set_timing(lbm_ctx* c, int32_t timing) {
  if (!c) return fail(LBM_EINVAL, "null context");
  c->timing = timing != 0;
  return LBM_OK;
}

int lbm_last_step_ms(lbm_ctx* c, double* ms) {
  if (!c || !ms) return fail(LBM_EINVAL, "null argument");
  if (c->last_ms < 0) return fail(LBM_ESTATE, "no timed step yet");
  *ms = c->last_ms;
  return LBM_OK;
}

static int read_result(lbm_ctx* c, double r[4]) {
  if (!c->checked) return fail(LBM_ESTATE, "no check step has run yet");
  HIPCHECK(hipStreamSynchronize(c->stream));
  HIPCHECK(hipMemcpy(r, c->result, 4 * sizeof(double), hipMemcpyDeviceToHost));
  return LBM_OK;
}

int lbm_average_last_two(lbm_ctx* c) {
  if (!c) return fail(LBM_EINVAL, "null context");
  const Geom g = make_geom(c);
  const long long n = 9LL * g.plane;
  HIPCHECK(launch_average(c->p.storage, c->lat[c->cur], c->lat[c->cur ^ 1], n,
                          (double)c->kf.scale, c->hist[c->cur], c->hist[c->cur ^ 1],
                          c->hist[0] ? 2LL * c->grid.ny : 0, c->stream));
  return LBM_OK;
}

int lbm_residual(lbm_ctx* c, double* r) {
  if (!c || !r) return fail(LBM_EINVAL, "null argument");
  double v[4];
  int rc = read_result(c, v);
  if (rc) return rc;
  if (!std::isfinite(v[0]) || !std::isfinite(v[1])) {
    *r = NAN;
    return fail(LBM_EUNSTABLE, "residual is not finite");
  }
  *r = v[1] > 0 ? std::sqrt(v[0] / v[1]) : (v[0] > 0 ? INFINITY : 0.0);
  return LBM_OK;
}

int lbm_mass(lbm_ctx* c, double* m) {
  if (!c || !m) return fail(LBM_EINVAL, "null argument");
  double v[4];
  int rc = read_result(c, v);
  if (rc) return rc;
  size_t fluid = (size_t)c->grid.nx * c->grid.ny;
  if (!c->h_solid.empty()) {
    fluid = 0;
    for (auto s : c->h_solid) fluid += s == 0;
  }
  *m = double(fluid) * c->p.rho0 + v[2];
  if (!std::isfinite(*m)) return fail(LBM_EUNSTABLE, "mass is not finite");
  return LBM_OK;
}

int lbm_guard_count(lbm_ctx* c, int64_t* n) {
  if (!c || !n) return fail(LBM_EINVAL, "null argument");
  double v[4];
  int rc = read_result(c, v);
  if (rc) return rc;
  *n = (int64_t)v[3];
  return LBM_OK;
}

int lbm_steps(lbm_ctx* c, int64_t* n) {
  if (!c || !n) return fail(LBM_EINVAL, "null argument");
  *n = c->t;
  return LBM_OK;
}

int lbm_fields(lbm_ctx* c, double* rho, double* ux, double* uy) {
  if (!c) return fail(LBM_EINVAL, "null context");
  const size_t n = (size_t)c->grid.nx * c->grid.ny;
  double* d = nullptr;
  HIPCHECK(hipMalloc(&d, 3 * n * sizeof(double)));
  int rc = export_common(c, nullptr, nullptr, nullptr, nullptr, d, d + n, d + 2 * n);
  if (rc == LBM_OK) {
    hipError_t e = hipStreamSynchronize(c->stream);
    double* h[3] = {rho, ux, uy};
    for (int i = 0; i < 3 && e == hipSuccess; ++i)
      if (h[i]) e = hipMemcpy(h[i], d + i * n, n * sizeof(double), hipMemcpyDeviceToHost);
    if (e != hipSuccess) rc = fail(LBM_EDEVICE, hipGetErrorString(e));
  }
  hipFree(d);
  return rc;
}

int lbm_fields_device(lbm_ctx* c, float* rho, float* ux, float* uy) {
  if (!c) return fail(LBM_EINVAL, "null context");
  const int rc = export_common(c, nullptr, rho, ux, uy, nullptr, nullptr, nullptr);
  if (rc) return rc;
  HIPCHECK(hipStreamSynchronize(c->stream));
  return LBM_OK;
}

int lbm_populations(lbm_ctx* c, double* f) {
  if (!c || !f) return fail(LBM_EINVAL, "null argument");
  const size_t n = (size_t)c->grid.nx * c->grid.ny;
  double* d = nullptr;
  HIPCHECK(hipMalloc(&d, 9 * n * sizeof(double)));
  int rc = export_common(c, d, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr);
  if (rc == LBM_OK) {
    hipError_t e = hipStreamSynchronize(c->stream);
    if (e == hipSuccess) e = hipMemcpy(f, d, 9 * n * sizeof(double), hipMemcpyDeviceToHost);
    if (e != hipSuccess) rc = fail(LBM_EDEVICE, hipGetErrorString(e));
  }
  hipFree(d);
  return rc;
}

static const char kMagic[8] = {'L', 'B', 'M', 'C', 'K', 'P', 'T', '1'};

int lbm_save(lbm_ctx* c, const char* path) {
  if (!c || !path) return fail(LBM_EINVAL, "null argument");
  HIPCHECK(hipStreamSynchronize(c->stream));
  const size_t n = (size_t)c->grid.nx * c->grid.ny;
  const Geom g = make_geom(c);
  std::vector<char> lat(9 * (size_t)g.plane * c->esize), hist(2 * (size_t)c->grid.ny * c->csize);
  HIPCHECK(hipMemcpy(lat.data(), c->lat[c->cur], lat.size(), hipMemcpyDeviceToHost));
  HIPCHECK(hipMemcpy(hist.data(), c->hist[c->cur], hist.size(), hipMemcpyDeviceToHost));
  std::vector<char> ub(2 * n * c->csize);
  HIPCHECK(hipMemcpy(ub.data(), c->ubuf, ub.size(), hipMemcpyDeviceToHost));
  FILE* fp = std::fopen(path, "wb");
  if (!fp) return fail(LBM_EINVAL, std::string("cannot open ") + path);
  int32_t hdr[8] = {c->grid.nx, c->grid.ny, c->p.storage, (int32_t)c->esize, 0, 0, 0, 0};
  int64_t t = c->t;
  bool ok = std::fwrite(kMagic, 1, 8, fp) == 8 && std::fwrite(hdr, sizeof hdr, 1, fp) == 1 &&
            std::fwrite(&t, sizeof t, 1, fp) == 1 &&
            std::fwrite(lat.data(), 1, lat.size(), fp) == lat.size() &&
            std::fwrite(hist.data(), 1, hist.size(), fp) == hist.size() &&
            std::fwrite(ub.data(), 1, ub.size(), fp) == ub.size();
  ok = (std::fclose(fp) == 0) && ok;
  return ok ? LBM_OK : fail(LBM_EDEVICE, "write failed");
}

int lbm_load(lbm_ctx* c, const char* path) {
  if (!c || !path) return fail(LBM_EINVAL, "null argument");
  FILE* fp = std::fopen(path, "rb");
  if (!fp) return fail(LBM_EINVAL, std::string("cannot open ") + path);
  char mg[8];
  int32_t hdr[8];
  int64_t t;
  const size_t n = (size_t)c->grid.nx * c->grid.ny;
  const Geom g = make_geom(c);
  std::vector<char> lat(9 * (size_t)g.plane * c->esize), hist(2 * (size_t)c->grid.ny * c->csize),
      ub(2 * n * c->csize);
  bool ok = std::fread(mg, 1, 8, fp) == 8 && std::memcmp(mg, kMagic, 8) == 0 &&
            std::fread(hdr, sizeof hdr, 1, fp) == 1 && hdr[0] == c->grid.nx &&
            hdr[1] == c->grid.ny && hdr[2] == c->p.storage && std::fread(&t, sizeof t, 1, fp) == 1 &&
            std::fread(lat.data(), 1, lat.size(), fp) == lat.size() &&
            std::fread(hist.data(), 1, hist.size(), fp) == hist.size() &&
            std::fread(ub.data(), 1, ub.size(), fp) == ub.size();
  std::fclose(fp);
  if (!ok) return fail(LBM_EINVAL, "checkpoint does not match this lattice");
  HIPCHECK(hipStreamSynchronize(c->stream));
  HIPCHECK(hipMemcpy(c->lat[0], lat.data(), lat.size(), hipMemcpyHostToDevice));
  HIPCHECK(hipMemcpy(c->lat[1], lat.data(), lat.size(), hipMemcpyHostToDevice));
  HIPCHECK(hipMemcpy(c->hist[0], hist.data(), hist.size(), hipMemcpyHostToDevice));
  HIPCHECK(hipMemcpy(c->hist[1], hist.data(), hist.size(), hipMemcpyHostToDevice));
  HIPCHECK(hipMemcpy(c->ubuf, ub.data(), ub.size(), hipMemcpyHostToDevice));
  c->cur = 0;
  c->t = t;
  c->checked = false;
  for (int i = 0; i < 2; ++i)
    if (c->graph[i]) {
      hipGraphExecDestroy(c->graph[i]);
      c->graph[i] = nullptr;
    }
  const int rc = set_rng_counter(c);
  if (rc) return rc;
  HIPCHECK(hipStreamSynchronize(c->stream));
  return LBM_OK;
}


int lbm_set_storage(lbm_ctx* c, int32_t storage, double storage_scale) {
  if (!c) return fail(LBM_EINVAL, "null context");
  if (storage < LBM_STORE_F64 || storage > LBM_STORE_F16) return fail(LBM_EINVAL, "unknown storage");
  double scale = 1.0;
  if (storage == LBM_STORE_BF16 || storage == LBM_STORE_F16) {
    scale = storage_scale > 0 ? storage_scale : (storage == LBM_STORE_F16 ? 4096.0 : 1.0);
    int e;
    if (std::frexp(scale, &e) != 0.5) return fail(LBM_EINVAL, "storage_scale must be a power of two");
  }
  HIPCHECK(hipStreamSynchronize(c->stream));
  const Geom g1 = make_geom(c);
  const int s1 = c->p.storage;
  const double inv1 = s1 == LBM_STORE_F64 ? double(c->kd.inv_scale) : double(c->kf.inv_scale);
  const size_t esize2 = storage_bytes(storage), csize2 = storage == LBM_STORE_F64 ? 8 : 4;
  {
    const int rc = check_lattice_bytes(c->grid.nx, c->grid.ny, esize2);
    if (rc) return rc;
  }
  const Geom g2 = make_geom_for(c->grid.nx, c->grid.ny, c->grid.side, esize2);
  const size_t np = (size_t)c->grid.nx * c->grid.ny;
  void* lat2[2] = {nullptr, nullptr};
  void* hist2[2] = {nullptr, nullptr};
  void* ubuf2 = nullptr;
  bool ok = true;
  for (int i = 0; ok && i < 2; ++i)
    ok = hipMalloc(&lat2[i], 9 * (size_t)g2.plane * esize2) == hipSuccess &&
         hipMemset(lat2[i], 0, 9 * (size_t)g2.plane * esize2) == hipSuccess &&
         hipMalloc(&hist2[i], 2 * (size_t)c->grid.ny * csize2) == hipSuccess;
  ok = ok && hipMalloc(&ubuf2, 2 * np * csize2) == hipSuccess;
  if (!ok) {
    for (int i = 0; i < 2; ++i) {
      hipFree(lat2[i]);
      hipFree(hist2[i]);
    }
    hipFree(ubuf2);
    return fail(LBM_ENOMEM, "allocation for the new storage failed");
  }
  const long long nf = (long long)(c->grid.nx + 2) * (c->grid.ny + 2);
  for (int i = 0; i < 2; ++i) {
    hipLaunchKernelGGL(convert_lattice_kernel, dim3(int((nf + 255) / 256)), dim3(256), 0, c->stream,
                       c->lat[i], s1, g1, inv1, lat2[i], (int)storage, g2, scale);
    const long long nh = 2LL * c->grid.ny;
    hipLaunchKernelGGL(convert_values_kernel, dim3(int((nh + 255) / 256)), dim3(256), 0, c->stream,
                       c->hist[i], int(c->csize == 8), hist2[i], int(csize2 == 8), nh);
  }
  hipLaunchKernelGGL(convert_values_kernel, dim3(int((2 * np + 255) / 256)), dim3(256), 0,
                     c->stream, c->ubuf, int(c->csize == 8), ubuf2, int(csize2 == 8),
                     (long long)(2 * np));
  HIPCHECK(hipGetLastError());
  HIPCHECK(hipStreamSynchronize(c->stream));
  for (int i = 0; i < 2; ++i) {
    hipFree(c->lat[i]);
    hipFree(c->hist[i]);
    c->lat[i] = lat2[i];
    c->hist[i] = hist2[i];
  }
  hipFree(c->ubuf);
  c->ubuf = ubuf2;
  c->p.storage = storage;
  c->p.storage_scale = storage_scale;
  c->esize = esize2;
  c->csize = csize2;
  c->kd = make_consts<double>(c->p, scale);
  c->kf = make_consts<float>(c->p, scale);
  for (int i = 0; i < 2; ++i)
    if (c->graph[i]) {
      hipGraphExecDestroy(c->graph[i]);
      c->graph[i] = nullptr;
    }
  const int rc = configure_multi(c);
  return rc ? rc : apply_force(c);
}

int lbm_set_force_field(lbm_ctx* c, const double* fx, const double* fy) {
  if (!c) return fail(LBM_EINVAL, "null context");
  if ((fx == nullptr) != (fy == nullptr))
    return fail(LBM_EINVAL, "force field: give both components or neither");
  const size_t n = (size_t)c->grid.nx * c->grid.ny;
  if (fx)
    for (size_t i = 0; i < n; ++i)
      if (!std::isfinite(fx[i]) || !std::isfinite(fy[i]))
        return fail(LBM_EINVAL, "force field holds a non-finite value");
  HIPCHECK(hipStreamSynchronize(c->stream));
  c->h_force.clear();
  if (fx) {
    c->h_force.assign(fx, fx + n);
    c->h_force.insert(c->h_force.end(), fy, fy + n);
  }
  for (int i = 0; i < 2; ++i)
    if (c->graph[i]) {
      hipGraphExecDestroy(c->graph[i]);
      c->graph[i] = nullptr;
    }
  return apply_force(c);
}

int lbm_set_launch(lbm_ctx* c, int32_t by, int32_t rows) {
  if (!c) return fail(LBM_EINVAL, "null context");
  bool known = false;
  for (int i = 0; i < kNumShapes; ++i) known |= kShapes[i].by == by && kShapes[i].rows == rows;
  if (!known) return fail(LBM_EINVAL, "unsupported launch shape");
  HIPCHECK(hipStreamSynchronize(c->stream));
  c->by = by;
  c->rows = rows;
  const int rc = configure_tiles(c);
  return rc ? rc : configure_multi(c);
}

int lbm_get_launch(lbm_ctx* c, int32_t* by, int32_t* rows) {
  if (!c || !by || !rows) return fail(LBM_EINVAL, "null argument");
  *by = c->by;
  *rows = c->rows;
  return LBM_OK;
}

}  // extern "C"
