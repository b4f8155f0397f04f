// Several time steps of the fused D2Q9 method in one launch (plain steps of
// the default kernel).
#pragma once

// One step reads and writes every population once, so a lattice that does not
// fit the caches is bound by memory and a small one by the launch and one
// memory round trip per step.  Here a block advances its tile T steps on
// chip.  The density gradient reaches one node further than the streaming, so
// a step needs its sources on a ring of two: the block starts from a region
// with a ring of 2 T - 1 nodes around the tile (64 columns, one per lane, and
// NR = NW * RPW rows, RPW per wavefront) and each step gives up two more.  The
// lattice between the steps lives in LDS with the layout of the lattice in
// memory: boundary nodes write their bounce-back values into the slots their
// neighbours pull from, nodes beyond a non-periodic side are mirrored onto
// the edge node (for the density only), across a periodic side the region
// simply continues.  Arithmetic, storage rounding (values go through the
// storage type between the steps) and the seeds of the stochastic rounding
// are those of the single step, so any mix of both gives the same bits as long
// as the densities are finite (the single step takes a density of +Inf for a
// solid node, here the mask decides; only a state that has diverged has one).
//
// Bound: vector instructions.  4096^2 FP32 issues them in 77 % of its cycles,
// 225 per 64 nodes of each row that a step collides, the ring's rows included;
// that is 269 per 64 nodes of the lattice and step (the single step with its
// halo work 283).  A pair moves 1.36 GB to and from HBM, two single steps 2.43
// GB.  1024^2 FP32: 75 % of the time, 314 instructions against 286, 79 MB
// against 154 MB.  Non-temporal stores, which the single step uses beyond the
// last-level cache, are slower here (4096^2 from rest 151 -> 184 us per step:
// the tiles' rows do not start on cache lines and neighbours' partial lines
// merge in L2).  Three or four steps
// save traffic that no longer bounds a large lattice and add ring, and in a
// small one a step inside the block costs 2.5-3 us at four wavefronts per SIMD
// (32^2 FP64 2.75 us per step in pairs, 2.9-6.0 in threes and fours; 256^2 FP32
// 2.68, 2.44-3.75).

#include "lbm_kernels.h"

namespace lbmk {

// Output tile of a launch shape.
template <int NW, int RPW, int T>
struct MultiTile {
  static constexpr int H = 2 * T - 1;             // ring of the region
  static constexpr int NR = NW * RPW;             // region rows
  static constexpr int TXO = kLanes - 2 * H, TYO = NR - 2 * H;
  static_assert(TYO > 0 && TXO > 0, "region");
};

template <class S, int NW, int RPW, int T, bool OBST, bool OUTL, bool CL, bool INT>
__device__ __forceinline__ void multi_tile(const typename S::T* __restrict__ fa,
                                           typename S::T* __restrict__ fb, const StepArgs& args,
                                           const Consts<typename S::C>& k, int tile,
                                           typename S::T (*s_f)[NW * RPW - 2][kLanes],
                                           typename S::C (*s_rho)[kLanes + 2]) {
  using C = typename S::C;
  using M = MultiTile<NW, RPW, T>;
  constexpr int H = M::H, NR = M::NR;
  const C SENT = C(HUGE_VALF);
  const Geom& g = args.g;
  const int lane = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(int(threadIdx.y));
  const int xb = tile % args.tiles_x * M::TXO - H;   // lattice column of lane 0
  const int yb = tile / args.tiles_x * M::TYO - H;   // lattice row of region row 0
  const int x = xb + lane;
  const bool px = periodic_x<CL>(g), py = periodic_y<CL>(g);
  const int gx = INT ? x : col_of<CL>(g, x);
  const bool inx = INT || px || (x >= 0 && x < g.nx);
  const C* hist_in = static_cast<const C*>(args.hist_in);
  const C* force = static_cast<const C*>(args.force);
  const bool has_force = args.has_force != 0;
  const int np = g.nx * g.ny;

  uint32_t rng_step = 0;
  if constexpr (S::kSR) {
    rng_step = __builtin_amdgcn_readfirstlane(
        __hip_atomic_load(args.rng + args.rng_slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    if (tile == 0 && lane == 0 && w == 0)
      __hip_atomic_store(args.rng + (args.rng_slot ^ 1), rng_step + uint32_t(T), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
  }

  // ---- the region from memory: all loads before any use
  C d[RPW][9];
  bool sol[RPW];
  int gy[RPW];
#pragma unroll
  for (int q = 0; q < RPW; ++q) {
    gy[q] = INT ? yb + w * RPW + q : row_of<CL>(g, yb + w * RPW + q);
    pull9<S>(fa, g, k, gx, gy[q], d[q]);
    sol[q] = OBST && !INT && args.solid[gy[q] * g.nx + gx];
  }
  __builtin_amdgcn_sched_barrier(0);
  // the outlet column's velocity per row (in LDS: one node per row has one,
  // registers for it in every lane cost FP64 spills)
  C(*s_uv)[2] = reinterpret_cast<C(*)[2]>(s_rho + NR);
  if (OUTL && !INT) {
#pragma unroll
    for (int q = 0; q < RPW; ++q)
      if (!sol[q] && gx == g.nx - 1) {
        C us, vs;
        outlet_links<S>(fa, g, k, has_force, force, hist_in, gy[q], d[q], us, vs);
        s_uv[w * RPW + q][0] = us;
        s_uv[w * RPW + q][1] = vs;
      }
  }
  // rows with a solid node: the others and their neighbours take the density
  // gradient without its tests (uniform per wavefront)
  int* s_any = reinterpret_cast<int*>(s_uv + NR);
#pragma unroll
  for (int q = 0; q < RPW; ++q) {
    s_rho[w * RPW + q][lane + 1] = sol[q] ? SENT : sum9<C>(d[q]);
    if (OBST && !INT) {
      const bool any = __builtin_amdgcn_ballot_w64(sol[q]) != 0;
      if (lane == 0) s_any[w * RPW + q] = any;
    }
  }
  __syncthreads();
  bool near[RPW];
#pragma unroll
  for (int q = 0; q < RPW; ++q) {
    near[q] = false;
    if (OBST && !INT) {
      const int r = w * RPW + q, r0 = r < 1 ? 0 : r - 1, r1 = r > NR - 2 ? NR - 1 : r + 1;
      near[q] = __builtin_amdgcn_readfirstlane(s_any[r0] | s_any[r] | s_any[r1]) != 0;
    }
  }

#pragma unroll
  for (int t = 0; t < T; ++t) {
    const bool last = t == T - 1;
    // ---- collide the rows this step still holds; all but the last step
    // write to LDS, the last one to memory
#pragma unroll
    for (int q = 0; q < RPW; ++q) {
      const int r = w * RPW + q, y = yb + r;
      if (r < 1 + 2 * t || r > NR - 2 - 2 * t) continue;   // uniform
      if (!INT && !py && (y < 0 || y >= g.ny)) continue;   // uniform
      const int ly = gy[q];
      bool on = inx;
      if (last) on = lane >= H && lane < kLanes - H && x < g.nx && y < g.ny;
      if (OBST && !INT) on = on && !sol[q];
      if (!on) continue;
      C drx, dry;
      unsigned solid_src = 0;
      if (OBST && !INT && near[q])
        density_gradient<C, true>(s_rho, r, lane + 1, uflag(k.stencil), drx, dry, solid_src);
      else
        density_gradient<C, false>(s_rho, r, lane + 1, uflag(k.stencil), drx, dry, solid_src);
      C fx = k.fx, fy = k.fy;
      if (has_force) {
        fx = force[ly * g.nx + gx];
        fy = force[np + ly * g.nx + gx];
      }
      C drho, ux, uy;
      collide<C, 0>(d[q], drx, dry, k, fx, fy, drho, ux, uy);
      if (OBST && !INT && near[q]) solid_src &= ~side_links<CL>(g, gx, ly);
      if (last) {
        double acc[4];
        finish_node<S, kPlain>(fb, args, k, d[q], gidx(g, x, y), y * g.nx + x, drho, ux, uy,
                                    0, acc, rng_step + uint32_t(t));
        if (!INT) {
          side_slots<S, CL>(fb, g, k, x, y, xb + H == 0, xb + kLanes - H >= g.nx, d[q]);
          if (OBST && near[q]) solid_slots<S>(fb, g, k, x, y, d[q], solid_src);
        }
        if (OUTL && !INT && x == g.nx - 1) {
          C* ho = static_cast<C*>(args.hist_out);
          ho[y] = s_uv[r][0];
          ho[g.ny + y] = s_uv[r][1];
        }
      } else {
        if constexpr (S::kSR) {
          const uint32_t h = hash32(uint32_t(gidx(g, gx, ly)) * 0x9E3779B1u ^
                                    hash32(rng_step + uint32_t(t)));
#pragma unroll
          for (int a = 0; a < 9; ++a)
            s_f[a][r - 1][lane] = S::enc_sr(d[q][a], k.scale, h + uint32_t(a) * 0x9E3779B9u);
        } else {
#pragma unroll
          for (int a = 0; a < 9; ++a) s_f[a][r - 1][lane] = S::enc(d[q][a], k.scale);
        }
        if (!INT) {
          // slots within the stored rows and columns (the others are beyond
          // what the next step pulls)
          auto put = [&](bool p, int a, int sx, int sy, C v) {
            const int rr = r - 1 + sy, cc = lane + sx;
            if (p && rr >= 0 && rr < NR - 2 && cc >= 0 && cc < kLanes)
              s_f[a][rr][cc] = S::enc(v, k.scale);
          };
          side_slots_to<C, CL, false>(g, k, gx, ly, xb <= 0, xb + kLanes >= g.nx, d[q], put);
          if (OBST && near[q]) {
#pragma unroll
            for (int a = 1; a < 9; ++a)
              put((solid_src >> a) & 1u, a, -ex_of(a), -ey_of(a), d[q][opp_of(a)]);
          }
        }
      }
    }
    if (last) break;
    __syncthreads();
    // ---- pull the next step's populations from LDS (the rows and columns
    // its collisions and their density ring need; nodes beyond a side from
    // the edge node)
    const int cc = INT ? lane : (px ? lane : gx - xb);
    const int c = cc < 1 ? 1 : (cc > kLanes - 2 ? kLanes - 2 : cc);
#pragma unroll
    for (int q = 0; q < RPW; ++q) {
      const int r = w * RPW + q;
      if (r < 2 + 2 * t || r > NR - 3 - 2 * t) continue;   // uniform
      const int rr = INT || py ? r : gy[q] - yb;
      const int row = rr < 2 ? 2 : (rr > NR - 3 ? NR - 3 : rr);
      auto pull = [&](int col, C f[9]) {
#pragma unroll
        for (int a = 0; a < 9; ++a)
          f[a] = S::dec(s_f[a][row - 1 - ey_of(a)][col - ex_of(a)], k.inv_scale);
      };
      pull(c, d[q]);
      if (OUTL && !INT && !sol[q] && gx == g.nx - 1) {
        C d2[9];
        const int c2 = c - 1 < 1 ? 1 : c - 1;
        pull(c2, d2);
        const int fi = gy[q] * g.nx + g.nx - 2;
        const C ffx = force[fi], ffy = force[np + fi];
        C us, vs;
        outlet_complete<C>(d2, g, k, has_force ? ffx : k.fx, has_force ? ffy : k.fy, s_uv[r][0],
                           s_uv[r][1], gy[q], d[q], us, vs);
        s_uv[r][0] = us;
        s_uv[r][1] = vs;
      }
      s_rho[r][lane + 1] = sol[q] ? SENT : sum9<C>(d[q]);
    }
    __syncthreads();
  }
}

// Wavefronts per SIMD the registers are limited for: FP64 with two rows per
// wavefront needs 135 without a limit, which leaves room for one block.
template <class S, int NW, int RPW>
constexpr int multi_waves() {
  return sizeof(typename S::C) == 8 && RPW == 2 ? 4 : 1;
}

// LDS bytes of a block: populations between the steps, densities, outlet
// velocities, rows with solid nodes.
template <class S, int NW, int RPW>
constexpr size_t multi_lds() {
  constexpr int NR = NW * RPW;
  return 9 * sizeof(typename S::T) * (NR - 2) * kLanes +
         sizeof(typename S::C) * NR * (kLanes + 2 + 2) + sizeof(int) * NR;
}

template <class S, int NW, int RPW, int T, bool OBST, bool OUTL, bool CL>
__global__ __launch_bounds__(kLanes* NW, (multi_waves<S, NW, RPW>()))
void multi_kernel(const typename S::T* __restrict__ fa, typename S::T* __restrict__ fb,
                  const StepArgs args, const uint8_t* __restrict__ fluid,
                  const Consts<typename S::C> k) {
  using M = MultiTile<NW, RPW, T>;
  extern __shared__ __align__(16) char smem[];
  using F = typename S::T[NW * RPW - 2][kLanes];
  using R = typename S::C[kLanes + 2];
  F* s_f = reinterpret_cast<F*>(smem);
  R* s_rho = reinterpret_cast<R*>(smem + 9 * sizeof(F));
  const int tile = xcd_tile(blockIdx.x, args.ntiles);
  // a region that keeps one node away from every side and holds no solid node
  // (fluid) has no boundary node
  const int x0 = tile % args.tiles_x * M::TXO - M::H, y0 = tile / args.tiles_x * M::TYO - M::H;
  if (x0 >= 1 && x0 + kLanes <= args.g.nx - 1 && y0 >= 1 && y0 + M::NR <= args.g.ny - 1 &&
      (!OBST || fluid[tile])) {
    multi_tile<S, NW, RPW, T, OBST, OUTL, CL, true>(fa, fb, args, k, tile, s_f, s_rho);
    return;
  }
  multi_tile<S, NW, RPW, T, OBST, OUTL, CL, false>(fa, fb, args, k, tile, s_f, s_rho);
}

// Launch shapes of the two-step kernel (shape index of launch_multi): NW x RPW
// wavefronts and rows per wavefront.
struct MultiShape {
  int nw, rpw;
};
constexpr MultiShape kMultiShapes[] = {{8, 1}, {12, 1}, {16, 1}, {8, 2}, {8, 4}};
constexpr int kMultiSteps = 2;
constexpr int kNumMultiShapes = sizeof(kMultiShapes) / sizeof(kMultiShapes[0]);

// kMultiSteps plain steps of the default kernel for storage code ST; a.tiles_x
// and a.ntiles describe the output tiles of the shape, fluid marks the tiles
// without solid nodes (lattices with a mask).  Returns false when the shape
// needs more LDS than a compute unit has.  Defined in lbm_multi.hip.
template <int ST>
bool launch_multi(int shape, const void* src, void* dst, const StepArgs& a,
                  const uint8_t* fluid, const void* consts, hipStream_t st);

}  // namespace lbmk
