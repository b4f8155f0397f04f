// Multi-step kernels of one storage type.  The build compiles this file once
// per storage, with LBM_STEP_STORAGE set to an LBM_STORE_* code.
#include "lbm_multi.h"

#if !defined(LBM_STEP_STORAGE)
#error "compile with -DLBM_STEP_STORAGE=<0..3>"
#endif

namespace lbmk {

namespace {

template <int ST>
struct StorageOf;
template <>
struct StorageOf<0> { using type = StoreF64; };
template <>
struct StorageOf<1> { using type = StoreF32; };
template <>
struct StorageOf<2> { using type = StoreBF16; };
template <>
struct StorageOf<3> { using type = StoreF16; };

using S = StorageOf<LBM_STEP_STORAGE>::type;
using T = S::T;
using C = S::C;

template <int NW, int RPW, bool OBST, bool OUTL, bool CL>
bool go_kernel(const void* src, void* dst, const StepArgs& a, const uint8_t* fluid,
               const Consts<C>& k, hipStream_t st) {
  constexpr size_t lds = multi_lds<S, NW, RPW>();
  if constexpr (lds > 160 * 1024) return false;
  auto* fn = multi_kernel<S, NW, RPW, kMultiSteps, OBST, OUTL, CL>;
  if (lds > 64 * 1024 &&
      hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) {
    (void)hipGetLastError();   // (handled: the caller steps singly)
    return false;
  }
  hipLaunchKernelGGL(fn, dim3(a.ntiles), dim3(kLanes, NW), lds, st, (const T*)src, (T*)dst, a,
                     fluid, k);
  return true;
}

template <int NW, int RPW>
bool go(const void* src, void* dst, const StepArgs& a, const uint8_t* fluid, const Consts<C>& k,
        hipStream_t st) {
  const bool obst = a.solid != nullptr;
  const bool outl = side_of(a.g, kE) == kOutlet;
  bool closed = true;
  for (int sd = 0; sd < 4; ++sd)
    closed = closed && (side_of(a.g, sd) == kWall || side_of(a.g, sd) == kLid);
  if (closed && obst) return go_kernel<NW, RPW, true, false, true>(src, dst, a, fluid, k, st);
  if (closed) return go_kernel<NW, RPW, false, false, true>(src, dst, a, fluid, k, st);
  if (obst && outl) return go_kernel<NW, RPW, true, true, false>(src, dst, a, fluid, k, st);
  if (obst) return go_kernel<NW, RPW, true, false, false>(src, dst, a, fluid, k, st);
  if (outl) return go_kernel<NW, RPW, false, true, false>(src, dst, a, fluid, k, st);
  return go_kernel<NW, RPW, false, false, false>(src, dst, a, fluid, k, st);
}

}  // namespace

template <>
bool launch_multi<LBM_STEP_STORAGE>(int shape, const void* src, void* dst, const StepArgs& a,
                                    const uint8_t* fluid, const void* consts, hipStream_t st) {
  const Consts<C>& k = *static_cast<const Consts<C>*>(consts);
  switch (shape) {
    case 0: return go<8, 1>(src, dst, a, fluid, k, st);
    case 1: return go<12, 1>(src, dst, a, fluid, k, st);
    case 2: return go<16, 1>(src, dst, a, fluid, k, st);
    case 3: return go<8, 2>(src, dst, a, fluid, k, st);
    default:   // (FP64 has no registers for four rows per wavefront)
      if constexpr (sizeof(C) == 4) return go<8, 4>(src, dst, a, fluid, k, st);
      return false;
  }
}

}  // namespace lbmk
