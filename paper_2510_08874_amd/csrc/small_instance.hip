// The kernels for small and skinny products (small_kernel.hpp), every shape, and the host
// functions that launch them.
#include "gemm_launch.hpp"
#include "ring_kernel.hpp"
#include "small_kernel.hpp"

namespace dmm {
namespace {

template <class SH>
hipError_t allow() {
  return hipFuncSetAttribute((const void *)small_gemm_kernel<SH>, hipFuncAttributeMaxDynamicSharedMemorySize, SH::LDS);
}

template <class SH>
bool launch(hipEvent_t behind, const SmallArgs &g, hipStream_t stream) {
  const unsigned tiles = (unsigned)g.tiles;
  const bool sum = g.runs > 1;
  const bool marked = launch_behind(sum ? nullptr : behind, small_gemm_kernel<SH>, tiles * (unsigned)g.runs, NT, SH::LDS, stream, g);
  if (!sum || hipPeekAtLastError() != hipSuccess) return marked;
  return launch_behind(behind, small_sum_kernel<SH>, tiles * (unsigned)(SH::TM * SH::TN / 1024), NT, 0, stream, g);
}

}  // namespace

hipError_t small_allow_lds() {
  hipError_t e = allow<RingSkinny>();
  if (e == hipSuccess) e = allow<RingSkinnyDeep>();
  if (e == hipSuccess) e = allow<RingHalf>();
  if (e == hipSuccess) e = allow<RingDeep>();
  if (e == hipSuccess) e = allow<RingPair>();
  if (e == hipSuccess) e = allow<SmallF32Tiny>();
  if (e == hipSuccess) e = allow<SmallF32>();
  if (e == hipSuccess) e = allow<SmallF32Split>();
  return e;
}

bool small_launch(hipEvent_t behind, int shape, const SmallArgs &g, int cus, hipStream_t stream) {
  const bool alone = g.tiles * g.runs <= cus;          // a CU for every workgroup
  switch (shape) {
    case SMALL_BF16_SKINNY: return alone ? launch<RingSkinnyDeep>(behind, g, stream) : launch<RingSkinny>(behind, g, stream);
    case SMALL_BF16_HALF: return launch<RingHalf>(behind, g, stream);
    case SMALL_BF16: return alone ? launch<RingDeep>(behind, g, stream) : launch<RingPair>(behind, g, stream);
    case SMALL_F32_SPLIT: return launch<SmallF32Split>(behind, g, stream);
    case SMALL_F32_TINY: return launch<SmallF32Tiny>(behind, g, stream);
    default: return launch<SmallF32>(behind, g, stream);
  }
}

}  // namespace dmm
