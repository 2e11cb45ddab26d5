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
void launch(const SmallArgs &g, hipStream_t stream) {
  const unsigned tiles = (unsigned)g.tiles;
  hipLaunchKernelGGL(small_gemm_kernel<SH>, dim3(tiles * (unsigned)g.runs), dim3(NT), SH::LDS, stream, g);
  if (g.runs > 1 && hipPeekAtLastError() == hipSuccess)
    hipLaunchKernelGGL(small_sum_kernel<SH>, dim3(tiles * (unsigned)(SH::TM * SH::TN / 1024)), dim3(NT), 0, stream, g);
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
  return e;
}

void small_launch(int shape, const SmallArgs &g, int cus, hipStream_t stream) {
  const bool alone = g.tiles * g.runs <= cus;          // a CU for every workgroup
  switch (shape) {
    case SMALL_BF16_SKINNY: return alone ? launch<RingSkinnyDeep>(g, stream) : launch<RingSkinny>(g, stream);
    case SMALL_BF16_HALF: return launch<RingHalf>(g, stream);
    case SMALL_BF16: return alone ? launch<RingDeep>(g, stream) : launch<RingPair>(g, stream);
    case SMALL_F32_TINY: return launch<SmallF32Tiny>(g, stream);
    default: return launch<SmallF32>(g, stream);
  }
}

}  // namespace dmm
