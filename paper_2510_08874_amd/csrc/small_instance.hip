// The kernels for small and skinny products (small_kernel.hpp), every shape, and the host
// functions that launch them.
#include "gemm_launch.hpp"
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
  hipError_t e = allow<SmallBf16Skinny>();
  if (e == hipSuccess) e = allow<SmallBf16Half>();
  if (e == hipSuccess) e = allow<SmallBf16>();
  if (e == hipSuccess) e = allow<SmallF32Tiny>();
  if (e == hipSuccess) e = allow<SmallF32>();
  return e;
}

void small_launch(int shape, const SmallArgs &g, hipStream_t stream) {
  switch (shape) {
    case SMALL_BF16_SKINNY: return launch<SmallBf16Skinny>(g, stream);
    case SMALL_BF16_HALF: return launch<SmallBf16Half>(g, stream);
    case SMALL_BF16: return launch<SmallBf16>(g, stream);
    case SMALL_F32_TINY: return launch<SmallF32Tiny>(g, stream);
    default: return launch<SmallF32>(g, stream);
  }
}

}  // namespace dmm
