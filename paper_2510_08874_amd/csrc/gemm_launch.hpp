// Host-side doors to the grouped-GEMM kernels.  Every instantiation of the kernels is compiled
// in an object file of its own (gemm_instance.hip, once per value of DMM_INSTANCE), so that they
// compile side by side; the rest of the library reaches them through these functions only.
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <tuple>

#include "gemm_kernel.hpp"

namespace dmm {

// A launch with the event (none: nullptr) that is to stand for its end.  Recorded by the launch itself an event costs the
// stream 0.2 us, by a call behind it 3 us (a host that waits for each call pays for it: 19 us instead of 17 for 256^3 fp32,
// 24 instead of 20 with a new plan).  True: it has been recorded; false: the runtime would not (it
// refuses such launches without saying so in a capture, where no event is given), or no event was given; the kernel
// has been launched, and the event is the caller's to record.  (launch_behind_only: nothing has been launched then.)
template <class... P, class... A>
bool launch_behind_only(hipEvent_t behind, void (*kernel)(P...), unsigned grid, unsigned block, size_t lds, hipStream_t stream, A... args) {
  std::tuple<P...> values(args...);
  void *at[sizeof...(P)];
  std::apply([&at](P &...v) { int i = 0; ((at[i++] = (void *)&v), ...); }, values);
  if (hipExtLaunchKernel((const void *)kernel, dim3(grid), dim3(block), at, lds, stream, nullptr, behind, 0) == hipSuccess) return true;
  (void)hipGetLastError();
  return false;
}
template <class... P, class... A>
bool launch_behind(hipEvent_t behind, void (*kernel)(P...), unsigned grid, unsigned block, size_t lds, hipStream_t stream, A... args) {
  if (behind && launch_behind_only(behind, kernel, grid, block, lds, stream, args...)) return true;
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(block), lds, stream, args...);
  return false;
}

// Per instantiation: allow the kernel its dynamic LDS on the current device; launch it.
#define DMM_DECLARE_GEMM(n)                                                                              \
  hipError_t gemm_allow_lds_##n();                                                                      \
  bool gemm_launch_##n(hipEvent_t behind, unsigned grid, hipStream_t stream, const ItemDev *items, const SegDev *segs,     \
                       const RedSrc *red, int n_items);
DMM_DECLARE_GEMM(0)   // bf16
DMM_DECLARE_GEMM(1)   // fp32
DMM_DECLARE_GEMM(2)   // bf16, epilogue that can add other replicas' partial sums
DMM_DECLARE_GEMM(3)   // fp32, the same
#undef DMM_DECLARE_GEMM

#define DMM_DECLARE_COMP(n)                                                                              \
  hipError_t gemm_allow_lds_##n();                                                                      \
  bool gemm_launch_##n(hipEvent_t behind, unsigned grid, hipStream_t stream, const CompItemDev *items, const PieceDev *a,  \
                       const PieceDev *b, const PieceDev *c, const int32_t *klen);
DMM_DECLARE_COMP(4)   // merged macro-tiles, bf16
DMM_DECLARE_COMP(5)   // merged macro-tiles, fp32
#undef DMM_DECLARE_COMP

// es = bytes per operand element (2 or 4); fuse = the instantiation whose epilogue can add partial sums
inline bool launch_grouped_gemm(hipEvent_t behind, int es, bool fuse, unsigned grid, hipStream_t stream, const ItemDev *items,
                                const SegDev *segs, const RedSrc *red, int n_items) {
  if (es == 2 && !fuse) return gemm_launch_0(behind, grid, stream, items, segs, red, n_items);
  if (es == 2) return gemm_launch_2(behind, grid, stream, items, segs, red, n_items);
  if (!fuse) return gemm_launch_1(behind, grid, stream, items, segs, red, n_items);
  return gemm_launch_3(behind, grid, stream, items, segs, red, n_items);
}

inline bool launch_grouped_gemm_comp(hipEvent_t behind, int es, unsigned grid, hipStream_t stream, const CompItemDev *items,
                                     const PieceDev *a, const PieceDev *b, const PieceDev *c, const int32_t *klen) {
  if (es == 2) return gemm_launch_4(behind, grid, stream, items, a, b, c, klen);
  return gemm_launch_5(behind, grid, stream, items, a, b, c, klen);
}

// The kernels for small and skinny products (small_kernel.hpp), by shape.
struct SmallArgs;
enum { SMALL_BF16_SKINNY, SMALL_BF16_HALF, SMALL_BF16, SMALL_F32_TINY, SMALL_F32, SMALL_F32_SPLIT, SMALL_SHAPES };
hipError_t small_allow_lds();
bool small_launch(hipEvent_t behind, int shape, const SmallArgs &g, int cus, hipStream_t stream);   // the product, and the sum of its partial tiles

}  // namespace dmm
