// Gathers a partitioned bf16 operand into dense rows (gfx950, device code only; included by
// exec.hip).  Large products whose operands lie in rows that are not 16-byte aligned, or in many
// K-segments, run the grouped GEMM on such a copy: every row of it starts at a multiple of 128
// bytes and K is one segment per replica of C, so no 64-byte row piece of a K step straddles two
// cache lines and no segment has a tail or a switch.
// Bound: HBM, one read and one write of the operands (12289 x 9973 and 9973 x 11003 in uneven
// packed tiles: 0.93 GB).  A thread moves 16 bytes of each of eight rows, all eight loads issued before
// the first store; reads are contiguous along the source's rows whatever their alignment.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gemm_kernel.hpp"
#include "small_kernel.hpp"

namespace dmm {

struct PackTile {          // one tile of the operand
  const char *ptr;
  int64_t pitch;           // bytes
};

struct PackJob {           // columns [col0, col0 + cols) of one tile row of an operand -> dense rows at dst
  char *dst;               // 16-byte aligned, like the pitch
  int64_t pitch;           // bytes
  int32_t rows, col0, cols;
  int32_t gc;              // tiles side by side
  int32_t cc, tiles;       // where the column cuts (in cuts[]) and the row's tiles (in tiles[]) begin
  int32_t first_block;     // the workgroups of the job begin here
  int32_t blocks_c;        // workgroups side by side
};

constexpr int PACK_ROWS = 8;
constexpr int PACK_COLS = 256 * 8;

__global__ __launch_bounds__(256) void pack_kernel(const PackJob *__restrict__ jobs, int n_jobs, const int32_t *__restrict__ cuts,
                                                   const PackTile *__restrict__ tiles) {
  // the last of `n` that does not lie behind `at`
  auto last_not_above = [](int n, int at, auto value) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (value(mid) <= at) lo = mid;
      else hi = mid - 1;
    }
    return lo;
  };
  const PackJob j = jobs[last_not_above(n_jobs, (int)blockIdx.x, [&](int x) { return jobs[x].first_block; })];
  const int b = (int)blockIdx.x - j.first_block, row0 = b / j.blocks_c * PACK_ROWS;
  const int at = (b % j.blocks_c * 256 + (int)threadIdx.x) * 8;          // column inside the job
  if (at >= j.cols) return;
  const int32_t *cc = cuts + j.cc;
  const PackTile *t = tiles + j.tiles;
  const int n = j.cols - at < 8 ? j.cols - at : 8;
  const int c = j.col0 + at;
  int tj = last_not_above(j.gc, c, [&](int x) { return cc[x]; });
  const int rows = j.rows - row0 < PACK_ROWS ? j.rows - row0 : PACK_ROWS;
  const gptr dst = (gptr)j.dst + ((int64_t)row0 * j.pitch + (int64_t)at * 2);
  typedef __attribute__((address_space(1))) u32x4 *gvec;
  // (rows past the block's end read its last row, so that the loads are free of branches)
  if (n == 8 && c + 8 <= cc[tj + 1]) {                                   // all eight columns in one tile
    const PackTile s = t[tj];
    const gptr p = (gptr)s.ptr + ((int64_t)row0 * s.pitch + (int64_t)(c - cc[tj]) * 2);
    u32x4 v[PACK_ROWS];
#pragma unroll
    for (int r = 0; r < PACK_ROWS; ++r) v[r] = *(const __attribute__((address_space(1))) u32x4_any *)(p + (r < rows ? r : rows - 1) * s.pitch);
#pragma unroll
    for (int r = 0; r < PACK_ROWS; ++r)
      if (r < rows) *(gvec)(dst + r * j.pitch) = v[r];
  } else {
    gptr p[8];
    int64_t pitch[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int col = c + (e < n ? e : n - 1);
      while (col >= cc[tj + 1]) ++tj;
      const PackTile s = t[tj];
      pitch[e] = s.pitch;
      p[e] = (gptr)s.ptr + ((int64_t)row0 * s.pitch + (int64_t)(col - cc[tj]) * 2);
    }
#pragma unroll 2
    for (int r = 0; r < rows; ++r) {
      unsigned u[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) u[e] = *(const __attribute__((address_space(1))) unsigned short *)(p[e] + r * pitch[e]);
      // (the last chunk of a row is written whole: the dense rows are padded to a multiple of 64 columns)
      *(gvec)(dst + r * j.pitch) = u32x4{u[0] | u[1] << 16, u[2] | u[3] << 16, u[4] | u[5] << 16, u[6] | u[7] << 16};
    }
  }
}

}  // namespace dmm
