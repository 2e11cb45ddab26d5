// Gathers a partitioned bf16 operand into dense rows (gfx950, device code only; included by
// exec.hip).  Large products whose operands lie in rows that are not 16-byte aligned, or in many
// K-segments, run the grouped GEMM on such a copy: every row of it starts at a multiple of 128
// bytes and K is one segment per replica of C, so no 64-byte row piece of a K step straddles two
// cache lines and no segment switch interrupts the K loop.
// Every K-segment of the operands keeps the K steps it has there: it starts at a multiple of a
// step and is filled up with zeros, in A's columns and in B's rows alike, as the macro-tile kernels
// do on the way to LDS.  The products on the copies are therefore those on the operands, step by
// step, and so are the sums, bit for bit.
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

struct PackRun {           // columns [start, start + len) of a copy's rows are columns [col, col + len) of a tile;
  int32_t start, len;      // what lies between two runs, and behind the last, is zero
  int32_t tile, col;
};

struct PackJob {           // rows of one tile row of an operand -> dense rows at dst
  char *dst;               // 16-byte aligned, like the pitch
  int64_t pitch;           // bytes
  int32_t rows, rows_out;  // rows copied, rows written (the others are zero)
  int32_t row;             // first row inside the tiles
  int32_t cols_out;        // columns written, up to the next multiple of eight
  int32_t runs, n_runs;    // in runs[]; the first run starts at 0
  int32_t tiles;           // where the tile row begins in tiles[]
  int32_t first_block;     // the workgroups of the job begin here
  int32_t blocks_c;        // workgroups side by side
  int32_t pad;
};

constexpr int PACK_ROWS = 8;
constexpr int PACK_COLS = 256 * 8;

__global__ __launch_bounds__(256) void pack_kernel(const PackJob *__restrict__ jobs, int n_jobs, const PackRun *__restrict__ all_runs,
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
  const int at = (b % j.blocks_c * 256 + (int)threadIdx.x) * 8;          // column of the copy
  if (at >= j.cols_out) return;
  const PackRun *runs = all_runs + j.runs;
  const PackTile *t = tiles + j.tiles;
  int x = last_not_above(j.n_runs, at, [&](int i) { return runs[i].start; });
  const PackRun u = runs[x];
  const int off = at - u.start, n = u.len - off;                         // the run has n columns from here on
  const bool alone = x + 1 == j.n_runs || runs[x + 1].start >= at + 8;   // no other run begins in the eight columns
  const int out = j.rows_out - row0 < PACK_ROWS ? j.rows_out - row0 : PACK_ROWS;
  const int rows = j.rows - row0 < out ? j.rows - row0 : out;            // of these rows hold values (may be 0 or less)
  const gptr dst = (gptr)j.dst + ((int64_t)row0 * j.pitch + (int64_t)at * 2);
  typedef __attribute__((address_space(1))) u32x4 *gvec;
  const u32x4 zero = {0u, 0u, 0u, 0u};
  if (rows <= 0 || (n <= 0 && alone)) {
    for (int r = 0; r < out; ++r) *(gvec)(dst + r * j.pitch) = zero;
  } else if (n >= 8 || (n > 0 && u.len >= 8 && alone)) {
    // all columns in one tile; at the end of a run the run's last eight columns are read and moved to the
    // front.  (Rows past the last read that one again, so that the loads are free of branches.)
    const int back = n >= 8 ? 0 : 8 - n;
    const PackTile s = t[u.tile];
    const gptr p = (gptr)s.ptr + ((int64_t)(j.row + row0) * s.pitch + (int64_t)(u.col + off - back) * 2);
    u32x4 v[PACK_ROWS];
#pragma unroll
    for (int r = 0; r < PACK_ROWS; ++r) v[r] = *(const __attribute__((address_space(1))) u32x4_any *)(p + (r < rows ? r : rows - 1) * s.pitch);
#pragma unroll
    for (int r = 0; r < PACK_ROWS; ++r)
      if (r < out) *(gvec)(dst + r * j.pitch) = r < rows ? drop_first(v[r], back) : zero;
  } else {
    // (columns without a value read the last one that has one)
    gptr p[8], last = nullptr;
    int64_t pitch[8], last_pitch = 0;
    unsigned have = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      while (x + 1 < j.n_runs && runs[x + 1].start <= at + e) ++x;
      const PackRun w = runs[x];
      const int o = at + e - w.start;
      if (o < w.len) {
        const PackTile s = t[w.tile];
        last_pitch = s.pitch;
        last = (gptr)s.ptr + ((int64_t)(j.row + row0) * s.pitch + (int64_t)(w.col + o) * 2);
        have |= 1u << e;
      }
      p[e] = last;
      pitch[e] = last_pitch;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (!(have & ((2u << e) - 1))) {                                   // nothing at or in front of it
        p[e] = last;
        pitch[e] = last_pitch;
      }
#pragma unroll 2
    for (int r = 0; r < rows; ++r) {
      unsigned q[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) q[e] = *(const __attribute__((address_space(1))) unsigned short *)(p[e] + r * pitch[e]);
#pragma unroll
      for (int e = 0; e < 8; ++e) q[e] = have >> e & 1 ? q[e] : 0u;
      *(gvec)(dst + r * j.pitch) = u32x4{q[0] | q[1] << 16, q[2] | q[3] << 16, q[4] | q[5] << 16, q[6] | q[7] << 16};
    }
    for (int r = rows; r < out; ++r) *(gvec)(dst + r * j.pitch) = zero;
  }
}

}  // namespace dmm
