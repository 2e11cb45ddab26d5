// GEMM kernels for products that 256 x 256 macro-tiles do not fill the device with (gfx950, device
// code only): small and skinny results, few macro-tiles, fp32 products cut into ragged pieces.
//
// What bounds such a product under the macro-tile kernels: CUs without a macro-tile, rows and
// columns of macro-tiles that hold nothing, and one workgroup per CU, whose waits nothing hides.
// Here a tile is 32 to 128 rows and columns, up to four workgroups share a CU, and a tile's K steps
// are dealt to as many workgroups as the device has room for.
//
// Tiles are cut from C as a whole, across the cuts of A, B and C: the slicing is kept in factored
// form (one A slice per row interval and K-segment, one B slice per K-segment and column
// interval, one C slice per row and column interval), and every thread looks up the slice that
// holds its own rows and its own chunk of columns.  A tile ends early at a column cut that is not
// a multiple of eight columns away from its start, so that a 16-byte chunk has one source.
//
// Here are the tables, the epilogue, the sum of partial tiles and the loop for fp32; the loop for bf16 is in
// ring_kernel.hpp.  The fp32 loop takes operands global -> registers -> LDS (two stages, one barrier per
// step): the register stage takes any alignment and lets K tails and column tails be zeroed on the way, so
// nothing is ever read past a slice.  Sums run over the same K-segments in the same order and through the
// same matrix instructions as in the macro-tile kernels, hence bitwise the same results, unless a
// tile's K steps are dealt to several workgroups or waves (their partial sums are then added in
// ascending k) or fp32 operands are taken apart into three bf16 (SmallF32Split: fewer roundings).
//
// Measured (kernel alone, us; macro-tile kernels -> these): fp32 256^3 50 -> 5.  Operands of one, two or three
// steps in flight made no difference.
#pragma once

#include "gemm_kernel.hpp"

namespace dmm {

struct SmallTile {         // one tile row (column) of C
  int32_t start, ext;      // first row (column), number of them
  int32_t first, pieces;   // first interval met, number of intervals met
  int32_t base;            // where that interval begins
  int32_t pad;
};

struct SmallStart {        // where a run of K steps begins
  int32_t seg, kpos;
};

struct SmallArgs {
  const SmallTile *rows, *cols;
  const int32_t *mc, *nc;              // boundaries of the row (column) intervals
  const SmallStart *starts;            // [runs]
  const int32_t *klen;                 // [S]
  const PieceDev *pa, *pb, *pc;        // A slice (i, s) at pa[i S + s], B slice (s, j) at pb[s NR + j], C slice (i, j) at pc[i NR + j]
  float *scratch;                      // runs > 1: partial tiles of the launch, number run * tiles + tile
  int32_t S, NR;
  int32_t tiles_m, tiles_n;
  int32_t runs, per;                   // a tile's K steps in `runs` ranges of `per` steps (the last may be shorter)
  int32_t first, tiles;                // tiles [first, first + tiles) are this launch's
  int32_t c_es;                        // bytes per element of C
  int32_t band;                        // tile rows of a band of the launch order (see small_tile_of)
  int32_t steps;                       // K steps of a tile
  int32_t pad;
};

typedef unsigned int u32x4_any __attribute__((ext_vector_type(4), aligned(2)));   // 16 bytes at any element's address
typedef __attribute__((address_space(3))) char *lds_ptr;

// ES bytes per operand element; TM x TN tile of C; BK elements of k per step; WM x WN waves over the
// tile, times WK waves over the matrix instructions of a step
// SPLIT: fp32 operands as three bf16 each (see split_planes)
// PARTS: the launch's tiles have PARTS times TM rows, and this is the loop over one of these parts
template <int ES_, int TM_, int TN_, int BK_, int WM_, int WN_, int WK_, int DEPTH_, int OCC_, bool SPLIT_ = false, int PARTS_ = 1>
struct SmallShape {
  static constexpr bool RING = false, SPLIT = SPLIT_;
  static constexpr int ES = ES_, TM = TM_, TN = TN_, BK = BK_, WM = WM_, WN = WN_, WK = WK_;
  static constexpr int PARTS = PARTS_;
  static constexpr int DEPTH = DEPTH_;                          // K steps whose operands are in flight
  static constexpr int OCC = OCC_;                              // workgroups per CU the LDS and registers leave room for
  static constexpr int PER = 16 / ES;
  static constexpr int A_CHUNKS = BK * ES / 16, B_CHUNKS = TN * ES / 16;   // 16-byte chunks per A row, per k row of B
  static constexpr int CA = TM * A_CHUNKS / NT, CB = BK * B_CHUNKS / NT;   // chunks per thread
  // row pitches in LDS that spread the fragment reads over all banks: 16 A rows read the same
  // chunk (pitch = 4 dwords off a multiple of 32); bf16 B: four k rows x 64 bytes per transposed read
  // (pitch = 64 bytes off a multiple of 128); fp32 B: rows k and k + 4 x 32 dwords (pitch = 8 off a multiple of 16)
  static constexpr int PLANES = SPLIT ? 3 : 1, LES = SPLIT ? 2 : ES;   // in LDS: so many copies, bytes per element
  static constexpr int A_PITCH = BK * LES + 16;
  static constexpr int B_PITCH = TN * LES + (LES == 2 ? 64 : 32);
  static constexpr int A_PLANE = TM * A_PITCH, B_PLANE = BK * B_PITCH;
  static constexpr int STAGE_BYTES = PLANES * (A_PLANE + B_PLANE);
  static constexpr int STAGES = SPLIT ? 1 : 2;
  static constexpr int T_PITCH = TN + 8;                         // floats: the finished tile in LDS
  static constexpr int TILE_BYTES = WK * TM * T_PITCH * 4;
  static constexpr int LDS = STAGES * STAGE_BYTES > TILE_BYTES ? STAGES * STAGE_BYTES : TILE_BYTES;
  static constexpr int MI = TM / WM / 32, NI = TN / WN / 32;     // 32 x 32 matrix tiles per wave
  static_assert(WM * WN * WK == NW && CA >= 1 && CB >= 1 && NT % A_CHUNKS == 0 && NT % B_CHUNKS == 0, "chunks are dealt evenly");
};

// the interval of a tile row (column) that holds `pos`, and where it begins
__device__ __forceinline__ int small_piece(const int32_t *bounds, const SmallTile &t, int pos, int *begin) {
  int i = t.first;
  *begin = t.base;
  for (int y = 1; y < t.pieces; ++y) {
    const int b = bounds[t.first + y];
    if (b <= pos) {
      i = t.first + y;
      *begin = b;
    }
  }
  return i;
}

// Where four columns of the tile, from column c on, go: the C slice that holds row r.  Looked up ahead of the
// K loop where registers allow: looked up row by row the stores of a 128 x 128 tile took 4 us instead of 1.8.
struct SmallOut {
  uint64_t at;             // address of the columns in the slice's first row
  unsigned pitch;
  int begin, end;          // the slice's rows
};
struct SmallOutLoad {      // the look-up under way: small_out_of is not called before the data are wanted
  PieceDev slice;
  int begin, end, n;       // the slice's rows; the column inside it
};
__device__ __forceinline__ SmallOutLoad small_out_load(const SmallArgs &g, const SmallTile &tr, const SmallTile &tc, int r, int c) {
  SmallOutLoad o;
  int n0;
  const int n = tc.start + c, i = small_piece(g.mc, tr, tr.start + r, &o.begin), j = small_piece(g.nc, tc, n, &n0);
  o.slice = g.pc[(int64_t)i * g.NR + j];
  o.end = i + 1 < tr.first + tr.pieces ? g.mc[i + 1] : tr.start + tr.ext;
  o.n = n - n0;
  return o;
}
__device__ __forceinline__ SmallOut small_out_of(const SmallArgs &g, const SmallOutLoad &o) {
  return SmallOut{(uint64_t)(uintptr_t)o.slice.ptr + (uint64_t)o.n * (unsigned)g.c_es, o.slice.pitch, o.begin, o.end};
}

// four columns of row r, from column c on
__device__ __forceinline__ void small_store4(const SmallArgs &g, const SmallTile &tr, const SmallTile &tc, SmallOut &o, int r, int c, f32x4 v) {
  if (tr.start + r >= o.end) o = small_out_of(g, small_out_load(g, tr, tc, r, c));
  const uint64_t at = o.at + (uint64_t)(tr.start + r - o.begin) * o.pitch;
  const int left = tc.ext - c;
  // (column pieces begin at multiples of eight columns of the tile: the four columns lie in one slice)
  if (g.c_es == 4) {
    gfloat_ptr p = (gfloat_ptr)(uintptr_t)at;
    if (left >= 4 && (at & 15) == 0) {
      *(__attribute__((address_space(1))) f32x4 *)p = v;
    } else {
#pragma unroll
      for (int x = 0; x < 4; ++x)
        if (x < left) p[x] = v[x];
    }
  } else {
    gushort_ptr p = (gushort_ptr)(uintptr_t)at;
    unsigned short e[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) e[x] = __builtin_bit_cast(unsigned short, (__bf16)v[x]);
    if (left >= 4 && (at & 7) == 0) {
      typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
      *(__attribute__((address_space(1))) u32x2 *)p = u32x2{e[0] | (unsigned)e[1] << 16, e[2] | (unsigned)e[3] << 16};
    } else {
#pragma unroll
      for (int x = 0; x < 4; ++x)
        if (x < left) p[x] = e[x];
    }
  }
}

constexpr int SMALL_BAND = 4;            // so that B columns that a few tile rows share are read by workgroups close to each other

// a / d for 0 <= a < 2^20, 0 < d (the compiler's division takes ten times as long, and a small product waits for it)
__device__ __forceinline__ int small_div(int a, int d) {
  return __builtin_amdgcn_readfirstlane((int)(((float)a + 0.5f) * __builtin_amdgcn_rcpf((float)d)));
}

// The tile row and tile column of a tile: bands of `band` tile rows, column by column inside a band.
__device__ __forceinline__ void small_tile_of(const SmallArgs &g, int tile, int *row, int *col) {
  const int whole = g.band * g.tiles_n, b = small_div(tile, whole), in = tile - b * whole, r0 = b * g.band;
  const int h = g.tiles_m - r0 < g.band ? g.tiles_m - r0 : g.band;
  *col = small_div(in, h);
  *row = r0 + (in - *col * h);
}

// The run and the tile of a workgroup.  Workgroup id mod 8 is the XCD: each XCD takes a contiguous eighth of
// the (run, tile) sequence, so that the workgroups that share an L2 share A rows, B columns and k ranges.
struct SmallPlace {
  int run, local, row, col;
  int slot;                // its partial tile's number
};
__device__ __forceinline__ SmallPlace small_place(const SmallArgs &g) {
  const int total = (int)gridDim.x, q8 = total >> 3, r8 = total & 7;
  const int xcd = blockIdx.x & 7, pos = blockIdx.x >> 3;
  const int id = xcd * q8 + (xcd < r8 ? xcd : r8) + pos;
  SmallPlace p;
  p.run = small_div(id, g.tiles);
  p.local = id - p.run * g.tiles;
  p.slot = id;
  small_tile_of(g, g.first + p.local, &p.row, &p.col);
  return p;
}

// The finished tile through LDS, four consecutive columns per thread.  value(i, j, e): element e of the lane's
// part of 32 x 32 tile (i, j), as the matrix instructions leave it.  Waves wk > 0 hold partial sums of the same elements.
template <class SH, class F>
__device__ __forceinline__ void small_epilogue(const SmallArgs &g, const SmallPlace &at, const SmallTile &tr, const SmallTile &tc, SmallOut &to,
                                               lds_ptr lds3, F &&value, int wm, int wn, int wk) {
  constexpr int MI = SH::MI, NI = SH::NI;
  const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
  __syncthreads();
  typedef __attribute__((address_space(3))) float *lds_float;
  const lds_float out = (lds_float)lds3 + wk * (SH::TM * SH::T_PITCH);
  static_for<MI>([&](auto ic) {
    static_for<NI>([&](auto jc) {
      static_for<16>([&](auto ec) {
        constexpr int i = decltype(ic)::value, j = decltype(jc)::value, e = decltype(ec)::value;
        out[(wm * (MI * 32) + i * 32 + 8 * (e >> 2) + 4 * half + (e & 3)) * SH::T_PITCH + wn * (NI * 32) + j * 32 + (lane & 31)] = value(ic, jc, ec);
      });
    });
  });
  __syncthreads();
  float *part = g.scratch + (int64_t)at.slot * (SH::TM * SH::TN);
  const int c = tid % (SH::TN / 4) * 4, r0 = tid / (SH::TN / 4);
  constexpr int STEP = NT / (SH::TN / 4);                 // rows from one of a thread's to the next
  if (c >= tc.ext || r0 >= tr.ext) return;
  auto value4 = [&](int r) __attribute__((always_inline)) {
    f32x4 v = *(const __attribute__((address_space(3))) f32x4 *)((lds_float)lds3 + r * SH::T_PITCH + c);
#pragma unroll
    for (int w = 1; w < SH::WK; ++w)
      v = v + *(const __attribute__((address_space(3))) f32x4 *)((lds_float)lds3 + (w * SH::TM + r) * SH::T_PITCH + c);
    return v;
  };
  // All of a thread's columns in one slice, at multiples of 16 bytes: an address and an increment.
  uint64_t p = to.at + (uint64_t)(tr.start + r0 - to.begin) * to.pitch, inc = (uint64_t)to.pitch * STEP;
  bool plain = g.c_es == 4 && tr.start + tr.ext <= to.end && tc.ext - c >= 4 && ((p | inc) & 15) == 0;
  if (g.runs > 1) {
    p = (uint64_t)(uintptr_t)(part + r0 * SH::TN + c);
    inc = (uint64_t)STEP * SH::TN * 4;
    plain = true;
  }
  if (plain) {
#pragma unroll
    for (int x = 0; x < SH::TM / STEP; ++x) {
      if (r0 + x * STEP < tr.ext) *(__attribute__((address_space(1))) f32x4 *)p = value4(r0 + x * STEP);
      p += inc;
    }
    return;
  }
  for (int r = r0; r < tr.ext; r += STEP) small_store4(g, tr, tc, to, r, c, value4(r));
}

// what a thread stores first, looked up ahead (nothing where partial tiles are stored)
template <class SH>
__device__ __forceinline__ SmallOutLoad small_first_out(const SmallArgs &g, const SmallTile &tr, const SmallTile &tc) {
  const int r = threadIdx.x / (SH::TN / 4), c = threadIdx.x % (SH::TN / 4) * 4;
  if (g.runs == 1 && r < tr.ext && c < tc.ext) return small_out_load(g, tr, tc, r, c);
  return SmallOutLoad{{nullptr, 0, 0u, 0u}, 0, 0, 0};
}

//                ES   TM   TN  BK WM WN WK DEPTH OCC
typedef SmallShape<4, 32, 32, 64, 1, 1, 4, 1, 4> SmallF32Tiny;
typedef SmallShape<4, 64, 64, 32, 2, 2, 1, 2, 4> SmallF32;
// What bounds the fp32 shapes is the fp32 matrix instruction, 64 cycles for 2 k of 32 x 32.  Taken as three bf16 each
// (exactly), eight bf16 products of 32 cycles do 16 k: 256 cycles instead of 512.  A 128 x 128 x 32 step is 2048 cycles
// of the matrix pipes and some 1200 of taking apart and LDS writes, which the CU's other workgroup fills with its
// matrix instructions (busy 54 % of the time): hence one LDS stage (60 KB; 68 KB with the finished tile), twice per CU.  Measured, us per call, the
// other fp32 kernels -> this one: 4096^3 950 (macro-tiles, 145 TFLOP/s) -> 860 (160); 2048^3 177 -> 127; 2501 x 1999 x 1777
// uneven 219 -> 172; 5612 x 1584 x 3264 597 -> 467.  Error against 64 bits: of sums of many terms 0.2 to 0.5 of the
// fp32 kernels', of single products the same (see multiply).
typedef SmallShape<4, 128, 128, 32, 2, 2, 1, 1, 2, true> SmallF32Split;
typedef SmallShape<4, 64, 128, 32, 2, 2, 1, 1, 2, false, 2> SmallF32Whole;   // for its tiles that cannot be split (all of them,
                                        // 2048 x 4096 x 2048: 503 us instead of 230; in 128 rows at once registers spill)

// An fp32 value as the sum of three bf16: the nearest one, the nearest one to what is left, and the rest, which has no
// more than 8 significant bits.  (To nearest, so that the second and third parts have either sign: cut off, all parts have
// the sign of the value, and the small products, which a long sum rounds away one by one, are missing from every sum
// of values of one sign: 159 units of 2^-24 at 4096^3 instead of 6.)  Nothing is lost; only bits below 2^-133, the
// smallest bf16, have no place, and they stand in the lower half of the rest: `lost` collects it.  A value that rounds to
// infinity leaves NaN behind.  (Neither the conversion nor the matrix pipe flushes denormals.)
struct SplitPlanes {
  unsigned p[3][2];                 // four values: plane, pairs of bf16
};
__device__ __forceinline__ unsigned to_bf16_pair(float x, float y) {
  unsigned r;
  asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(r) : "v"(x), "v"(y));
  return r;
}
__device__ __forceinline__ SplitPlanes split_planes(u32x4 v, unsigned &lost) {
  SplitPlanes s;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const unsigned u0 = v[2 * h], u1 = v[2 * h + 1];
    const float x0 = __builtin_bit_cast(float, u0), x1 = __builtin_bit_cast(float, u1);
    const unsigned first = to_bf16_pair(x0, x1);
    const float y0 = x0 - __builtin_bit_cast(float, first << 16), y1 = x1 - __builtin_bit_cast(float, first & 0xFFFF0000u);
    const unsigned second = to_bf16_pair(y0, y1);
    const float z0 = y0 - __builtin_bit_cast(float, second << 16), z1 = y1 - __builtin_bit_cast(float, second & 0xFFFF0000u);
    const unsigned rest0 = __builtin_bit_cast(unsigned, z0), rest1 = __builtin_bit_cast(unsigned, z1);
    lost |= rest0 | rest1;
    s.p[0][h] = first;
    s.p[1][h] = second;
    s.p[2][h] = __builtin_amdgcn_perm(rest1, rest0, 0x07060302u);   // the upper halves of two words
  }
  return s;
}

// (SPLIT: true if the tile is not to be had this way: an operand or a sum is infinite or not a number, or bits were lost.
// Nothing has been stored then.)
template <class SH>
__device__ __forceinline__ bool staged_gemm(const SmallArgs &g, char *lds, const int tid, const int part = 0) {
  constexpr int ES = SH::ES, BK = SH::BK, PER = SH::PER, CA = SH::CA, CB = SH::CB, DEPTH = SH::DEPTH, MI = SH::MI, NI = SH::NI;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wk = wave % SH::WK, wn = wave / SH::WK % SH::WN, wm = wave / SH::WK / SH::WN;
  SmallPlace at = small_place(g);
  SmallTile tr = g.rows[at.row];
  const SmallTile tc = g.cols[at.col];
  if constexpr (SH::PARTS > 1) {
    at.slot = at.slot * SH::PARTS + part;
    tr.start += part * SH::TM;
    tr.ext = tr.ext - part * SH::TM < SH::TM ? tr.ext - part * SH::TM : SH::TM;
  }
  const int S = g.S, NR = g.NR;
  const SmallStart start = g.starts[at.run];
  const int t0 = at.run * g.per, n = g.steps - t0 < g.per ? g.steps - t0 : g.per;   // at least 1: the host sees to it

  // ---- this thread's chunks ------------------------------------------------------------
  const int ak = tid % SH::A_CHUNKS * PER;                // first k of its A chunks inside a step
  const int bn = tid % SH::B_CHUNKS * PER;                // first column of its B chunks inside the tile
  const int bk = tid / SH::B_CHUNKS;                      // k row of its first B chunk
  constexpr int A_ROWS = NT / SH::A_CHUNKS, B_ROWS = NT / SH::B_CHUNKS;   // rows from one chunk to the next
  // Where its A rows lie.  (SPLIT: in places of its own in LDS, behind the stage: registers are short there.)
  struct RowAt {
    int slice, row;                                       // the A slice, at segment 0; row inside the slice's tile part
  };
  static_assert(!SH::SPLIT || SH::LDS >= SH::STAGE_BYTES + CA * NT * (int)sizeof(RowAt), "room behind the stage");
  RowAt rows[SH::SPLIT ? 1 : CA];
  typedef __attribute__((address_space(3))) RowAt *row_ptr;
  const row_ptr own_rows = (row_ptr)((lds_ptr)(lds_void_ptr)lds + SH::STAGES * SH::STAGE_BYTES) + tid;
  auto row_at = [&](int x) __attribute__((always_inline)) -> RowAt {
    if constexpr (SH::SPLIT) return RowAt{own_rows[x * NT].slice, own_rows[x * NT].row};
    else return rows[x];
  };
#pragma unroll
  for (int x = 0; x < CA; ++x) {
    int row = tid / SH::A_CHUNKS + x * A_ROWS;
    row = tr.start + (row < tr.ext ? row : tr.ext - 1);   // (rows past the tile's end read its last row; never stored)
    int m0;
    const int slice = small_piece(g.mc, tr, row, &m0) * S;
    if constexpr (SH::SPLIT) {
      own_rows[x * NT].slice = slice;
      own_rows[x * NT].row = row - m0;
    } else {
      rows[x] = RowAt{slice, row - m0};
    }
  }
  int bvalid = tc.ext - bn;                               // columns of its chunk that exist
  bvalid = bvalid < 0 ? 0 : bvalid < PER ? bvalid : PER;
  const bool edge = tc.ext < SH::TN;
  int bp;                                                 // its B slice, at segment 0
  unsigned bcol;                                          // byte column inside the slice
  {
    const int col = tc.start + (bvalid > 0 ? bn : 0);
    int n0;
    bp = small_piece(g.nc, tc, col, &n0);
    bcol = (unsigned)(col - n0) * ES;
  }

  // ---- cursor over the K steps whose loads are issued ------------------------------------
  // The descriptors of the segment after the cursor's are fetched a segment ahead: loads return in
  // order, so waiting for a descriptor asked for just now would wait for all operands in flight.
  // (SPLIT: not ahead, for the same shortage of registers; the CU's other workgroup multiplies meanwhile.)
  int seg = 0, krem = 0;                                  // segment; elements of it left
  gptr pa[CA], pb;
  unsigned bpitch = 0;
  PieceDev na[CA], nb;                                    // descriptors of the coming segment
  int nlen = 0;
  // Which of its chunks a thread may read in full where only the first elements count (a K tail, the
  // last columns): all but those that would cross the end of a tile buffer.
  unsigned asafe = 0;                                     // bit x: A chunk x of the segment's last step
  bool bsafe = false;                                     // the B chunk of the segment's last k row
  bool quick = true;                                      // the chunks of all its other rows, in every lane
  auto fetch = [&](int s) {
#pragma unroll
    for (int x = 0; x < CA; ++x) na[x] = g.pa[row_at(x).slice + s];
    nb = g.pb[bp + (int64_t)s * NR];
    nlen = g.klen[s];
  };
  auto open = [&](int kpos) __attribute__((always_inline)) {                             // the cursor enters the segment fetched last
    if constexpr (SH::SPLIT) fetch(seg);
    krem = nlen - kpos;
    const int64_t last = (int64_t)((nlen - 1) / BK) * (BK * ES) + ak * ES;
    asafe = 0;
#pragma unroll
    for (int x = 0; x < CA; ++x) {
      const int64_t off = (int64_t)row_at(x).row * na[x].pitch;
      pa[x] = (gptr)na[x].ptr + (off + (int64_t)(kpos + ak) * ES);
      asafe |= (na[x].room - off - last >= 16 ? 1u : 0u) << x;
    }
    bpitch = nb.pitch;
    pb = (gptr)nb.ptr + ((int64_t)(kpos + bk) * bpitch + bcol);
    bsafe = nb.room - (int64_t)(nlen - 1) * bpitch - bcol >= 16;
    quick = !edge || __builtin_amdgcn_ballot_w64(bpitch < 16) == 0;
    if (!SH::SPLIT && seg + 1 < S) fetch(seg + 1);
  };
  seg = start.seg;
  if (!SH::SPLIT) fetch(seg);
  open(start.kpos);
  u32x4 ra[DEPTH][CA], rb[DEPTH][CB];                     // operands of DEPTH steps in flight
  int rk[DEPTH];                                          // elements of the segment left at those steps
  auto load16 = [](gptr p) -> u32x4 { return *(const __attribute__((address_space(1))) u32x4_any *)p; };
  auto load_step = [&](u32x4 (&va)[CA], u32x4 (&vb)[CB], int &left_k, bool more) __attribute__((always_inline)) {
    left_k = krem;
    if (__builtin_expect(krem > BK ? quick : krem == BK && !edge, 1)) {
#pragma unroll
      for (int x = 0; x < CA; ++x) va[x] = load16(pa[x]);
      gptr p = pb;
#pragma unroll
      for (int x = 0; x < CB; ++x) {
        vb[x] = load16(p);
        p += (int64_t)B_ROWS * bpitch;
      }
    } else {
      // the segment's last step: what is read past the segment in k is zeroed on the way to LDS, so
      // that no load is waited for here (columns past the tile's end stay as they are, or are zeroed there)
      const int an = krem - ak;
#pragma unroll
      for (int x = 0; x < CA; ++x) {
        va[x] = u32x4{0u, 0u, 0u, 0u};
        if (an >= PER || (an > 0 && (asafe >> x & 1))) va[x] = load16(pa[x]);
        else if (an > 0) va[x] = load_partial<ES>(pa[x], an);
      }
      gptr p = pb;
#pragma unroll
      for (int x = 0; x < CB; ++x) {
        const int left = krem - (bk + x * B_ROWS);        // k rows of the segment from this one on
        vb[x] = u32x4{0u, 0u, 0u, 0u};
        if (left > 0 && bvalid > 0) {
          if (bvalid == PER || bsafe || (left > 1 && bpitch >= 16)) vb[x] = load16(p);
          else vb[x] = load_partial<ES>(p, bvalid);
        }
        p += (int64_t)B_ROWS * bpitch;
      }
    }
    if (!more) return;
    krem -= BK;
    if (krem <= 0) {
      ++seg;
      open(0);
    } else {
#pragma unroll
      for (int x = 0; x < CA; ++x) pa[x] += BK * ES;
      pb += (int64_t)BK * bpitch;
    }
  };
  const lds_ptr lds3 = (lds_ptr)(lds_void_ptr)lds;
  unsigned lost = 0;
  auto write_step = [&](int stage, u32x4 (&va)[CA], u32x4 (&vb)[CB], int left_k) __attribute__((always_inline)) {
    if (__builtin_expect(left_k < BK, 0)) {
#pragma unroll
      for (int x = 0; x < CA; ++x) va[x] = keep_first<ES>(va[x], left_k - ak);
    }
    const lds_ptr sa = lds3 + stage * SH::STAGE_BYTES, sb = sa + SH::PLANES * SH::A_PLANE;
    if constexpr (SH::SPLIT) {
      typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
#pragma unroll
      for (int x = 0; x < CA; ++x) {
        const SplitPlanes s = split_planes(va[x], lost);
#pragma unroll
        for (int p = 0; p < 3; ++p)
          *(__attribute__((address_space(3))) u32x2 *)(sa + p * SH::A_PLANE + (tid / SH::A_CHUNKS + x * A_ROWS) * SH::A_PITCH + ak * 2) = u32x2{s.p[p][0], s.p[p][1]};
      }
      // (columns past the tile's end, the padding of a row among them, have no say in how the tile is multiplied)
      if (edge) {
#pragma unroll
        for (int x = 0; x < CB; ++x) vb[x] = keep_first<ES>(vb[x], bvalid);
      }
#pragma unroll
      for (int x = 0; x < CB; ++x) {
        const SplitPlanes s = split_planes(vb[x], lost);
#pragma unroll
        for (int p = 0; p < 3; ++p)
          *(__attribute__((address_space(3))) u32x2 *)(sb + p * SH::B_PLANE + (bk + x * B_ROWS) * SH::B_PITCH + bn * 2) = u32x2{s.p[p][0], s.p[p][1]};
      }
    } else {
#pragma unroll
      for (int x = 0; x < CA; ++x)
        *(__attribute__((address_space(3))) u32x4 *)(sa + (tid / SH::A_CHUNKS + x * A_ROWS) * SH::A_PITCH + ak * ES) = va[x];
#pragma unroll
      for (int x = 0; x < CB; ++x)
        *(__attribute__((address_space(3))) u32x4 *)(sb + (bk + x * B_ROWS) * SH::B_PITCH + bn * ES) = vb[x];
    }
  };

  // ---- the K loop: step t is multiplied while the loads of the DEPTH steps after it travel -----------------
  floatx16 acc[MI][NI], small[SH::SPLIT ? MI : 1][SH::SPLIT ? NI : 1];   // SPLIT: sums of a1 b1; of the other products
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        acc[i][j][e] = 0.f;
        if constexpr (SH::SPLIT) small[i][j][e] = 0.f;
      }
  const int a_row = wm * (MI * 32) + (lane & 31), half = lane >> 5;
  auto multiply = [&](int stage) __attribute__((always_inline)) {
    const lds_ptr sa = lds3 + stage * SH::STAGE_BYTES, sb = sa + SH::PLANES * SH::A_PLANE;
    if constexpr (SH::SPLIT) {
      // a b = a1 b1 + (a1 b2 + a2 b1 + a2 b2 + a1 b3 + a3 b1 + a2 b3 + a3 b2); what is left out, a3 b3, is 2^-32 of a product
      // and less.  (Without a2 b3 and a3 b2, 2^-24 and less: a row of A with one element had errors of 0.95 units of 2^-24
      // instead of 0.54 at the worst mantissas, for 15 % of the time.)  The products in brackets are summed up by themselves: next to
      // the sum of a1 b1 they would be rounded to its last bit, and round it eight times in 16 k instead of twice.
      const int gr = lane >> 4, li = lane & 15;
#pragma unroll
      for (int q = 0; q < BK / 16; ++q) {
        bf16x8 fb[3][NI];
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
          for (int j = 0; j < NI; ++j) {
            union { short4_t h[2]; bf16x8 v; } u;
#pragma unroll
            for (int h = 0; h < 2; ++h)
              u.h[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                  (lds_short4_ptr)(sb + p * SH::B_PLANE + (q * 16 + (gr >> 1) * 8 + (li >> 2) + 4 * h) * SH::B_PITCH +
                                   (wn * (NI * 32) + j * 32 + (gr & 1) * 16 + (li & 3) * 4) * 2));
            fb[p][j] = u.v;
          }
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          bf16x8 fa[MI];
#pragma unroll
          for (int i = 0; i < MI; ++i)
            fa[i] = *(const __attribute__((address_space(3))) bf16x8 *)(sa + p * SH::A_PLANE + (a_row + i * 32) * SH::A_PITCH + q * 32 + half * 16);
#pragma unroll
          for (int x = 0; x < (p < 2 ? 3 : 2); ++x)
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
              for (int j = 0; j < NI; ++j) {
                floatx16 &sum = p + x == 0 ? acc[i][j] : small[i][j];
                sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[x][j], sum, 0, 0, 0);
              }
          DMM_SCHED_BARRIER;       // (no plane of A is read before the one before is used up: registers)
        }
      }
    } else {
#pragma unroll
      for (int q = 0; q < BK / 8 / SH::WK; ++q) {
        const int qq = q * SH::WK + wk;
        f32x4 fa[MI];
#pragma unroll
        for (int i = 0; i < MI; ++i)
          fa[i] = *(const __attribute__((address_space(3))) f32x4 *)(sa + (a_row + i * 32) * SH::A_PITCH + qq * 32 + half * 16);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int j = 0; j < NI; ++j) {
            const float fb = *(const __attribute__((address_space(3))) float *)(sb + (qq * 8 + half * 4 + e) * SH::B_PITCH +
                                                                               (wn * (NI * 32) + j * 32 + (lane & 31)) * 4);
#pragma unroll
            for (int i = 0; i < MI; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i][e], fb, acc[i][j], 0, 0, 0);
          }
      }
    }
  };
  static_for<DEPTH>([&](auto dc) {
    constexpr int d = decltype(dc)::value;
    if (d < n) load_step(ra[d], rb[d], rk[d], d + 1 < n);
  });
  if constexpr (SH::SPLIT) {
    static_assert(!SH::SPLIT || DEPTH == 1, "one stage, one step in flight: the CU's other workgroup multiplies meanwhile");
    for (int t = 0; t < n; ++t) {
      if (t > 0) __syncthreads();                         // (every wave has read the stage)
      write_step(0, ra[0], rb[0], rk[0]);
      if (t + 1 < n) load_step(ra[0], rb[0], rk[0], t + 2 < n);
      __syncthreads();
      multiply(0);
    }
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) acc[i][j] = acc[i][j] + small[i][j];
    // infinities and NaN of the operands have made NaN of the sums
    unsigned bad = lost & 0xFFFFu;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int r = wm * (MI * 32) + i * 32 + 8 * (e >> 2) + 4 * half + (e & 3), c = wn * (NI * 32) + j * 32 + (lane & 31);
          const float sum = acc[i][j][e];
          const bool finite = (__builtin_bit_cast(unsigned, sum) & 0x7F800000u) != 0x7F800000u;
          bad |= r < tr.ext && c < tc.ext && !finite;
        }
    if (__syncthreads_or(bad != 0)) return true;
  } else {
    for (int t = 0; t < n; t += DEPTH) {
      static_for<DEPTH>([&](auto dc) {
        constexpr int d = decltype(dc)::value;
        if (t + d < n) {
          // (the stage's last readers multiplied step t + d - 2 and have passed the barrier of the step between)
          write_step((t + d) & 1, ra[d], rb[d], rk[d]);
          if (t + d + DEPTH < n) load_step(ra[d], rb[d], rk[d], t + d + DEPTH + 1 < n);
          __syncthreads();
          multiply((t + d) & 1);
        }
      });
    }
  }

  // (not ahead of the loop here: its registers would be in the loop's way)
  const SmallOutLoad to_load = small_first_out<SH>(g, tr, tc);
  SmallOut to = small_out_of(g, to_load);
  small_epilogue<SH>(g, at, tr, tc, to, lds3, [&](auto ic, auto jc, auto ec) { return acc[decltype(ic)::value][decltype(jc)::value][decltype(ec)::value]; },
                     wm, wn, wk);
  return false;
}

// The partial tiles of every tile, added up in ascending k.  A workgroup takes 1024 elements.
template <class SH>
__global__ __launch_bounds__(NT) void small_sum_kernel(const SmallArgs g) {
  constexpr int BLOCKS = SH::TM * SH::TN / 1024;
  const int local = blockIdx.x / BLOCKS, x = (blockIdx.x % BLOCKS) * NT + threadIdx.x;
  int row, col;
  small_tile_of(g, g.first + local, &row, &col);
  const SmallTile tr = g.rows[row], tc = g.cols[col];
  const int r = x / (SH::TN / 4), c = x % (SH::TN / 4) * 4;
  if (r >= tr.ext || c >= tc.ext) return;
  typedef const __attribute__((address_space(1))) f32x4 *gvec;
  const int64_t step = (int64_t)g.tiles * (SH::TM * SH::TN);
  const SmallOutLoad to_load = small_out_load(g, tr, tc, r, c);
  const float *p = g.scratch + (int64_t)local * (SH::TM * SH::TN) + r * SH::TN + c;
  f32x4 s = *(gvec)p;
  constexpr int QB = 8;                                   // runs whose loads are in flight at a time
  for (int q0 = 1; q0 < g.runs; q0 += QB) {
    f32x4 v[QB];
#pragma unroll
    for (int q = 0; q < QB; ++q)
      if (q0 + q < g.runs) v[q] = *(gvec)(p + (q0 + q) * step);
#pragma unroll
    for (int q = 0; q < QB; ++q)
      if (q0 + q < g.runs) s = s + v[q];
  }
  SmallOut to = small_out_of(g, to_load);
  small_store4(g, tr, tc, to, r, c, s);
}

// What the host's choice between them knows of a shape: microseconds per K step and tile, measured.
struct SmallKind {
  int es, tm, tn, bk, occ;
  double step;        // per workgroup where `occ` of them share every CU
  double alone;       // from a step to the next where a workgroup has a CU to itself
};
template <class SH>
constexpr SmallKind small_kind(double step, double alone) {
  return {SH::ES, SH::TM, SH::TN, SH::BK, SH::OCC, step, alone};
}

}  // namespace dmm
