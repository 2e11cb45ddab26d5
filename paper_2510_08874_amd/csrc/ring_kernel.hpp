// The bf16 loop of the kernels for small and skinny products (small_kernel.hpp): tiles of 32, 64 and 128 x 128.
//
// What bounds a 128 x 128 tile: a step of 64 k is 512 cycles of the matrix pipes, 64 KB of LDS reads (512
// cycles), 32 KB of LDS writes and 32 load instructions that take the CU's memory pipeline 16 to 20 cycles
// each.  Done one after the other, as a loop that stages operands in registers does them, they made 1900 cycles a
// step.  So here operands go straight into a ring of LDS stages, and the loads of a later step, the LDS reads and
// the matrix instructions of a step are interleaved by hand; a fragment is read one or two sub-steps of 16 k in front
// of its use.  One barrier per step: behind it the step's stage may be read, and the stage of the step
// before, whose reads every wave has waited for, may be filled again.
//
// A few rows against many columns are bound by memory: what counts is how much is on its way, so the
// 32-row tiles have three stages where each has a CU to itself, and two where three share one.
//
// The last step of a K-segment is loaded with the lanes whose chunks lie in it, zeros for the others.  A chunk that
// would reach past the segment (past the end of a tile buffer) is read as many elements further in front and moved
// to its place when it has landed.  (Loaded element by element, as rows shorter than a chunk still are, a tail cost 2.6 us.)
//
// Measured, kernel us, register-staged loop -> this one: 2048^3 38 -> 27 (a step 0.9 -> 0.5, of which the loads alone,
// 45 bytes per CU and cycle from L2, take 0.4), 1024 x 16384 x 1024 with the sum of its runs 59 (eight of them) -> 47 (four);
// us per call 1536^3 29 -> 18, 17 x 11429 x 13568 77 -> 60, 21 x 10368 x 31384 134 -> 106 (6.1 TB/s), 32 x 12288 x 49152 226
// either way (5.4 TB/s).
#pragma once

#include "small_kernel.hpp"

namespace dmm {

// TM x 128 tile of C, WM x WN waves over it; NST stages; OCC workgroups per CU
template <int TM_, int WM_, int NST_, int LAG_, int OCC_, int DESC_>
struct RingShape {
  static constexpr bool RING = true;
  static constexpr int ES = 2, TM = TM_, TN = 128, BK = 64, WM = WM_, WN = NW / WM_, WK = 1, OCC = OCC_;
  static constexpr int NST = NST_;
  static constexpr int LAG = LAG_;                               // sub-steps of 16 k from a fragment's read to its use
  static constexpr int A_BYTES = TM * BK * ES, STAGE_BYTES = A_BYTES + BK * TN * ES;
  static constexpr int DESC = DESC_;                             // bytes of LDS for slice descriptors, behind the stages
  static constexpr int T_PITCH = TN + 8;
  static constexpr int LDS = NST * STAGE_BYTES + DESC;
  static constexpr int MI = TM / WM / 32, NI = TN / WN / 32;     // 32 x 32 matrix tiles per wave
  static constexpr int LA = A_BYTES / 1024 / NW, LB = BK * TN * ES / 1024 / NW;   // 1 KB loads per wave and step
  static_assert(LDS >= TM * T_PITCH * 4, "the finished tile goes through the stages");
  static_assert(MI * NI <= 4 && LA >= 1 && NST >= 2 && NST <= 9 && (LA + LB) * (NST - 2) < 64, "accumulators, loads per wave, the counter of loads");
  static_assert(DESC >= (TM + TN / 8) * 24 + 4, "room for the slices of a segment");
};

// 16-byte chunk positions in a stage.  A: rows of 128 bytes, the chunk XOR-ed with a function of the row that
// spreads 16 rows reading one logical chunk over all banks.  B: k rows of 256 bytes, 64-byte segments XOR-ed
// with k & 3: the four k rows of a transposed read fall into different banks.
__device__ __forceinline__ int ring_a_swizzle(int row) { return (row >> 1) & 7; }

// The partial sums of a lane: accumulator registers a0 .. a63 by name (tile (i, j) of the wave's 2 x 2 owns
// 16 of them), as in the macro-tile kernels and for the same reason.
#define DMM_RING_ACC "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", "a10", "a11", "a12", "a13", "a14", "a15", "a16", "a17", "a18", "a19", "a20", "a21", "a22", "a23", "a24", "a25", "a26", "a27", "a28", "a29", "a30", "a31", "a32", "a33", "a34", "a35", "a36", "a37", "a38", "a39", "a40", "a41", "a42", "a43", "a44", "a45", "a46", "a47", "a48", "a49", "a50", "a51", "a52", "a53", "a54", "a55", "a56", "a57", "a58", "a59", "a60", "a61", "a62", "a63"

// all partial sums = 0: 0 * 0 + 0 through the matrix pipe
template <int T>
__device__ __forceinline__ void ring_acc_clear_tile(u32x4 z) {
  asm volatile("v_mfma_f32_32x32x16_bf16 a[%1:%2], %0, %0, 0" : : "v"(z), "n"(16 * T), "n"(16 * T + 15) : DMM_RING_ACC);
}
__device__ __forceinline__ void ring_acc_clear() {
  u32x4 z = {0u, 0u, 0u, 0u};
  asm volatile("s_nop 7" : "+v"(z));      // (the pipe must not read the zeros in the very next cycles)
  static_for<4>([&](auto tc) { ring_acc_clear_tile<decltype(tc)::value>(z); });
}

// A lane's slot of 16 bytes := the first n elements at p, zeros behind them.
__device__ __forceinline__ void ring_fill(lds_ptr slot, gptr p, int n) {
  *(__attribute__((address_space(3))) u32x4 *)slot = u32x4{0u, 0u, 0u, 0u};
#pragma clang loop unroll(disable)
  for (int e = 0; e < n; ++e)
    ((__attribute__((address_space(3))) unsigned short *)slot)[e] = ((const __attribute__((address_space(1))) unsigned short *)p)[e];
}

template <class SH>
__device__ __forceinline__ void ring_gemm(const SmallArgs &g, char *lds) {
  constexpr int BK = SH::BK, NST = SH::NST, STAGE_B = SH::STAGE_BYTES, A_B = SH::A_BYTES, MI = SH::MI, NI = SH::NI, PER = 8;
  constexpr int LA = SH::LA, LB = SH::LB, LT = LA + LB;   // 1 KB loads per wave and step
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = wave % SH::WN, wm = wave / SH::WN;
  const SmallPlace at = small_place(g);
  const SmallTile tr = g.rows[at.row], tc = g.cols[at.col];
  const int S = g.S, NR = g.NR, R = tr.pieces, Q = tc.pieces;
  const SmallStart start = g.starts[at.run];
  const int t0 = at.run * g.per, n = g.steps - t0 < g.per ? g.steps - t0 : g.per;   // at least 1: the host sees to it
  const unsigned lds_base = (unsigned)(uintptr_t)(lds_void_ptr)lds;
  const lds_ptr lds3 = (lds_ptr)(lds_void_ptr)lds;

  // ---- slice descriptors of a window of segments, in LDS -----------------------------------
  // (a segment switch that read them from memory would wait for all operands in flight: loads return in order)
  const int W = SH::DESC / ((R + Q) * (int)sizeof(PieceDev) + 4);
  PieceDev *const ad = (PieceDev *)(lds + NST * STAGE_B);
  PieceDev *const bd = ad + W * R;
  int32_t *const klen_s = (int32_t *)(bd + W * Q);
  int w0 = 0;                                             // the window's first segment
  auto stage_descriptors = [&](int first) {
    w0 = first;
    const int m = S - first < W ? S - first : W;
    if (R == 1) {
      for (int x = tid; x < m; x += NT) ad[x] = g.pa[(int64_t)tr.first * S + first + x];
    } else {
      for (int x = tid; x < m * R; x += NT) ad[x] = g.pa[(int64_t)(tr.first + x % R) * S + first + x / R];
    }
    if (Q == 1) {
      for (int x = tid; x < m; x += NT) bd[x] = g.pb[(int64_t)(first + x) * NR + tc.first];
    } else {
      for (int x = tid; x < m * Q; x += NT) bd[x] = g.pb[(int64_t)(first + x / Q) * NR + tc.first + x % Q];
    }
    for (int x = tid; x < m; x += NT) klen_s[x] = g.klen[first + x];
  };
  int seg = start.seg;
  const SmallOutLoad out_load = small_first_out<SH>(g, tr, tc);
  stage_descriptors(seg);

  // ---- this lane's chunks: load i of the wave fills KB number 4 i + wave of a stage's A and B -----------
  const int ak = ((lane & 7) ^ ring_a_swizzle(wave * 8 + (lane >> 3))) * PER;     // first k of its A chunks inside a step
  const int bn = ((((lane & 15) >> 2) ^ (lane >> 4)) << 2 | (lane & 3)) * PER;    // first column of its B chunks inside the tile
  const int bk = wave * 4 + (lane >> 4);                                          // k row of its first B chunk; 16 rows on to the next
  int ap[LA], bp;                                         // row pieces of its A rows, column piece of its B chunks
  unsigned arow[LA], bcol;                                 // row, byte column inside the slice
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    int row = (i * NW + wave) * 8 + (lane >> 3);
    row = tr.start + (row < tr.ext ? row : tr.ext - 1);   // (rows past the tile's end read its last row; never stored)
    int m0;
    ap[i] = small_piece(g.mc, tr, row, &m0) - tr.first;
    arow[i] = (unsigned)(row - m0);
  }
  {
    const int col = tc.start + (bn < tc.ext ? bn : 0);    // (columns past the tile's end: any; never stored)
    int n0;
    bp = small_piece(g.nc, tc, col, &n0) - tc.first;
    bcol = (unsigned)(col - n0) * 2;
  }
  __syncthreads();
  SmallOut out = small_out_of(g, out_load);

  // ---- cursor over the steps whose loads are issued ----------------------------------------
  // A step is loaded as it is, or as the segment's last one (K tail, chunks of B that would cross the end of a
  // tile buffer in the segment's last row), or, where that has no room to move, slowly.
  enum { PLAIN, LAST, SLOW };
  gptr pa[LA], pb[LB];
  int64_t bstep = 0;                                      // bytes a step advances in B
  int left = 0, krem = 0;                                 // steps (elements) of the segment left
  bool last_odd = false, last_slow = false, all_slow = false;   // what the segment's last step is, what all of them are
  bool b_past = false;                                    // some lane's chunk of B crosses the end of a tile buffer
  int b_back = 0;                                         // ... this lane's, by so many elements
  uint64_t a_mask = 0, b_mask[LB] = {};                    // the lanes that take part in the loads of the segment's last step
  const bool even = R == 1 && tr.ext == SH::TM;           // all A rows in one slice, 32 rows from one of a lane's to the next
  auto kind = [&]() __attribute__((always_inline)) -> int {
    return all_slow || (left == 1 && last_slow) ? SLOW : left == 1 && last_odd ? LAST : PLAIN;
  };
  auto open = [&](int kpos) __attribute__((always_inline)) {                             // the cursor enters segment `seg` at kpos
    if (seg - w0 >= W) {
      __syncthreads();
      stage_descriptors(seg);
      __syncthreads();
    }
    const int ls = seg - w0, klen = __builtin_amdgcn_readfirstlane(klen_s[ls]);
    krem = klen - kpos;
    left = (krem + BK - 1) / BK;
    const PieceDev d = bd[ls * Q + bp];
    if (even) {
      const PieceDev *e = ad + ls;
      const int64_t pitch32 = (int64_t)e->pitch * 32;
      pa[0] = (gptr)e->ptr + ((int64_t)arow[0] * e->pitch + (kpos + ak) * 2);
#pragma unroll
      for (int i = 1; i < LA; ++i) pa[i] = pa[i - 1] + pitch32;
    } else {
#pragma unroll
      for (int i = 0; i < LA; ++i) {
        const PieceDev *e = ad + ls * R + ap[i];
        pa[i] = (gptr)e->ptr + ((int64_t)arow[i] * e->pitch + (kpos + ak) * 2);
      }
    }
    const int64_t pitch = d.pitch;
    bstep = pitch * BK;
    pb[0] = (gptr)d.ptr + ((kpos + bk) * pitch + bcol);
#pragma unroll
    for (int i = 1; i < LB; ++i) pb[i] = pb[i - 1] + pitch * 16;
    // A chunk of B crosses the end of its tile buffer in the segment's last row at most, if rows are 16 bytes and more.
    // It is read as many elements further in front as cross, a chunk of A with a K tail likewise, and moved when it has landed.
    const int64_t room = d.room - (klen - 1) * pitch - bcol;
    b_back = room < 16 ? 8 - (int)(room >> 1) : 0;
    b_past = __builtin_amdgcn_ballot_w64(room < 16) != 0;
    last_odd = klen % BK != 0 || b_past;
    last_slow = (klen < PER && klen % BK != 0) || __builtin_amdgcn_ballot_w64((klen - 1) * pitch + bcol < 2 * b_back) != 0;
    all_slow = __builtin_amdgcn_ballot_w64(pitch < 16) != 0;
  };
  // The cursor has come to a step: its segment if it is the first, what is different if it is the last.
  auto arrive = [&]() __attribute__((always_inline)) {
    if (left == 0) {
      ++seg;
      open(0);
    }
    if (kind() != LAST) return;
    const int valid = krem - ak;
    a_mask = __builtin_amdgcn_ballot_w64(valid > 0);
#pragma unroll
    for (int i = 0; i < LA; ++i)
      if (valid > 0 && valid < PER) pa[i] -= (PER - valid) * 2;
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      if (bk + 16 * i == krem - 1) pb[i] -= b_back * 2;
      b_mask[i] = __builtin_amdgcn_ballot_w64(bk + 16 * i < krem);
    }
  };
  // Per step in flight a byte of what is to be moved when it has landed: elements of A's row inside the segment if
  // no multiple of eight, 128 if chunks of B are; and this lane's chunk of B, and by how many elements.
  typedef std::conditional_t<(NST > 5), uint64_t, unsigned> Bytes;
  Bytes moves = 0, b_moves = 0;
  auto pass = [&]() __attribute__((always_inline)) {      // the loads of the cursor's step have been issued
    moves <<= 8;
    b_moves <<= 8;
    if (kind() == LAST) {
      moves |= (unsigned)((krem % PER ? krem : 0) | (b_past ? 128 : 0));
#pragma unroll
      for (int i = 0; i < LB; ++i)
        if (bk + 16 * i == krem - 1) b_moves |= (unsigned)(b_back | i << 4);
    }
    --left;
    krem -= BK;
  };
  auto slow_step = [&](int stage) __attribute__((always_inline)) {
    const int ls = seg - w0, kpos = __builtin_amdgcn_readfirstlane(klen_s[ls]) - krem;
    const unsigned to = __builtin_amdgcn_readfirstlane(lds_base + stage * STAGE_B + wave * 1024);
    const lds_ptr slot = lds3 + stage * STAGE_B + wave * 1024 + lane * 16;
    const int valid = krem - ak;
#pragma unroll
    for (int i = 0; i < LA; ++i) {
      const bool ok = valid >= PER;                       // (then the chunk lies inside the segment)
      const uint64_t mask = __builtin_amdgcn_ballot_w64(ok);
      load_to_lds_16_masked_v<0>(pa[i], to + i * (NW * 1024), (unsigned)mask, (unsigned)(mask >> 32));
      if (!ok) ring_fill(slot + i * (NW * 1024), pa[i], valid);
      pa[i] += BK * 2;
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      const PieceDev d = bd[ls * Q + bp];
      const int64_t room = d.room - ((int64_t)(kpos + bk + 16 * i) * d.pitch + bcol);
      const bool in = bk + 16 * i < krem, ok = in && room >= 16;
      const uint64_t mask = __builtin_amdgcn_ballot_w64(ok);
      load_to_lds_16_masked_v<0>(pb[i], to + A_B + i * (NW * 1024), (unsigned)mask, (unsigned)(mask >> 32));
      if (!ok) ring_fill(slot + A_B + i * (NW * 1024), pb[i], in ? (int)(room >> 1) : 0);
      pb[i] += bstep;
    }
  };
  auto place = [&](int stage) -> unsigned { return __builtin_amdgcn_readfirstlane(lds_base + stage * STAGE_B + wave * 1024); };
  // number j of the cursor step's loads, into the stage at `to`
  auto load = [&](auto kind_tag, auto jc, unsigned to) __attribute__((always_inline)) {
    constexpr int j = decltype(jc)::value, IMM = j < LA ? j * (NW * 1024) : A_B + (j - LA) * (NW * 1024);
    gptr &p = j < LA ? pa[j < LA ? j : 0] : pb[j < LA ? 0 : j - LA];
    if constexpr (decltype(kind_tag)::value == LAST) {
      const uint64_t mask = j < LA ? a_mask : b_mask[j < LA ? 0 : j - LA];
      load_to_lds_16_masked_v<IMM>(p, to, (unsigned)mask, (unsigned)(mask >> 32));   // (the address is not needed any more)
    } else {
      load_to_lds_16_plain_v<IMM>(p, to);
      p += j < LA ? (int64_t)(BK * 2) : bstep;
    }
  };
  auto zero_tail = [&](int stage) __attribute__((always_inline)) {     // what lies behind the segment in its last step
    const lds_ptr slot = lds3 + stage * STAGE_B + wave * 1024 + lane * 16;
    const u32x4 zero = {0u, 0u, 0u, 0u};
    if (ak >= krem) {
#pragma unroll
      for (int i = 0; i < LA; ++i) *(__attribute__((address_space(3))) u32x4 *)(slot + i * (NW * 1024)) = zero;
    }
#pragma unroll
    for (int i = 0; i < LB; ++i)
      if (bk + 16 * i >= krem) *(__attribute__((address_space(3))) u32x4 *)(slot + A_B + i * (NW * 1024)) = zero;
  };

  // ---- fragments ----------------------------------------------------------------------------
  constexpr int SUB = BK / 16;                            // sub-steps
  constexpr int LAG = SH::LAG, SETS = LAG == 1 ? 2 : 4;   // fragments of SETS sub-steps are held
  bf16x8 fa[SETS][MI];
  union BFrag { short4_t h[2]; bf16x8 v; } fb[SETS][NI];
  const bf16x8 none = {};
#pragma unroll
  for (int q = 0; q < SETS; ++q) {
#pragma unroll
    for (int i = 0; i < MI; ++i) fa[q][i] = none;
#pragma unroll
    for (int j = 0; j < NI; ++j) fb[q][j].v = none;
  }
  ring_acc_clear();
  const int half = lane >> 5, gr = lane >> 4, li = lane & 15;
  int a_at[SUB], b_at[NI];                                // this lane's places in a stage
#pragma unroll
  for (int q = 0; q < SUB; ++q) {
    const int row = wm * (MI * 32) + (lane & 31);
    a_at[q] = row * (BK * 2) + ((q * 2 + half) ^ ring_a_swizzle(row)) * 16;
  }
#pragma unroll
  for (int j = 0; j < NI; ++j) {
    const int k = (gr >> 1) * 8 + (li >> 2), col = wn * (NI * 32) + j * 32 + (gr & 1) * 16 + (li & 3) * 4, c = col >> 3;
    b_at[j] = A_B + k * 256 + (((c >> 2) ^ (k & 3)) << 2 | (c & 3)) * 16 + (col & 7) * 2;
  }
  auto read_a = [&](lds_ptr st, int q, int i) __attribute__((always_inline)) {
    fa[q % SETS][i] = *(const __attribute__((address_space(3))) bf16x8 *)(st + a_at[q] + i * (32 * BK * 2));
  };
  auto read_b = [&](lds_ptr st, int q, int j) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
      fb[q % SETS][j].h[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(st + b_at[j] + (q * 16 + 4 * h) * 256));
  };
  auto mfma = [&](auto qc, auto ic, auto jc) __attribute__((always_inline)) {
    constexpr int q = decltype(qc)::value, i = decltype(ic)::value, j = decltype(jc)::value;
    constexpr int T = i * NI + j, X = q % SETS;
    const bf16x8 x = fa[X][i], y = fb[X][j].v;
    asm volatile("v_mfma_f32_32x32x16_bf16 a[%2:%3], %0, %1, a[%2:%3]" : : "v"(x), "v"(y), "n"(16 * T), "n"(16 * T + 15)
                 : "memory", DMM_RING_ACC);
  };

  // ---- the K loop ------------------------------------------------------------------------
  constexpr std::integral_constant<int, PLAIN> plain{};
  constexpr std::integral_constant<int, LAST> last{};
  constexpr std::integral_constant<int, -1> nothing{};
  open(start.kpos);
  arrive();
#pragma clang loop unroll(disable)
  for (int t = 0; t < NST - 1; ++t) {
    if (t < n) {
      const int k = kind();
      if (k == PLAIN) {
        static_for<LT>([&](auto jc) __attribute__((always_inline)) { load(plain, jc, place(t)); });
      } else if (k == LAST) {
        static_for<LT>([&](auto jc) __attribute__((always_inline)) { load(last, jc, place(t)); });
        zero_tail(t);
      } else {
        slow_step(t);
      }
      pass();
      if (t + 1 < n) arrive();
    } else {
      moves <<= 8;
      b_moves <<= 8;
    }
  }
  auto iteration = [&](auto kind_tag, int stage, unsigned to) __attribute__((always_inline)) {
    constexpr bool LOADS = decltype(kind_tag)::value >= 0;
    const lds_ptr st = lds3 + stage * STAGE_B;
    static_for<SUB>([&](auto qc) __attribute__((always_inline)) {
      constexpr int q = decltype(qc)::value;
      constexpr std::integral_constant<int, (q + SUB - LAG) % SUB> m{};   // the sub-step multiplied (of the step before for q < LAG)
      constexpr int SLOTS = MI * NI, FIRST = q * LT / SUB, LOADS_Q = (q + 1) * LT / SUB - FIRST;
      static_for<SLOTS>([&](auto xc) __attribute__((always_inline)) {
        constexpr int x = decltype(xc)::value;
        mfma(m, std::integral_constant<int, x % MI>{}, std::integral_constant<int, x / MI>{});
        // one A and one B fragment behind the first matrix instruction, one of the others behind each of the next
        if constexpr (x == 0) {
          read_a(st, q, 0);
          read_b(st, q, 0);
        } else if constexpr (x < MI) {
          read_a(st, q, x);
        } else if constexpr (x - MI + 1 < NI) {
          read_b(st, q, x - MI + 1);
        }
        if constexpr (LOADS)
          static_for<(x + 1) * LOADS_Q / SLOTS - x * LOADS_Q / SLOTS>([&](auto lc) __attribute__((always_inline)) {
            load(kind_tag, std::integral_constant<int, FIRST + x * LOADS_Q / SLOTS + decltype(lc)::value>{}, to);
          });
        DMM_SCHED_BARRIER;
      });
    });
  };
  int stage = 0, t = 0;
  auto next_stage = [&] {
    ++t;
    stage = __builtin_amdgcn_readfirstlane(stage + 1 == NST ? 0 : stage + 1);
  };
  while (t < n) {
    // step t is in: its loads have landed where no more than those of the steps behind it are under way
    const int behind = n - 1 - t;
    if (behind >= NST - 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LT * (NST - 2)) : "memory");
    static_for<NST - 2>([&](auto xc) {
      if (behind == decltype(xc)::value) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LT * decltype(xc)::value) : "memory");
    });
    const unsigned move = __builtin_amdgcn_readfirstlane((unsigned)(moves >> (8 * (NST - 2))) & 255u);
    if (__builtin_expect(move != 0, 0)) {
      typedef __attribute__((address_space(3))) u32x4 *slot_ptr;
      const lds_ptr slot = lds3 + stage * STAGE_B + wave * 1024 + lane * 16;
      const int valid = (int)(move & 127u) - ak;
      if (valid > 0 && valid < PER) {
#pragma unroll
        for (int i = 0; i < LA; ++i) {
          const slot_ptr p = (slot_ptr)(slot + i * (NW * 1024));
          *p = drop_first(*p, PER - valid);
        }
      }
      const unsigned b = (unsigned)(b_moves >> (8 * (NST - 2))) & 255u;
      if (b & 15u) {
        const slot_ptr p = (slot_ptr)(slot + A_B + (b >> 4) * (NW * 1024));
        *p = drop_first(*p, (int)(b & 15u));
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    const int to = stage == 0 ? NST - 1 : stage - 1;      // the stage of the step before, free now
    const int ahead = n - (t + NST - 1);                  // steps whose loads have not been issued
    if (ahead > 0) {
      const int k = kind();
      if (k == PLAIN) {
        iteration(plain, stage, place(to));
      } else if (k == LAST) {
        zero_tail(to);
        iteration(last, stage, place(to));
      } else {
        slow_step(to);
        iteration(nothing, stage, 0u);
      }
      pass();
      if (ahead > 1) arrive();                            // (in front of the barrier: nobody waits for it)
    } else {
      iteration(nothing, stage, 0u);
      moves <<= 8;
      b_moves <<= 8;
    }
    next_stage();
    // Then as many steps as need none of this: what is loaded meanwhile is followed by a step of the same
    // segment and is loaded as it is, and no step in flight has something to be moved.
    int quiet = left - 1 < ahead - 1 ? left - 1 : ahead - 1;
    quiet = __builtin_amdgcn_readfirstlane(moves != 0 || all_slow ? 0 : quiet);
    if (quiet <= 0) continue;
    left -= quiet;
    krem -= quiet * BK;
    const bool more = quiet < ahead - 1;
#pragma clang loop unroll(disable)
    for (; quiet > 0; --quiet) {
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(LT * (NST - 2)) : "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      iteration(plain, stage, place(stage == 0 ? NST - 1 : stage - 1));
      next_stage();
    }
    if (more) arrive();
  }
  static_for<LAG>([&](auto qc) {
    static_for<MI>([&](auto ic) { static_for<NI>([&](auto jc) { mfma(std::integral_constant<int, SUB - LAG + decltype(qc)::value>{}, ic, jc); }); });
  });
  // (the last results leave the matrix pipe before other instructions read them)
  asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");
  small_epilogue<SH>(g, at, tr, tc, out, lds3, [](auto ic, auto jc, auto ec) {
    return acc_read<16 * (decltype(ic)::value * NI + decltype(jc)::value) + decltype(ec)::value>();
  }, wm, wn, 0);
}

// The launch: either loop.
template <class SH>
__global__ __launch_bounds__(NT, SH::OCC) void small_gemm_kernel(const SmallArgs g) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  if constexpr (SH::RING) ring_gemm<SH>(g, lds);
  else if constexpr (!SH::SPLIT) staged_gemm<SH>(g, lds, threadIdx.x);
  else if (staged_gemm<SH>(g, lds, threadIdx.x)) {
    typedef SmallF32Whole Part;
    static_assert(SH::LDS >= Part::LDS && SH::TM == Part::TM * Part::PARTS && SH::TN == Part::TN && SH::BK == Part::BK, "the same launch");
    const int ext = g.rows[small_place(g).row].ext;
#pragma clang loop unroll(disable)
    for (int part = 0; part * Part::TM < ext; ++part) {
      int tid = threadIdx.x;
      asm volatile("" : "+v"(tid));      // (nothing worked out for this loop is kept in registers through the other one)
      if (part > 0) __syncthreads();     // (the part before has left the LDS)
      staged_gemm<Part>(g, lds, tid, part);
    }
  }
}

// The "deep" ones run where every workgroup has a CU to itself (us per call, two stages -> deep: 2048^3 33 -> 28, 21 x 10368
// x 31384 147 -> 109; with more workgroups the other way round: 2560^3 46 and 52, 32 x 12288 x 49152 in two runs 225 and 228).
//                TM  WM NST LAG OCC
typedef RingShape<128, 2, 4, 2, 1, 24 * 1024> RingDeep;
typedef RingShape<128, 2, 2, 1, 2, 16 * 1024> RingPair;
typedef RingShape<64, 2, 3, 1, 2, 8 * 1024> RingHalf;
typedef RingShape<32, 1, 3, 1, 2, 16 * 1024> RingSkinnyDeep;
typedef RingShape<32, 1, 2, 1, 3, 12 * 1024> RingSkinny;

}  // namespace dmm
