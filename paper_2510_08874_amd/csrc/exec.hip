// Device-facing half of the library (gfx950 only): the entry points that turn a plan plus
// tile pointers into device work tables and launch the grouped GEMM (gemm_kernel.hpp), the
// replica sum, the replica broadcast and the measurement aids (aux_kernels.hpp), on top of the
// pools and the uploader of device_state.hpp.
#include <hip/hip_runtime.h>
#include <rocprofiler-sdk-roctx/roctx.h>

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <utility>
#include <vector>

#include "aux_kernels.hpp"
#include "device_state.hpp"
#include "gemm_kernel.hpp"
#include "gemm_launch.hpp"
#include "pack_kernel.hpp"
#include "plan_internal.h"
#include "ring_kernel.hpp"
#include "small_kernel.hpp"

namespace dmm {

namespace {

static_assert(kMaxPieces == PMAX && kDescBytes == DESC_LDS - DESC_GEO && sizeof(PieceDev) == 24 &&
                  kPieceAlign * 2 >= 16 && 2 * (PMAX + 1) * 4 <= 128 && 128 + PMAX * PMAX * 24 <= DESC_GEO && kMacroTile == BM && kMacroTile == BN,
              "the planner's limits for merged macro-tiles describe the kernel's descriptor area");

// A named range on the calling thread for tracing tools (rocprofv3 --marker-trace), closed when
// the object goes out of scope: "dmm_execute" with "tables" (host assembly of the work tables and
// their upload), "gemm" and "replica_sum" (the launches) inside it, "dmm_reduce_replicas", ...
struct TraceRange {
  explicit TraceRange(const char *name) { roctxRangePushA(name); }
  ~TraceRange() { end(); }
  void end() {                        // (ranges nest: end them in reverse order of their construction)
    if (open_) roctxRangePop();
    open_ = false;
  }
  TraceRange(const TraceRange &) = delete;
  TraceRange &operator=(const TraceRange &) = delete;

 private:
  bool open_ = true;
};

// Whether the current device lets one workgroup have the stages plus the descriptor area (the
// merged macro-tile kernels); decided in ensure_state.
bool g_comp_ok[64] = {};

int ensure_state(dmm_plan_t *P) {
  // the kernels' LDS size has to be allowed once per device
  static std::mutex mu;
  static bool done[64] = {};
  int device = 0;
  DMM_HIP(hipGetDevice(&device));
  if (device < 0 || device >= 64) return DMM_EINVAL;
  {
    std::lock_guard<std::mutex> g(mu);
    if (!done[device]) {
      DMM_HIP(gemm_allow_lds_0());
      DMM_HIP(gemm_allow_lds_1());
      DMM_HIP(gemm_allow_lds_2());
      DMM_HIP(gemm_allow_lds_3());
      DMM_HIP(small_allow_lds());
      const bool ok = gemm_allow_lds_4() == hipSuccess && gemm_allow_lds_5() == hipSuccess;
      if (!ok) (void)hipGetLastError();
      g_comp_ok[device] = ok;
      done[device] = true;
    }
  }
  if (!P->dev) {
    P->dev = new (std::nothrow) DeviceState;
    if (!P->dev) return DMM_ENOMEM;
  }
  return DMM_OK;
}

// Compute units of the current device (queried once per device).
int device_cus(int *out) {
  static std::mutex mu;
  static int cus[64] = {};
  int dev = 0;
  DMM_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64) return DMM_EINVAL;
  std::lock_guard<std::mutex> g(mu);
  if (!cus[dev]) {
    hipDeviceProp_t prop;
    DMM_HIP(hipGetDeviceProperties(&prop, dev));
    cus[dev] = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 1;
  }
  *out = cus[dev];
  return DMM_OK;
}

int timing_events(hipEvent_t ev[2]) {
  for (int i = 0; i < 2; ++i)
    if (!ev[i]) DMM_HIP(hipEventCreate(&ev[i]));
  return DMM_OK;
}

// ld >= width for every non-empty tile of a matrix
int check_lds(const Grid &G, const int64_t *ld) {
  for (int32_t rep = 0; rep < G.c; ++rep)
    for (int32_t ti = 0; ti < G.gr; ++ti)
      for (int32_t tj = 0; tj < G.gc; ++tj) {
        const int64_t w = G.cc[tj + 1] - G.cc[tj], h = G.rc[ti + 1] - G.rc[ti];
        if (w > 0 && h > 0 && ld[G.table_index(rep, ti, tj)] < w) return DMM_ELD;
      }
  return DMM_OK;
}

// The replica sum in two halves, so that dmm_execute can put the table upload in front of the
// GEMM launch and nothing but the launch itself behind it.
// Appends the replica sum's tables to *h at byte offset `base` (a multiple of 8).
int build_reduce(dmm_plan_t *P, void *const *c_tiles, const int64_t *c_ld, int32_t origin, std::vector<char> *hp,
                 size_t base, RedLaunch *L) {
  const Grid &C = P->C;
  L->n_items = 0;
  if (C.c <= 1) return DMM_OK;
  const int nparts = C.c;
  std::vector<RedTile> tiles;
  std::vector<RedItem> items;
  std::vector<const float *> parts;
  std::vector<int64_t> part_ld;
  bool vec_ok = true;
  for (int32_t ti = 0; ti < C.gr; ++ti)
    for (int32_t tj = 0; tj < C.gc; ++tj) {
      const int64_t rows = C.rc[ti + 1] - C.rc[ti], cols = C.cc[tj + 1] - C.cc[tj];
      if (rows <= 0 || cols <= 0) continue;
      RedTile t;
      const int64_t oi = C.table_index(origin, ti, tj);
      t.out = (float *)c_tiles[oi];
      t.ldo = c_ld[oi];
      t.part_begin = (int64_t)parts.size();
      t.rows = (int32_t)rows;
      t.cols = (int32_t)cols;
      if (!t.out) return DMM_EINVAL;
      if (((uintptr_t)t.out & 15) || (t.ldo & 3) || (cols & 3)) vec_ok = false;
      for (int32_t rep = 0; rep < nparts; ++rep) {
        const int64_t pi = C.table_index(rep, ti, tj);
        const float *pp = (const float *)c_tiles[pi];
        if (!pp) return DMM_EINVAL;
        if (((uintptr_t)pp & 15) || (c_ld[pi] & 3)) vec_ok = false;
        parts.push_back(pp);
        part_ld.push_back(c_ld[pi]);
      }
      // blocks of rows holding about RED_ELEMS elements each
      int64_t per = (RED_ELEMS + cols - 1) / cols;
      if (per < 1) per = 1;
      for (int64_t r = 0; r < rows; r += per) {
        RedItem it;
        it.tile = (int32_t)tiles.size();
        it.row0 = (int32_t)r;
        it.nrows = (int32_t)(rows - r < per ? rows - r : per);
        it.pad = 0;
        items.push_back(it);
      }
      tiles.push_back(t);
    }
  if (items.empty()) return DMM_OK;
  // items | tiles | part pointers | part lds   (all 8-byte aligned)
  const size_t o_items = base;
  const size_t o_tiles = o_items + items.size() * sizeof(RedItem);
  const size_t o_parts = o_tiles + tiles.size() * sizeof(RedTile);
  const size_t o_lds = o_parts + parts.size() * sizeof(void *);
  const size_t total = o_lds + part_ld.size() * sizeof(int64_t);
  std::vector<char> &h = *hp;
  h.resize(total);
  std::memcpy(h.data() + o_items, items.data(), items.size() * sizeof(RedItem));
  std::memcpy(h.data() + o_tiles, tiles.data(), tiles.size() * sizeof(RedTile));
  std::memcpy(h.data() + o_parts, parts.data(), parts.size() * sizeof(void *));
  std::memcpy(h.data() + o_lds, part_ld.data(), part_ld.size() * sizeof(int64_t));
  L->n_items = items.size();
  L->o_items = o_items;
  L->o_tiles = o_tiles;
  L->o_parts = o_parts;
  L->o_lds = o_lds;
  L->nparts = nparts;
  L->vec_ok = vec_ok;
  return DMM_OK;
}

// The replica sum's (or the broadcast's) tables alone, uploaded through the plan's second buffer.
int stage_reduce(dmm_plan_t *P, void *const *c_tiles, const int64_t *c_ld, int32_t origin, hipStream_t stream,
                 RedLaunch *L) {
  std::vector<char> &h = P->dev->host;
  h.clear();
  int rc = build_reduce(P, c_tiles, c_ld, origin, &h, 0, L);
  if (rc || L->n_items == 0) return rc;
  if ((rc = P->dev->red_table.upload(h.data(), h.size(), stream, P->dev->uses))) return rc;
  L->dev_base = P->dev->red_table.dev();
  return DMM_OK;
}

// *marked: `behind` (if any) has been recorded by the launch.
int fire_reduce(dmm_plan_t *P, const RedLaunch &L, hipStream_t stream, bool timed, hipEvent_t behind, bool *marked) {
  if (L.n_items == 0) return DMM_OK;
  int rc;
  char *d = L.dev_base;
  const size_t o_items = L.o_items, o_tiles = L.o_tiles, o_parts = L.o_parts, o_lds = L.o_lds;
  const int nparts = L.nparts;
  const bool vec_ok = L.vec_ok;
  if (timed) {
    if ((rc = timing_events(P->dev->t_red))) return rc;
    DMM_HIP(hipEventRecord(P->dev->t_red[0], stream));
  }
  *marked = launch_behind(behind, reduce_replicas_kernel, (unsigned)L.n_items, RED_NT, 0, stream, (const RedItem *)(d + o_items),
                          (const RedTile *)(d + o_tiles), (const float *const *)(d + o_parts), (const int64_t *)(d + o_lds), nparts,
                          vec_ok ? 1 : 0);
  DMM_HIP(hipGetLastError());
  if (timed) {
    DMM_HIP(hipEventRecord(P->dev->t_red[1], stream));
    P->dev->red_timed = true;
  }
  return DMM_OK;
}

// Device tables of the merged macro-tiles, appended to *hp (empty on entry):
//   CompItemDev[items] | PieceDev a[...] | PieceDev b[...] | PieceDev c[...] | int32 klen[...]
// A slices are numbered (replica, row interval, segment), B slices (replica, segment, column
// interval), C slices (replica, row interval, column interval).
// K steps a run of a macro-tile cut along K has at least (see build_group_exec): 64 with bf16
// operands, measured; a K step of fp32 operands keeps the matrix pipes busy eight times as long
// (128 MFMAs of 64 cycles against 32 of 32), so there a run of the same duration is 8 steps.
constexpr int32_t MIN_RUN = 64;
inline int32_t min_run_steps(int64_t es) { return es == 4 ? MIN_RUN / 8 : MIN_RUN; }

// Scratch buffer of the plan for `need` bytes of partial tiles; orders this call behind the plan's earlier ones.
int acquire_split_buffer(dmm_plan_t *P, size_t need, hipStream_t stream) {
  // the scratch buffer is shared by all calls on this plan: order this call behind the others
  // (a no-op when all are on the same stream)
  int rc = P->dev->uses.order(stream);
  if (rc) return rc;
  if (need > P->dev->split_cap) {
    // growing: earlier calls on this plan may still use the old buffer
    if (P->dev->split_buf) {
      DMM_HIP(hipStreamSynchronize(stream));
      scratch_pool().release(&P->dev->split_buf, &P->dev->split_cap);
    }
    return scratch_pool().acquire(need, &P->dev->split_buf, &P->dev->split_cap);
  }
  return DMM_OK;
}

int build_merged_tables(dmm_plan_t *P, int64_t es, int64_t bk, int64_t c_es, const void *const *a_tiles,
                        const int64_t *a_ld, const void *const *b_tiles, const int64_t *b_ld, void *const *c_tiles,
                        const int64_t *c_ld, int cus, bool uncut, hipStream_t stream, std::vector<char> *hp, MergedLaunch *L) {
  const Merged &G = P->merged;
  const Grid &A = P->A, &B = P->B, &C = P->C;
  const size_t MR = G.mc.size() - 1, NR = G.nc.size() - 1;
  // tile that holds a cut point (the last tile whose lower cut is not above it: skips empty tiles)
  auto holder = [](const std::vector<int64_t> &cuts, int64_t x) {
    return (int32_t)(std::upper_bound(cuts.begin(), cuts.end() - 1, x) - cuts.begin()) - 1;
  };
  std::vector<int32_t> a_ti(MR), c_ti(MR), b_tj(NR), c_tj(NR);
  for (size_t i = 0; i < MR; ++i) { a_ti[i] = holder(A.rc, G.mc[i]); c_ti[i] = holder(C.rc, G.mc[i]); }
  for (size_t j = 0; j < NR; ++j) { b_tj[j] = holder(B.cc, G.nc[j]); c_tj[j] = holder(C.cc, G.nc[j]); }
  std::vector<PieceDev> pa, pb, pc;
  std::vector<int32_t> klen;
  std::vector<int32_t> a0(G.reps.size()), b0(G.reps.size()), c0(G.reps.size()), k0(G.reps.size()), steps(G.reps.size());
  std::vector<std::vector<int32_t>> steps_before(G.reps.size());   // K steps in front of every segment, per replica
  auto piece = [](const void *base, int64_t ld, int64_t r, int64_t c, int64_t h, int64_t w, int64_t esz) {
    PieceDev d;
    const int64_t off = r * ld + c;
    d.ptr = (const char *)base + off * esz;
    d.room = ((h - 1) * ld + w - off) * esz;
    d.pitch = (uint32_t)(ld * esz);
    d.pad = 0;
    return d;
  };
  for (size_t rep = 0; rep < G.reps.size(); ++rep) {
    const MergedRep &R = G.reps[rep];
    const size_t S = R.kc.size() - 1;
    a0[rep] = (int32_t)pa.size();
    b0[rep] = (int32_t)pb.size();
    c0[rep] = (int32_t)pc.size();
    k0[rep] = (int32_t)klen.size();
    std::vector<int32_t> a_tj(S), b_ti(S);
    int32_t nsteps = 0;
    for (size_t s = 0; s < S; ++s) {
      a_tj[s] = holder(A.cc, R.kc[s]);
      b_ti[s] = holder(B.rc, R.kc[s]);
      klen.push_back((int32_t)(R.kc[s + 1] - R.kc[s]));
      steps_before[rep].push_back(nsteps);
      nsteps += (int32_t)((R.kc[s + 1] - R.kc[s] + bk - 1) / bk);
    }
    steps_before[rep].push_back(nsteps);
    steps[rep] = nsteps;
    for (size_t i = 0; i < MR; ++i)
      for (size_t s = 0; s < S; ++s) {
        const int32_t ti = a_ti[i], tj = a_tj[s];
        const int64_t idx = A.table_index(R.a_rep, ti, tj);
        if (!a_tiles[idx]) return DMM_EINVAL;
        pa.push_back(piece(a_tiles[idx], a_ld[idx], G.mc[i] - A.rc[ti], R.kc[s] - A.cc[tj], A.rc[ti + 1] - A.rc[ti],
                           A.cc[tj + 1] - A.cc[tj], es));
      }
    for (size_t s = 0; s < S; ++s)
      for (size_t j = 0; j < NR; ++j) {
        const int32_t ti = b_ti[s], tj = b_tj[j];
        const int64_t idx = B.table_index(R.b_rep, ti, tj);
        if (!b_tiles[idx]) return DMM_EINVAL;
        pb.push_back(piece(b_tiles[idx], b_ld[idx], R.kc[s] - B.rc[ti], G.nc[j] - B.cc[tj], B.rc[ti + 1] - B.rc[ti],
                           B.cc[tj + 1] - B.cc[tj], es));
      }
    for (size_t i = 0; i < MR; ++i)
      for (size_t j = 0; j < NR; ++j) {
        const int32_t ti = c_ti[i], tj = c_tj[j];
        const int64_t idx = C.table_index((int32_t)rep, ti, tj);
        if (!c_tiles[idx]) return DMM_EINVAL;
        pc.push_back(piece(c_tiles[idx], c_ld[idx], G.mc[i] - C.rc[ti], G.nc[j] - C.cc[tj], C.rc[ti + 1] - C.rc[ti],
                           C.cc[tj + 1] - C.cc[tj], c_es));
      }
  }
  std::vector<CompItemDev> items(G.items.size());
  for (size_t x = 0; x < G.items.size(); ++x) {
    const MergedItem &w = G.items[x];
    const size_t S = G.reps[(size_t)w.rep].kc.size() - 1;
    CompItemDev d;
    std::memset(&d, 0, sizeof(d));
    d.m_ext = w.m_ext;
    d.n_ext = w.n_ext;
    d.R = w.R;
    d.Q = w.Q;
    d.S = (int32_t)S;
    d.nsteps = steps[(size_t)w.rep];
    d.c_es = (int32_t)c_es;
    d.a_first = a0[(size_t)w.rep] + w.mr0 * (int32_t)S;
    d.a_stride = (int32_t)S;
    d.b_first = b0[(size_t)w.rep] + w.nr0;
    d.b_stride = (int32_t)NR;
    d.c_first = c0[(size_t)w.rep] + w.mr0 * (int32_t)NR + w.nr0;
    d.c_stride = (int32_t)NR;
    d.k_first = k0[(size_t)w.rep];
    for (int32_t p = 0; p <= w.R; ++p) d.rb[p] = (int32_t)(G.mc[(size_t)(w.mr0 + p)] - w.m0);
    for (int32_t q = 0; q <= w.Q; ++q) d.cb[q] = (int32_t)(G.nc[(size_t)(w.nr0 + q)] - w.n0);
    items[x] = d;
  }
  // K-split of the last round, as for the per-group macro-tiles: the last W % cus macro-tiles, if
  // they are at most half a round, are cut into runs of at least min_run_steps() K steps; every run writes
  // a plain partial tile to the scratch buffer, and the partial tiles of a macro-tile are added up
  // piece by piece (one FixItem per row piece and column piece, each with its own C slice).
  std::vector<FixItem> fixes;
  size_t n_runs = 0;
  const size_t n_whole = items.size();
  // one FixItem per (row piece, column piece) of a macro-tile whose `runs` partial tiles start at
  // partial tile number `first_part`
  auto fix_pieces = [&](const CompItemDev &whole, size_t first_part, int32_t runs) {
    for (int32_t p = 0; p < whole.R; ++p)
      for (int32_t q = 0; q < whole.Q; ++q) {
        const int32_t r0 = std::max(whole.rb[p], 0), r1 = std::min(whole.rb[p + 1], whole.m_ext);
        const int32_t q0 = std::max(whole.cb[q], 0), q1 = std::min(whole.cb[q + 1], whole.n_ext);
        const PieceDev &cp = pc[(size_t)(whole.c_first + p * whole.c_stride + q)];
        FixItem f;
        f.dst = (void *)(cp.ptr + (int64_t)(r0 - whole.rb[p]) * cp.pitch + (int64_t)(q0 - whole.cb[q]) * c_es);
        f.ldc = (int64_t)cp.pitch / c_es;
        f.parts = (const float *)(uintptr_t)(first_part * sizeof(float) * BM * BN);   // offset for now
        f.m_ext = r1 - r0;
        f.n_ext = q1 - q0;
        f.nparts = runs;
        f.c_es = (int32_t)c_es;
        f.row0 = r0;
        f.col0 = q0;
        fixes.push_back(f);
      }
  };
  // Cutting macro-tiles along K.  Two reasons, one mechanism: (a) the plan asks for it (G.window:
  // the descriptors of all of a macro-tile's segments would not fit beside eight pieces per axis),
  // (b) the macro-tiles fill the device badly: at most half a round of them in all, or a last round
  // that is at most half full (then its macro-tiles only), as for the per-group macro-tiles.  A run
  // is a range of at least min_run_steps() K steps; its workgroup stages the descriptors of the segments
  // the range touches only, starts `first_step` steps into the first of them and writes a plain
  // partial tile.  Launch order: the first run of every macro-tile in the macro-tiles' own order,
  // then the second of every one, ...
  auto desc_bytes = [](int64_t segs, int64_t pieces) { return 4 * ((segs + 3) & ~(int64_t)3) + 24 * segs * pieces; };
  std::vector<int32_t> want(n_whole, 1);                 // runs wanted per macro-tile
  size_t total = 0;
  for (size_t x = 0; x < n_whole; ++x) {
    if (G.window > 0 && items[x].S > G.window) want[x] = (items[x].S + G.window - 1) / G.window;
    total += (size_t)want[x];
  }
  if (uncut) {
    // (and the plan has no windows)
  } else if (total <= (size_t)cus / 2) {
    const int32_t f = (int32_t)((size_t)cus / total);
    for (size_t x = 0; x < n_whole; ++x) want[x] *= f;
  } else if (G.window == 0) {
    const size_t tail = n_whole % (size_t)cus;
    if (tail > 0 && tail <= (size_t)cus / 2)
      for (size_t x = n_whole - tail; x < n_whole; ++x) want[x] = (int32_t)((size_t)cus / tail);
  }
  std::vector<CompItemDev> later;
  for (size_t x = 0; x < n_whole; ++x) {
    const CompItemDev whole = items[x];
    const std::vector<int32_t> &before = steps_before[(size_t)G.items[x].rep];
    const int32_t least = G.window > 0 && whole.S > G.window ? (whole.S + G.window - 1) / G.window : 1;
    int32_t runs = std::max(least, std::min(want[x], whole.nsteps / min_run_steps(es)));
    if (runs < 2) continue;
    // ranges of `per` steps; more runs if some range touches more segments than fit
    int32_t per = 0;
    for (;; ++runs) {
      per = (whole.nsteps + runs - 1) / runs;
      bool fits = true;
      for (int32_t t0 = 0; t0 < whole.nsteps && fits; t0 += per) {
        const int32_t t1 = std::min(t0 + per, whole.nsteps);
        const int64_t lo = std::upper_bound(before.begin(), before.end(), t0) - before.begin() - 1;
        const int64_t hi = std::upper_bound(before.begin(), before.end(), t1 - 1) - before.begin() - 1;
        fits = desc_bytes(hi - lo + 1, whole.R + whole.Q) <= kDescBytes;
      }
      if (fits || per == 1) break;
    }
    runs = (whole.nsteps + per - 1) / per;
    if (runs < 2) continue;
    fix_pieces(whole, n_runs, runs);
    for (int32_t j = 0; j < runs; ++j) {
      const int32_t t0 = j * per, t1 = std::min(t0 + per, whole.nsteps);
      const int32_t lo = (int32_t)(std::upper_bound(before.begin(), before.end(), t0) - before.begin()) - 1;
      const int32_t hi = (int32_t)(std::upper_bound(before.begin(), before.end(), t1 - 1) - before.begin()) - 1;
      CompItemDev r = whole;
      r.S = hi - lo + 1;
      r.a_first = whole.a_first + lo;
      r.b_first = whole.b_first + lo * whole.b_stride;
      r.k_first = whole.k_first + lo;
      r.first_step = t0 - before[(size_t)lo];
      r.nsteps = t1 - t0;
      r.scratch = (float *)(uintptr_t)((n_runs + (size_t)j) * sizeof(float) * BM * BN);   // offset for now
      r.pad = 1 + j;                                                                        // marks the offset; run number + 1
      if (j == 0) items[x] = r;
      else later.push_back(r);
    }
    n_runs += (size_t)runs;
  }
  std::stable_sort(later.begin(), later.end(), [](const CompItemDev &a, const CompItemDev &b) { return a.pad < b.pad; });
  for (CompItemDev &r : later) r.pad = 1;
  for (CompItemDev &r : items)
    if (r.pad > 0) r.pad = 1;
  items.insert(items.end(), later.begin(), later.end());
  if (n_runs > 0) {
    int rc = acquire_split_buffer(P, n_runs * sizeof(float) * BM * BN, stream);
    if (rc) return rc;
    for (CompItemDev &d : items)
      if (d.pad == 1) {
        d.scratch = (float *)(P->dev->split_buf + (uintptr_t)d.scratch);
        d.pad = 0;
      }
    for (FixItem &f : fixes) f.parts = (const float *)(P->dev->split_buf + (uintptr_t)f.parts);
  }
  L->n_items = items.size();
  L->n_fix = fixes.size();
  L->o_a = items.size() * sizeof(CompItemDev);
  L->o_b = L->o_a + pa.size() * sizeof(PieceDev);
  L->o_c = L->o_b + pb.size() * sizeof(PieceDev);
  L->o_k = L->o_c + pc.size() * sizeof(PieceDev);
  L->o_fix = (L->o_k + klen.size() * sizeof(int32_t) + 7) & ~(size_t)7;
  L->total = L->o_fix + fixes.size() * sizeof(FixItem);
  std::vector<char> &h = *hp;
  h.assign(L->total, 0);
  std::memcpy(h.data(), items.data(), items.size() * sizeof(CompItemDev));
  std::memcpy(h.data() + L->o_a, pa.data(), pa.size() * sizeof(PieceDev));
  std::memcpy(h.data() + L->o_b, pb.data(), pb.size() * sizeof(PieceDev));
  std::memcpy(h.data() + L->o_c, pc.data(), pc.size() * sizeof(PieceDev));
  std::memcpy(h.data() + L->o_k, klen.data(), klen.size() * sizeof(int32_t));
  if (!fixes.empty()) std::memcpy(h.data() + L->o_fix, fixes.data(), fixes.size() * sizeof(FixItem));
  return DMM_OK;
}

}  // namespace
}  // namespace dmm

extern "C" {

int dmm_last_hip_error(void) { return dmm::g_last_hip_error; }

int dmm_measure_mfma_rate(float milliseconds, int random_operands, float *tflops, float *shader_mhz) {
  using namespace dmm;
  if (!(milliseconds > 0.f) || milliseconds > 1000.f) return DMM_EINVAL;
  int dev = 0;
  hipDeviceProp_t prop;
  DMM_HIP(hipGetDevice(&dev));
  DMM_HIP(hipGetDeviceProperties(&prop, dev));
  const int blocks = prop.multiProcessorCount;      // one block of four waves per CU
  unsigned long long *d_cycles = nullptr;
  float *d_sink = nullptr;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  int rc = DMM_OK;
  auto fail = [&](hipError_t e) {
    if (e != hipSuccess && rc == DMM_OK) {
      g_last_hip_error = (int)e;
      rc = DMM_EHIP;
    }
    return e != hipSuccess;
  };
  std::vector<unsigned long long> h((size_t)blocks);
  float ms = 0.f;
  double cyc = 0.0;
  int iters = 4000;                                 // first pass: ~1 ms, to size the second
  if (fail(hipMalloc((void **)&d_cycles, sizeof(unsigned long long) * (size_t)blocks))) goto done;
  if (fail(hipMalloc((void **)&d_sink, sizeof(float)))) goto done;
  if (fail(hipEventCreate(&e0)) || fail(hipEventCreate(&e1))) goto done;
  for (int pass = 0; pass < 2; ++pass) {
    if (fail(hipEventRecord(e0, nullptr))) goto done;
    hipLaunchKernelGGL(mfma_rate_kernel, dim3((unsigned)blocks), dim3(256), 0, nullptr, d_cycles, d_sink, iters,
                       random_operands);
    if (fail(hipGetLastError())) goto done;
    if (fail(hipEventRecord(e1, nullptr)) || fail(hipEventSynchronize(e1))) goto done;
    if (fail(hipEventElapsedTime(&ms, e0, e1))) goto done;
    if (pass == 0) {
      double scale = (double)milliseconds / (ms > 1e-3f ? ms : 1e-3f);
      double want = iters * scale;
      if (want > 2.0e8) want = 2.0e8;
      iters = (int)(want / 4) * 4;
      if (iters < 4) iters = 4;
    }
  }
  if (fail(hipMemcpy(h.data(), d_cycles, sizeof(unsigned long long) * (size_t)blocks, hipMemcpyDeviceToHost))) goto done;
  for (unsigned long long c : h) cyc += (double)c;
  cyc /= blocks;
  // per block: 4 waves x iters x 8 MFMAs x 32 * 32 * 16 * 2 flop
  if (tflops) *tflops = (float)((double)blocks * 4.0 * iters * 8.0 * 32768.0 / (ms * 1e-3) / 1e12);
  if (shader_mhz) *shader_mhz = (float)(cyc / (ms * 1e-3) / 1e6);
done:
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  if (d_cycles) (void)hipFree(d_cycles);
  if (d_sink) (void)hipFree(d_sink);
  return rc;
}

namespace dmm {
namespace {

struct ExecArgs {
  int dtype;
  int64_t es, bk, c_es;
  const void *const *a_tiles;
  const int64_t *a_ld;
  const void *const *b_tiles;
  const int64_t *b_ld;
  void *const *c_tiles;
  const int64_t *c_ld;
  uint32_t flags;
  int device;
  bool uncut;                   // no list is cut along K (see choose_dense)
};

// Work tables of the merged macro-tiles:  merged tables | replica-sum tables, one copy.
int build_merged_exec(dmm_plan_t *P, const ExecArgs &x, hipStream_t stream, ExecLayout *L) {
  int rc;
  RedLaunch red;
  MergedLaunch ml;
  std::vector<char> &h = P->dev->host;
  h.clear();
  int cus = 0;
  if ((rc = device_cus(&cus))) return rc;
  if ((rc = build_merged_tables(P, x.es, x.bk, x.c_es, x.a_tiles, x.a_ld, x.b_tiles, x.b_ld, x.c_tiles, x.c_ld, cus, x.uncut, stream, &h, &ml)))
    return rc;
  if (!(x.flags & DMM_NO_REDUCE) && (rc = build_reduce(P, x.c_tiles, x.c_ld, 0, &h, ml.total, &red))) return rc;
  if ((rc = P->dev->gemm_table.upload(h.data(), h.size(), stream, P->dev->uses))) return rc;
  red.dev_base = P->dev->gemm_table.dev();
  L->merged = true;
  L->ml = ml;
  L->red = red;
  L->uses_split = ml.n_fix > 0;
  return DMM_OK;
}

// Work tables of the per-group macro-tiles.  The tables of all kernels go up in one copy in front
// of the GEMM launch, so that nothing but the launches separates them:
// ItemDev[] | SegDev[] | FixItem[] | RedSrc[] | replica-sum tables.
int build_group_exec(dmm_plan_t *P, const ExecArgs &x, hipStream_t stream, ExecLayout *L) {
  int rc;
  const int64_t es = x.es, bk = x.bk, c_es = x.c_es;
  const void *const *a_tiles = x.a_tiles;
  const void *const *b_tiles = x.b_tiles;
  void *const *c_tiles = x.c_tiles;
  const int64_t *a_ld = x.a_ld, *b_ld = x.b_ld, *c_ld = x.c_ld;
  const uint32_t flags = x.flags;
  if ((rc = materialize(P))) return rc;
    RedLaunch red;
  const size_t n_plan_items = P->items.size();
  const size_t n_segs = P->tasks.size();
  std::vector<SegDev> hs(n_segs);
  std::vector<ItemDev> hi(n_plan_items);
  std::vector<FixItem> fixes;
  // segments in grouped order: segment index = position in `order`
  for (size_t pos = 0; pos < n_segs; ++pos) {
    const dmm_task &t = P->tasks[P->order[pos]];
    const int64_t ai = P->A.table_index(t.a_rep, t.a_ti, t.a_tj);
    const int64_t bi = P->B.table_index(t.b_rep, t.b_ti, t.b_tj);
    if (!a_tiles[ai] || !b_tiles[bi]) return DMM_EINVAL;
    SegDev sg;
    sg.lda = a_ld[ai];
    sg.ldb = b_ld[bi];
    sg.a = (const char *)a_tiles[ai] + ((t.m0 - P->A.rc[t.a_ti]) * sg.lda + (t.k0 - P->A.cc[t.a_tj])) * es;
    sg.b = (const char *)b_tiles[bi] + ((t.k0 - P->B.rc[t.b_ti]) * sg.ldb + (t.n0 - P->B.cc[t.b_tj])) * es;
    // bytes that may be read from the segment's origin to the end of the tile buffer
    // ((rows - 1) * ld + cols elements are guaranteed to exist)
    const int64_t a_h = P->A.rc[t.a_ti + 1] - P->A.rc[t.a_ti], a_w = P->A.cc[t.a_tj + 1] - P->A.cc[t.a_tj];
    const int64_t b_h = P->B.rc[t.b_ti + 1] - P->B.rc[t.b_ti], b_w = P->B.cc[t.b_tj + 1] - P->B.cc[t.b_tj];
    sg.a_bytes = ((a_h - 1) * sg.lda + a_w - ((t.m0 - P->A.rc[t.a_ti]) * sg.lda + (t.k0 - P->A.cc[t.a_tj]))) * es;
    sg.b_bytes = ((b_h - 1) * sg.ldb + b_w - ((t.k0 - P->B.rc[t.b_ti]) * sg.ldb + (t.n0 - P->B.cc[t.b_tj]))) * es;
    sg.klen = (int32_t)(t.k1 - t.k0);
    sg.pad = 0;
    hs[pos] = sg;
  }
  for (size_t i = 0; i < n_plan_items; ++i) {
    const dmm_work_item &w = P->items[i];
    const int64_t ci = P->C.table_index(w.c_rep, w.c_ti, w.c_tj);
    if (!c_tiles[ci]) return DMM_EINVAL;
    ItemDev d;
    d.ldc = c_ld[ci];
    d.c = (char *)c_tiles[ci] + ((w.m0 - P->C.rc[w.c_ti]) * d.ldc + (w.n0 - P->C.cc[w.c_tj])) * c_es;
    if (w.group >= 0) {
      const Group &G = P->groups[(size_t)w.group];
      d.seg_begin = (int32_t)G.first;
      d.nsteps = 0;
      for (int64_t q = 0; q < G.count; ++q) d.nsteps += (int32_t)((hs[(size_t)(G.first + q)].klen + bk - 1) / bk);
      d.m_off = (int32_t)(w.m0 - G.m0);
      d.n_off = (int32_t)(w.n0 - G.n0);
    } else {
      d.seg_begin = 0;
      d.nsteps = 0;
      d.m_off = d.n_off = 0;
    }
    d.m_ext = w.m_ext;
    d.n_ext = w.n_ext;
    d.first_step = 0;
    d.c_es = (int32_t)c_es;
    d.red_first = d.red_count = 0;
    hi[i] = d;
  }
  // K-split of the last round (see sum_parts_kernel): with W working items on `cus` CUs the
  // last W % cus of them run alone; if they are few, each is cut into up to cus / (W % cus) runs
  // of at least min_run_steps() K steps.  Run 0 takes the item's place in the launch order, the others
  // go to the end; all of them write to the scratch buffer.  A run pays a prologue and an
  // epilogue of its own (about 13 K steps' worth) and the pass that adds the runs up is one more
  // launch: measured with bf16 operands, runs of 32 steps lose (2048^3: 45 -> 66 us), so a run is
  // 64 steps at least (8 of fp32 operands, the same duration).
  int cus = 0;
  if ((rc = device_cus(&cus))) return rc;
  size_t working = 0;
  for (const ItemDev &d : hi) working += d.nsteps > 0;
  const size_t tail = x.uncut ? 0 : working % (size_t)cus;
  size_t n_runs = 0;
  if (tail > 0 && tail <= (size_t)cus / 2) {
    const int32_t max_runs = (int32_t)((size_t)cus / tail);
    size_t seen = 0;
    for (size_t i = n_plan_items; i-- > 0 && seen < tail;) {
      if (hi[i].nsteps <= 0) continue;
      ++seen;
      int32_t runs = std::min(max_runs, hi[i].nsteps / min_run_steps(es));
      if (runs < 2) continue;
      const int32_t per = (hi[i].nsteps + runs - 1) / runs;
      runs = (hi[i].nsteps + per - 1) / per;
      const ItemDev whole = hi[i];
      FixItem f;
      f.dst = whole.c;
      f.ldc = whole.ldc;
      f.parts = (const float *)(uintptr_t)(n_runs * sizeof(float) * BM * BN);   // offset for now, base added below
      f.m_ext = whole.m_ext;
      f.n_ext = whole.n_ext;
      f.nparts = runs;
      f.c_es = whole.c_es;
      f.row0 = f.col0 = 0;
      fixes.push_back(f);
      for (int32_t j = 0; j < runs; ++j) {
        ItemDev r = whole;
        r.c = (void *)(uintptr_t)((n_runs + (size_t)j) * sizeof(float) * BM * BN);        // offset for now
        r.ldc = BN;
        r.first_step = j * per;
        r.nsteps = std::min(per, whole.nsteps - j * per);
        r.c_es = -4;                                                                        // fp32; negative marks "c is a scratch offset"
        if (j == 0) hi[i] = r;
        else hi.push_back(r);
      }
      n_runs += (size_t)runs;
    }
  }
  if (n_runs > 0) {
    if ((rc = acquire_split_buffer(P, n_runs * sizeof(float) * BM * BN, stream))) return rc;
    for (ItemDev &d : hi)
      if (d.c_es < 0) {
        d.c = (void *)(P->dev->split_buf + (uintptr_t)d.c);
        d.c_es = 4;
      }
    for (FixItem &f : fixes) f.parts = (const float *)(P->dev->split_buf + (uintptr_t)f.parts);
  }
  // Fused replica sum: the macro-tiles of replicas 1, 2, ... go first, those of replica 0 behind
  // them, and these add the others' partial sums to their own before they store.  No replica-sum
  // kernel runs.  (Not together with the K-split, whose runs store through a scratch buffer.)
  // One launch where the list can be laid out so that every macro-tile of replica 0 finds the
  // partial sums of its region written by its own workgroup earlier in the same launch (workgroup
  // w walks items w, w + grid, ... in order, and a wave reads back exactly the elements it stored
  // itself); otherwise two launches, replica 0's second (stream order: every partial sum is
  // complete by then).
  const bool fuse = !(flags & (DMM_SEPARATE_REDUCE | DMM_NO_REDUCE)) && P->C.c > 1 && n_runs == 0;
  std::vector<RedSrc> reds;
  size_t n_first = hi.size();               // items of the first launch
  bool one_launch = false;
  if (fuse) {
    std::vector<ItemDev> others, origin;
    others.reserve(hi.size());
    origin.reserve(hi.size());
    std::vector<std::vector<uint32_t>> of_rep((size_t)P->C.c);     // per replica: plan items in list order
    for (size_t i = 0; i < n_plan_items; ++i) {
      const dmm_work_item &w = P->items[i];
      of_rep[(size_t)w.c_rep].push_back((uint32_t)i);
      if (w.c_rep != 0) {
        others.push_back(hi[i]);
        continue;
      }
      ItemDev d = hi[i];
      d.red_first = (int32_t)reds.size();
      d.red_count = P->C.c - 1;
      for (int32_t r = 1; r < P->C.c; ++r) {
        const int64_t idx = P->C.table_index(r, w.c_ti, w.c_tj);
        if (!c_tiles[idx]) return DMM_EINVAL;
        RedSrc src;
        src.ld = c_ld[idx];
        src.p = (const float *)c_tiles[idx] + (w.m0 - P->C.rc[w.c_ti]) * src.ld + (w.n0 - P->C.cc[w.c_tj]);
        reds.push_back(src);
      }
      origin.push_back(d);
    }
    n_first = others.size();
    // One launch?  Every replica has to have as many macro-tiles as replica 0, the k-th of each
    // covering the region of replica 0's k-th, and that number has to be a whole number of rounds
    // of the grid: then the list can be laid out so that workgroup w (which walks positions w,
    // w + grid, ...) meets the partial sums of a region before it meets replica 0's macro-tile of it.
    const size_t grid = std::min<size_t>(n_plan_items, (size_t)cus);
    const size_t n0 = of_rep[0].size();
    one_launch = grid > 0 && n0 > 0 && n0 % grid == 0;
    for (int32_t r = 1; r < P->C.c && one_launch; ++r) {
      if (of_rep[(size_t)r].size() != n0) one_launch = false;
      for (size_t k = 0; k < n0 && one_launch; ++k) {
        const dmm_work_item &o = P->items[of_rep[0][k]], &s = P->items[of_rep[(size_t)r][k]];
        if (o.c_ti != s.c_ti || o.c_tj != s.c_tj || o.m0 != s.m0 || o.n0 != s.n0 || o.m_ext != s.m_ext || o.n_ext != s.n_ext)
          one_launch = false;
      }
    }
    if (one_launch) {
      // Chunk j = macro-tiles j grid .. (j + 1) grid - 1 of every replica (a round of the planner's
      // order: the 32 workgroups of an XCD on one block of neighbouring tiles).  Per workgroup and
      // chunk: `o` = the other replicas' macro-tiles, `s` = replica 0's, which adds their partial
      // sums.  All workgroups in step would read their partial sums at the same moments, at the
      // memory's pace with the matrix pipes idle; so the XCDs alternate between two schedules,
      //   o0 s0 o1 s1 o2 s2 ...      and      o0 o1 s0 o2 s1 ... s(last),
      // whose `s` fall into different rounds except the last (cfg4, four chunks: 2 % off the step
      // against o0 o1 o2 o3 s0 s1 s2 s3 everywhere; the first schedule everywhere: 1 % on).
      const size_t Q = n0 / grid;
      std::vector<ItemDev> laid(hi.size());
      std::vector<std::pair<bool, size_t>> seq;                      // (is s, chunk)
      for (size_t w = 0; w < grid; ++w) {
        seq.clear();
        if (((w % 8) & 1) == 0 || Q < 2) {
          for (size_t j = 0; j < Q; ++j) {
            seq.push_back({false, j});
            seq.push_back({true, j});
          }
        } else {
          seq.push_back({false, 0});
          for (size_t j = 0; j < Q; ++j) {
            if (j + 1 < Q) seq.push_back({false, j + 1});
            seq.push_back({true, j});
          }
        }
        size_t t = 0;
        for (const auto &e : seq) {
          const size_t k = e.second * grid + w;
          if (e.first) laid[(t++) * grid + w] = origin[k];
          else
            for (int32_t r = 1; r < P->C.c; ++r) laid[(t++) * grid + w] = hi[of_rep[(size_t)r][k]];
        }
      }
      hi = std::move(laid);
    } else {
      hi = std::move(others);
      hi.insert(hi.end(), origin.begin(), origin.end());
    }
  }
  const size_t n_items = hi.size();
  const size_t o_segs = n_items * sizeof(ItemDev);
  const size_t o_fix = o_segs + n_segs * sizeof(SegDev);
  const size_t o_red = o_fix + fixes.size() * sizeof(FixItem);
  const size_t total = n_items > 0 ? o_red + reds.size() * sizeof(RedSrc) : 0;
  std::vector<char> &h = P->dev->host;
  h.clear();
  h.resize(total);
  if (n_items > 0) {
    std::memcpy(h.data(), hi.data(), n_items * sizeof(ItemDev));
    std::memcpy(h.data() + o_segs, hs.data(), n_segs * sizeof(SegDev));
    if (!fixes.empty()) std::memcpy(h.data() + o_fix, fixes.data(), fixes.size() * sizeof(FixItem));
    if (!reds.empty()) std::memcpy(h.data() + o_red, reds.data(), reds.size() * sizeof(RedSrc));
  }
  if (!(flags & DMM_NO_REDUCE) && !fuse && (rc = build_reduce(P, c_tiles, c_ld, 0, &h, total, &red))) return rc;
  if (!h.empty()) {
    if ((rc = P->dev->gemm_table.upload(h.data(), h.size(), stream, P->dev->uses))) return rc;
    red.dev_base = P->dev->gemm_table.dev();
  }
  L->merged = false;
  L->n_items = n_items;
  L->o_segs = o_segs;
  L->o_fix = o_fix;
  L->o_red = o_red;
  L->n_first = n_first;
  L->n_fix = fixes.size();
  L->fuse = fuse;
  L->one_launch = one_launch;
  L->uses_split = n_runs > 0;
  L->n_runs = n_runs;
  L->red = red;
  return DMM_OK;
}

// ---- small and skinny products (small_kernel.hpp) ------------------------------------------------

struct SmallPlan {
  int shape = -1;
  int32_t runs = 1, per = 0;
  std::vector<int64_t> mc, nc, kc;
  std::vector<Extent> rows, cols;
};

constexpr int64_t kSmallMost = 1 << 20;    // workgroups of a launch (small_div)

constexpr SmallKind kSmall[SMALL_SHAPES] = {
    small_kind<RingSkinny>(0.25, 0.46), small_kind<RingHalf>(0.31, 0.46), small_kind<RingPair>(0.44, 0.62),
    small_kind<SmallF32Tiny>(0.39, 0.72), small_kind<SmallF32>(0.52, 0.78), small_kind<SmallF32Split>(1.55, 2.0),
};

int64_t count_steps(const std::vector<int64_t> &kc, int64_t bk) {
  int64_t n = 0;
  for (size_t s = 0; s + 1 < kc.size(); ++s) n += (kc[s + 1] - kc[s] + bk - 1) / bk;
  return n;
}

// The share of an operand's columns in K-segments (column intervals) that begin inside their tile's rows
// at positions that are not multiples of 16 bytes.
double cut_misaligned(const Grid &G, const std::vector<int64_t> &cuts) {
  int64_t odd = 0;
  for (size_t i = 0; i + 1 < cuts.size(); ++i) {
    const int64_t in = cuts[i] - *(std::upper_bound(G.cc.begin(), G.cc.end(), cuts[i]) - 1);
    if (in & 7) odd += cuts[i + 1] - cuts[i];
  }
  return (double)odd / (double)std::max<int64_t>(1, cuts.back());
}

// segments whose last step is a K tail
int64_t count_tails(const std::vector<int64_t> &kc, int64_t bk) {
  int64_t n = 0;
  for (size_t s = 0; s + 1 < kc.size(); ++s) n += (kc[s + 1] - kc[s]) % bk != 0;
  return n;
}

// Whether (and how) the kernels for small products run this call: the estimated time of the best of
// their shapes and numbers of runs against that of the macro-tile kernels.  The line between the two
// depends on how many macro-tiles there are for the CUs, how much of them is product, how long K is and
// how many segments it has, so it is drawn by an estimate and not by a size.  Measured, us per call
// with macro-tiles -> with these kernels: fp32 256^3 54 -> 8.6; bf16 3072^3 (144 macro-tiles) 69 against 80: stays;
// 868 x 6784 x 8448 160 -> 117; 2700 x 1630 x 2180 uneven 101 -> 57; 425 x 2623 x 41280 137 against 152: stays;
// 64 x 5760 x 4960 61 -> 19; fp32 577 x 28352 x 512 216 -> 176.  Between these shapes, us in tiles of 32, 64 and 128
// rows: 128 x 8960 x 8576 60, 49, 40; 64 x 6615 x 45440 177, 146, 156; 640 x 247 x 384 11, 12, 16 (a 128-row tile's prologue
// and epilogue take 5 us longer, which shows where they do not fill the CUs); 900 x 333 x 1100 14, 16, 19.
// fp32 in tiles of 64 rows and of 128, taken apart: 1024^3 34, 38; 3840 x 1006 x 594 in 16 column strips (tiles 37 wide)
// 102, 124; 512 x 8416 x 848 78, 69; 2432 x 4256 x 600 uneven 148, 137; 5612 x 1584 x 3264 597, 467.  Below K = 512 or 16
// tiles there is no time to win: a call is its launches.
void choose_small(dmm_plan_t *P, const ExecArgs &x, int cus, SmallPlan *best) {
  const Grid &A = P->A, &B = P->B, &C = P->C;
  const int64_t M = C.rows, K = A.cols, N = C.cols, lim = (int64_t)1 << 30;
  if (P->dense_copy || C.c != 1 || M <= 0 || K <= 0 || N <= 0 || M >= lim || K >= lim || N >= lim) return;
  if ((P->flags & DMM_MERGE_ALWAYS) || (x.flags & DMM_NO_MERGE)) return;      // the caller named a work list
  SmallPlan c;
  c.mc = merged_cuts({&A.rc, &C.rc});
  c.nc = merged_cuts({&B.cc, &C.cc});
  c.kc = merged_cuts({&A.cc, &B.rc});
  const double mr = (double)c.mc.size(), nr = (double)c.nc.size(), sr = (double)c.kc.size();
  if (mr * sr + sr * nr + mr * nr > 65536.0) return;
  size_t items = 0;
  if (P->merged.valid) items = P->merged.items.size();
  else
    for (const dmm_work_item &w : P->items) items += w.group >= 0;
  if (x.es == 2 && M >= 2048 && N >= 2048 && items >= 2 * (size_t)cus) return;   // two full rounds of macro-tiles: theirs
  // Microseconds.  The macro-tile kernels: rounds of macro-tiles, the last one cut along K where it is
  // at most half full; a K step costs more the fuller the device (its clock falls), every item a
  // prologue and an epilogue, every segment a switch.
  const double segs = (double)(c.kc.size() - 1);
  const int64_t big_steps = count_steps(c.kc, x.bk), tail = (int64_t)(items % (size_t)cus), full = (int64_t)items / cus;
  const int64_t big_runs = tail > 0 && tail <= cus / 2 ? std::max<int64_t>(1, std::min<int64_t>(cus / tail, big_steps / min_run_steps(x.es))) : 1;
  const double fill = full > 0 ? 1.0 : (double)(tail * big_runs) / cus;
  const double big_step = (x.es == 2 ? 0.46 + 0.31 * fill : 3.9) * (P->merged.valid ? 1.06 : 1.0);
  const double item = 6 + (x.es == 2 ? 1.5 * segs + 2.5 * (double)count_tails(c.kc, x.bk) : 1.5 * segs);
  double least = 4 + (double)full * ((double)big_steps * big_step + item);
  if (tail > 0) {
    least += (double)((big_steps + big_runs - 1) / big_runs) * big_step + item;
    if (big_runs > 1) least += 4 + 2.0 * (double)(tail * big_runs) * sizeof(float) * BM * BN / 12e6;
  }
  least *= x.es == 2 ? 0.93 : 0.97;                                            // (not for a tie)
  // These kernels: rounds of `occ` workgroups per CU, operands at no more than 5.6 TB/s (7.5 from the last-level cache:
  // 82 x 2944 x 33024 in 264 workgroups 42, in 792 and their sum 56), and a second launch that adds the partial tiles up.
  const double bytes = (double)x.es * ((double)M * K + (double)K * N) + (double)x.c_es * (double)M * N;
  // (long K at odd places: 4985 x 9842 x 3072 in uneven tiles, packed, 440 with macro-tiles and 550 with these)
  const double odd = std::max(cut_misaligned(A, c.kc), cut_misaligned(B, c.nc)) > 0.1 ? (K >= 7680 ? 1.6 : 1.25) : 1.0;
  for (int k = 0; k < SMALL_SHAPES; ++k) {
    const SmallKind &s = kSmall[k];
    if (s.es != (int)x.es) continue;
    c.rows = tile_axis(c.mc, 1 << 30, 1, s.tm);
    c.cols = tile_axis(c.nc, 1 << 30, kPieceAlign, s.tn);
    const int64_t tiles = (int64_t)(c.rows.size() * c.cols.size()), steps = count_steps(c.kc, s.bk);
    const int64_t tails = count_tails(c.kc, s.bk);
    if (tiles >= kSmallMost || (k == SMALL_F32_SPLIT && (K < 512 || tiles < 16))) continue;
    // B comes again for every tile row but the first: from memory (64 x 6615 x 45440 in 32 x 128 tiles 187 us, in
    // 64 x 128 tiles 161), or, where the last-level cache holds it, from there.
    const double b_bytes = (double)x.es * (double)K * N;
    const double mem = bytes / (x.es == 2 && bytes < 256e6 ? 7.5e6 : 5.6e6) + (double)(c.rows.size() - 1) * b_bytes / (b_bytes > 128e6 ? 6.5e6 : 14e6);
    // Rounding grows with the root of the number of terms in a chain of sums.  The split kernel rounds once where the others
    // round eight times: over drawn products it has 0.3 times their error (median; normal and uniform operands), and with at
    // least 0.15 times as many chains as there would be otherwise never more than it (0.91 at most, operands of one sign).
    const int64_t least_runs = k != SMALL_F32_SPLIT ? 1 : (int64_t)std::ceil(0.15 * std::max(
        (double)items / ((double)full * cus + (double)tail / (double)big_runs),
        best->shape < 0 ? 1.0 : (double)best->runs * (best->shape == SMALL_F32_TINY ? SmallF32Tiny::WK : 1)));
    // a run has at least 256 (fp32: 128) elements of k, and the partial tiles fit 64 MB, which is
    // what the macro-tile kernels use at most
    const int64_t least_per = (s.es == 2 ? 256 : 128) / s.bk;
    for (int64_t r = 1; r <= std::max<int64_t>(1, std::min<int64_t>(64, steps / least_per)); ++r) {
      const int64_t per = (steps + r - 1) / r, runs = (steps + per - 1) / per;
      if (runs != r || r < least_runs || runs * tiles >= kSmallMost) continue;
      const int64_t part_bytes = runs * tiles * s.tm * s.tn * 4;
      if (runs > 1 && part_bytes > (int64_t)64 << 20) break;
      const int64_t per_cu = (tiles * runs + cus - 1) / cus, whole = per_cu / s.occ, rest = per_cu % s.occ;
      double t = (double)whole * ((double)per * std::max(s.step * s.occ, s.alone) + 2);
      if (rest > 0) t += (double)per * std::max(s.step * (double)rest, s.alone) + 2;
      if (s.es == 2) {
        if (k == SMALL_BF16 && per_cu == 1) t = (double)per * (0.36 + 0.12 * (double)(tiles * runs) / cus) + 2;   // (the ring of four stages)
        // K-segments that begin at odd places; a switch, and what a K tail costs
        t = t * odd + (double)(whole + (rest > 0)) * (0.4 * segs + (s.tm == 32 ? 0.75 : 0.9) * (double)tails) / (double)runs;
        t += k == SMALL_BF16 ? (tiles * runs < 140 ? 6 : 1.5) : 1;
      } else {
        t += segs / (double)runs + (k == SMALL_F32_SPLIT ? 5 : 0);
      }
      // Operands from memory take as long as on the CU that loads most of them, where 200 CUs (160 that hold more, smaller
      // workgroups) keep memory busy: 40 x 10240 x 11088 in 176 workgroups 40, in 264 54; 43 x 13723 x 16385 in 270 136, in
      // 405 104; 32-row tiles, 2 x 3328 x 34716 in 272 41, in 816 49; 8 x 14848 x 16652 in 272 122, in 680 96.
      const double share = (s.tm == 32 ? 160.0 : 200.0) * (double)per_cu / (double)(tiles * runs);
      t = 4 + std::max(t, s.es == 2 ? mem * std::max(1.0, share) : mem);
      // (a second launch: 640 x 384 x 832 uncut 10, in two runs 14; 8 x 2496 x 18432 17, 23)
      if (runs > 1) t += (x.es == 2 ? 6 : 4) + 2.0 * (double)part_bytes / 12e6;
      if (t < least) {
        least = t;
        best->shape = k;
        best->runs = (int32_t)runs;
        best->per = (int32_t)per;
        best->rows = c.rows;
        best->cols = c.cols;
      }
    }
  }
  best->mc = c.mc;
  best->nc = c.nc;
  best->kc = c.kc;
}

// Work tables of the kernels for small products:
//   SmallTile rows[] | cols[] | PieceDev a[] | b[] | c[] | SmallStart starts[] | int32 mc[] | nc[] | klen[]
// DMM_EINVAL where a tile that the op list names has no pointer.
int build_small_exec(dmm_plan_t *P, const ExecArgs &x, const SmallPlan &sp, hipStream_t stream, ExecLayout *L) {
  int rc = DMM_OK;
  const Grid &A = P->A, &B = P->B, &C = P->C;
  const SmallKind &kind = kSmall[sp.shape];
  const size_t MR = sp.mc.size() - 1, NR = sp.nc.size() - 1, S = sp.kc.size() - 1;
  auto holder = [](const std::vector<int64_t> &cuts, int64_t at) {
    return (int32_t)(std::upper_bound(cuts.begin(), cuts.end() - 1, at) - cuts.begin()) - 1;
  };
  SmallLaunch &l = L->small;
  l.o_rows = 0;
  l.o_cols = l.o_rows + sp.rows.size() * sizeof(SmallTile);
  l.o_a = l.o_cols + sp.cols.size() * sizeof(SmallTile);
  l.o_b = l.o_a + MR * S * sizeof(PieceDev);
  l.o_c = l.o_b + S * NR * sizeof(PieceDev);
  l.o_starts = l.o_c + MR * NR * sizeof(PieceDev);
  l.o_mc = l.o_starts + (size_t)sp.runs * sizeof(SmallStart);
  l.o_nc = l.o_mc + (MR + 1) * 4;
  l.o_klen = l.o_nc + (NR + 1) * 4;
  const size_t total = (l.o_klen + S * 4 + 7) & ~(size_t)7;   // (whole words: table_kernel)
  std::vector<char> &h = P->dev->host;
  h.assign(total, 0);
  auto tiles = [&](size_t at, const std::vector<Extent> &v, const std::vector<int64_t> &cuts) {
    SmallTile *t = (SmallTile *)(h.data() + at);
    for (size_t i = 0; i < v.size(); ++i) t[i] = {(int32_t)v[i].start, v[i].ext, v[i].first, v[i].pieces, (int32_t)cuts[(size_t)v[i].first], 0};
  };
  tiles(l.o_rows, sp.rows, sp.mc);
  tiles(l.o_cols, sp.cols, sp.nc);
  auto piece = [](const void *base, int64_t ld, int64_t r, int64_t c, int64_t hh, int64_t w, int64_t esz) {
    PieceDev d;
    const int64_t off = r * ld + c;
    d.ptr = (const char *)base + off * esz;
    d.room = ((hh - 1) * ld + w - off) * esz;
    d.pitch = (uint32_t)(ld * esz);
    d.pad = 0;
    return d;
  };
  std::vector<int32_t> a_ti(MR), c_ti(MR), b_tj(NR), c_tj(NR), a_tj(S), b_ti(S);
  for (size_t i = 0; i < MR; ++i) { a_ti[i] = holder(A.rc, sp.mc[i]); c_ti[i] = holder(C.rc, sp.mc[i]); }
  for (size_t j = 0; j < NR; ++j) { b_tj[j] = holder(B.cc, sp.nc[j]); c_tj[j] = holder(C.cc, sp.nc[j]); }
  for (size_t s = 0; s < S; ++s) { a_tj[s] = holder(A.cc, sp.kc[s]); b_ti[s] = holder(B.rc, sp.kc[s]); }
  PieceDev *pa = (PieceDev *)(h.data() + l.o_a), *pb = (PieceDev *)(h.data() + l.o_b), *pc = (PieceDev *)(h.data() + l.o_c);
  for (size_t i = 0; i < MR; ++i)
    for (size_t s = 0; s < S; ++s) {
      const int64_t idx = A.table_index(0, a_ti[i], a_tj[s]);
      if (!x.a_tiles[idx]) return DMM_EINVAL;
      pa[i * S + s] = piece(x.a_tiles[idx], x.a_ld[idx], sp.mc[i] - A.rc[a_ti[i]], sp.kc[s] - A.cc[a_tj[s]],
                            A.rc[a_ti[i] + 1] - A.rc[a_ti[i]], A.cc[a_tj[s] + 1] - A.cc[a_tj[s]], x.es);
    }
  for (size_t s = 0; s < S; ++s)
    for (size_t j = 0; j < NR; ++j) {
      const int64_t idx = B.table_index(0, b_ti[s], b_tj[j]);
      if (!x.b_tiles[idx]) return DMM_EINVAL;
      pb[s * NR + j] = piece(x.b_tiles[idx], x.b_ld[idx], sp.kc[s] - B.rc[b_ti[s]], sp.nc[j] - B.cc[b_tj[j]],
                             B.rc[b_ti[s] + 1] - B.rc[b_ti[s]], B.cc[b_tj[j] + 1] - B.cc[b_tj[j]], x.es);
    }
  for (size_t i = 0; i < MR; ++i)
    for (size_t j = 0; j < NR; ++j) {
      const int64_t idx = C.table_index(0, c_ti[i], c_tj[j]);
      if (!x.c_tiles[idx]) return DMM_EINVAL;
      pc[i * NR + j] = piece(x.c_tiles[idx], x.c_ld[idx], sp.mc[i] - C.rc[c_ti[i]], sp.nc[j] - C.cc[c_tj[j]],
                             C.rc[c_ti[i] + 1] - C.rc[c_ti[i]], C.cc[c_tj[j] + 1] - C.cc[c_tj[j]], x.c_es);
    }
  int32_t *mc = (int32_t *)(h.data() + l.o_mc), *nc = (int32_t *)(h.data() + l.o_nc), *klen = (int32_t *)(h.data() + l.o_klen);
  for (size_t i = 0; i <= MR; ++i) mc[i] = (int32_t)sp.mc[i];
  for (size_t j = 0; j <= NR; ++j) nc[j] = (int32_t)sp.nc[j];
  SmallStart *starts = (SmallStart *)(h.data() + l.o_starts);
  int32_t before = 0, run = 0;                            // K steps in front of the segment
  for (size_t s = 0; s < S; ++s) {
    klen[s] = (int32_t)(sp.kc[s + 1] - sp.kc[s]);
    const int32_t steps = (klen[s] + kind.bk - 1) / kind.bk;
    for (; run < sp.runs && run * sp.per < before + steps; ++run) starts[run] = {(int32_t)s, (run * sp.per - before) * kind.bk};
    before += steps;
  }
  l.steps = before;
  l.shape = sp.shape;
  l.segs = (int32_t)S;
  l.nr = (int32_t)NR;
  l.tiles_m = (int32_t)sp.rows.size();
  l.tiles_n = (int32_t)sp.cols.size();
  l.runs = sp.runs;
  l.per = sp.per;
  l.c_es = (int32_t)x.c_es;
  // Partial tiles: how K is cut does not depend on free memory, so where there is no room for those of all
  // tiles at once, the tiles are taken in several launches.
  l.batch = l.tiles_m * l.tiles_n;
  if (sp.runs > 1)
    for (;;) {
      rc = acquire_split_buffer(P, (size_t)sp.runs * (size_t)l.batch * (size_t)(kind.tm * kind.tn) * sizeof(float), stream);
      if (rc != DMM_ENOMEM || l.batch == 1) break;
      (void)hipGetLastError();
      l.batch = (l.batch + 1) / 2;
    }
  if (rc) return rc;
  if ((rc = P->dev->gemm_table.upload(h.data(), h.size(), stream, P->dev->uses))) return rc;
  L->uses_split = sp.runs > 1;
  return DMM_OK;
}

// ---- products on dense copies of their operands (pack_kernel.hpp) -----------------------------------

// Whether rows of its tiles begin at positions that are not multiples of 16 bytes.
bool placed_misaligned(const Grid &G, const void *const *tiles, const int64_t *ld) {
  for (int32_t i = 0; i < G.gr; ++i)
    for (int32_t j = 0; j < G.gc; ++j)
      if (G.rc[i + 1] > G.rc[i] && G.cc[j + 1] > G.cc[j]) {
        const int64_t x = G.table_index(0, i, j);
        if (((uintptr_t)tiles[x] & 15) || (ld[x] & 7)) return true;
      }
  return false;
}

// How the copies hold K: one share per replica of C, each of `len` columns of A's copy (rows of B's).
// The K-segments of a share start at multiples of a K step and are filled up with zeros; where the
// shares differ in length, zeros stand in front (sums that start at zero do not change by adding zero).
struct DenseShape {
  std::vector<int64_t> shares;        // where the shares begin in K, and K
  std::vector<int64_t> kc;            // the segments' cuts
  std::vector<int32_t> share;         // of every segment
  std::vector<int64_t> at;            // where a segment begins inside its share of the copy
  int64_t len = 0;
};

void dense_shape(const dmm_plan_t *P, int64_t bk, DenseShape *shape) {
  DenseShape &d = *shape;
  const int64_t K = P->A.cols, c = P->C.c;
  for (int64_t r = 0; r <= c; ++r) d.shares.push_back(r * K / c);
  d.kc = merged_cuts({&P->A.cc, &P->B.rc, &d.shares});
  std::vector<int64_t> len((size_t)c, 0);
  for (size_t s = 0; s + 1 < d.kc.size(); ++s) {
    const int32_t r = (int32_t)(std::upper_bound(d.shares.begin(), d.shares.end(), d.kc[s]) - d.shares.begin()) - 1;
    d.share.push_back(r);
    d.at.push_back(len[(size_t)r]);
    len[(size_t)r] += (d.kc[s + 1] - d.kc[s] + bk - 1) / bk * bk;
  }
  for (int64_t l : len) d.len = std::max(d.len, l);
  for (size_t s = 0; s < d.at.size(); ++s) d.at[s] += d.len - len[(size_t)d.share[s]];
}

constexpr int64_t kDenseMost = (int64_t)2 << 30;      // bytes of copies a product may ask for

// leading dimension of a copy with that many columns
int64_t dense_ld(int64_t cols) { return (cols + 63) & ~(int64_t)63; }

int64_t dense_bytes(const dmm_plan_t *P, const DenseShape &d) {
  return 2 * P->C.c * (P->C.rows * dense_ld(d.len) + d.len * dense_ld(P->C.cols));
}

// Whether macro-tiles of a list of `n` would be cut along K to fill its last round.
bool last_round_is_cut(int64_t n, int64_t steps, int64_t es, int cus) {
  const int64_t tail = n % cus;
  return tail > 0 && tail <= cus / 2 && steps >= 2 * min_run_steps(es);
}

// Whether a segment list is too long for a merged macro-tile's descriptors (which is then cut along K).
bool in_windows(const dmm_plan_t *P) {
  if (!P->merged.valid || P->merged.window <= 0) return false;
  for (const MergedRep &R : P->merged.reps)
    if ((int64_t)R.kc.size() - 1 > P->merged.window) return true;
  return false;
}

// Whether a large bf16 product runs on dense copies of A and B: the estimated time of the copy plus
// the macro-tiles on it against that of the macro-tiles on the operands as they are.  The copies
// must not show in the result, since a call takes them or not by where its operands lie and by what
// memory is free: they hold the very K steps of the operands (pack_kernel.hpp) and their list is
// never cut along K, so the bits are those of the product's own list uncut.  Where that list would be
// cut, the shape alone decides: either such a product always runs uncut (*uncut: on the copies, or on
// its own list where it cannot have them), or it never runs on copies.
// A K step takes 1.27 of the time where segments (a tenth of them and more) begin at odd places, else 1.12 where
// rows do (8102 x 4002 x 8102 in 2 x 2 tiles packed against padded rows: 544 and 486 us), a segment another step and a half, a
// macro-tile that spans tiles 1.13; the copy runs at 4.5 TB/s and more (0.93 GB in 171 us).  Measured, us per call on the operands -> on
// copies: 12289 x 9973 x 11003 in uneven packed tiles 3040 -> 2320, the same with rows padded to 16 bytes
// 2750 -> 2330; 8192^3 in block-cyclic tiles of 128 1035 -> 980, of 256 960 -> 940; 6784 x 3003 x 7824 in
// 100 x 100 ones, packed, 1890 -> 985; 12223 x 8751 x 2891 uneven (three rounds either way) and 11441 x 9344 x 4245
// in column blocks of 530 and 531 (four rounds and a cut one, 1173; five on copies, 1570) stay.
bool choose_dense(const dmm_plan_t *P, const ExecArgs &x, bool given, int cus, bool *uncut) {
  const Grid &A = P->A, &B = P->B, &C = P->C;
  const int64_t M = C.rows, K = A.cols, N = C.cols, lim = (int64_t)1 << 30;
  if (x.es != 2 || P->dense_copy || (P->flags & DMM_MERGE_ALWAYS) || (x.flags & DMM_NO_MERGE)) return false;
  if (P->merged.valid && !g_comp_ok[x.device]) return false;
  if ((P->flags & (DMM_STATIONARY_B | DMM_STATIONARY_A)) && (A.c != 1 || B.c != 1 || C.c != 1)) return false;   // (their replicas do not split K)
  if (M < 1024 || N < 1024 || K < 1024 * (int64_t)C.c || M >= lim || K >= lim || N >= lim) return false;
  if (A.tiles_per_rep() + B.tiles_per_rep() > 65536) return false;
  const double bytes = 2.0 * ((double)M * K + (double)K * N);
  if (bytes > (double)kDenseMost) return false;
  size_t items = 0;
  if (P->merged.valid) items = P->merged.items.size();
  else
    for (const dmm_work_item &w : P->items) items += w.group >= 0;
  if (items < (size_t)cus) return false;
  DenseShape d;
  dense_shape(P, x.bk, &d);
  if (dense_bytes(P, d) > kDenseMost) return false;
  int64_t dense_items = 0, merged_items = 0;
  for (int32_t i = 0; i < C.gr; ++i)
    for (int32_t j = 0; j < C.gc; ++j)
      dense_items += ((C.rc[i + 1] - C.rc[i] + kMacroTile - 1) / kMacroTile) * ((C.cc[j + 1] - C.cc[j] + kMacroTile - 1) / kMacroTile);
  // (what dmm_plan will choose: merged macro-tiles end at column cuts that are not aligned)
  merged_items = (int64_t)(tile_axis(merged_cuts({&C.rc}), kMaxPieces, 1, kMacroTile).size() *
                           tile_axis(merged_cuts({&C.cc}), kMaxPieces, kPieceAlign, kMacroTile).size());
  const bool merge = g_comp_ok[x.device] && merged_items * 10 <= dense_items * 9;
  const std::vector<int64_t> nc = merged_cuts({&B.cc, &C.cc});
  const int64_t steps = d.len / x.bk;                                 // (of the longest share)
  const double segs = (double)(d.kc.size() - 1) / C.c, us = 0.72;
  // rounds of macro-tiles; the own list's last one is cut along K where it is at most half full
  const bool cut = last_round_is_cut((int64_t)items, steps, x.es, cus);
  auto rounds = [&](int64_t n) { return (double)((n + cus - 1) / cus); };
  double own = rounds((int64_t)items);
  if (cut) {
    const int64_t tail = (int64_t)items % cus;
    own += 1.0 / (double)std::min<int64_t>(cus / tail, steps / min_run_steps(x.es)) - 1.0;
  }
  own *= ((double)steps + 1.5 * segs) * us * (P->merged.valid ? 1.13 : 1.0);
  const double then = rounds((merge ? merged_items : dense_items) * C.c) * ((double)steps + 1.5) * us * (merge ? 1.08 : 1.0) +
                      ((double)dense_bytes(P, d) + bytes) / 4.5e6 + 5;
  const bool odd = std::max(cut_misaligned(A, d.kc), cut_misaligned(B, nc)) > 0.1;
  if (odd) own *= 1.27;
  // (not for a tie: of per-group lists the estimate is good to a tenth; 8832 x 10112 x 2847 uneven, 0.93 by the
  // estimate, took 655 us on copies and 567 on its operands)
  const double much = P->merged.valid ? 0.93 : 0.88;
  const bool by_shape = then < much * own;
  if (cut || in_windows(P)) {
    *uncut = by_shape;
    return by_shape && given;
  }
  if (!given) return false;
  return by_shape || (!odd && then < much * 1.12 * own && (placed_misaligned(A, x.a_tiles, x.a_ld) || placed_misaligned(B, x.b_tiles, x.b_ld)));
}

int stage(dmm_plan_t *P, ExecArgs &x, hipStream_t stream, ExecLayout *L);

// The tables of the product on the copies.
int stage_dense(dmm_plan_t *P, const ExecArgs &x, hipStream_t stream, ExecLayout *L) {
  DeviceState &D = *P->dev;
  const void *b = D.pack_b;
  ExecArgs in = x;
  in.a_tiles = D.pack_a.data();
  in.a_ld = D.pack_lda.data();
  in.b_tiles = &b;
  in.b_ld = &D.pack_ldb;
  in.uncut = true;
  return stage(D.dense, in, stream, L);
}

// Launches the copy, whose tables are in place.
int launch_copy(dmm_plan_t *P, const ExecArgs &x, hipStream_t stream) {
  int rc;
  DeviceState &D = *P->dev;
  const bool timed = (x.flags & DMM_TIMING) != 0;
  if (timed) {
    if ((rc = timing_events(D.t_pack))) return rc;
    DMM_HIP(hipEventRecord(D.t_pack[0], stream));
  }
  TraceRange tr("copy_operands");
  const char *d = D.pack_table.dev();
  hipLaunchKernelGGL(pack_kernel, dim3((unsigned)D.pack_blocks), dim3(256), 0, stream, (const PackJob *)d, D.pack_jobs,
                     (const PackRun *)(d + D.pack_o_runs), (const PackTile *)(d + D.pack_o_tiles));
  DMM_HIP(hipGetLastError());
  D.pack_launched = true;
  if (timed) DMM_HIP(hipEventRecord(D.t_pack[1], stream));
  return DMM_OK;
}

// Gives back everything that is there for products on copies.
void drop_dense(dmm_plan_t *P, hipStream_t stream) {
  DeviceState &D = *P->dev;
  if (D.pack_kept) return;
  if (D.dense) dmm_plan_destroy(D.dense);       // (waits for the calls on copies)
  D.dense = nullptr;
  D.pack_table.release();
  pack_pool().give_back(&D.pack, stream);
}

// A buffer of D.pack_need bytes for the copies of this call.
int take_copies(DeviceState &D, hipStream_t stream) {
  if (D.pack_kept) return D.dense->dev->uses.order(stream);
  int rc;
  if (!D.pack.p && (rc = pack_pool().acquire(D.pack_need, stream, D.pack_at, &D.pack))) return rc;
  D.pack_kept = is_capturing(stream);                       // (the graph may run any time from now on)
  return DMM_OK;
}

// The plan on the copies, the copies' buffer, the tables of the copy and, while the copy runs already,
// those of the product on it (70 us of host work for 8192^3 in 128 x 128 tiles).  With them in
// place a call cannot run out of memory any more.  DMM_ENOMEM: no room (if it was the last tables that
// had none, the copy was for nothing).
int build_dense_exec(dmm_plan_t *P, const ExecArgs &x, hipStream_t stream, ExecLayout *L) {
  int rc;
  DeviceState &D = *P->dev;
  const Grid &A = P->A, &B = P->B, &C = P->C;
  const int64_t M = C.rows, N = C.cols;
  DenseShape d;
  dense_shape(P, x.bk, &d);
  if (!D.dense) {
    const int64_t len = d.len * C.c, all_m[2] = {0, M}, all_k[2] = {0, len}, all_n[2] = {0, N};
    std::vector<int64_t> shares;        // (the planner's own split of K: the shares are of one length)
    for (int32_t r = 0; r <= C.c; ++r) shares.push_back(r * d.len);
    const dmm_matrix_desc a = {M, len, 1, C.c, all_m, shares.data(), 1, 1, 1}, b = {len, N, 1, 1, all_k, all_n, 1, 1, 1},
                          c = {M, N, C.gr, C.gc, C.rc.data(), C.cc.data(), C.pr, C.pc, C.c};
    if ((rc = dmm_plan(&a, &b, &c, P->nranks, 0, &D.dense))) return rc;
    D.dense->dense_copy = true;
  }
  if ((rc = ensure_state(D.dense))) return rc;
  const int64_t lda = dense_ld(d.len), share_bytes = 2 * M * lda, need = dense_bytes(P, d);
  D.pack_ldb = dense_ld(N);
  D.pack_need = (size_t)need;
  if ((rc = take_copies(D, stream))) return rc;
  D.pack_at = D.pack.p;
  std::vector<PackRun> runs;
  std::vector<PackTile> tiles;
  std::vector<PackJob> jobs;
  int32_t blocks = 0;
  auto operand = [&](const Grid &G, const void *const *ptr, const int64_t *ld) {
    for (int64_t i = 0; i < G.tiles_per_rep(); ++i) tiles.push_back({(const char *)ptr[i], ld[i] * 2});
  };
  // `rows_out` rows of a copy, `rows` of them from a tile row; runs [first_run, end) say where their columns come from
  auto job = [&](int64_t first_tile, int64_t row, int64_t rows, int64_t rows_out, size_t first_run, int64_t cols_out, char *dst, int64_t ld) {
    PackJob j;
    std::memset(&j, 0, sizeof(j));
    j.dst = dst;
    j.pitch = ld * 2;
    j.rows = (int32_t)rows;
    j.rows_out = (int32_t)rows_out;
    j.row = (int32_t)row;
    j.cols_out = (int32_t)cols_out;
    j.runs = (int32_t)first_run;
    j.n_runs = (int32_t)(runs.size() - first_run);
    j.tiles = (int32_t)first_tile;
    j.first_block = blocks;
    j.blocks_c = (int32_t)((cols_out + PACK_COLS - 1) / PACK_COLS);
    blocks += j.blocks_c * (int32_t)((rows_out + PACK_ROWS - 1) / PACK_ROWS);
    jobs.push_back(j);
  };
  auto holder = [](const std::vector<int64_t> &cuts, int64_t pos) {
    return (int32_t)(std::upper_bound(cuts.begin(), cuts.end() - 1, pos) - cuts.begin()) - 1;
  };
  const size_t S = d.kc.size() - 1;
  operand(A, x.a_tiles, x.a_ld);
  D.pack_a.clear();
  D.pack_lda.assign((size_t)C.c, lda);
  for (int32_t r = 0; r < C.c; ++r) {
    const size_t first = runs.size();
    char *dst = D.pack.p + r * share_bytes;
    for (size_t s = 0; s < S; ++s)
      if (d.share[s] == r) {
        if (runs.size() == first && d.at[s] > 0) runs.push_back({0, 0, 0, 0});
        const int32_t tj = holder(A.cc, d.kc[s]);
        runs.push_back({(int32_t)d.at[s], (int32_t)(d.kc[s + 1] - d.kc[s]), tj, (int32_t)(d.kc[s] - A.cc[tj])});
      }
    for (int32_t i = 0; i < A.gr; ++i) {
      const int64_t h = A.rc[i + 1] - A.rc[i];
      if (h > 0) job((int64_t)i * A.gc, 0, h, h, first, d.len, dst + 2 * A.rc[i] * lda, lda);
    }
    D.pack_a.push_back(dst);
  }
  const int64_t b_tile = (int64_t)tiles.size();
  const size_t b_runs = runs.size();
  operand(B, x.b_tiles, x.b_ld);
  D.pack_b = D.pack.p + C.c * share_bytes;
  for (int32_t k = 0; k < B.gc; ++k)
    if (B.cc[k + 1] > B.cc[k]) runs.push_back({(int32_t)B.cc[k], (int32_t)(B.cc[k + 1] - B.cc[k]), k, 0});
  for (size_t s = 0; s < S; ++s) {
    const int64_t base = d.share[s] * d.len, len = d.kc[s + 1] - d.kc[s];
    const bool first = s == 0 || d.share[s - 1] != d.share[s], last = s + 1 == S || d.share[s + 1] != d.share[s];
    const int32_t ti = holder(B.rc, d.kc[s]);
    if (first && d.at[s] > 0) job(b_tile, 0, 0, d.at[s], b_runs, N, D.pack_b + 2 * base * D.pack_ldb, D.pack_ldb);
    job(b_tile + (int64_t)ti * B.gc, d.kc[s] - B.rc[ti], len, (last ? d.len : d.at[s + 1]) - d.at[s], b_runs, N,
        D.pack_b + 2 * (base + d.at[s]) * D.pack_ldb, D.pack_ldb);
  }
  D.pack_jobs = (int)jobs.size();
  D.pack_blocks = blocks;
  D.pack_o_tiles = jobs.size() * sizeof(PackJob);
  D.pack_o_runs = D.pack_o_tiles + tiles.size() * sizeof(PackTile);
  std::vector<char> &h = D.host;
  h.assign(D.pack_o_runs + runs.size() * sizeof(PackRun), 0);
  std::memcpy(h.data(), jobs.data(), jobs.size() * sizeof(PackJob));
  std::memcpy(h.data() + D.pack_o_tiles, tiles.data(), tiles.size() * sizeof(PackTile));
  std::memcpy(h.data() + D.pack_o_runs, runs.data(), runs.size() * sizeof(PackRun));
  if ((rc = D.pack_table.upload(h.data(), h.size(), stream, D.dense->dev->uses))) return rc;
  if ((rc = launch_copy(P, x, stream))) return rc;
  ExecLayout product;
  if ((rc = stage_dense(P, x, stream, &product))) {
    const int rc2 = D.dense->dev->uses.mark(stream);      // (of the copy)
    return rc2 ? rc2 : rc;
  }
  L->dense = true;
  return DMM_OK;
}

// Whether every tile that the call's own work list would read has a pointer, and every tile of the
// first replicas of A and B: the kernels for small products and the copies read only these
// (replicas are copies of each other, Section 3); what the other work lists refuse is refused all
// the same, and what they accept they get.
bool operands_given(const dmm_plan_t *P, const ExecArgs &x) {
  auto given = [](const Grid &G, const void *const *tiles, int32_t rep) {
    for (int32_t i = 0; i < G.gr; ++i)
      for (int32_t j = 0; j < G.gc; ++j)
        if (G.rc[i + 1] > G.rc[i] && G.cc[j + 1] > G.cc[j] && !tiles[G.table_index(rep, i, j)]) return false;
    return true;
  };
  if (!given(P->A, x.a_tiles, 0) || !given(P->B, x.b_tiles, 0)) return false;
  if (P->merged.valid) {
    for (const MergedRep &R : P->merged.reps)
      if (!given(P->A, x.a_tiles, R.a_rep) || !given(P->B, x.b_tiles, R.b_rep)) return false;
    return true;
  }
  for (const dmm_task &t : P->tasks)
    if (!x.a_tiles[P->A.table_index(t.a_rep, t.a_ti, t.a_tj)] || !x.b_tiles[P->B.table_index(t.b_rep, t.b_ti, t.b_tj)]) return false;
  return true;
}

// The launches of one dmm_execute, from the device table the layout describes.
int launch_exec(dmm_plan_t *P, const ExecLayout &L, int64_t es, hipStream_t stream, bool timed) {
  int rc;
  // the event that stands for the call goes with its last launch
  hipEvent_t behind = nullptr;
  bool marked = false;
  if ((rc = P->dev->uses.claim(stream, &behind))) return rc;
  const hipEvent_t behind_gemm = L.red.n_items > 0 ? nullptr : behind;
  char *d = P->dev->gemm_table.dev();
  if (L.small.shape >= 0) {
    const SmallLaunch &l = L.small;
    SmallArgs g;
    g.rows = (const SmallTile *)(d + l.o_rows);
    g.cols = (const SmallTile *)(d + l.o_cols);
    g.mc = (const int32_t *)(d + l.o_mc);
    g.nc = (const int32_t *)(d + l.o_nc);
    g.starts = (const SmallStart *)(d + l.o_starts);
    g.klen = (const int32_t *)(d + l.o_klen);
    g.pa = (const PieceDev *)(d + l.o_a);
    g.pb = (const PieceDev *)(d + l.o_b);
    g.pc = (const PieceDev *)(d + l.o_c);
    g.scratch = (float *)P->dev->split_buf;
    g.S = l.segs;
    g.NR = l.nr;
    g.tiles_m = l.tiles_m;
    g.tiles_n = l.tiles_n;
    g.runs = l.runs;
    g.per = l.per;
    g.c_es = l.c_es;
    g.band = es == 2 ? SMALL_BAND : 1;
    g.steps = l.steps;
    g.pad = 0;
    int cus = 0;
    if ((rc = device_cus(&cus))) return rc;
    TraceRange gemm("gemm");
    if (timed) {
      if ((rc = timing_events(P->dev->t_gemm))) return rc;
      DMM_HIP(hipEventRecord(P->dev->t_gemm[0], stream));
    }
    for (g.first = 0; g.first < l.tiles_m * l.tiles_n; g.first += l.batch) {
      g.tiles = std::min(l.batch, l.tiles_m * l.tiles_n - g.first);
      marked = small_launch(g.first + g.tiles < l.tiles_m * l.tiles_n ? nullptr : behind_gemm, l.shape, g, cus, stream);
      DMM_HIP(hipGetLastError());
    }
    if (timed) {
      DMM_HIP(hipEventRecord(P->dev->t_gemm[1], stream));
      P->dev->gemm_timed = true;
    }
    P->dev->ran_merged = false;
    P->dev->ran_small = l.shape;
    P->dev->small_runs = l.runs;
    // (the waves of the one shape share a tile's K steps, those of the other add up 16 k at a time)
    P->dev->ran_k_split = l.runs > 1 || l.shape == SMALL_F32_TINY || l.shape == SMALL_F32_SPLIT;
    P->dev->ran_fused = 0;
  } else if (L.merged) {
    const MergedLaunch &ml = L.ml;
    TraceRange gemm("gemm");
    if (timed) {
      if ((rc = timing_events(P->dev->t_gemm))) return rc;
      DMM_HIP(hipEventRecord(P->dev->t_gemm[0], stream));
    }
    marked = launch_grouped_gemm_comp(ml.n_fix > 0 ? nullptr : behind_gemm, (int)es, (unsigned)ml.n_items, stream, (const CompItemDev *)d, (const PieceDev *)(d + ml.o_a),
                             (const PieceDev *)(d + ml.o_b), (const PieceDev *)(d + ml.o_c), (const int32_t *)(d + ml.o_k));
    DMM_HIP(hipGetLastError());
    if (ml.n_fix > 0) {
      marked = launch_behind(behind_gemm, sum_parts_kernel, (unsigned)(ml.n_fix * (BM / FIX_ROWS)), 256, 0, stream, (const FixItem *)(d + ml.o_fix));
      DMM_HIP(hipGetLastError());
    }
    if (timed) {
      DMM_HIP(hipEventRecord(P->dev->t_gemm[1], stream));
      P->dev->gemm_timed = true;
    }
    gemm.end();
    P->dev->ran_merged = true;
    P->dev->ran_k_split = ml.n_fix > 0;
    P->dev->ran_fused = 0;
  } else {
    P->dev->ran_merged = false;
    if (L.n_items > 0) {
      int cus = 0;
      if ((rc = device_cus(&cus))) return rc;
      const size_t n_items = L.n_items, n_first = L.n_first;
      const bool fuse = L.fuse, one_launch = L.one_launch;
      TraceRange gemm("gemm");
      const ItemDev *di = (const ItemDev *)d;
      const SegDev *ds = (const SegDev *)(d + L.o_segs);
      if (timed) {
        if ((rc = timing_events(P->dev->t_gemm))) return rc;
        DMM_HIP(hipEventRecord(P->dev->t_gemm[0], stream));
      }
      const RedSrc *dr = (const RedSrc *)(d + L.o_red);
      // {first item, count} per launch
      const size_t part[2][2] = {{0, one_launch ? n_items : n_first}, {n_first, one_launch ? 0 : n_items - n_first}};
      for (int l = 0; l < 2; ++l) {
        if (part[l][1] == 0) continue;
        const bool sums = fuse && (l == 1 || one_launch);   // the launch whose macro-tiles add the other replicas' partial sums
        // one workgroup per CU at most: workgroup w walks items w, w + grid, w + 2 grid, ... of its launch
        const int count = (int)part[l][1];
        const bool ends = L.n_fix == 0 && (l == 1 || part[1][1] == 0);
        marked = launch_grouped_gemm(ends ? behind_gemm : nullptr, (int)es, sums, (unsigned)std::min(count, cus), stream, di + part[l][0], ds, dr, count);
        DMM_HIP(hipGetLastError());
        if (timed && fuse && !one_launch && l == 0 && part[1][1] > 0) {
          if (!P->dev->t_mid) DMM_HIP(hipEventCreate(&P->dev->t_mid));
          DMM_HIP(hipEventRecord(P->dev->t_mid, stream));
          P->dev->mid_timed = true;
          P->dev->launch_flops[0] = P->dev->launch_flops[1] = 0.0;
          for (const dmm_task &t : P->tasks)
            P->dev->launch_flops[t.c_rep == 0 ? 1 : 0] += 2.0 * (double)(t.m1 - t.m0) * (double)(t.n1 - t.n0) * (double)(t.k1 - t.k0);
        }
      }
      if (L.n_fix > 0) {
        marked = launch_behind(behind_gemm, sum_parts_kernel, (unsigned)(L.n_fix * (BM / FIX_ROWS)), 256, 0, stream, (const FixItem *)(d + L.o_fix));
        DMM_HIP(hipGetLastError());
      }
      if (timed) {
        DMM_HIP(hipEventRecord(P->dev->t_gemm[1], stream));
        P->dev->gemm_timed = true;
      }
    }
    P->dev->ran_k_split = L.n_runs > 0;
    P->dev->ran_fused = !L.fuse ? 0 : L.one_launch ? 1 : 2;
  }
  {
    TraceRange tr("replica_sum");
    if ((rc = fire_reduce(P, L.red, stream, timed, behind, &marked))) return rc;
  }
  return marked ? DMM_OK : P->dev->uses.mark(stream);
}

int launch_dense(dmm_plan_t *P, const ExecArgs &x, hipStream_t stream, bool timed) {
  int rc;
  DeviceState &D = *P->dev;
  ExecLayout product;
  if (!D.pack_launched && (rc = launch_copy(P, x, stream))) return rc;
  // (the tables are in place: this orders the stream behind them)
  if ((rc = stage_dense(P, x, stream, &product)) || (rc = launch_exec(D.dense, product, x.es, stream, timed))) return rc;
  dmm_execute_report r;
  if ((rc = dmm_plan_last_execute(D.dense, &r))) return rc;
  D.ran_merged = r.ran_merged != 0;
  D.ran_k_split = r.ran_k_split != 0;
  D.ran_fused = r.ran_fused;
  D.ran_dense = true;
  return DMM_OK;
}

// Decides what a call runs and puts its work tables in place.
int stage(dmm_plan_t *P, ExecArgs &x, hipStream_t stream, ExecLayout *L) {
  int rc;
  DeviceState &D = *P->dev;
  D.gemm_timed = D.red_timed = D.mid_timed = false;
  D.ran_dense = D.pack_launched = false;
  D.ran_small = -1;
  // The call's inputs, side by side: when they are those of the plan's last dmm_execute, the
  // device table of that call is still in place and describes this one too (DMM_TIMING changes
  // nothing in it), so the assembly of the tables and their upload are skipped.
  std::vector<char> &key = D.key_scratch;
  key.clear();
  auto put = [&key](const void *p, size_t bytes) { key.insert(key.end(), (const char *)p, (const char *)p + bytes); };
  const int64_t head[3] = {x.dtype, (int64_t)(x.flags & ~DMM_TIMING), x.device};
  put(head, sizeof head);
  const size_t na = (size_t)(P->A.c * P->A.tiles_per_rep()), nb = (size_t)(P->B.c * P->B.tiles_per_rep()),
               nc = (size_t)(P->C.c * P->C.tiles_per_rep());
  put(x.a_tiles, na * sizeof(void *));
  put(x.a_ld, na * sizeof(int64_t));
  put(x.b_tiles, nb * sizeof(void *));
  put(x.b_ld, nb * sizeof(int64_t));
  put(x.c_tiles, nc * sizeof(void *));
  put(x.c_ld, nc * sizeof(int64_t));
  if (D.exec_cached && key == D.exec_key) {
    *L = D.exec_layout;
    D.table_reused = true;
    // (the scratch buffer of macro-tiles cut along K is shared by all calls on this plan)
    if (!L->dense) return (rc = D.gemm_table.order_behind_copy(stream)) || !L->uses_split ? rc : D.uses.order(stream);
    if (!(rc = take_copies(D, stream)) && D.pack.p == D.pack_at) return D.pack_table.order_behind_copy(stream);
    if (rc && rc != DMM_ENOMEM) return rc;
    *L = ExecLayout();             // the copies get another place, or none
  }
  D.exec_cached = false;
  D.table_reused = false;
  TraceRange tables("tables");
  SmallPlan sp;
  int cus = 0;
  if ((rc = device_cus(&cus))) return rc;
  const bool given = operands_given(P, x);
  if (given) choose_small(P, x, cus, &sp);
  bool built = false;
  if ((given && sp.shape >= 0) || choose_dense(P, x, given, cus, &x.uncut)) {
    rc = sp.shape >= 0 ? build_small_exec(P, x, sp, stream, L) : build_dense_exec(P, x, stream, L);
    if (rc == DMM_ENOMEM) {
      // no room for copies (or for anything): the call's own work list, which may do with less
      (void)hipGetLastError();
      if (sp.shape < 0) drop_dense(P, stream);
      *L = ExecLayout();
    } else {
      built = true;
    }
  }
  if (!built) {
    if (P->merged.valid && !(x.flags & DMM_NO_MERGE) && g_comp_ok[x.device] && !(x.uncut && in_windows(P))) rc = build_merged_exec(P, x, stream, L);
    else rc = build_group_exec(P, x, stream, L);
  }
  if (rc) return rc;
  D.exec_key = key;
  D.exec_layout = *L;
  D.exec_cached = true;
  return DMM_OK;
}

}  // namespace
}  // namespace dmm

int dmm_execute(dmm_plan_t *P, int dtype, const void *const *a_tiles, const int64_t *a_ld,
                const void *const *b_tiles, const int64_t *b_ld, void *const *c_tiles, const int64_t *c_ld,
                uint32_t flags, void *hip_stream) {
  using namespace dmm;
  if (!P || !a_tiles || !a_ld || !b_tiles || !b_ld || !c_tiles || !c_ld) return DMM_EINVAL;
  if (dtype != DMM_BF16 && dtype != DMM_F32) return DMM_EINVAL;
  if (flags & ~(DMM_NO_REDUCE | DMM_TIMING | DMM_C_BF16 | DMM_NO_MERGE | DMM_SEPARATE_REDUCE)) return DMM_EINVAL;
  const bool timed = (flags & DMM_TIMING) != 0;
  // bf16 C tiles only where a tile receives a final sum: partial sums of a replicated C stay fp32
  if ((flags & DMM_C_BF16) && P->C.c != 1) return DMM_EINVAL;
  const int64_t c_es = (flags & DMM_C_BF16) ? 2 : 4;
  int rc;
  if ((rc = check_lds(P->A, a_ld)) || (rc = check_lds(P->B, b_ld)) || (rc = check_lds(P->C, c_ld))) return rc;
  const int64_t es = dtype == DMM_BF16 ? 2 : 4;
  const int64_t bk = dtype == DMM_BF16 ? Shape<2>::BK : Shape<4>::BK;
  // the kernel addresses a macro-tile's rows with 32-bit byte offsets, built as a 24-bit
  // multiply of (row, pitch): every row pitch has to stay below 2^24 bytes
  constexpr int64_t MAX_PITCH = (int64_t)1 << 24;
  for (int64_t i = 0; i < P->A.c * P->A.tiles_per_rep(); ++i)
    if (a_ld[i] * es >= MAX_PITCH) return DMM_ELD;
  for (int64_t i = 0; i < P->B.c * P->B.tiles_per_rep(); ++i)
    if (b_ld[i] * es >= MAX_PITCH) return DMM_ELD;
  for (int64_t i = 0; i < P->C.c * P->C.tiles_per_rep(); ++i)
    if (c_ld[i] * c_es >= MAX_PITCH) return DMM_ELD;
  hipStream_t stream = (hipStream_t)hip_stream;
  TraceRange whole("dmm_execute");
  try {
    if ((rc = ensure_state(P))) return rc;
    int device = 0;
    DMM_HIP(hipGetDevice(&device));
    ExecArgs x = {dtype, es, bk, c_es, a_tiles, a_ld, b_tiles, b_ld, c_tiles, c_ld, flags, device, false};
    ExecLayout L;
    struct HandBack {                  // the copies' buffer, behind all that was enqueued
      DeviceState &D;
      hipStream_t stream;
      ~HandBack() {
        if (D.pack_launched && !D.ran_dense && D.dense) (void)D.dense->dev->uses.mark(stream);   // (a copy whose product failed)
        if (!D.pack_kept) pack_pool().give_back(&D.pack, stream);
      }
    } hand_back = {*P->dev, stream};
    if ((rc = stage(P, x, stream, &L))) return rc;
    if (L.dense) return launch_dense(P, x, stream, timed);
    return launch_exec(P, L, es, stream, timed);
  } catch (const std::bad_alloc &) {
    return DMM_ENOMEM;
  }
}

int dmm_plan_gemm_launch_ms(dmm_plan_t *P, float ms[2], double flops[2]) {
  using namespace dmm;
  if (!P || !ms || !flops) return DMM_EINVAL;
  ms[0] = ms[1] = -1.f;
  flops[0] = flops[1] = 0.0;
  if (P->dev && P->dev->ran_dense) return dmm_plan_gemm_launch_ms(P->dev->dense, ms, flops);
  if (!P->dev || !P->dev->gemm_timed || !P->dev->mid_timed) return DMM_OK;
  DMM_HIP(hipEventSynchronize(P->dev->t_gemm[1]));
  DMM_HIP(hipEventElapsedTime(&ms[0], P->dev->t_gemm[0], P->dev->t_mid));
  DMM_HIP(hipEventElapsedTime(&ms[1], P->dev->t_mid, P->dev->t_gemm[1]));
  flops[0] = P->dev->launch_flops[0];
  flops[1] = P->dev->launch_flops[1];
  return DMM_OK;
}

int dmm_plan_last_execute(const dmm_plan_t *P, dmm_execute_report *out) {
  if (!out) return DMM_EINVAL;
  *out = dmm_execute_report{0, 0, 0, 0};
  if (!P || !P->dev) return DMM_OK;
  out->ran_merged = P->dev->ran_merged ? 1 : 0;
  out->ran_k_split = P->dev->ran_k_split ? 1 : 0;
  out->ran_fused = P->dev->ran_fused;
  out->table_reused = P->dev->table_reused ? 1 : 0;
  return DMM_OK;
}

int dmm_plan_last_kernels(const dmm_plan_t *P, dmm_kernel_report *out) {
  using namespace dmm;
  if (!out) return DMM_EINVAL;
  *out = dmm_kernel_report{0, 0, 0, 0};
  if (!P || !P->dev) return DMM_OK;
  if (P->dev->ran_small >= 0) {
    out->small_rows = kSmall[P->dev->ran_small].tm;
    out->small_cols = kSmall[P->dev->ran_small].tn;
    out->small_runs = P->dev->small_runs;
  }
  out->ran_dense = P->dev->ran_dense ? 1 : 0;
  return DMM_OK;
}

int dmm_plan_elapsed_ms(dmm_plan_t *P, float *gemm_ms, float *reduce_ms) {
  using namespace dmm;
  if (!P) return DMM_EINVAL;
  float g = -1.f, r = -1.f;
  if (P->dev && P->dev->ran_dense) {
    // (the copy of the operands counts as part of the product)
    float ms = 0.f;
    int rc = dmm_plan_elapsed_ms(P->dev->dense, &g, &r);
    if (rc) return rc;
    if (g >= 0.f) {
      DMM_HIP(hipEventElapsedTime(&ms, P->dev->t_pack[0], P->dev->t_pack[1]));
      g += ms;
    }
  }
  if (P->dev && P->dev->gemm_timed) {
    DMM_HIP(hipEventSynchronize(P->dev->t_gemm[1]));
    DMM_HIP(hipEventElapsedTime(&g, P->dev->t_gemm[0], P->dev->t_gemm[1]));
  }
  if (P->dev && P->dev->red_timed) {
    DMM_HIP(hipEventSynchronize(P->dev->t_red[1]));
    DMM_HIP(hipEventElapsedTime(&r, P->dev->t_red[0], P->dev->t_red[1]));
  }
  if (gemm_ms) *gemm_ms = g;
  if (reduce_ms) *reduce_ms = r;
  return DMM_OK;
}

int dmm_reduce_replicas(dmm_plan_t *P, void *const *c_tiles, const int64_t *c_ld, int32_t origin_replica,
                        void *hip_stream) {
  using namespace dmm;
  if (!P || !c_tiles || !c_ld) return DMM_EINVAL;
  if (origin_replica < 0 || origin_replica >= P->C.c) return DMM_EINVAL;
  int rc;
  if ((rc = check_lds(P->C, c_ld))) return rc;
  TraceRange whole("dmm_reduce_replicas");
  try {
    if ((rc = ensure_state(P))) return rc;
    RedLaunch red;
    if ((rc = stage_reduce(P, c_tiles, c_ld, origin_replica, (hipStream_t)hip_stream, &red))) return rc;
    hipEvent_t behind = nullptr;
    bool marked = false;
    if (P->C.c > 1 && (rc = P->dev->uses.claim((hipStream_t)hip_stream, &behind))) return rc;
    if ((rc = fire_reduce(P, red, (hipStream_t)hip_stream, false, behind, &marked))) return rc;
    return P->C.c > 1 && !marked ? P->dev->uses.mark((hipStream_t)hip_stream) : DMM_OK;
  } catch (const std::bad_alloc &) {
    return DMM_ENOMEM;
  }
}

int dmm_broadcast_replica(dmm_plan_t *P, void *const *c_tiles, const int64_t *c_ld, int32_t origin_replica,
                          void *hip_stream) {
  using namespace dmm;
  if (!P || !c_tiles || !c_ld) return DMM_EINVAL;
  if (origin_replica < 0 || origin_replica >= P->C.c) return DMM_EINVAL;
  int rc;
  if ((rc = check_lds(P->C, c_ld))) return rc;
  TraceRange whole("dmm_broadcast_replica");
  try {
    if ((rc = ensure_state(P))) return rc;
    hipStream_t stream = (hipStream_t)hip_stream;
    RedLaunch L;
    if ((rc = stage_reduce(P, c_tiles, c_ld, origin_replica, stream, &L))) return rc;
    if (L.n_items == 0) return DMM_OK;
    char *d = L.dev_base;
    hipEvent_t behind = nullptr;
    if ((rc = P->dev->uses.claim(stream, &behind))) return rc;
    const bool marked = launch_behind(behind, broadcast_replica_kernel, (unsigned)L.n_items, RED_NT, 0, stream, (const RedItem *)(d + L.o_items),
                                      (const RedTile *)(d + L.o_tiles), (float *const *)(d + L.o_parts), (const int64_t *)(d + L.o_lds),
                                      L.nparts, L.vec_ok ? 1 : 0);
    DMM_HIP(hipGetLastError());
    return marked ? DMM_OK : P->dev->uses.mark(stream);
  } catch (const std::bad_alloc &) {
    return DMM_ENOMEM;
  }
}

}  // extern "C"

// ------------------------------------------------------------------ no allocation: static tables

// The replica sum's work tables for dmm_reduce_replicas_static.  In host code this name stands in
// for the symbol only: the memory is reached through the address hipGetSymbolAddress returns on
// each device (static_scratch below), never through the name.
static __device__ __align__(256) unsigned char scratch[DMM_STATIC_SCRATCH_BYTES];

namespace dmm {
namespace {

// Device address of `scratch` on the current device (every GPU holds its own copy), looked up
// once per device.
int static_scratch(char **out) {
  static std::mutex mu;
  static char *ptr[64] = {};
  int dev = 0;
  DMM_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64) return DMM_EINVAL;
  std::lock_guard<std::mutex> g(mu);
  if (!ptr[dev]) {
    void *p = nullptr;
    DMM_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return DMM_EHIP;
    ptr[dev] = (char *)p;
  }
  *out = ptr[dev];
  return DMM_OK;
}

// The tables of build_reduce, laid out the same way (items | tiles | part pointers | part lds),
// written into `dst` (capacity `cap` bytes) without any allocation: sizes first, then the records.
int build_reduce_in_place(const dmm_plan_t *P, void *const *c_tiles, const int64_t *c_ld, int32_t origin, char *dst,
                          size_t cap, RedLaunch *L, size_t *bytes) {
  const Grid &C = P->C;
  L->n_items = 0;
  *bytes = 0;
  if (C.c <= 1) return DMM_OK;
  const int nparts = C.c;
  auto rows_per_item = [](int64_t cols) { int64_t per = (RED_ELEMS + cols - 1) / cols; return per < 1 ? (int64_t)1 : per; };
  size_t n_tiles = 0, n_items = 0;
  for (int32_t ti = 0; ti < C.gr; ++ti)
    for (int32_t tj = 0; tj < C.gc; ++tj) {
      const int64_t rows = C.rc[ti + 1] - C.rc[ti], cols = C.cc[tj + 1] - C.cc[tj];
      if (rows <= 0 || cols <= 0) continue;
      const int64_t per = rows_per_item(cols);
      ++n_tiles;
      n_items += (size_t)((rows + per - 1) / per);
    }
  if (n_items == 0) return DMM_OK;
  const size_t o_items = 0;
  const size_t o_tiles = o_items + n_items * sizeof(RedItem);
  const size_t o_parts = o_tiles + n_tiles * sizeof(RedTile);
  const size_t o_lds = o_parts + n_tiles * (size_t)nparts * sizeof(void *);
  const size_t total = o_lds + n_tiles * (size_t)nparts * sizeof(int64_t);
  if (total > cap) return DMM_ELIMIT;
  RedItem *items = (RedItem *)(dst + o_items);
  RedTile *tiles = (RedTile *)(dst + o_tiles);
  const float **parts = (const float **)(dst + o_parts);
  int64_t *part_ld = (int64_t *)(dst + o_lds);
  bool vec_ok = true;
  size_t t_idx = 0, i_idx = 0;
  for (int32_t ti = 0; ti < C.gr; ++ti)
    for (int32_t tj = 0; tj < C.gc; ++tj) {
      const int64_t rows = C.rc[ti + 1] - C.rc[ti], cols = C.cc[tj + 1] - C.cc[tj];
      if (rows <= 0 || cols <= 0) continue;
      RedTile t;
      const int64_t oi = C.table_index(origin, ti, tj);
      t.out = (float *)c_tiles[oi];
      t.ldo = c_ld[oi];
      t.part_begin = (int64_t)(t_idx * (size_t)nparts);
      t.rows = (int32_t)rows;
      t.cols = (int32_t)cols;
      if (!t.out) return DMM_EINVAL;
      if (((uintptr_t)t.out & 15) || (t.ldo & 3) || (cols & 3)) vec_ok = false;
      for (int32_t rep = 0; rep < nparts; ++rep) {
        const int64_t pi = C.table_index(rep, ti, tj);
        const float *pp = (const float *)c_tiles[pi];
        if (!pp) return DMM_EINVAL;
        if (((uintptr_t)pp & 15) || (c_ld[pi] & 3)) vec_ok = false;
        parts[t_idx * (size_t)nparts + (size_t)rep] = pp;
        part_ld[t_idx * (size_t)nparts + (size_t)rep] = c_ld[pi];
      }
      const int64_t per = rows_per_item(cols);
      for (int64_t r = 0; r < rows; r += per) {
        RedItem it;
        it.tile = (int32_t)t_idx;
        it.row0 = (int32_t)r;
        it.nrows = (int32_t)(rows - r < per ? rows - r : per);
        it.pad = 0;
        items[i_idx++] = it;
      }
      tiles[t_idx++] = t;
    }
  L->n_items = n_items;
  L->o_items = o_items;
  L->o_tiles = o_tiles;
  L->o_parts = o_parts;
  L->o_lds = o_lds;
  L->nparts = nparts;
  L->vec_ok = vec_ok;
  *bytes = total;
  return DMM_OK;
}

}  // namespace
}  // namespace dmm

extern "C" int dmm_reduce_replicas_static(dmm_plan_t *P, void *const *c_tiles, const int64_t *c_ld,
                                          int32_t origin_replica, void *hip_stream) {
  using namespace dmm;
  if (!P || !c_tiles || !c_ld) return DMM_EINVAL;
  if (origin_replica < 0 || origin_replica >= P->C.c) return DMM_EINVAL;
  int rc;
  if ((rc = check_lds(P->C, c_ld))) return rc;
  hipStream_t stream = (hipStream_t)hip_stream;
  char *dev = nullptr;
  if ((rc = static_scratch(&dev))) return rc;
  // Fixed host buffers for all callers, taken in turn, one for the length of a call.  The copy
  // below reads pageable memory out (or stages it) before hipMemcpyAsync returns; taking four
  // buffers in turn means that even a copy that lagged behind its call would have to lag by four
  // calls to find its source overwritten.
  static std::mutex mu;
  constexpr int SLOTS = 4;
  alignas(16) static char slots[SLOTS][DMM_STATIC_SCRATCH_BYTES];
  static int next_slot = 0;
  std::lock_guard<std::mutex> g(mu);
  char *staging = slots[next_slot];
  RedLaunch L;
  size_t bytes = 0;
  if ((rc = build_reduce_in_place(P, c_tiles, c_ld, origin_replica, staging, DMM_STATIC_SCRATCH_BYTES, &L, &bytes))) return rc;
  if (L.n_items == 0) return DMM_OK;
  next_slot = (next_slot + 1) % SLOTS;
  DMM_HIP(hipMemcpyAsync(dev, staging, bytes, hipMemcpyHostToDevice, stream));
  hipLaunchKernelGGL(reduce_replicas_kernel, dim3((unsigned)L.n_items), dim3(RED_NT), 0, stream,
                     (const RedItem *)(dev + L.o_items), (const RedTile *)(dev + L.o_tiles),
                     (const float *const *)(dev + L.o_parts), (const int64_t *)(dev + L.o_lds), L.nparts, L.vec_ok ? 1 : 0);
  DMM_HIP(hipGetLastError());
  return DMM_OK;
}
