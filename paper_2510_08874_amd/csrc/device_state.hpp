// Host-side device resources of the library (included by exec.hip): error bookkeeping, the
// slab and scratch pools, the work-table uploader and the per-plan device state.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "dmm.h"
#include "gemm_launch.hpp"

namespace dmm {

// ------------------------------------------------------------------ host state

thread_local int g_last_hip_error = 0;

#define DMM_HIP(call)                            \
  do {                                           \
    hipError_t e_ = (call);                      \
    if (e_ != hipSuccess) {                      \
      g_last_hip_error = (int)e_;                \
      return DMM_EHIP;                           \
    }                                            \
  } while (0)

// A stream as the calling thread means it: hipStreamPerThread names another one in every thread.
struct StreamKey {
  hipStream_t stream = nullptr;
  uint64_t thread = 0;                 // (a number of our own: the system's are used again)

  static StreamKey of(hipStream_t stream) {
    static std::atomic<uint64_t> threads{0};
    static thread_local const uint64_t mine = ++threads;
    return {stream, stream == hipStreamPerThread ? mine : 0};
  }
  bool operator==(const StreamKey &o) const { return stream == o.stream && thread == o.thread; }
};

bool is_capturing(hipStream_t stream) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &status) != hipSuccess) (void)hipGetLastError();
  return status == hipStreamCaptureStatusActive;
}

// The calls of a plan whose kernels may still be running: an event behind the last call on each of
// the streams it was used on.  Whoever writes a buffer that those kernels use waits for all of them
// (one event for the plan would forget a stream as soon as the next call came on another).  A stream
// is not made to wait for its own event: it is in order by itself, and while it is being captured the
// runtime refuses to let it wait for what was recorded on it before.
class Uses {
 public:
  // behind everything the call enqueued on `stream`
  int mark(hipStream_t stream) {
    Entry *e = nullptr;
    const int rc = entry(stream, &e);
    if (rc) return rc;
    DMM_HIP(hipEventRecord(e->ev, stream));
    return DMM_OK;
  }
  // The event that the call's last launch on `stream` is to record; none: mark() then.  That is while the stream is being
  // captured, on hipStreamPerThread and hipStreamLegacy (launches that record events are documented for streams and for
  // the null stream only), and for one call of 32 in any case: of a stream of launches that record events themselves the runtime
  // keeps what it had for each until the host waits or an event is recorded behind them, and then works that off beside
  // the caller.  (256^3 fp32, after 20000 calls without a wait: the first calls of new plans took 60 to 130 us instead of 25, and
  // each of the 20000 8.2 us instead of 6.)  Every 8th, 32nd or 128th call made no difference.
  int claim(hipStream_t stream, hipEvent_t *ev) {
    static std::atomic<unsigned> calls{0};
    *ev = nullptr;
    if (stream == hipStreamPerThread || stream == hipStreamLegacy) return DMM_OK;
    if (calls.fetch_add(1, std::memory_order_relaxed) % 32 == 31 || is_capturing(stream)) return DMM_OK;
    Entry *e = nullptr;
    const int rc = entry(stream, &e);
    if (!rc) *ev = e->ev;
    return rc;
  }
  // orders what follows on `stream` behind all of them
  int order(hipStream_t stream) const {
    const StreamKey key = StreamKey::of(stream);
    for (int i = 0; i < n_; ++i)
      if (!(uses_[i].key == key)) DMM_HIP(hipStreamWaitEvent(stream, uses_[i].ev, 0));
    return DMM_OK;
  }
  // blocks until they have finished (all of them, also where one reports an error)
  int wait() const {
    int rc = DMM_OK;
    for (int i = 0; i < n_; ++i) {
      const hipError_t e = hipEventSynchronize(uses_[i].ev);
      if (e == hipSuccess) continue;
      g_last_hip_error = (int)e;
      rc = DMM_EHIP;
    }
    return rc;
  }
  void destroy() {
    for (int i = 0; i < n_; ++i) (void)hipEventDestroy(uses_[i].ev);
    n_ = 0;
  }

 private:
  static constexpr int kMost = 8;
  struct Entry {
    StreamKey key;
    hipEvent_t ev = nullptr;
  };
  // that of `stream`
  int entry(hipStream_t stream, Entry **out) {
    const StreamKey key = StreamKey::of(stream);
    Entry *e = nullptr;
    for (int i = 0; i < n_ && !e; ++i)
      if (uses_[i].key == key) e = &uses_[i];
    if (!e && n_ < kMost) {
      e = &uses_[n_];
      DMM_HIP(hipEventCreateWithFlags(&e->ev, hipEventDisableTiming));
      ++n_;
    } else if (!e) {
      // more streams than entries: the new event takes over from the one of another stream by
      // being recorded behind it too
      e = &uses_[next_];
      next_ = (next_ + 1) % kMost;
      DMM_HIP(hipStreamWaitEvent(stream, e->ev, 0));
    }
    e->key = key;
    *out = e;
    return DMM_OK;
  }
  Entry uses_[kMost] = {};
  int n_ = 0, next_ = 0;
};

// Buffers for dense copies of operands (pack_kernel.hpp), up to 2 GiB each, shared by all plans.  The
// copies live for one call: it takes a buffer, enqueues the copy and the product on it, and hands
// the buffer back behind them.  Calls on one stream share a buffer in stream order, calls on different
// streams have buffers of their own as long as all of a device's stay within 2 GiB, and wait for
// each other beyond that.  (More than 2 GiB are held only where that many are taken at one time, or
// kept for a captured graph.)
class PackPool {
 public:
  struct Lease {
    char *p = nullptr;
    size_t cap = 0;
    int device = 0;
    StreamKey stream;                  // that of the last call, behind which `done` is recorded
    hipEvent_t done = nullptr;
  };
  // A buffer for what is enqueued on `stream` from now on; the one at `last` if that is there, since
  // the caller has tables for it.  DMM_ENOMEM (nothing recorded): there is no room, the caller does without.
  int acquire(size_t bytes, hipStream_t stream, const char *last, Lease *out) {
    int device = 0;
    DMM_HIP(hipGetDevice(&device));
    if (device < 0 || device >= 64) return DMM_EINVAL;
    const StreamKey key = StreamKey::of(stream);
    std::lock_guard<std::mutex> g(mu_);
    int own = -1, any = -1;
    for (int i = 0; i < (int)free_.size(); ++i) {
      const Lease &e = free_[(size_t)i];
      if (e.device != device || e.cap < bytes) continue;
      if (e.p == last) return take(i, stream, out);
      if (e.stream == key && (own < 0 || e.cap < free_[(size_t)own].cap)) own = i;
      if (any < 0) any = i;                                  // (the one that has been free for longest)
    }
    if (own >= 0) return take(own, stream, out);
    const size_t want = (bytes + ((size_t)32 << 20) - 1) >> 25 << 25;
    if (held(device) + want <= kMost && allocate(want, device, out)) return DMM_OK;
    if (any >= 0) return take(any, stream, out);
    while (held(device) + want > kMost && drop_oldest(device)) {}
    if (allocate(want, device, out)) return DMM_OK;
    while (drop_oldest(device)) {}
    return allocate(want, device, out) ? DMM_OK : DMM_ENOMEM;
  }
  // behind everything on `stream` that uses it
  void give_back(Lease *l, hipStream_t stream) {
    if (!l->p) return;
    l->stream = StreamKey::of(stream);
    if (hipEventRecord(l->done, stream) != hipSuccess) (void)hipStreamSynchronize(stream);
    put(l);
  }
  // of a buffer that no call uses any more
  void put(Lease *l) {
    if (!l->p) return;
    std::lock_guard<std::mutex> g(mu_);
    free_.push_back(*l);
    out_[l->device] -= l->cap;
    *l = Lease();
  }
  // Gives up the buffers of a device that no call has at this moment; false: there are none.
  bool trim(int device) {
    std::lock_guard<std::mutex> g(mu_);
    bool any = false;
    while (drop_oldest(device)) any = true;
    return any;
  }

 private:
  static constexpr size_t kMost = (size_t)2 << 30;
  int take(int i, hipStream_t stream, Lease *out) {
    if (!(free_[(size_t)i].stream == StreamKey::of(stream))) DMM_HIP(hipStreamWaitEvent(stream, free_[(size_t)i].done, 0));
    *out = free_[(size_t)i];
    out_[out->device] += out->cap;
    free_.erase(free_.begin() + i);
    return DMM_OK;
  }
  static bool across_line(const char *p, size_t bytes) {
    return ((uintptr_t)p >> 32) != (((uintptr_t)p + bytes - 1) >> 32);
  }
  bool allocate(size_t bytes, int device, Lease *out) {
    Lease l;
    l.cap = bytes;
    l.device = device;
    if (hipEventCreateWithFlags(&l.done, hipEventDisableTiming) != hipSuccess || hipMalloc((void **)&l.p, bytes) != hipSuccess) {
      (void)hipGetLastError();
      if (l.done) (void)hipEventDestroy(l.done);
      return false;
    }
    // Not across a multiple of 2^32: the merged macro-tile kernel loads a K-segment that such a line runs
    // through step by step, and all of K is one segment on copies (4096 x 5888 x 6600: 1085 instead of 400 us).
    if (across_line(l.p, bytes)) {
      char *other = nullptr;
      if (hipMalloc((void **)&other, bytes) != hipSuccess) (void)hipGetLastError();
      else if (across_line(other, bytes)) (void)hipFree(other);
      else {
        (void)hipFree(l.p);
        l.p = other;
      }
    }
    *out = l;
    out_[device] += bytes;
    return true;
  }
  bool drop_oldest(int device) {
    for (size_t i = 0; i < free_.size(); ++i)
      if (free_[i].device == device) {
        const Lease l = free_[i];
        (void)hipEventSynchronize(l.done);
        (void)hipFree(l.p);
        (void)hipEventDestroy(l.done);
        free_.erase(free_.begin() + (long)i);
        return true;
      }
    return false;
  }
  size_t held(int device) const {
    size_t n = out_[device];
    for (const Lease &e : free_)
      if (e.device == device) n += e.cap;
    return n;
  }
  std::mutex mu_;
  std::vector<Lease> free_;            // in the order in which they came back
  size_t out_[64] = {};                // bytes that calls have
};

PackPool &pack_pool() {
  static PackPool *p = new PackPool;   // never destroyed, like the slab pool
  return *p;
}

// hipMalloc on the current device; where there is no room, buffers that only wait for another product on
// copies are given up for it.
hipError_t device_malloc(char **p, size_t bytes) {
  hipError_t e = hipMalloc((void **)p, bytes);
  int device = 0;
  if (e == hipErrorOutOfMemory && hipGetDevice(&device) == hipSuccess && pack_pool().trim(device)) {
    (void)hipGetLastError();
    e = hipMalloc((void **)p, bytes);
  }
  return e;
}

// One device buffer plus two pinned staging slots and their events.  Slabs are
// recycled through a process-wide pool (in the spirit of the memory pool of
// Section 4.2: allocate once, sub-allocate from the CPU side), so creating and
// destroying plans in a loop does not hit hipMalloc / hipHostMalloc each time.
struct Slab {
  int device = -1;       // the device its buffer and events belong to
  char *dev = nullptr;
  char *pinned[2] = {nullptr, nullptr};
  hipEvent_t ev[2] = {nullptr, nullptr};
  size_t cap = 0;
  // Host copy of what the device buffer holds (empty: unknown).  It stays with the slab through
  // the pool, so a new plan whose tables equal those of a destroyed one (plan + execute in a
  // loop over the same buffers) finds them already on the device and uploads nothing.
  std::vector<char> *mirror = nullptr;
};

class SlabPool {
 public:
  int acquire(size_t bytes, Slab *out) {
    int device = 0;
    DMM_HIP(hipGetDevice(&device));
    {
      std::lock_guard<std::mutex> g(mu_);
      int best = -1;
      for (size_t i = 0; i < free_.size(); ++i)
        if (free_[i].device == device && free_[i].cap >= bytes &&
            (best < 0 || free_[i].cap < free_[(size_t)best].cap))
          best = (int)i;
      if (best >= 0) {
        *out = free_[(size_t)best];
        free_.erase(free_.begin() + best);
        return DMM_OK;
      }
    }
    size_t want = 64 * 1024;
    while (want < bytes) want *= 2;
    Slab s;
    hipError_t e = device_malloc(&s.dev, want);
    for (int i = 0; i < 2 && e == hipSuccess; ++i) {
      e = hipHostMalloc((void **)&s.pinned[i], want, hipHostMallocDefault);
      if (e == hipSuccess) e = hipEventCreateWithFlags(&s.ev[i], hipEventDisableTiming);
    }
    if (e != hipSuccess) {
      destroy(&s);
      g_last_hip_error = (int)e;
      return e == hipErrorOutOfMemory ? DMM_ENOMEM : DMM_EHIP;
    }
    s.cap = want;
    s.device = device;
    s.mirror = new (std::nothrow) std::vector<char>;
    if (!s.mirror) {
      destroy(&s);
      return DMM_ENOMEM;
    }
    *out = s;
    return DMM_OK;
  }
  // The caller guarantees that no stream work still uses the slab.
  void release(Slab *s) {
    if (!s->dev) return;
    std::lock_guard<std::mutex> g(mu_);
    if (free_.size() < 16) free_.push_back(*s);
    else destroy(s);
    *s = Slab();
  }

 private:
  static void destroy(Slab *s) {
    delete s->mirror;
    if (s->dev) (void)hipFree(s->dev);
    for (int i = 0; i < 2; ++i) {
      if (s->pinned[i]) (void)hipHostFree(s->pinned[i]);
      if (s->ev[i]) (void)hipEventDestroy(s->ev[i]);
    }
    *s = Slab();
  }
  std::mutex mu_;
  std::vector<Slab> free_;
};

SlabPool &pool() {
  static SlabPool *p = new SlabPool;   // never destroyed: outlives the HIP runtime teardown order
  return *p;
}

// One stream per device for work-table uploads (default priority, created on first use and
// kept for the life of the process): a table copy then overlaps whatever the caller's stream
// is still running, instead of queueing behind it.
int copy_stream(hipStream_t *out) {
  static std::mutex mu;
  static hipStream_t streams[64] = {};
  int dev = 0;
  DMM_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64) return DMM_EINVAL;
  std::lock_guard<std::mutex> g(mu);
  if (!streams[dev]) DMM_HIP(hipStreamCreateWithFlags(&streams[dev], hipStreamNonBlocking));
  *out = streams[dev];
  return DMM_OK;
}

// A small table travels as the argument of a kernel that writes it: on the caller's own stream, one launch, where the
// copy takes the host a copy, two events and two waits (2048^3 in 2 x 2 tiles, a new plan and other buffers
// every time: 42 -> 34 us a call, 27 of host work -> 12).
constexpr size_t kTableWords = 448;
struct TableArg {
  uint64_t word[kTableWords];
};
__global__ __launch_bounds__(256) void table_kernel(TableArg, uint64_t *dst, int words) {
  // (read where the launch has put the argument; taken by its name it would go through private memory)
  const auto *src = (const __attribute__((address_space(4))) uint64_t *)__builtin_amdgcn_kernarg_segment_ptr();
  for (int i = threadIdx.x; i < words; i += 256) dst[i] = src[i];
}

// upload() copies host bytes to the slab's device buffer (on the copy stream, or with table_kernel) and makes the
// caller's stream wait for that copy; it skips the copy when those bytes are already resident.
// `readers` are the calls whose kernels may still read the device buffer: the copy waits for them.
struct Uploader {
  Slab slab;
  bool ev_used[2] = {false, false};
  int cur = 0;
  StreamKey copied_on;                   // where the copy behind ev[cur] was made

  char *dev() const { return slab.dev; }
  int upload(const void *src, size_t bytes, hipStream_t stream, const Uses &readers) {
    if (bytes == 0) return DMM_OK;
    if (bytes > slab.cap) {
      // growing: the old slab may still be read by enqueued work of this plan
      int rc;
      if (slab.dev) {
        if ((rc = readers.wait())) return rc;
        DMM_HIP(hipStreamSynchronize(stream));
        release();
      }
      if ((rc = pool().acquire(bytes, &slab))) return rc;
      ev_used[0] = ev_used[1] = false;
    }
    std::vector<char> &resident = *slab.mirror;
    if (resident.size() == bytes && std::memcmp(resident.data(), src, bytes) == 0) {
      // already resident; the caller's stream (possibly another one than last time) still has to
      // be ordered behind the copy that put it there, if this uploader made that copy (a copy made
      // for an earlier owner of the slab finished before the slab went back to the pool)
      return order_behind_copy(stream);
    }
    resident.clear();                      // unknown contents until the copy below has been enqueued
    if (bytes <= sizeof(TableArg) && bytes % 8 == 0 && stream != hipStreamPerThread && stream != hipStreamLegacy && !is_capturing(stream)) {
      // (behind the readers on other streams, and behind a copy that a call made and failed to use)
      int rc = readers.order(stream);
      if (rc || (rc = order_behind_copy(stream))) return rc;
      TableArg table;
      std::memcpy(table.word, src, bytes);
      if (launch_behind_only(slab.ev[cur ^ 1], table_kernel, 1, 256, 0, stream, table, (uint64_t *)slab.dev, (int)(bytes / 8))) {
        cur ^= 1;
        ev_used[cur] = true;
        copied_on = StreamKey::of(stream);
        resident.assign((const char *)src, (const char *)src + bytes);
        return DMM_OK;
      }
    }
    const int next = cur ^ 1;
    if (ev_used[next]) DMM_HIP(hipEventSynchronize(slab.ev[next]));  // slot last used two uploads ago
    std::memcpy(slab.pinned[next], src, bytes);
    hipStream_t cs = nullptr;
    int rc = copy_stream(&cs);
    if (rc) return rc;
    // (behind the readers, and behind a copy on a caller's stream whose call failed to use it: late, it would
    // write the old table over this one)
    if ((rc = readers.order(cs)) || (rc = order_behind_copy(cs))) return rc;
    DMM_HIP(hipMemcpyAsync(slab.dev, slab.pinned[next], bytes, hipMemcpyHostToDevice, cs));
    DMM_HIP(hipEventRecord(slab.ev[next], cs));
    cur = next;                            // (only now: a call that fails above leaves the last copy known)
    ev_used[cur] = true;
    copied_on = StreamKey::of(cs);
    DMM_HIP(hipStreamWaitEvent(stream, slab.ev[cur], 0));
    resident.assign((const char *)src, (const char *)src + bytes);
    return DMM_OK;
  }
  // Orders `stream` behind the copy that put the resident bytes in place (for a caller that knows
  // by other means that they are the bytes it wants).
  int order_behind_copy(hipStream_t stream) {
    if (slab.dev && ev_used[cur] && !(copied_on == StreamKey::of(stream))) DMM_HIP(hipStreamWaitEvent(stream, slab.ev[cur], 0));
    return DMM_OK;
  }
  // The caller guarantees that no stream work still uses the slab: in particular its last copy has
  // completed, so the mirror describes the buffer.
  void release() {
    // (a call that failed between the upload and its launches may have left the copy in flight)
    if (slab.dev && ev_used[cur]) (void)hipEventSynchronize(slab.ev[cur]);
    pool().release(&slab);
  }
};

// Device-only buffers for the partial sums of K-split items, recycled like the slabs.
class ScratchPool {
 public:
  int acquire(size_t bytes, char **out, size_t *cap) {
    int device = 0;
    DMM_HIP(hipGetDevice(&device));
    {
      std::lock_guard<std::mutex> g(mu_);
      int best = -1;
      for (size_t i = 0; i < free_.size(); ++i)
        if (free_[i].device == device && free_[i].cap >= bytes &&
            (best < 0 || free_[i].cap < free_[(size_t)best].cap))
          best = (int)i;
      if (best >= 0) {
        *out = free_[(size_t)best].p;
        *cap = free_[(size_t)best].cap;
        free_.erase(free_.begin() + best);
        return DMM_OK;
      }
    }
    size_t want = (size_t)4 << 20;
    while (want < bytes) want *= 2;
    char *p = nullptr;
    hipError_t e = device_malloc(&p, want);
    if (e != hipSuccess) {
      g_last_hip_error = (int)e;
      return e == hipErrorOutOfMemory ? DMM_ENOMEM : DMM_EHIP;
    }
    *out = p;
    *cap = want;
    return DMM_OK;
  }
  // The caller guarantees that no stream work still uses the buffer (and is on its device).
  void release(char **p, size_t *cap) {
    if (!*p) return;
    int device = 0;
    (void)hipGetDevice(&device);
    std::lock_guard<std::mutex> g(mu_);
    if (free_.size() < 8) free_.push_back({*p, *cap, device});
    else (void)hipFree(*p);
    *p = nullptr;
    *cap = 0;
  }

 private:
  struct Entry {
    char *p;
    size_t cap;
    int device;
  };
  std::mutex mu_;
  std::vector<Entry> free_;
};

ScratchPool &scratch_pool() {
  static ScratchPool *p = new ScratchPool;   // never destroyed, like the slab pool
  return *p;
}

// Where the replica sum's (or the broadcast's) tables sit in a device buffer.
struct RedLaunch {
  char *dev_base = nullptr;   // device address of the buffer the offsets below refer to
  size_t n_items = 0;
  size_t o_items = 0, o_tiles = 0, o_parts = 0, o_lds = 0;
  int nparts = 0;
  bool vec_ok = true;
};

// Where the merged macro-tiles' tables sit in the plan's device table.
struct MergedLaunch {
  size_t n_items = 0, o_a = 0, o_b = 0, o_c = 0, o_k = 0, o_fix = 0, n_fix = 0, total = 0;
};

// Where the tables of the kernels for small products sit in the plan's device table, and the rest of
// their arguments.
struct SmallLaunch {
  int shape = -1;               // SMALL_* (gemm_launch.hpp)
  size_t o_rows = 0, o_cols = 0, o_mc = 0, o_nc = 0, o_starts = 0, o_klen = 0, o_a = 0, o_b = 0, o_c = 0;
  int32_t segs = 0, nr = 0, tiles_m = 0, tiles_n = 0, runs = 1, per = 0, steps = 0, c_es = 4;
  int32_t batch = 0;            // tiles per launch: all of them where there is room for their partial sums
};

// What the launches of a dmm_execute need to know besides the device table itself.
struct ExecLayout {
  bool merged = false;
  MergedLaunch ml;                                                       // merged macro-tiles
  size_t n_items = 0, o_segs = 0, o_fix = 0, o_red = 0, n_first = 0, n_fix = 0;   // per-group macro-tiles
  bool fuse = false, one_launch = false;
  bool dense = false;           // the operands are copied first and DeviceState::dense runs the product
  SmallLaunch small;            // shape >= 0: these kernels run the product
  size_t n_runs = 0;
  bool uses_split = false;      // some macro-tiles store through the plan's scratch buffer
  RedLaunch red;                // the replica-sum launch behind the GEMM (n_items == 0: none)
};

struct DeviceState {
  // A product that runs on dense copies of its operands: the plan it runs as, whose `uses` stand for these
  // calls, where the copies are, and the tables of the kernel that makes them.
  dmm_plan_t *dense = nullptr;
  PackPool::Lease pack;                // the copies' buffer, during a call
  bool pack_kept = false;              // ... for as long as the plan lives: a captured graph refers to it
  const char *pack_at = nullptr;       // where the tables say that the copies are
  size_t pack_need = 0;
  Uploader pack_table;
  int pack_jobs = 0, pack_blocks = 0;
  size_t pack_o_tiles = 0, pack_o_runs = 0;
  char *pack_b = nullptr;              // the copy of B
  std::vector<const void *> pack_a;    // the copy of A, one tile per replica of C
  std::vector<int64_t> pack_lda;
  int64_t pack_ldb = 0;
  bool pack_launched = false;          // the copy of this call is under way
  bool ran_dense = false;              // the last dmm_execute did so
  int ran_small = -1, small_runs = 0;  // ... ran the kernels for small products: their shape, its tiles in so many ranges of K
  hipEvent_t t_pack[2] = {nullptr, nullptr};
  char *split_buf = nullptr;   // partial sums of K-split items
  size_t split_cap = 0;
  Uploader gemm_table;   // [ItemDev x items][SegDev x segments]
  Uploader red_table;    // [RedItem][RedTile][part pointers][part lds]
  std::vector<char> host;  // scratch for table assembly
  Uses uses;                          // marked after the last launch of every call
  hipEvent_t t_gemm[2] = {nullptr, nullptr}, t_red[2] = {nullptr, nullptr};  // DMM_TIMING
  hipEvent_t t_mid = nullptr;         // ... between the two GEMM launches of a fused replica sum
  bool gemm_timed = false, red_timed = false, mid_timed = false;
  double launch_flops[2] = {0.0, 0.0};  // 2 m n k of the ops behind each of those two launches
  bool ran_merged = false;            // the last dmm_execute ran the merged macro-tiles
  bool ran_k_split = false;           // ... and cut macro-tiles along K
  int ran_fused = 0;                  // ... and fused the replica sum into the GEMM: in 1 launch, in 2; 0 = not
  // The inputs of the last successful dmm_execute (element type, flags, device, the six pointer
  // and leading-dimension arrays) and the layout of the device table it left in gemm_table: a call
  // with the same inputs launches from that table as it stands.
  std::vector<char> exec_key, key_scratch;
  ExecLayout exec_layout;
  bool exec_cached = false;
  bool table_reused = false;          // the last dmm_execute did
};

void destroy_device_state(DeviceState *d) {
  if (!d) return;
  // wait for this plan's own work only, then hand the buffers back to the pool
  (void)d->uses.wait();
  if (d->dense) dmm_plan_destroy(d->dense);
  d->pack_table.release();
  pack_pool().put(&d->pack);
  for (int i = 0; i < 2; ++i)
    if (d->t_pack[i]) (void)hipEventDestroy(d->t_pack[i]);
  d->gemm_table.release();
  d->red_table.release();
  scratch_pool().release(&d->split_buf, &d->split_cap);
  d->uses.destroy();
  for (int i = 0; i < 2; ++i) {
    if (d->t_gemm[i]) (void)hipEventDestroy(d->t_gemm[i]);
    if (d->t_red[i]) (void)hipEventDestroy(d->t_red[i]);
  }
  if (d->t_mid) (void)hipEventDestroy(d->t_mid);
  delete d;
}

}  // namespace dmm
