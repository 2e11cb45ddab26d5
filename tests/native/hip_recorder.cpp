// A stand-in for the HIP runtime that runs no kernel: loaded in front of the library under test it
// keeps a record of what the library enqueues where, and answers which of two operations is ordered
// behind the other (stream order, events, host synchronisation).  Device memory is host memory
// that is never read by anything but copies; its amount can be limited.  Test infrastructure: no GPU.
#include <hip/hip_runtime_api.h>

#include <cxxabi.h>
#include <sys/mman.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {

struct Op {
  std::string name;             // kernel, "copy", "event"
  void *stream;
  uint64_t arg, bytes;          // kernel: first eight bytes of its first argument; copy: destination and size
  uint64_t more[3] = {0, 0, 0}; // pack_kernel: its other arguments; copy: 1 if table_kernel makes it
  unsigned blocks = 0;
  std::vector<int> behind;
  int done_at = -1;             // known on the host to have finished before operation number done_at was enqueued
};
struct Stream {
  int last = -1;
  std::vector<int> waits;
  bool capturing = false;
  int since = 0;                // operations in front of the capture
};

std::vector<Op> ops;
std::map<void *, Stream> streams;
std::map<void *, int> events;                       // the record it stands for, -1: none yet
std::map<const void *, std::string> kernels;
std::map<const void *, void *> symbols;
std::map<void *, size_t> memory;
size_t live = 0, limit = ~(size_t)0;
int wait_in = -1;                                   // waits for an event until one reports an error and does not wait
bool launches_fail = false;                         // of all kernels but table_kernel
int fail_in = -1, fail_n = 0;                       // allocations until some fail, and how many do
uint64_t next_at = 0;                               // where the next large allocation goes
hipError_t last_error = hipSuccess;
dim3 cfg_grid, cfg_block;
size_t cfg_lds;
hipStream_t cfg_stream;

hipError_t fail(hipError_t e) { return last_error = e; }

void *fresh() {
  static char *next = (char *)0x1000;
  return next += 16;
}

hipStream_t real(hipStream_t s) {                   // hipStreamPerThread: a stream of the calling thread's own
  static thread_local hipStream_t mine = nullptr;
  if (s == hipStreamLegacy) return nullptr;
  if (s != hipStreamPerThread) return s;
  if (!mine) mine = (hipStream_t)fresh();
  return mine;
}

int enqueue(const std::string &name, void *stream, uint64_t arg, uint64_t bytes) {
  Stream &s = streams[stream];
  Op o;
  o.name = name;
  o.stream = stream;
  o.arg = arg;
  o.bytes = bytes;
  if (s.last >= 0) o.behind.push_back(s.last);
  o.behind.insert(o.behind.end(), s.waits.begin(), s.waits.end());
  s.waits.clear();
  ops.push_back(o);
  return s.last = (int)ops.size() - 1;
}

void finish(int i) {                                // the host has waited for operation i
  if (i < 0 || ops[(size_t)i].done_at >= 0) return;
  ops[(size_t)i].done_at = (int)ops.size();
  for (int b : ops[(size_t)i].behind) finish(b);
}

void finish_all() {
  for (size_t i = 0; i < ops.size(); ++i) finish((int)i);
}

bool before(int a, int b) {                         // a has finished when b starts, whatever the device does
  std::vector<int> todo = {b};
  std::vector<char> seen((size_t)std::max(a, b) + 1, 0);
  while (!todo.empty()) {
    const int x = todo.back();
    todo.pop_back();
    if (x == a || (ops[(size_t)a].done_at >= 0 && ops[(size_t)a].done_at <= x)) return true;
    for (int y : ops[(size_t)x].behind)             // (what an operation is behind has been enqueued earlier)
      if (!seen[(size_t)y] && y >= a) {
        seen[(size_t)y] = 1;
        todo.push_back(y);
      }
  }
  return false;
}

}  // namespace

extern "C" {

// ---- for the test -----------------------------------------------------------------------------------
int rec_count() { return (int)ops.size(); }
const char *rec_name(int i) { return ops[(size_t)i].name.c_str(); }
uint64_t rec_stream(int i) { return (uint64_t)ops[(size_t)i].stream; }
uint64_t rec_arg(int i) { return ops[(size_t)i].arg; }
uint64_t rec_bytes(int i) { return ops[(size_t)i].bytes; }
uint64_t rec_more(int i, int k) { return ops[(size_t)i].more[k]; }
unsigned rec_blocks(int i) { return ops[(size_t)i].blocks; }
int rec_before(int a, int b) { return before(a, b); }
uint64_t rec_new_stream() { return (uint64_t)fresh(); }
void rec_finish_stream(uint64_t s) { finish(streams[(void *)s].last); }
void rec_set_capturing(uint64_t s, int on) {
  streams[(void *)s].capturing = on != 0;
  streams[(void *)s].since = (int)ops.size();
}
void rec_set_limit(uint64_t bytes) { limit = bytes; }
void rec_next_at(uint64_t p) { next_at = p; }
uint64_t rec_live() { return live; }
void rec_fail_allocations(int in, int n) {
  fail_in = in;
  fail_n = n;
}
void rec_fail_wait(int in) { wait_in = in; }
void rec_fail_launches(int on) { launches_fail = on != 0; }
int rec_failed() { return fail_in < 0; }

// ---- the runtime ------------------------------------------------------------------------------------
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *device, unsigned, void *, void *, dim3 *, dim3 *, int *) {
  int status = 0;
  char *s = abi::__cxa_demangle(device, nullptr, nullptr, &status);
  std::string n = status == 0 ? s : device;
  free(s);
  n = n.substr(0, n.find('('));
  n = n.substr(0, n.find('<'));
  const size_t at = n.rfind("dmm::");
  kernels[host] = at == std::string::npos ? n : n.substr(at + 5);
}
void __hipRegisterVar(void **, void *var, char *, char *, int, size_t size, int, int) { symbols[var] = calloc(1, size); }
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
  cfg_grid = grid;
  cfg_block = block;
  cfg_lds = lds;
  cfg_stream = stream;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *stream) {
  *grid = cfg_grid;
  *block = cfg_block;
  *lds = cfg_lds;
  *stream = cfg_stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3, void **args, size_t, hipStream_t stream) {
  stream = real(stream);
  if (kernels[f] == "table_kernel") {               // (table, where to, words): a copy on the caller's stream
    void *to = *(void **)args[1];
    const size_t bytes = 8 * (size_t)*(int *)args[2];
    memcpy(to, args[0], bytes);
    ops[(size_t)enqueue("copy", stream, (uint64_t)to, bytes)].more[0] = 1;
    return hipSuccess;
  }
  if (launches_fail) return fail(hipErrorLaunchFailure);
  uint64_t first;
  memcpy(&first, args[0], sizeof first);
  Op &o = ops[(size_t)enqueue(kernels[f], stream, first, 0)];
  o.blocks = grid.x;
  if (o.name == "pack_kernel") {                    // (jobs, number of them, runs, tiles)
    o.more[0] = *(int *)args[1];
    memcpy(&o.more[1], args[2], 8);
    memcpy(&o.more[2], args[3], 8);
  }
  return hipSuccess;
}
// (the event is recorded by the launch; in a capture the runtime refuses)
hipError_t hipExtLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t stream, hipEvent_t before, hipEvent_t behind, int) {
  if (stream == hipStreamPerThread || stream == hipStreamLegacy) abort();   // (not documented for these)
  if (before || streams[real(stream)].capturing) return fail(hipErrorStreamCaptureUnsupported);
  const hipError_t e = hipLaunchKernel(f, grid, block, args, lds, stream);
  if (behind && e == hipSuccess) events[behind] = streams[real(stream)].last;
  return e;
}
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
  memset(p, 0, sizeof *p);
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetLastError() {
  hipError_t e = last_error;
  last_error = hipSuccess;
  return e;
}
hipError_t hipPeekAtLastError() { return last_error; }
hipError_t hipGetSymbolAddress(void **p, const void *s) { *p = symbols[s]; return hipSuccess; }

hipError_t hipMalloc(void **p, size_t n) {
  if (fail_in <= 0 && fail_n > 0) {
    fail_in = -1;
    --fail_n;
    return fail(hipErrorOutOfMemory);
  }
  if (fail_in > 0) --fail_in;
  if (live + n > limit) return fail(hipErrorOutOfMemory);
  void *at = n >= (size_t)32 << 20 ? (void *)next_at : nullptr;
  if (at) next_at = 0;
  void *m = mmap(at, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE | (at ? MAP_FIXED_NOREPLACE : 0), -1, 0);
  if (m == MAP_FAILED) return fail(hipErrorOutOfMemory);
  // (not across a multiple of 2^32 unless the test wants it there: where the system puts it changes from run to run)
  const uint64_t line = (((uint64_t)m >> 32) + 1) << 32;
  for (uint64_t up = 0; !at && n < (size_t)1 << 32 && (uint64_t)m + n > line && up < 16; ++up) {
    void *other = mmap((void *)(line - ((up + 1) << 32)), n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE | MAP_FIXED_NOREPLACE, -1, 0);
    if (other == MAP_FAILED) continue;
    munmap(m, n);
    m = other;
    break;
  }
  memory[*p = m] = n;
  live += n;
  return hipSuccess;
}
hipError_t hipFree(void *p) {
  finish_all();                                     // (it waits for the device)
  auto it = memory.find(p);
  if (it == memory.end()) return fail(hipErrorInvalidValue);
  munmap(p, it->second);
  live -= it->second;
  memory.erase(it);
  return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = malloc(n); return *p ? hipSuccess : fail(hipErrorOutOfMemory); }
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
  finish_all();
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t stream) {
  memcpy(d, s, n);
  enqueue("copy", real(stream), (uint64_t)d, n);
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)fresh(); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
  Stream &t = streams[real(s)];
  finish(t.last);
  for (int w : t.waits) finish(w);
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *status) {
  *status = streams[real(s)].capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
  *e = (hipEvent_t)fresh();
  events[*e] = -1;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { events.erase(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  events[e] = enqueue("event", real(s), (uint64_t)e, 0);
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  if (wait_in >= 0 && wait_in-- == 0) return fail(hipErrorUnknown);
  finish(events[e]);
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
  const int i = events[e];
  return i < 0 || ops[(size_t)i].done_at >= 0 ? hipSuccess : hipErrorNotReady;   // (not an error to be read back later)
}
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0.125f; return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  const int i = events[e];
  s = real(s);
  if (i >= 0 && streams[s].capturing && ops[(size_t)i].stream == s && i < streams[s].since) return fail(hipErrorStreamCaptureIsolation);
  if (i >= 0) streams[s].waits.push_back(i);
  return hipSuccess;
}

}  // extern "C"
