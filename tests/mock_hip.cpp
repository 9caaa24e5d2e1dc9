// A HIP runtime without a device, for the host code of the library alone
// (test_device_memory_cpu.py): it counts the work that calls queue on each
// stream and what of it the host has waited for, and allocations.  Kernel
// launches are generated stubs that end in mock_launch.
#include <cstdint>
#include <cstring>
#include <map>

typedef int hipError_t;
typedef void* hipStream_t;
typedef void* hipEvent_t;

namespace {
struct Event {
  hipStream_t stream = nullptr;
  long seq = 0;
};
std::map<hipStream_t, long> queued, waited;  // launches on a stream; of these, finished for the host
std::map<hipStream_t, bool> recording;
std::map<void*, size_t> live;
long graph_work = 0;  // launches recorded into a graph, which may replay until the device is waited for
long fail_in = -1, mallocs = 0, frees = 0;
uintptr_t next_address = uintptr_t(1) << 40;
size_t capacity = ~size_t(0);

void finish(hipStream_t s, long seq) {
  if (waited[s] < seq) waited[s] = seq;
}
void finish_all() {
  for (auto& q : queued) finish(q.first, q.second);
  graph_work = 0;
}
size_t used() {
  size_t n = 0;
  for (auto& l : live) n += l.second;
  return n;
}
hipError_t queue(hipStream_t s) {
  if (fail_in >= 0 && fail_in-- == 0) return 719;  // hipErrorLaunchFailure
  if (recording[s]) ++graph_work;
  else ++queued[s];
  return 0;
}
}  // namespace

extern "C" {
hipError_t mock_launch(hipStream_t s) { return queue(s); }
// for the test: fail the n-th launch from now; work on s the host has not waited for; and so on
void mock_fail_in(long n) { fail_in = n; }
long mock_pending(hipStream_t s) { return queued[s] - waited[s]; }
long mock_graph_work() { return graph_work; }
void mock_record(hipStream_t s, int on) { recording[s] = on != 0; }
long mock_mallocs() { return mallocs; }
long mock_frees() { return frees; }
size_t mock_used() { return used(); }
void mock_capacity(size_t n) { capacity = n; }

hipError_t hipGetDevice(int* d) { *d = 0; return 0; }
hipError_t hipSetDevice(int) { return 0; }
hipError_t hipGetLastError() { return 0; }
const char* hipGetErrorString(hipError_t) { return "mock"; }
hipError_t hipMalloc(void** p, size_t n) {
  for (auto& r : recording)
    if (r.second) return 900;  // hipErrorStreamCaptureUnsupported
  if (used() + n > capacity) return 2;
  *p = reinterpret_cast<void*>(next_address);
  next_address += (n + 4095) / 4096 * 4096;
  live[*p] = n;
  ++mallocs;
  return 0;
}
hipError_t hipFree(void* p) {
  if (!live.erase(p)) return 1;
  ++frees;
  finish_all();
  return 0;
}
hipError_t hipMemcpyAsync(void* d, const void*, size_t n, int kind, hipStream_t s) {
  if (kind == 2 && !recording[s]) memset(d, 0xff, n);  // to the host: "no zero pivot"
  return queue(s);
}
hipError_t hipMemcpy2DAsync(void*, size_t, const void*, size_t, size_t, size_t, int, hipStream_t s) { return queue(s); }
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t s) { return queue(s); }
hipError_t hipStreamSynchronize(hipStream_t s) {
  if (recording[s]) return 900;
  finish(s, queued[s]);
  return 0;
}
hipError_t hipDeviceSynchronize() { finish_all(); return 0; }
hipError_t hipStreamIsCapturing(hipStream_t s, int* st) { *st = recording[s]; return 0; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = new Event(); return 0; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { delete static_cast<Event*>(e); return 0; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0; return 0; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  *static_cast<Event*>(e) = Event{s, recording[s] ? 0 : queued[s]};
  return 0;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  finish(static_cast<Event*>(e)->stream, static_cast<Event*>(e)->seq);
  return 0;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return 0; }
}

namespace hodlr {
size_t scratch_capacity() { return size_t(64) << 20; }
hipError_t scratch_device_ptr(void** p) { *p = reinterpret_cast<void*>(4096); return 0; }
int aca_tile_elems() { return 1024; }
int aca_block_class(int, int, int) { return 3; }
int aca_own_launches(const int64_t (&)[4], const int64_t (&)[4], const int64_t (&)[4]) { return 0; }
}  // namespace hodlr
