// A stand-in for the HIP runtime calls that the one-shot entry points make:
// "device" memory is host memory, copies are made at once, kernels do
// nothing, and streams, events and captures are counters that a test sets
// and reads.  Loaded before libtt.so, so that its symbols are found first.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <vector>

namespace {
struct Event {
  hipStream_t stream = nullptr;
  int device = 0;
  bool ready = true;
};
struct Node {  // of the captured graph, in order
  void* dst = nullptr;
  const void* src = nullptr;
  size_t bytes = 0;
  hipHostFn_t fn = nullptr;
  void* arg = nullptr;
};
struct UserObject {
  void* ptr;
  hipHostFn_t destroy;
};
std::set<hipStream_t> blocked;      // streams whose work does not end
std::vector<Event*> events;
std::map<hipStream_t, int> device_of;
hipStream_t capturing = nullptr;
bool invalidated = false;           // a call that is not allowed was made while a stream captured
thread_local hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;
std::vector<Node> graph;
std::vector<UserObject*> retained;
int waits = 0, launches = 0, host_allocs = 0, host_frees = 0;
std::vector<const void*> sources;   // of the copies and launches that took host memory, in order
int fail_record = 0;

// calls on events and memory invalidate a capture of any stream, unless the
// thread has said that they are no part of it
hipError_t unsafe() {
  if (capturing && mode != hipStreamCaptureModeRelaxed) {
    invalidated = true;
    return hipErrorStreamCaptureUnsupported;
  }
  return hipSuccess;
}
}  // namespace

extern "C" {
// ------------------------------------------------------- what a test drives
void fake_block(void* s) { blocked.insert((hipStream_t)s); }
void fake_unblock(void* s) {
  blocked.erase((hipStream_t)s);
  for (Event* e : events)
    if (e->stream == (hipStream_t)s) e->ready = true;
}
void fake_stream_device(void* s, int device) { device_of[(hipStream_t)s] = device; }
void fake_capture(void* s) { capturing = (hipStream_t)s; }
int fake_invalidated() { return invalidated; }
int fake_waits() { return waits; }
int fake_launches() { return launches; }
int fake_host_allocs() { return host_allocs; }
int fake_host_frees() { return host_frees; }
int fake_sources() { return (int)sources.size(); }
const void* fake_source(int k) { return sources[k]; }
void fake_fail_record(int n) { fail_record = n; }
int fake_graph_host_functions() {
  int n = 0;
  for (const Node& x : graph) n += x.fn != nullptr;
  return n;
}
int fake_retained() { return (int)retained.size(); }
// one replay; returns the sum of the bytes copied
long fake_replay() {
  long sum = 0;
  for (const Node& x : graph) {
    if (x.fn) x.fn(x.arg);
    for (size_t k = 0; k < x.bytes; ++k) sum += ((uint8_t*)x.dst)[k] = ((const uint8_t*)x.src)[k];
  }
  return sum;
}
void fake_destroy_graph() {
  for (UserObject* o : retained) {
    o->destroy(o->ptr);
    delete o;
  }
  retained.clear();
  graph.clear();
}

// ------------------------------------------------------------- the runtime
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {  // (a macro: the current revision's name)
  std::memset(p, 0, sizeof(*p));
  std::strcpy(p->gcnArchName, "gfx950");
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t* d) {
  *d = device_of.count(s) ? device_of[s] : 0;
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipPeekAtLastError() { return hipSuccess; }

hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
  *st = capturing && s == capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamGetCaptureInfo_v2(hipStream_t s, hipStreamCaptureStatus* st, unsigned long long* id, hipGraph_t* g,
                                      const hipGraphNode_t** deps, size_t* n) {
  (void)hipStreamIsCapturing(s, st);
  if (id) *id = 1;
  if (g) *g = *st == hipStreamCaptureStatusActive ? (hipGraph_t)&graph : nullptr;
  if (deps) *deps = nullptr;
  if (n) *n = 0;
  return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) {
  std::swap(*m, mode);
  return hipSuccess;
}
hipError_t hipUserObjectCreate(hipUserObject_t* o, void* ptr, hipHostFn_t destroy, unsigned, unsigned) {
  *o = (hipUserObject_t) new UserObject{ptr, destroy};
  return hipSuccess;
}
hipError_t hipUserObjectRelease(hipUserObject_t o, unsigned) {
  auto* u = (UserObject*)o;
  u->destroy(u->ptr);
  delete u;
  return hipSuccess;
}
hipError_t hipGraphRetainUserObject(hipGraph_t, hipUserObject_t o, unsigned, unsigned) {
  retained.push_back((UserObject*)o);
  return hipSuccess;
}

hipError_t hipMallocAsync(void** p, size_t n, hipStream_t) {
  *p = std::malloc(n);
  return hipSuccess;
}
hipError_t hipFreeAsync(void*, hipStream_t) { return hipSuccess; }  // (kept: replays write it)
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static void* array = std::malloc(32u << 20);
  *p = array;
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  if (unsafe() != hipSuccess) return hipErrorStreamCaptureUnsupported;
  ++host_allocs;
  *p = std::malloc(n);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {  // waits for the whole device
  if (unsafe() != hipSuccess) return hipErrorStreamCaptureUnsupported;
  ++host_frees;
  waits += !blocked.empty();
  std::free(p);
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  events.push_back(new Event());
  *e = (hipEvent_t)events.back();
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
  if (unsafe() != hipSuccess) return hipErrorStreamCaptureUnsupported;
  return ((Event*)e)->ready ? hipSuccess : hipErrorNotReady;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  auto* x = (Event*)e;
  if (fail_record > 0 && fail_record--) return hipErrorUnknown;
  if (x->device != (device_of.count(s) ? device_of[s] : 0)) return hipErrorInvalidHandle;
  x->stream = s;
  x->ready = !blocked.count(s);
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  if (unsafe() != hipSuccess) return hipErrorStreamCaptureUnsupported;
  if (((Event*)e)->ready) return hipSuccess;
  ++waits;  // for good
  return hipErrorUnknown;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
  if (!blocked.count(s)) return hipSuccess;
  ++waits;
  return hipErrorUnknown;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t s) {
  sources.push_back(src);
  if (capturing && s == capturing)
    graph.push_back(Node{dst, src, n, nullptr, nullptr});
  else
    std::memcpy(dst, src, n);
  return hipSuccess;
}
hipError_t hipLaunchHostFunc(hipStream_t s, hipHostFn_t fn, void* arg) {
  if (capturing && s == capturing)
    graph.push_back(Node{nullptr, nullptr, 0, fn, arg});
  else if (!blocked.count(s))
    fn(arg);
  return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s) {
  *g = *b = dim3{1, 1, 1};
  *lds = 0;
  *s = nullptr;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) {
  ++launches;
  return hipSuccess;
}
}
