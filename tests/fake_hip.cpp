// A HIP runtime that runs nothing and writes down what it is asked, for tests
// of the library's host code without a GPU: loaded with RTLD_GLOBAL before
// libflb.so, whose calls then come here.  "Device" memory is untouched host
// memory, kernels are log lines, and work is finished by waiting for it.
//
// Log, one line each: K <stream> <kernel> <grid> (a launch), C ... (the same, into a
// captured graph), G <stream> <branches> (a replay), M <bytes> (an allocation), S <stream>
// <steps> (a wait for a stream with that many step launches pending), P <stream>
// (an event asked for while step launches recorded before it are pending).
#include <hip/hip_runtime.h>

#include <sys/mman.h>

#include <cstring>
#include <map>
#include <mutex>
#include <set>
#include <string>

namespace {
struct Stream {
  int id, device, steps = 0;
  bool capturing = false;
};
struct Event {
  int device;
  Stream* on = nullptr;
  bool steps = false, captured = false;
};
std::recursive_mutex mu;
std::string text;
std::map<const void*, std::string> names;
std::map<void*, size_t> blocks;
std::map<Stream*, bool> streams;
size_t total = (size_t)288 << 30, used = 0;
int next_id = 1, fail_in = 0;
std::string fail_name;
hipError_t last = hipSuccess;
thread_local int current = 0;
Stream null_stream{0, 0};
std::set<Stream*> captured;  // streams with launches in the current capture
struct Graph {
  size_t branches;
};

Stream* of(hipStream_t s) { return s ? (Stream*)s : &null_stream; }
void put(const std::string& s) { text += s + "\n"; }
using Lock = std::lock_guard<std::recursive_mutex>;
hipError_t error(hipError_t e) { return last = e; }
void* map(size_t n) {
  void* p = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE,
                 -1, 0);
  return p == MAP_FAILED ? nullptr : p;
}
}  // namespace

extern "C" {
const char* fake_log() { return text.c_str(); }
void fake_clear() { text.clear(); }
void fake_memory(size_t bytes) { total = bytes; }
// The n-th launch from now on of a kernel whose name holds `name` fails.
void fake_fail(const char* name, int n) {
  fail_name = name;
  fail_in = n;
}

struct Config {
  dim3 grid, block;
  size_t lds;
  hipStream_t st;
};
static thread_local Config config;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t st) {
  config = Config{g, b, lds, st};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* st) {
  *g = config.grid, *b = config.block, *lds = config.lds, *st = config.st;
  return hipSuccess;
}
void** __hipRegisterFatBinary(const void*) {
  static void* h;
  return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*,
                           void*, void*, int*) {
  names[f] = name;
}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}

hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void**, size_t lds, hipStream_t st) {
  Lock lk(mu);
  Stream* s = of(st);
  const std::string& n = names[f];
  if (g.x * (size_t)g.y * g.z == 0 || b.x * b.y * b.z > 1024 || lds > 163840)
    return error(hipErrorInvalidConfiguration);
  if (fail_in > 0 && n.find(fail_name) != std::string::npos && --fail_in == 0)
    return error(hipErrorLaunchFailure);
  put((s->capturing ? "C " : "K ") + std::to_string(s->id) + " " + n + " " +
      std::to_string(g.x));
  if (s->capturing) captured.insert(s);
  if (!s->capturing && n.find("step") != std::string::npos) ++s->steps;
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void**, const void*) { return error(hipErrorInvalidSymbol); }
const char* hipGetErrorString(hipError_t) { return "fake"; }
hipError_t hipGetLastError() {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}

hipError_t hipGetDevice(int* d) { return *d = current, hipSuccess; }
hipError_t hipSetDevice(int d) { return current = d, hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 163840;
  return hipSuccess;
}

hipError_t hipMalloc(void** p, size_t n) {
  Lock lk(mu);
  if (used + n > total || !(*p = map(n))) return error(hipErrorOutOfMemory);
  blocks[*p] = n;
  used += n;
  put("M " + std::to_string(n));
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  Lock lk(mu);
  used -= blocks[p];
  munmap(p, blocks[p]);
  blocks.erase(p);
  return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* f, size_t* t) {
  Lock lk(mu);
  return *f = total - used, *t = total, hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  return (*p = map(n)) ? hipSuccess : error(hipErrorOutOfMemory);
}
hipError_t hipHostFree(void*) { return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  return memcpy(d, s, n), hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  return memcpy(d, s, n), hipSuccess;
}
hipError_t hipMemset(void* p, int v, size_t n) { return memset(p, v, n), hipSuccess; }
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t) {
  return memset(p, v, n), hipSuccess;
}

hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  Lock lk(mu);
  Stream* n = new Stream{next_id++, current};
  streams[n] = true;
  return *s = (hipStream_t)n, hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  Lock lk(mu);
  streams.erase((Stream*)s);
  delete (Stream*)s;
  return hipSuccess;
}
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t* d) {
  return *d = of(s)->device, hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
  Lock lk(mu);
  put("S " + std::to_string(of(s)->id) + " " + std::to_string(of(s)->steps));
  of(s)->steps = 0;
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  Lock lk(mu);
  if (((Event*)e)->captured) of(s)->capturing = true;
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
  captured.clear();
  return of(s)->capturing = true, hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  Lock lk(mu);
  for (auto& s : streams) s.first->capturing = false;
  return *g = (hipGraph_t) new Graph{captured.size()}, hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t g, hipGraphNode_t*, char*, size_t) {
  return *x = (hipGraphExec_t) new Graph(*(Graph*)g), hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t s) {
  Lock lk(mu);
  put("G " + std::to_string(of(s)->id) + " " + std::to_string(((Graph*)x)->branches));
  ++of(s)->steps;
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { return delete (Graph*)g, hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t x) { return delete (Graph*)x, hipSuccess; }

hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  return *e = (hipEvent_t) new Event{current}, hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { return delete (Event*)e, hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  Lock lk(mu);
  Event* v = (Event*)e;
  if (v->device != of(s)->device) return error(hipErrorInvalidHandle);
  v->on = of(s);
  v->steps = of(s)->steps > 0;
  v->captured = of(s)->capturing;
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
  Lock lk(mu);
  Event* v = (Event*)e;
  if (!v->steps || v->on->steps == 0) return hipSuccess;
  put("P " + std::to_string(v->on->id));
  v->on->steps = 0;
  return hipErrorNotReady;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  if (((Event*)e)->on) ((Event*)e)->on->steps = 0;
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = 1.f, hipSuccess; }
}
