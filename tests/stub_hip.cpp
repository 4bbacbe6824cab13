// A HIP runtime without a device for tests of the library's host code: every
// call the library makes is answered, written to a log and, on request, made
// to fail.  Preloaded in front of the real runtime; kernels do not run.
#include <hip/hip_runtime_api.h>

#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>

namespace {
std::mutex mu;
std::string text, fail_name;
int fail_at = 0;
uintptr_t next_handle = 0x1000;
struct Symbol { std::string name; int module; };
std::map<const void*, Symbol>& symbols() {  // kernels and device variables
  static std::map<const void*, Symbol> k;
  return k;
}
// code objects: bytes of static device memory, and whether anything of it was used (loaded)
struct Module { size_t bytes; bool used; } modules[256];
void* handles[256];
int nmodules = 0;
int module_of(void** m) { return (int)(m - handles); }
const char* use(const void* f) {
  Symbol& s = symbols()[f];
  modules[s.module].used = true;
  return s.name.c_str();
}

hipError_t note(const char* name, const char* fmt = "", ...) {
  std::lock_guard<std::mutex> lk(mu);
  char line[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(line, sizeof line, fmt, ap);
  va_end(ap);
  const bool fails = fail_name == name && --fail_at == 0;
  text += std::string(name) + " " + line + (fails ? " FAILS\n" : "\n");
  return fails ? hipErrorUnknown : hipSuccess;
}
thread_local struct { dim3 g, b; size_t s; hipStream_t st; } config;

template <class T>
void handle(T* out) { *out = (T)(next_handle += 0x10); }
}  // namespace

extern "C" {
const char* stub_log() { return text.c_str(); }
void stub_clear() { text.clear(); }
// the nth call of `name` from now on fails
void stub_fail(const char* name, int nth) { fail_name = name; fail_at = nth; }

// static device memory of the code objects used so far
size_t stub_loaded_bytes() {
  size_t n = 0;
  for (int i = 0; i < nmodules; ++i) n += modules[i].used ? modules[i].bytes : 0;
  return n;
}

void** __hipRegisterFatBinary(const void*) { return &handles[nmodules++]; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void** m, void* v, char*, char* name, int, size_t bytes, int, int) {
  symbols()[v] = {name, module_of(m)};
  modules[module_of(m)].bytes += bytes;
}
void __hipRegisterFunction(void** m, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*,
                           int*) {
  symbols()[f] = {name, module_of(m)};
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t st) {
  config = {g, b, s, st};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, hipStream_t* st) {
  *g = config.g; *b = config.b; *s = config.s; *st = config.st;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3, void**, size_t, hipStream_t s) {
  return note("kernel", "%s %u %p", use(f), g.x, (void*)s);
}
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return note("device_sync"); }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  memset(p, 0, sizeof *p);
  strcpy(p->gcnArchName, "stub");
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipFuncGetAttributes(hipFuncAttributes* a, const void* f) { use(f); memset(a, 0, sizeof *a); return hipSuccess; }
hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute, int) { use(f); return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 8; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* v) { use(v); handle(p); return hipSuccess; }
hipError_t hipMemcpyToSymbolAsync(const void* v, const void*, size_t, size_t, hipMemcpyKind, hipStream_t) {
  use(v);
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { handle(e); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { handle(e); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t s) { return note("event_record", "%p", (void*)s); }
hipError_t hipEventSynchronize(hipEvent_t) { return note("event_sync"); }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { handle(s); return note("stream_create", "%p", (void*)*s); }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { return note("stream_sync", "%p", (void*)s); }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return note("capture"); }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { handle(g); return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* g, hipGraph_t, hipGraphNode_t*, char*, size_t) { handle(g); return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return note("graph_destroy"); }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t s) { return note("graph_launch", "%p", (void*)s); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(n, 1); return note("host_malloc", "%p %zu", *p, n); }
hipError_t hipHostFree(void* p) { free(p); return note("host_free", "%p", p); }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void*, size_t n, hipMemcpyKind k, hipStream_t s) {
  return note(k == hipMemcpyDeviceToHost ? "download" : k == hipMemcpyHostToDevice ? "upload" : "copy", "%p %zu %p", d, n, (void*)s);
}
}
