// Stand-in for the HIP runtime, for tests of the library's host side on the
// CPU (tests/test_host_calls.py): device memory is host memory,
// kernels do not run, one gfx950 device of 256 CUs, and every call of
// interest is a line of the log. mock_fail_malloc(n, k): from now on the k
// next allocations of at least n bytes fail.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>

namespace {
std::string g_log, g_out;
std::map<const void*, std::string> g_kernel;
std::set<const void*> g_live;      // streams
size_t g_fail_bytes = 0;
int g_fail_count = 0;
uintptr_t g_next = 0x1000;
dim3 g_grid, g_block;
size_t g_shared = 0;
hipStream_t g_stream = nullptr;

void note(const char* call, const void* a = nullptr) {
  char line[96];
  std::snprintf(line, sizeof line, "%s %p\n", call, a);
  g_log += line;
}
template <typename T>
hipError_t make(T* out) {
  *out = reinterpret_cast<T>(g_next += 0x10);
  return hipSuccess;
}
hipError_t on_stream(const char* call, hipStream_t s) {
  note(call, s);
  if (s && !g_live.count(s)) note("DEAD_STREAM", s);
  return hipSuccess;
}
}  // namespace

extern "C" {
const char* mock_log() {
  g_out.swap(g_log);
  g_log.clear();
  return g_out.c_str();
}
void mock_fail_malloc(size_t bytes, int count) {
  g_fail_bytes = bytes;
  g_fail_count = count;
}

void** __hipRegisterFatBinary(const void*) {
  static void* h;
  return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* fn, char*, const char* name, unsigned, void*, void*,
                           void*, void*, int*) {
  g_kernel[fn] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t m, hipStream_t s) {
  g_grid = g; g_block = b; g_shared = m; g_stream = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* m, hipStream_t* s) {
  *g = g_grid; *b = g_block; *m = g_shared; *s = g_stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* fn, dim3 g, dim3, void**, size_t lds, hipStream_t s) {
  g_log += "launch " + std::to_string(g.x) + " " + std::to_string(lds) + " " + g_kernel[fn] + "\n";
  return on_stream("on", s);
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }

hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {
  std::memset(p, 0, sizeof *p);
  std::strcpy(p->gcnArchName, "gfx950:sramecc+:xnack-");
  p->multiProcessorCount = 256;
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "mock error"; }
hipError_t hipGetLastError() { return hipSuccess; }

hipError_t hipMalloc(void** p, size_t n) {
  if (g_fail_count > 0 && n >= g_fail_bytes) {
    --g_fail_count;
    *p = nullptr;
    return hipErrorOutOfMemory;
  }
  *p = std::aligned_alloc(4096, (n + 4095) & ~(size_t)4095);
  note("hipMalloc", reinterpret_cast<void*>(n));
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) {
  note("hipFree", p);
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemset(void* d, int v, size_t n) {
  std::memset(d, v, n);
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static void* scratch = std::aligned_alloc(4096, 64 << 20);
  *p = scratch;
  return hipSuccess;
}

hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  make(s);
  g_live.insert(*s);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  on_stream("hipStreamDestroy", s);
  g_live.erase(s);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) { return on_stream("hipStreamSynchronize", s); }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* c) {
  *c = hipStreamCaptureStatusNone;
  return on_stream("hipStreamIsCapturing", s);
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
  return on_stream("hipStreamBeginCapture", s);
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g) {
  make(g);
  return on_stream("hipStreamEndCapture", s);
}
hipError_t hipDeviceSynchronize() { note("hipDeviceSynchronize"); return hipSuccess; }

hipError_t hipEventCreate(hipEvent_t* e) { return make(e); }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return make(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t s) { return on_stream("hipEventRecord", s); }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 1.0f;
  return hipSuccess;
}

hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  return make(e);
}
hipError_t hipGraphExecUpdate(hipGraphExec_t, hipGraph_t, hipGraphNode_t*,
                              hipGraphExecUpdateResult* r) {
  *r = hipGraphExecUpdateSuccess;
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t s) { return on_stream("hipGraphLaunch", s); }
hipError_t hipGraphExecDestroy(hipGraphExec_t e) { note("hipGraphExecDestroy", e); return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t g) { note("hipGraphDestroy", g); return hipSuccess; }
}
