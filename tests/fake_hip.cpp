// A stand-in for the HIP runtime on a machine without a GPU: device memory is
// host memory, kernels are only noted, streams and events are numbers.  It lets
// the library's host code run through its C entry points, with copies and host
// allocations that fail on demand and a log of what was enqueued where.
// Loaded before the library, with its symbols global.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>
#include <string>

namespace {

struct State {
  std::string log;
  std::map<const void *, std::string> kernels;
  std::map<void *, size_t> sizes;
  long streams = 0, events = 0;
};
State &st() {
  static State *s = new State;
  return *s;
}
bool g_log = false;
long g_fail_copy = 0;   // the n-th copy from now fails (0: none)
size_t g_fail_new = 0;  // host allocations of at least this size fail (0: none)
thread_local bool g_own = false;  // an allocation of the stand-in itself
thread_local struct {
  dim3 grid, block;
  size_t shmem;
  hipStream_t stream;
} g_call;

void note(const char *what, const void *a, size_t n) {
  if (!g_log) return;
  char line[256];
  snprintf(line, sizeof line, "%s %ld %zu\n", what, (long)(intptr_t)a, n);
  g_own = true;
  st().log += line;
  g_own = false;
}
hipError_t copy(void *d, const void *s, size_t n, hipStream_t q, const char *what) {
  note(what, q, n);
  if (g_fail_copy > 0 && --g_fail_copy == 0) return hipErrorInvalidValue;
  std::memmove(d, s, n);
  return hipSuccess;
}
const char *kind_name(hipMemcpyKind k) {
  return k == hipMemcpyHostToDevice ? "to_device"
                                    : (k == hipMemcpyDeviceToHost ? "to_host" : "on_device");
}

}  // namespace

// host allocations of the library
void *operator new(size_t n) {
  if (g_fail_new && !g_own && n >= g_fail_new) throw std::bad_alloc();
  void *p = std::malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

extern "C" {

void fake_fail_copy(long n) { g_fail_copy = n; }
void fake_fail_new(size_t n) { g_fail_new = n; }
void fake_log_start() {
  st().log.clear();
  g_log = true;
}
const char *fake_log_stop() {
  g_log = false;
  return st().log.c_str();
}

void **__hipRegisterFatBinary(const void *) {
  static void *handle = nullptr;
  return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *,
                           void *, void *, void *, int *) {
  st().kernels[host] = name;
}
void __hipRegisterVar(void **, void *var, char *, char *, int, size_t size, int, int) {
  st().sizes[var] = size;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, hipStream_t s) {
  g_call = {grid, block, shmem, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shmem, hipStream_t *s) {
  *grid = g_call.grid;
  *block = g_call.block;
  *shmem = g_call.shmem;
  *s = g_call.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3, dim3, void **, size_t, hipStream_t s) {
  char what[192];
  snprintf(what, sizeof what, "kernel %s", st().kernels[f].c_str());
  note(what, s, 0);
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **out, const void *var) {
  *out = std::calloc(1, st().sizes.count((void *)var) ? st().sizes[(void *)var] : 1 << 21);
  return *out ? hipSuccess : hipErrorOutOfMemory;
}

hipError_t hipGetDeviceCount(int *n) {
  *n = 1;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) {
  std::memset(p, 0, sizeof *p);
  std::strcpy(p->gcnArchName, "gfx950");
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "stand-in error"; }

hipError_t hipMalloc(void **p, size_t n) {
  *p = std::calloc(1, n ? n : 1);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void *p) { return hipFree(p); }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind k) {
  return copy(d, s, n, nullptr, kind_name(k));
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t q) {
  return copy(d, s, n, q, kind_name(k));
}
hipError_t hipMemset(void *d, int v, size_t n) {
  std::memset(d, v, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { return hipMemset(d, v, n); }

hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
  *s = (hipStream_t)(intptr_t)++st().streams;
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
  note("wait", s, 0);
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  note("wait_event", s, (size_t)(intptr_t)e);
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
  *g = (hipGraph_t)1;
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t) {
  *e = (hipGraphExec_t)1;
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t s) {
  note("graph", s, 0);
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }

hipError_t hipEventCreate(hipEvent_t *e) {
  *e = (hipEvent_t)(intptr_t)++st().events;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  note("record_event", s, (size_t)(intptr_t)e);
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
  *ms = 1.0f;
  return hipSuccess;
}

}  // extern "C"
