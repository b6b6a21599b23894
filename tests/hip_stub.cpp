// A HIP runtime of host functions that only keeps a record, for tests of the
// library's host side without a GPU: loaded with RTLD_GLOBAL before libdomino.so,
// it takes the place of the real runtime in it.  "Device" addresses are never
// dereferenced.  Streams are plain numbers; those listed by stub_capture() capture.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <vector>

namespace {
std::map<const void *, std::string> g_names;  // host stub -> kernel name (mangled)
std::string g_log;
std::map<std::string, int> g_fail;  // entry point -> calls left that fail
std::set<hipStream_t> g_capturing;
size_t g_next = 1 << 20;
struct Config {
  dim3 grid, block;
  size_t lds;
  hipStream_t st;
};
std::vector<Config> g_cfg;

bool failing(const char *fn) {
  auto it = g_fail.find(fn);
  return it != g_fail.end() && it->second > 0 && it->second-- > 0;
}
template <typename... A>
void note(const char *fmt, A... a) {
  char buf[768];
  snprintf(buf, sizeof(buf), fmt, a...);
  g_log += buf;
}
void *fresh() { return (void *)(g_next += 4096); }
}  // namespace

extern "C" {
const char *stub_log() { return g_log.c_str(); }
void stub_clear() { g_log.clear(); }
void stub_fail(const char *fn, int calls) { g_fail[fn] = calls; }
void stub_capture(hipStream_t st, int on) {
  if (on) g_capturing.insert(st);
  else g_capturing.erase(st);
}

void **__hipRegisterFatBinary(const void *) { return (void **)fresh(); }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *) {
  g_names[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t st) {
  g_cfg.push_back({grid, block, lds, st});
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *st) {
  const Config c = g_cfg.back();
  g_cfg.pop_back();
  *grid = c.grid;
  *block = c.block;
  *lds = c.lds;
  *st = c.st;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *fn, dim3 g, dim3 b, void **, size_t, hipStream_t st) {
  if (failing("hipLaunchKernel")) return hipErrorUnknown;
  note("launch %s %u %u %u %u %zu\n", g_names[fn].c_str(), g.x, g.y, g.z, b.x, (size_t)st);
  return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t) {
  *p = fresh();
  return hipSuccess;
}
hipError_t hipFree(void *) { return hipSuccess; }
hipError_t hipMemcpy(void *, const void *, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *, const void *, size_t n, hipMemcpyKind, hipStream_t st) {
  note("copy %zu %zu\n", n, (size_t)st);
  return hipSuccess;
}
hipError_t hipMemcpy2DAsync(void *, size_t, const void *, size_t, size_t, size_t, hipMemcpyKind, hipStream_t) {
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetDevice(int *d) {
  if (failing("hipGetDevice")) return hipErrorUnknown;
  *d = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) {
  *v = 256;
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipGetSymbolAddress(void **p, const void *) {
  *p = fresh();
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) {
  *n = 1;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
  *s = (hipStream_t)fresh();
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t st, hipStreamCaptureStatus *s) {
  *s = g_capturing.count(st) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) {
  *e = (hipEvent_t)fresh();
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
  if (failing("hipEventCreateWithFlags")) return hipErrorOutOfMemory;
  return hipEventCreate(e);
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
  *ms = 0.f;
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t st) {
  if (failing("hipEventRecord")) return hipErrorUnknown;
  note("record %zu\n", (size_t)st);
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t st, hipEvent_t, unsigned) {
  if (failing("hipStreamWaitEvent")) return hipErrorUnknown;
  note("wait %zu\n", (size_t)st);
  return hipSuccess;
}
}
