// A HIP runtime that runs no kernel, linked with the library's host code (both compiled for the
// host alone) so that what the host decides can be tested without a GPU: which kernels it
// launches on which streams, what waits for what, what happens when an allocation fails or a
// stream captures.  "Device" memory is host memory.  Streams are idle unless held; a virtual
// clock advances by a settable cost per launch, and events take its time.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "rod_kernels.hpp"

namespace {
struct Event {
  hipStream_t stream = nullptr;
  bool recorded = false, captured = false;
  double at = 0.0;
};
struct Launch {
  std::string name;
  hipStream_t stream;
  unsigned grid;
};
std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}
std::map<uintptr_t, size_t> blocks;   // allocations
std::set<hipStream_t> held, capturing;
std::vector<Launch> launches;
std::vector<std::pair<std::string, double>> costs;
int waits, syncs, queries, broken_captures;
long long fail_malloc = -1;   // allocations until one fails
bool strict;                  // another thread captures in the global mode
bool implicit;                // the null stream's capture status is not to be had
hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;
double now_us;
hipError_t last = hipSuccess;
hipError_t ret(hipError_t e) {
  if (e != hipSuccess) last = e;
  return e;
}
struct Config {
  dim3 grid, block;
  size_t shared;
  hipStream_t stream;
} config;
hipError_t unsafe_call() {   // a call that a capture in the global mode does not allow
  if (!strict || mode == hipStreamCaptureModeRelaxed) return hipSuccess;
  ++broken_captures;
  return ret(hipErrorStreamCaptureUnsupported);
}
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) {
  static void* h;
  return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* fn, char*, const char* name, unsigned, void*, void*,
                           void*, void*, int*) {
  names()[fn] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream) {
  config = {grid, block, shared, stream};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* stream) {
  *grid = config.grid, *block = config.block, *shared = config.shared, *stream = config.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* fn, dim3 grid, dim3, void**, size_t, hipStream_t stream) {
  launches.push_back({names()[fn], stream, grid.x});
  for (const auto& c : costs)
    if (launches.back().name.find(c.first) != std::string::npos) now_us += c.second;
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipDeviceSynchronize() { ++syncs; return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = 2;
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
  if (fail_malloc >= 0 && fail_malloc-- == 0) return ret(hipErrorOutOfMemory);
  *p = calloc(1, n);
  blocks[(uintptr_t)*p] = n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  blocks.erase((uintptr_t)p);
  free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static void* scratch = malloc(64u << 20);
  *p = scratch;
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemset(void* d, int v, size_t n) { memset(d, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { memset(d, v, n); return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  auto it = blocks.upper_bound((uintptr_t)p);
  if (it == blocks.begin()) return ret(hipErrorInvalidValue);
  --it;
  if ((uintptr_t)p >= it->first + it->second) return ret(hipErrorInvalidValue);
  a->type = hipMemoryTypeDevice;
  a->device = 0;
  return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t* base, size_t* n, hipDeviceptr_t p) {
  auto it = --blocks.upper_bound((uintptr_t)p);
  *base = (hipDeviceptr_t)it->first, *n = it->second;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  static uintptr_t next = 0x100000;
  *s = (hipStream_t)(next += 16);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
  if (capturing.count(s)) return ret(hipErrorStreamCaptureUnsupported);
  ++syncs;
  held.erase(s);
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
  if (implicit && !s) return ret(hipErrorStreamCaptureImplicit);
  *st = capturing.count(s) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) {
  std::swap(*m, mode);
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  Event& ev = *(Event*)e;
  if (ev.captured != (capturing.count(s) != 0) && ev.recorded) {
    ++broken_captures;
    return ret(hipErrorStreamCaptureIsolation);
  }
  ++waits;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t) new Event; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { delete (Event*)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  *(Event*)e = {s, true, capturing.count(s) != 0, now_us};
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
  const Event& ev = *(Event*)e;
  ++queries;
  if (hipError_t r = unsafe_call()) return r;
  if (ev.captured) return ret(hipErrorCapturedEvent);
  return ev.recorded && held.count(ev.stream) ? ret(hipErrorNotReady) : hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  Event& ev = *(Event*)e;
  if (ev.captured) return ret(hipErrorCapturedEvent);
  held.erase(ev.stream);
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
  if (((Event*)a)->captured || ((Event*)b)->captured) return ret(hipErrorCapturedEvent);
  *ms = (float)((((Event*)b)->at - ((Event*)a)->at) * 1e-3);
  return hipSuccess;
}
hipError_t hipGetLastError() {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t) { return "error of the test's runtime"; }

// ---- what the tests set and read
void stub_reset() {
  held.clear(), capturing.clear(), launches.clear(), costs.clear();
  waits = syncs = queries = broken_captures = 0;
  fail_malloc = -1, strict = implicit = false, mode = hipStreamCaptureModeGlobal, now_us = 0.0, last = hipSuccess;
}
void stub_hold(hipStream_t s, int on) { on ? (void)held.insert(s) : (void)held.erase(s); }
void stub_capture(hipStream_t s, int on) { on ? (void)capturing.insert(s) : (void)capturing.erase(s); }
void stub_strict(int on) { strict = on; }
void stub_implicit(int on) { implicit = on; }
void stub_fail_malloc(long long after) { fail_malloc = after; }
void stub_cost(const char* part, double us) { costs.push_back({part, us}); }
int stub_waits() { return waits; }
int stub_syncs() { return syncs; }
int stub_queries() { return queries; }
int stub_broken_captures() { return broken_captures; }
int stub_allocations() { return (int)blocks.size(); }
int stub_launches() { return (int)launches.size(); }
const char* stub_launch(int i, hipStream_t* s, unsigned* grid) {
  *s = launches[i].stream, *grid = launches[i].grid;
  return launches[i].name.c_str();
}
int chunk_mark_behind(uint32_t mark, uint32_t target) { return corde::mark_behind(mark, target); }
uint32_t chunk_first_mark() { return corde::kFirstMark; }
uint32_t chunk_launch_marks(int n_steps, int every) { return corde::launch_marks(n_steps, every); }
}
