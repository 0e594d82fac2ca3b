// A stand-in for the HIP runtime on a machine without a GPU: the library's host code
// linked against it runs its checks, allocations and launches, no kernel runs, and the
// test sets what the runtime answers (a capture in progress, memory that runs out).
// "Device" memory is zeroed host memory.
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <string>

extern "C" {
// set by the test
int sim_capturing = 0;                  // streams are being captured
size_t sim_limit = (size_t)1 << 40;     // bytes of device memory
// read by the test
size_t sim_used = 0;                    // bytes of device memory allocated
int sim_allocs = 0, sim_frees = 0, sim_device_waits = 0;
int sim_ordered_allocs = 0;             // of those, in stream order
int sim_uploads = 0;                    // host-to-device copies since the last device allocation
}

namespace {
std::map<const void*, std::string>& kernels() {
  static std::map<const void*, std::string> k;
  return k;
}
std::map<void*, size_t>& blocks() {
  static std::map<void*, size_t> b;
  return b;
}
dim3 g_grid, g_block;
size_t g_shared;
hipStream_t g_stream;
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) {
  static void* module = nullptr;
  return &module;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*,
                           int*) {
  kernels()[host] = name;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t s) {
  g_grid = grid;
  g_block = block;
  g_shared = shared;
  g_stream = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* s) {
  *grid = g_grid;
  *block = g_block;
  *shared = g_shared;
  *s = g_stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t) {
  // the counts of a closed surface, so that a synchronised build ends well:
  // k_stats_out(ecls, ne, vbits, nv, stats, host)
  if (kernels()[f].find("k_stats_out") != std::string::npos) (*(int64_t**)args[5])[0] = *(int64_t*)args[1];
  return hipSuccess;
}

hipError_t hipMalloc(void** p, size_t bytes) {
  if (sim_used + bytes > sim_limit) return hipErrorOutOfMemory;
  *p = calloc(1, bytes ? bytes : 1);
  blocks()[*p] = bytes;
  sim_used += bytes;
  sim_allocs++;
  sim_uploads = 0;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (!p) return hipSuccess;
  auto b = blocks().find(p);
  if (b == blocks().end()) return hipErrorInvalidValue;
  sim_used -= b->second;
  blocks().erase(b);
  free(p);
  sim_frees++;
  return hipSuccess;
}
hipError_t hipMallocAsync(void** p, size_t bytes, hipStream_t) {
  sim_ordered_allocs++;
  return hipMalloc(p, bytes);
}
hipError_t hipFreeAsync(void* p, hipStream_t) {
  sim_frees--;  // waits for nothing
  return hipFree(p);
}
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned) {
  *p = calloc(1, bytes);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  free(p);
  return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) {
  *d = h;
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind kind) {
  if (kind == hipMemcpyHostToDevice) sim_uploads++;
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind kind, hipStream_t) {
  return hipMemcpy(d, s, n, kind);
}
hipError_t hipDeviceSynchronize(void) {
  sim_device_waits++;
  return sim_capturing ? hipErrorStreamCaptureUnsupported : hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {  // the null stream is never captured
  return s && sim_capturing ? hipErrorStreamCaptureUnsupported : hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* st) {
  *st = sim_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode*) { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipGetDeviceCount(int* n) {
  *n = 1;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  memset(p, 0, sizeof(*p));
  strcpy(p->gcnArchName, "gfx950");
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 256;
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = 4;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void**, const void*) { return hipErrorInvalidSymbol; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "simulated"; }
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = nullptr;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 0.f;
  return hipSuccess;
}
}
