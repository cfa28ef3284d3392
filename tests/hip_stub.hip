// HIP runtime for host-logic tests without a GPU: device memory is host memory, kernels do nothing
// but the two a solve's host loop lives on (the state's upload and the control step's progress
// word).  Loaded with RTLD_GLOBAL before the library, whose runtime calls then come here.
#include "fftc_internal.h"

#include <stdlib.h>
#include <string.h>

#include <map>
#include <string>

using fftc::DevState;

namespace {
std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}
struct Config {
  dim3 grid, block;
  size_t lds;
  hipStream_t s;
} g_cfg;
unsigned* g_word = nullptr;        // of the solve under way
unsigned g_tests = 0, g_last = 0;  // its equilibrium tests so far; the one that ends it
long long g_seq = 0, g_launch_at = 0, g_sync_at = 0;
int g_errors_after = -1, g_sync_fails = 0, g_slabs = 0;
}  // namespace

extern "C" {

// what the tests set and read
void stub_reset(int tests_to_end, int errors_after, int sync_fails) {
  g_last = (unsigned)tests_to_end;
  g_errors_after = errors_after;   // hipGetLastError calls that succeed, -1: all
  g_sync_fails = sync_fails;
}
void* stub_word() { return g_word; }
int stub_slabs() { return g_slabs; }
int stub_drained() { return g_sync_at > g_launch_at; }

void** __hipRegisterFatBinary(const void*) {
  static void* module = nullptr;
  return &module;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  names()[f] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) {
  g_cfg = Config{grid, block, lds, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s) {
  *grid = g_cfg.grid;
  *block = g_cfg.block;
  *lds = g_cfg.lds;
  *s = g_cfg.s;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t) {
  g_launch_at = ++g_seq;
  const std::string& name = names()[f];
  if (name.find("k_set_state") != std::string::npos) {
    g_word = ((const DevState*)args[1])->progress;
    g_tests = 0;
  } else if (name.find("k_control") != std::string::npos && g_word) {
    ++g_tests;
    *g_word = g_tests | (g_tests >= g_last ? fftc::kProgressDone : 0u);
  }
  return hipSuccess;
}
hipError_t hipGetLastError() {
  if (g_errors_after < 0) return hipSuccess;
  return g_errors_after-- > 0 ? hipSuccess : hipErrorUnknown;
}
const char* hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipStreamSynchronize(hipStream_t) {
  if (g_sync_fails) return hipErrorUnknown;
  g_sync_at = ++g_seq;
  return hipSuccess;
}
hipError_t hipStreamQuery(hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t) {
  memmove(dst, src, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* dst, int v, size_t n, hipStream_t) {
  memset(dst, v, n);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  ++g_slabs;
  *p = calloc(1, n);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void* p) {
  --g_slabs;
  free(p);
  return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode*) { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 256;
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = 2;
  return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t*, const void*) { return hipErrorInvalidValue; }
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = (hipEvent_t)1;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 1.0f;
  return hipSuccess;
}

}  // extern "C"
