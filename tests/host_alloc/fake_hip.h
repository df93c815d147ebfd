// A HIP runtime for host tests: an executable that defines these functions and exports
// them (-rdynamic) takes them in the place of the runtime's, so that libgps.so runs its host
// paths without a GPU.  Device memory is host memory under a limit, kernels are counted by
// name and not run, graphs are empty, and every solve state that the host reads back (a short
// copy whose first word is the done flag) says done.
#pragma once

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

#include <hip/hip_runtime_api.h>

namespace fake {
inline std::map<void*, size_t> blocks;         // device allocations
inline size_t used = 0, peak = 0, limit = ~size_t(0);
inline int frees = 0, late = 0;                // frees, and allocations after one
inline std::map<std::string, int> launches;    // by kernel name (mangled)
// (the library registers its kernels before this executable's objects are constructed)
inline std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> n;
  return n;
}

inline int count(const char* part) {
  int n = 0;
  for (const auto& l : launches)
    if (l.first.find(part) != std::string::npos) n += l.second;
  return n;
}
}  // namespace fake

extern "C" {

void** __hipRegisterFatBinary(const void*) {
  static void* handle = nullptr;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device_name, unsigned,
                           void*, void*, void*, void*, int*) {
  fake::names()[host] = device_name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}

static thread_local dim3 g_grid, g_block;
static thread_local size_t g_shared;
static thread_local hipStream_t g_stream;
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
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void**, size_t, hipStream_t) {
  ++fake::launches[fake::names()[f]];
  return hipSuccess;
}
hipError_t hipExtLaunchKernel(const void* f, dim3 g, dim3 b, void** a, size_t n, hipStream_t s,
                              hipEvent_t, hipEvent_t, int) {
  return hipLaunchKernel(f, g, b, a, n, s);
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }

#undef hipMalloc
#undef hipHostMalloc
hipError_t hipMalloc(void** p, size_t n) {
  *p = nullptr;
  if (n > fake::limit - fake::used || fake::used > fake::limit) return hipErrorOutOfMemory;
  *p = std::calloc(n, 1);
  fake::blocks[*p] = n;
  fake::used += n;
  if (fake::used > fake::peak) fake::peak = fake::used;
  if (fake::frees > 0) ++fake::late;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  const auto b = fake::blocks.find(p);
  if (p == nullptr) return hipSuccess;
  if (b == fake::blocks.end()) std::abort();
  ++fake::frees;
  fake::used -= b->second;
  fake::blocks.erase(b);
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  *p = std::calloc(n, 1);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind kind, hipStream_t) {
  std::memcpy(d, s, n);
  const int done = 1;
  if (kind == hipMemcpyDeviceToHost && n < 512) std::memcpy(d, &done, sizeof(done));
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void**, const void*) { return hipErrorInvalidSymbol; }
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = reinterpret_cast<hipStream_t>(std::malloc(1));
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  std::free(s);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  *g = nullptr;
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  *e = reinterpret_cast<hipGraphExec_t>(std::malloc(1));
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t e) {
  std::free(e);
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = reinterpret_cast<hipEvent_t>(std::malloc(1));
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
  std::free(e);
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 1.0f;
  return hipSuccess;
}

}  // extern "C"
