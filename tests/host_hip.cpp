// A HIP runtime for the host alone: device memory is host memory, kernels do
// not run, and every launch is recorded by kernel name and first argument. With
// it loaded before the library, the library's host code (plans, queues,
// workspaces, clears) runs on any machine and a test reads what it launched.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}
std::string& launches() {
  static std::string s;
  return s;
}
std::map<void*, size_t>& blocks() {
  static std::map<void*, size_t> m;
  return m;
}
int fail_cooperative = 0;                    // the n-th next cooperative launch fails (0: none)
struct Config {
  dim3 grid, block;
  size_t shmem;
  hipStream_t stream;
} config;

void record(const void* f, void** args) {
  char first[32];
  std::snprintf(first, sizeof first, " %p\n", args ? *(void**)args[0] : nullptr);
  launches() += names()[f] + first;
}
}  // namespace

extern "C" {

const char* host_hip_launches() { return launches().c_str(); }
void host_hip_reset() { launches().clear(); }
size_t host_hip_bytes() {                    // of device memory held now
  size_t n = 0;
  for (const auto& b : blocks()) n += b.second;
  return n;
}
void host_hip_fail_cooperative(int n) { fail_cooperative = n; }

void** __hipRegisterFatBinary(const void*) {
  static void* handle = nullptr;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, dim3*, dim3*,
                           int*) {
  names()[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, hipStream_t stream) {
  config = {grid, block, shmem, stream};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shmem, hipStream_t* stream) {
  *grid = config.grid;
  *block = config.block;
  *shmem = config.shmem;
  *stream = config.stream;
  return hipSuccess;
}

hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t) {
  record(f, args);
  return hipSuccess;
}
hipError_t hipLaunchCooperativeKernel(const void* f, dim3, dim3, void** args, unsigned, hipStream_t) {
  if (fail_cooperative > 0 && --fail_cooperative == 0) return hipErrorLaunchFailure;
  record(f, args);
  return hipSuccess;
}

hipError_t hipMalloc(void** p, size_t n) {
  *p = std::calloc(1, n);
  if (!*p) return hipErrorOutOfMemory;
  blocks()[*p] = n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  blocks().erase(p);
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemset(void* p, int v, size_t n) {
  std::memset(p, v, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t) { return hipMemset(p, v, n); }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static double scratch[4096];
  *p = scratch;
  return hipSuccess;
}

hipError_t hipGetDeviceCount(int* n) {
  *n = 1;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 100000;
  return hipSuccess;
}
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {
  std::memset(p, 0, sizeof *p);
  p->multiProcessorCount = 256;
  p->totalGlobalMem = (size_t)288 << 30;
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = 1;
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = nullptr;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 0.f;
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "host"; }

}  // extern "C"
