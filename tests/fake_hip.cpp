// A stand-in for the HIP calls that the library's host code makes, for tests of that code without
// a GPU: "device" memory is zeroed host memory, copies are immediate and kernels do nothing.
// fake_limit sets the size from which hipMalloc fails, fake_allow how many of its calls succeed;
// fake_on_read a function called after each copy to the host, which may change what it reads;
// fake_log returns the calls so far, one "name value" a line.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <string>

namespace {
size_t limit = ~(size_t)0, allow = ~(size_t)0;
void (*on_read)(void*, size_t) = nullptr;
std::string calls;
hipError_t last = hipSuccess;

void note(const char* what, size_t v) { calls += std::string(what) + " " + std::to_string(v) + "\n"; }
}  // namespace

extern "C" {

void fake_limit(size_t bytes) { limit = bytes; }
void fake_allow(size_t count) { allow = count; }
void fake_on_read(void (*f)(void*, size_t)) { on_read = f; }
const char* fake_log() { return calls.c_str(); }

void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, hipStream_t* st) {
  *g = *b = dim3(1);
  *s = 0;
  *st = nullptr;
  return hipSuccess;
}

hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  std::memset(p, 0, sizeof(*p));
  p->multiProcessorCount = 256;
  p->sharedMemPerBlock = 160 * 1024;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 100000; return hipSuccess; }

hipError_t hipMalloc(void** p, size_t n) {
  note("malloc", n);
  if (n >= limit || allow == 0) return last = hipErrorOutOfMemory;
  --allow;
  *p = std::calloc(1, n);
  return hipSuccess;
}
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  note("host", n);
  *p = std::calloc(1, n);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }

hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) {
  std::memcpy(d, s, n);
  if (k == hipMemcpyDeviceToHost && on_read) on_read(d, n);
  return hipSuccess;
}
hipError_t hipMemcpy2DAsync(void*, size_t, const void*, size_t, size_t, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)std::malloc(1); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.0f; return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 1; return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipLaunchCooperativeKernel(const void*, dim3 g, dim3, void**, unsigned, hipStream_t) {
  note("cooperative", g.x);
  return hipSuccess;
}
hipError_t hipGetLastError() { const hipError_t e = last; last = hipSuccess; return e; }
const char* hipGetErrorString(hipError_t) { return "error"; }
}
