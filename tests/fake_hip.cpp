// A HIP runtime for tests of the library's host code: memory from the heap,
// copies at once, launches that do nothing.  Loaded before libstarmap.so, whose
// calls then come here.
//   FAKE_LDS             bytes of LDS per workgroup (default 160 KiB)
//   fake_failing_copies  copies that fail from now on
//   fake_device          the current device
// A launch with more than 64 KiB of LDS fails where its kernel was not opted in
// to them on the current device.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <utility>

static std::map<std::pair<int, const void*>, size_t> opted_in;
static hipError_t last = hipSuccess;
static struct {
  dim3 grid, block;
  size_t lds;
  hipStream_t stream;
} launch;

extern "C" {
int fake_failing_copies = 0, fake_device = 0;
hipError_t hipGetDevice(int* d) { *d = fake_device; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  const char* lds = std::getenv("FAKE_LDS");
  *v = a == hipDeviceAttributeMaxSharedMemoryPerBlock ? (lds ? std::atoi(lds) : 160 * 1024) : 256;
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) { return posix_memalign(p, 256, n + 256) ? hipErrorOutOfMemory : hipSuccess; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  if (fake_failing_copies > 0 && fake_failing_copies--) return hipErrorInvalidValue;
  std::memcpy(d, s, n);
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "an error"; }
hipError_t hipStreamCreate(hipStream_t* s) { *s = reinterpret_cast<hipStream_t>(std::malloc(1)); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { std::free(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = reinterpret_cast<hipEvent_t>(std::malloc(1)); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { std::free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute a, int v) {
  if (a == hipFuncAttributeMaxDynamicSharedMemorySize) opted_in[{fake_device, f}] = size_t(v);
  return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) {
  launch = {g, b, lds, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s) {
  *g = launch.grid, *b = launch.block, *lds = launch.lds, *s = launch.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void**, size_t lds, hipStream_t) {
  if (lds > 64 * 1024 && opted_in[{fake_device, f}] < lds) last = hipErrorInvalidValue;
  return last;
}
hipError_t hipGetLastError() {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
}
