// The trainer's C entries (closure.cpp) on the host, with launches that only
// record Adam's bias correction, or fail where the command line says so.
//   FAIL...   per training step the number of the launch that fails (0: none);
//             prints the step's return code, and the correction 1 - beta1^t of
//             its update if that was launched
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>

#include "../include/starmap.h"
#include "mlp.hpp"

static int fail_at = 0, launched = 0;
static hipError_t launch() { return ++launched == fail_at ? hipErrorInvalidValue : hipSuccess; }
static float updated = -1.f;

extern "C" {
hipError_t hipMalloc(void** p, size_t n) { return (*p = std::malloc(n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "an error"; }
}

namespace starmap {
namespace detail {
int fail(int code, const std::string&) { return code; }
}  // namespace detail
int mlp_row_blocks(int) { return 1; }
int mlp_sum_chunks(int) { return 1; }
hipError_t launch_mlp_rows(const MlpRows&, bool, hipStream_t) { return launch(); }
hipError_t launch_mlp_grad(const MlpGrad&, hipStream_t) { return launch(); }
hipError_t launch_mlp_update(const MlpGrad&, float*, const MlpAdam& a, const double*, double*, hipStream_t) {
  const hipError_t e = launch();
  if (e == hipSuccess) updated = a.c1;
  return e;
}
hipError_t launch_adam(const MlpAdam& a, const float*, hipStream_t) {
  const hipError_t e = launch();
  if (e == hipSuccess) updated = a.c1;
  return e;
}
}  // namespace starmap

int main(int argc, char** argv) {
  starmap_mlp* n = nullptr;
  if (starmap_mlp_create(32, nullptr, &n)) return 1;
  static float x[32 * 128], t[32 * 6];
  for (int i = 1; i < argc; ++i) {
    fail_at = std::atoi(argv[i]);
    launched = 0;
    updated = -1.f;
    const int rc = starmap_mlp_train_step(n, x, t, 32, 1e-3, nullptr);
    std::printf("%d %.9g\n", rc, double(updated));
  }
  starmap_mlp_destroy(n);
  return 0;
}
