// Decay and source planes of time-separable data, formed on the device once
// per step (time-dependent data are frozen at t + dt/2 for a step, Sect. 5.7):
// each output plane is a short linear combination of basis planes g_i whose
// time factors a_i(t + dt/2) arrive as kernel arguments.  Per output point one
// read per entry and one write; on the small grids that such runs have, the
// time is the launch and the chain of reads record -> entries -> basis.  So one
// launch forms decay and source planes, a record holds what an output needs,
// and up to four entries' planes are read together.  A P_7 run on 128^2 cells
// with four absorbers, two pulses and scattering by order: 28.7 -> 23.2 us per
// step of three sweeps.
#include "device.hpp"
#include "kernels.hpp"

namespace starmap {

namespace {

constexpr int kThreads = 256;
constexpr int kPerThread = 4;

// acc += the next K entries' planes, all in flight before the first is used.
template <int K, typename C>
__device__ __forceinline__ void add_entries(C (&acc)[kPerThread], const CombineArgs& a, int e, int64_t base) {
  const cptr<int> ent = (cptr<int>)a.entries;
  C coef[K], g[K][kPerThread];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int b = ent[3 * (e + k)], term = ent[3 * (e + k) + 1], sign = ent[3 * (e + k) + 2];
    coef[k] = C(double(sign) * (term >= 0 ? a.a[term] : 1.0));
    const C* p = static_cast<const C*>(a.basis) + int64_t(b) * a.plane_stride;
#pragma unroll
    for (int r = 0; r < kPerThread; ++r) g[k][r] = p[min(base + r * kThreads, a.plane_stride - 1)];
  }
#pragma unroll
  for (int k = 0; k < K; ++k)
#pragma unroll
    for (int r = 0; r < kPerThread; ++r) acc[r] = fma(coef[k], g[k][r], acc[r]);
}

// blockIdx.y: one output, of the decay list and then of the source list;
// blockIdx.x: kThreads * kPerThread consecutive points of the plane.  The entry
// range is uniform over the block.
template <typename C, typename To>
__global__ void __launch_bounds__(kThreads) combine_kernel(CombineArgs a) {
  const bool src = int(blockIdx.y) >= a.nlist[0];
  const int4 rec = src ? rec4((cptr<int>)a.list[1], int(blockIdx.y) - a.nlist[0])
                       : rec4((cptr<int>)a.list[0], int(blockIdx.y));
  const int64_t base = int64_t(blockIdx.x) * (kThreads * kPerThread) + threadIdx.x;
  C acc[kPerThread];
#pragma unroll
  for (int r = 0; r < kPerThread; ++r) acc[r] = C(((cptr<double>)a.cst)[rec.w]);
  int e = rec.y;
  const int end = e + rec.z;
  for (; end - e >= 4; e += 4) add_entries<4>(acc, a, e, base);
  switch (end - e) {
    case 3: add_entries<3>(acc, a, e, base); break;
    case 2: add_entries<2>(acc, a, e, base); break;
    case 1: add_entries<1>(acc, a, e, base); break;
  }
#pragma unroll
  for (int r = 0; r < kPerThread; ++r) {
    const int64_t i = base + r * kThreads, at = int64_t(rec.x) * a.plane_stride + i;
    if (i >= a.plane_stride) continue;
    if (src)
      static_cast<To*>(a.sources)[at] = from_c<To>(acc[r]);
    else
      static_cast<C*>(a.decay)[at] = acc[r];
  }
}

template <typename C, typename To>
hipError_t launch_t(const CombineArgs& a, hipStream_t stream) {
  const int64_t per_block = kThreads * kPerThread;
  const dim3 grid(unsigned((a.plane_stride + per_block - 1) / per_block), unsigned(a.nlist[0] + a.nlist[1]));
  hipLaunchKernelGGL((combine_kernel<C, To>), grid, dim3(kThreads), 0, stream, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_combine(int storage, const CombineArgs& a, hipStream_t stream) {
  if (a.nlist[0] < 0 || a.nlist[1] < 0 || a.nlist[0] + a.nlist[1] < 1 || a.nlist[0] + a.nlist[1] > 65535 ||
      a.plane_stride < 1)
    return hipErrorInvalidValue;
  switch (storage) {
    case STORE_FP64: return launch_t<double, double>(a, stream);
    case STORE_FP32: return launch_t<float, float>(a, stream);
    case STORE_BF16: return launch_t<float, bf16>(a, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace starmap
