// Learned closure of the P_5 hierarchy on gfx950: the network's training
// kernels (BF16 MFMA matrix products with FP32 accumulation, GELU, loss,
// Adam), the extraction of training samples from a high-order state, and the
// fused closure kernel that evaluates the network at every point of a P_5
// state before an odd sweep.
//
// The closure replaces the order-6 flux the P_N truncation drops (the moment
// system is closed by zeroing order N + 1, Sect. 2) with a network of the
// local order-4/5 data:
//   inputs  : 3 x 3 array stencils of the eleven order-4/5 moments divided by
//             their norm nu, log10(sigma_a + 0.01), log10(sigma_s + 0.01),
//             zero padding to 128;
//   network : 128 -> 128 -> 128 -> 6, GELU after the hidden layers;
//   output  : g = nu * y / dx added to the residual of the six order-5 moments.
// Matrix-product operands are rounded to bfloat16 (nearest, ties to even);
// accumulation, biases and activations before rounding are FP32.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cmath>
#include <cstdint>

#include "device.hpp"
#include "mlp.hpp"

namespace starmap {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// ------------------------------------------------------------ scalar helpers
__device__ __forceinline__ uint32_t bf16_bits(float v) { return from_c<bf16>(v).bits; }

// Correctly rounded double -> bfloat16: round to odd into FP32 (24 bits, at
// least two more than bfloat16 keeps), then to nearest even.
__device__ __forceinline__ uint32_t bf16_bits(double v) {
  float f = __double2float_rz(v);
  if (double(f) != v) f = __uint_as_float(__float_as_uint(f) | 1u);
  return bf16_bits(f);
}

__device__ __forceinline__ float bf16_value(uint32_t bits) { return __uint_as_float(bits << 16); }

// The same rounding (nearest, ties to even) by the conversion instruction.
__device__ __forceinline__ uint32_t bf16_hw(float v) {
  return __builtin_bit_cast(uint16_t, static_cast<__bf16>(v));
}
__device__ __forceinline__ uint32_t bf16_in(float v) { return bf16_hw(v); }
__device__ __forceinline__ uint32_t bf16_in(double v) { return bf16_bits(v); }

// Two of them, packed.
__device__ __forceinline__ uint32_t bf16_hw2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{lo, hi}), bf16x2));
}

// GELU z Phi(z), Phi the standard normal distribution function, with erf
// from Abramowitz & Stegun, Handbook of Mathematical Functions, formula 7.1.26
// (|error| <= 1.5e-7 on the real line).  Training and inference use this one
// definition.  The formula's coefficients are halved (exactly), so that erf / 2
// comes out without a multiplication by a half.
__device__ __forceinline__ float normal_cdf(float z) {
  const float x = fabsf(z) * 0.70710678118654752f;
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, x, 1.0f));
  const float half_poly =
      t * fmaf(t, fmaf(t, fmaf(t, fmaf(t, 0.5f * 1.061405429f, 0.5f * -1.453152027f), 0.5f * 1.421413741f),
                       0.5f * -0.284496736f), 0.5f * 0.254829592f);
  const float half_erf_abs = fmaf(-half_poly, __expf(-x * x), 0.5f);
  return 0.5f + copysignf(half_erf_abs, z);
}
__device__ __forceinline__ float gelu(float z) { return z * normal_cdf(z); }
// d/dz z Phi(z) = Phi(z) + z phi(z)
__device__ __forceinline__ float gelu_grad(float z) {
  return normal_cdf(z) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

__device__ __forceinline__ f32x4 mfma16(uint4 a, uint4 b, f32x4 c) {
  // D[i][j] += sum_k A[i][k] B[k][j], 16 x 16 x 32: lane l holds A[l % 16][8 (l / 16) + e]
  // and B[8 (l / 16) + e][l % 16] (e = 0..7), and D[4 (l / 16) + r][l % 16] (r = 0..3)
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                  0, 0, 0);
}

__device__ __forceinline__ uint4 pack8(const uint32_t (&h)[8]) {
  return make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16));
}

// ------------------------------------------------------------ training
// A training step is three launches: the rows of the batch through the network
// and back (mlp_rows_kernel), the weight gradients' split partials and the
// column sums (mlp_grad_kernel), and their sums with the Adam update
// (mlp_update_kernel).  The arrays a step moves are a few MB, so launches and
// chains of memory round trips bound it: one product, epilogue or column sum
// per launch (25 of them), with products whose loads waited for one another,
// took 293 us per step at 4096 rows; these three take 40 us.
constexpr int TR = 16;                   // rows of the batch per block
constexpr int LDT = CLOSURE_HIDDEN + 8;  // LDS row of one row's activations (bf16), padded
constexpr int KT = 32;                   // rows per k step of the weight gradients

typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));  // callers' arrays: float alignment

// eight consecutive values as bfloat16
__device__ __forceinline__ uint4 bf16_row8(const float* p) {
  const f32x4u v0 = *reinterpret_cast<const f32x4u*>(p), v1 = *reinterpret_cast<const f32x4u*>(p + 4);
  const uint32_t h[8] = {bf16_bits(v0[0]), bf16_bits(v0[1]), bf16_bits(v0[2]), bf16_bits(v0[3]),
                         bf16_bits(v1[0]), bf16_bits(v1[1]), bf16_bits(v1[2]), bf16_bits(v1[3])};
  return pack8(h);
}

// Transposed activations as the weight gradients read them: per k step of 32
// rows of the batch [unit][row], so that a lane's eight rows of one unit are one
// 16-byte load and a wave's loads are 1 KiB together.
__device__ __forceinline__ int64_t t_index(int b, int units, int unit) {
  return int64_t(b / KT) * (units * KT) + unit * KT + (b % KT);
}
__device__ __forceinline__ void store_transposed(const uint16_t* S, uint16_t* T, int b0) {
  const int unit = int(threadIdx.x) >> 1, half = 8 * (int(threadIdx.x) & 1);
  uint32_t h[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) h[e] = S[(half + e) * LDT + unit];
  *reinterpret_cast<uint4*>(&T[t_index(b0 + half, CLOSURE_HIDDEN, unit)]) = pack8(h);
}

// Rows of the batch through the network (TRAIN: and the loss's gradient back to
// the pre-activations).  A workgroup keeps all weights in registers and loops
// over blocks of 16 rows; wave w owns hidden units [32 w, 32 w + 32).  Products
// are computed transposed as in the closure kernel, H^T = W X^T; the
// pre-activations stay in registers until the backward products need them.
// Only what the weight gradients and the biases' sums read goes to memory.
template <bool TRAIN>
__global__ void __launch_bounds__(256, 2) mlp_rows_kernel(const MlpRows g) {
  __shared__ __align__(16) uint16_t Xs[TR * LDT], H1[TR * LDT], H2[TR * LDT], D2[TR * LDT], D1[TR * LDT];
  __shared__ __align__(16) uint16_t Ys[TR * 8];
  const int tid = int(threadIdx.x), lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pt = lane & 15, grp = lane >> 4, fk = 8 * grp, u0 = 32 * w;
  const float* P = g.params;

  // weight fragments (A operands): rows are the outputs of each product
  uint4 w1[2][4], w2[2][4], w2t[2][4], w3[4], w3t[2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int row = u0 + 16 * i + pt;
      w1[i][ks] = bf16_row8(P + OFF_W1 + row * CLOSURE_IN + 32 * ks + fk);
      w2[i][ks] = bf16_row8(P + OFF_W2 + row * CLOSURE_HIDDEN + 32 * ks + fk);
    }
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    const uint4 v = bf16_row8(P + OFF_W3 + min(pt, CLOSURE_OUT - 1) * CLOSURE_HIDDEN + 32 * ks + fk);
    w3[ks] = pt < CLOSURE_OUT ? v : make_uint4(0, 0, 0, 0);
  }
  if constexpr (TRAIN) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int unit = u0 + 16 * i + pt;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        uint32_t h[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) h[e] = bf16_bits(P[OFF_W2 + (32 * ks + fk + e) * CLOSURE_HIDDEN + unit]);
        w2t[i][ks] = pack8(h);
      }
      uint32_t h[8] = {};
#pragma unroll
      for (int e = 0; e < CLOSURE_OUT; ++e) h[e] = bf16_bits(P[OFF_W3 + e * CLOSURE_HIDDEN + unit]);
      const uint4 v = pack8(h);
      w3t[i] = grp == 0 ? v : make_uint4(0, 0, 0, 0);
    }
  }
  // biases of the lane's outputs: units u0 + 16 i + 4 grp + r, outputs 4 grp + r
  f32x4 b1[2], b2[2], b3;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      b1[i][r] = P[OFF_B1 + u0 + 16 * i + 4 * grp + r];
      b2[i][r] = P[OFF_B2 + u0 + 16 * i + 4 * grp + r];
    }
#pragma unroll
  for (int r = 0; r < 4; ++r) b3[r] = P[OFF_B3 + min(4 * grp + r, CLOSURE_OUT - 1)];

  // a layer: the lane's four units x two tiles of point pt
  auto product = [&](const uint4 (&wf)[2][4], const uint16_t* S, f32x4 (&acc)[2]) {
    acc[0] = acc[1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const uint4 x = *reinterpret_cast<const uint4*>(&S[pt * LDT + 32 * ks + fk]);
#pragma unroll
      for (int i = 0; i < 2; ++i) acc[i] = mfma16(wf[i][ks], x, acc[i]);
    }
  };
  auto put = [&](uint16_t* S, int i, const float (&v)[4]) {
    *reinterpret_cast<uint2*>(&S[pt * LDT + u0 + 16 * i + 4 * grp]) =
        make_uint2(bf16_bits(v[0]) | (bf16_bits(v[1]) << 16), bf16_bits(v[2]) | (bf16_bits(v[3]) << 16));
  };

  double loss = 0.0;
  const float scale = 2.0f / float(int64_t(g.B) * CLOSURE_OUT);
  const int nblk = (g.B + TR - 1) / TR;
  for (int blk = int(blockIdx.x); blk < nblk; blk += int(gridDim.x)) {
    const int b0 = blk * TR, b = b0 + pt;
    const bool live = b < g.B;
    float tv[4] = {};
    if (TRAIN && w == 0 && live) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (4 * grp + r < CLOSURE_OUT) tv[r] = g.t[int64_t(b) * CLOSURE_OUT + 4 * grp + r];
    }
    {  // rows past the batch are zeros (and so are their activations below)
      const int row = tid >> 4, col = 8 * (tid & 15);
      uint4 v = make_uint4(0, 0, 0, 0);
      if (b0 + row < g.B) v = bf16_row8(g.x + int64_t(b0 + row) * CLOSURE_IN + col);
      *reinterpret_cast<uint4*>(&Xs[row * LDT + col]) = v;
    }
    __syncthreads();
    f32x4 z1[2], z2[2];
    product(w1, Xs, z1);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      float v[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        z1[i][r] += b1[i][r];
        v[r] = live ? gelu(z1[i][r]) : 0.f;
      }
      put(H1, i, v);
    }
    if constexpr (TRAIN) store_transposed(Xs, g.xt, b0);
    __syncthreads();
    product(w2, H1, z2);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      float v[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        z2[i][r] += b2[i][r];
        v[r] = live ? gelu(z2[i][r]) : 0.f;
      }
      put(H2, i, v);
    }
    if constexpr (TRAIN) store_transposed(H1, g.h1t, b0);
    __syncthreads();
    if (w == 0) {
      f32x4 y = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
        y = mfma16(w3[ks], *reinterpret_cast<const uint4*>(&H2[pt * LDT + 32 * ks + fk]), y);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int o = 4 * grp + r;
        const float yv = y[r] + b3[r];
        if constexpr (TRAIN) {
          const float d = yv - tv[r];
          const float dy = live && o < CLOSURE_OUT ? scale * d : 0.f;
          if (o < 8) {
            Ys[pt * 8 + o] = uint16_t(bf16_bits(dy));
            g.dyt[t_index(b, 8, o)] = uint16_t(bf16_bits(dy));
          }
          if (live && o < CLOSURE_OUT) {
            g.dy[int64_t(b) * CLOSURE_OUT + o] = dy;
            loss += double(d) * double(d);
          }
        } else if (live && o < CLOSURE_OUT) {
          g.y[int64_t(b) * CLOSURE_OUT + o] = yv;
        }
      }
    }
    if constexpr (TRAIN) {
      store_transposed(H2, g.h2t, b0);
      __syncthreads();
      // dZ2 = (dY W3) * gelu'(Z2), dZ1 = (dZ2 W2) * gelu'(Z1)
      uint4 yf = *reinterpret_cast<const uint4*>(&Ys[pt * 8]);
      if (grp) yf = make_uint4(0, 0, 0, 0);
      auto back = [&](const f32x4 (&acc)[2], const f32x4 (&z)[2], uint16_t* S, float* out) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          float v[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = live ? acc[i][r] * gelu_grad(z[i][r]) : 0.f;
          put(S, i, v);
          if (live)
            *reinterpret_cast<float4*>(&out[int64_t(b) * CLOSURE_HIDDEN + u0 + 16 * i + 4 * grp]) =
                make_float4(v[0], v[1], v[2], v[3]);
        }
      };
      f32x4 acc[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) acc[i] = mfma16(w3t[i], yf, f32x4{0.f, 0.f, 0.f, 0.f});
      back(acc, z2, D2, g.dz2);
      __syncthreads();
      product(w2t, D2, acc);
      back(acc, z1, D1, g.dz1);
      store_transposed(D2, g.dz2t, b0);
      __syncthreads();
      store_transposed(D1, g.dz1t, b0);
    }
    // (the next block writes Xs, H1, H2 and Ys behind barriers that follow every
    // read of them here; H2, read by wave 0 above, waits for the next block's
    // two barriers, and D1 for more)
  }
  if constexpr (TRAIN) {
    if (w == 0) {
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) loss += __shfl_xor(loss, d);
      if (lane == 0) g.lpart[blockIdx.x] = loss;
    }
  }
}

// Sum of n values in order, the loads of 16 in flight together.
__device__ __forceinline__ float sum_strided(const float* q, int n, int step) {
  float a = 0.f;
  int z = 0;
  for (; z + 16 <= n; z += 16) {
    float v[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) v[e] = q[int64_t(z + e) * step];
#pragma unroll
    for (int e = 0; e < 16; ++e) a += v[e];
  }
  for (; z < n; ++z) a += q[int64_t(z) * step];
  return a;
}

// Weight gradients, G (M x 128) = D^T A over the batch, as partials per split of
// kchunk rows, and partial column sums of the unrounded dZ1, dZ2 and dY (the
// biases' gradients) per chunk of 256 rows.  A workgroup is one 64 x 64 tile of
// W1 or W2 (or all of W3) of one split, fragments straight from memory (the
// operands are laid out for it: no LDS, every load of eight k steps in flight
// together), or 64 columns of a chunk's sums.
constexpr int CS_ROWS = 256;
constexpr int GRAD_TILES = 9;  // four of W1, four of W2, W3
constexpr int SUM_TILES = 5;   // dZ1 and dZ2 64 columns each, dY
__global__ void __launch_bounds__(256) mlp_grad_kernel(const MlpGrad g) {
  __shared__ float s[4][64];
  const int tid = int(threadIdx.x), lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  int id = int(blockIdx.x);
  if (id < g.splits * GRAD_TILES) {
    const int z = id / GRAD_TILES, tile = id - z * GRAD_TILES;
    const int layer = tile >> 2;  // 0: W1, 1: W2, 2: W3
    const uint16_t* D = layer == 0 ? g.dz1t : layer == 1 ? g.dz2t : g.dyt;
    const uint16_t* A = layer == 0 ? g.xt : layer == 1 ? g.h1t : g.h2t;
    const int units = layer == 2 ? 8 : CLOSURE_HIDDEN;
    const int m0 = layer == 2 ? 0 : (tile >> 1 & 1) * 64 + (w >> 1) * 32;
    const int n0 = layer == 2 ? 32 * w : (tile & 1) * 64 + (w & 1) * 32;
    const int pt = lane & 15, fk = 8 * (lane >> 4);
    const int kb = z * g.kchunk, ke = min(g.B, kb + g.kchunk);
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // (rows of W3 past its eight repeat the last one and are not stored)
    auto frag = [&](const uint16_t* T, int n, int unit, int k) {
      return *reinterpret_cast<const uint4*>(&T[t_index(k + fk, n, min(unit, n - 1))]);
    };
    auto step = [&](const uint4 (&a)[2], const uint4 (&b)[2]) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = mfma16(a[i], b[j], acc[i][j]);
    };
    constexpr int DEEP = 8;  // k steps whose loads are in flight together
    int k = kb;
    for (; k + DEEP * KT <= ke; k += DEEP * KT) {
      uint4 a[DEEP][2], b[DEEP][2];
#pragma unroll
      for (int d = 0; d < DEEP; ++d)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          a[d][i] = frag(D, units, m0 + 16 * i + pt, k + d * KT);
          b[d][i] = frag(A, CLOSURE_HIDDEN, n0 + 16 * i + pt, k + d * KT);
        }
#pragma unroll
      for (int d = 0; d < DEEP; ++d) step(a[d], b[d]);
    }
    for (; k < ke; k += KT) {
      uint4 a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a[i] = frag(D, units, m0 + 16 * i + pt, k);
        b[i] = frag(A, CLOSURE_HIDDEN, n0 + 16 * i + pt, k);
        if (k + fk >= ke) a[i] = b[i] = make_uint4(0, 0, 0, 0);  // eight rows past the batch
      }
      step(a, b);
    }
    float* P = g.part + int64_t(z) * CLOSURE_PARAMS + (layer == 0 ? OFF_W1 : layer == 1 ? OFF_W2 : OFF_W3);
    const int M = layer == 2 ? CLOSURE_OUT : CLOSURE_HIDDEN;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = m0 + 16 * i + 4 * (lane >> 4) + r, n = n0 + 16 * j + pt;
          if (m < M) P[m * CLOSURE_HIDDEN + n] = acc[i][j][r];
        }
    return;
  }
  id -= g.splits * GRAD_TILES;
  const int chunk = id / SUM_TILES, part = id - chunk * SUM_TILES;
  const float* X = part < 2 ? g.dz1 : part < 4 ? g.dz2 : g.dy;
  const int N = part < 4 ? CLOSURE_HIDDEN : CLOSURE_OUT;
  const int c = (part < 4 ? (part & 1) * 64 : 0) + lane;
  const int r0 = chunk * CS_ROWS, r1 = min(g.B, r0 + CS_ROWS);
  float a = 0.f;
  if (c < N) a = sum_strided(X + int64_t(r0 + w) * N + c, r1 > r0 + w ? (r1 - r0 - w + 3) / 4 : 0, 4 * N);
  s[w][lane] = a;
  __syncthreads();
  if (w == 0 && c < N)
    g.cpart[int64_t(chunk) * SUM_COLS + (part >> 1) * CLOSURE_HIDDEN + c] =
        ((s[0][lane] + s[1][lane]) + s[2][lane]) + s[3][lane];
}

// Adam with bias correction; c1 = 1 - beta1^t, c2 = 1 - beta2^t.
__device__ __forceinline__ void adam(const MlpAdam& a, int i, float gi) {
  const float mi = a.b1 * a.m[i] + (1.f - a.b1) * gi;
  const float vi = a.b2 * a.v[i] + (1.f - a.b2) * gi * gi;
  a.m[i] = mi;
  a.v[i] = vi;
  a.p[i] -= a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
}
__global__ void __launch_bounds__(256) adam_kernel(const MlpAdam a, const float* grads) {
  const int i = int(blockIdx.x) * 256 + int(threadIdx.x);
  if (i < CLOSURE_PARAMS) adam(a, i, grads[i]);
}

// Sums of the partials in split (chunk) order: the gradient, then (with a.p) the
// Adam update; the last workgroup sums the loss.
__global__ void __launch_bounds__(256) mlp_update_kernel(const MlpGrad g, float* __restrict__ grads, const MlpAdam a,
                                                         const double* __restrict__ lpart, const int nloss,
                                                         double* __restrict__ loss) {
  if (blockIdx.x == gridDim.x - 1) {
    __shared__ double s[256];
    double v = 0.0;
    for (int i = int(threadIdx.x); i < nloss; i += 256) v += lpart[i];
    s[threadIdx.x] = v;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
      if (int(threadIdx.x) < w) s[threadIdx.x] += s[threadIdx.x + w];
      __syncthreads();
    }
    if (threadIdx.x == 0) loss[0] = s[0] * (1.0 / double(int64_t(g.B) * CLOSURE_OUT));
    return;
  }
  const int i = int(blockIdx.x) * 256 + int(threadIdx.x);
  if (i >= CLOSURE_PARAMS) return;
  // biases lie behind their layer's weights
  int col = -1;
  if (i >= OFF_B3)
    col = 2 * CLOSURE_HIDDEN + i - OFF_B3;
  else if (i >= OFF_B2 && i < OFF_W3)
    col = CLOSURE_HIDDEN + i - OFF_B2;
  else if (i >= OFF_B1 && i < OFF_W2)
    col = i - OFF_B1;
  const float* q = col < 0 ? g.part + i : g.cpart + col;
  const int n = col < 0 ? g.splits : (g.B + CS_ROWS - 1) / CS_ROWS, step = col < 0 ? CLOSURE_PARAMS : SUM_COLS;
  const float acc = sum_strided(q, n, step);
  grads[i] = acc;
  if (a.p) adam(a, i, acc);
}

// ------------------------------------------------------------ closure inputs
// Public index a of a moment's array along an axis -> internal storage index
// (nodes of a periodic axis are stored modulo n).
__device__ __forceinline__ int internal_index(int a, int node, int periodic, int n) {
  return (node && periodic) ? (a + 1) % n : a;
}

// The 99 stencil values at evaluation point (i, j) (moment, then b, then a)
// and the two material inputs.
template <typename T, typename C>
__device__ __forceinline__ void stencil_value(const T* __restrict__ U, const ClosureGeo& G, int p, int i, int j,
                                              int a, int b, C* out) {
  const int ii = min(max(i + a, 0), G.pnx[p] - 1);
  const int jj = min(max(j + b, 0), G.pny[p] - 1);
  const int X = internal_index(ii, G.nodex[p], G.px, G.nx);
  const int Y = internal_index(jj, G.nodey[p], G.py, G.ny);
  *out = to_c(U[int64_t(G.k[p]) * G.plane_stride + int64_t(Y) * G.pitch + X]);
}

template <typename C>
__device__ __forceinline__ void sigma_inputs(const C* __restrict__ decay, const ClosureGeo& G, int i, int j, C* fa,
                                             C* fs) {
  const int ci = min(i, G.nx - 1), cj = min(j, G.ny - 1);
  const int64_t o = int64_t(cj) * G.pitch + ci;
  const C sa = decay[int64_t(G.dk_a) * G.plane_stride + o];
  const C st = decay[int64_t(G.dk_t) * G.plane_stride + o];
  *fa = log10(sa + C(0.01));
  *fs = log10((st - sa) + C(0.01));
}

// Training samples from a state of order >= 6: inputs (count x 128, FP32) and
// targets F_k dx / nu (count x 6) at cells (i, j).  targ may be null (inputs
// only); nu_out, if not null, receives nu per sample.
//
// One wave per sample: the lanes gather the 99 stencil values side by side, all
// add their squares in order from LDS (a sum split over lanes would round
// otherwise), and write the row of inputs together.  Latency bounds it; one
// thread per sample walked 198 loads and 128 strided stores one after another:
// 79 us for 512 samples of a P_31 state, now 7.6.
constexpr int kStencil = 9 * CLOSURE_PLANES;
template <typename T>
__global__ void __launch_bounds__(256) closure_samples_kernel(const T* __restrict__ U,
                                                              const typename ComputeOf<T>::type* __restrict__ decay,
                                                              const ClosureGeo G, const int* __restrict__ pts,
                                                              int count, float* __restrict__ feat,
                                                              float* __restrict__ targ, float* __restrict__ nu_out) {
  using C = typename ComputeOf<T>::type;
  __shared__ C stencils[4][kStencil];
  const int lane = int(threadIdx.x) & 63, w = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  const int s = int(blockIdx.x) * 4 + w;
  if (s >= count) return;
  C* const st = stencils[w];
  const int i = pts[2 * s], j = pts[2 * s + 1];
  C v[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int q = min(lane + 64 * h, kStencil - 1);  // moment, then b, then a
    stencil_value(U, G, q / 9, i, j, q % 3 - 1, q / 3 % 3 - 1, &v[h]);
  }
  C fa, fs;
  sigma_inputs(decay, G, i, j, &fa, &fs);
#pragma unroll
  for (int h = 0; h < 2; ++h)
    if (lane + 64 * h < kStencil) st[lane + 64 * h] = v[h];
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  C ss = C(0);
#pragma unroll 33
  for (int q = 0; q < kStencil; ++q) ss += st[q] * st[q];
  const C nu = sqrt(ss) + C(CLOSURE_EPS);
  float* const f = feat + int64_t(s) * CLOSURE_IN;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int q = lane + 64 * h;
    f[q] = q < kStencil ? float(v[h] / nu) : q == kStencil ? float(fa) : q == kStencil + 1 ? float(fs) : 0.f;
  }
  if (nu_out && lane == 0) nu_out[s] = float(nu);
  if (!targ || lane >= CLOSURE_OUT) return;
  // targets, one lane each: the order-6 part of the odd residual at the order-5 points
  const int o = lane;
  const int X = internal_index(i, G.out_nodex[o], G.px, G.nx);
  const int Y = internal_index(j, G.out_nodey[o], G.py, G.ny);
  C d[4], m[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const ClosureTerm ct = G.term[o][min(t, max(G.nterm[o] - 1, 0))];
    const T* up = U + int64_t(ct.k) * G.plane_stride;
    // the input shares the output's index along the other axis
    const bool alongx = ct.axis == 0;
    const int z = alongx ? X : Y, n = alongx ? G.nx : G.ny, per = alongx ? G.px : G.py;
    const int lo = ct.cell ? map_axis(z - 1, n, per, 1) : map_axis(z, n, per, 0);
    const int hi = ct.cell ? map_axis(z, n, per, 1) : map_axis(z + 1, n, per, 0);
    const int64_t row = int64_t(Y) * G.pitch;
    d[t] = (to_c(up[alongx ? row + hi : int64_t(hi) * G.pitch + X]) -
            to_c(up[alongx ? row + lo : int64_t(lo) * G.pitch + X])) / C(alongx ? G.dx : G.dy);
    m[t] = C(ct.m);
  }
  C F = C(0);
#pragma unroll
  for (int t = 0; t < 4; ++t)
    if (t < G.nterm[o]) F -= m[t] * d[t];
  targ[int64_t(s) * CLOSURE_OUT + o] = float(F * C(G.dx) / nu);
}

// ------------------------------------------------------------ closure network
// The closure terms g = nu y / dx of every evaluation point of the
// (nx + 1) x (ny + 1) index domain, into the closure planes of the order-5
// moments (which the odd sweep then reads like source planes).
//
// One workgroup of 16 waves per compute unit keeps the network in LDS; every
// wave takes blocks of 16 points through all of it by itself: gather and
// normalise the inputs, three layers of MFMA products, the outputs.  The layers
// are computed transposed, H^T = W X^T: the weights are the A operand, the
// activations the B operand, read from the wave's own LDS rows [point][unit],
// and each lane's four outputs (consecutive units of one point) go back there
// with one 8-byte write.  Once the weights are staged no wave waits for
// another, and the stencil's values stay in registers between the sum of their
// squares and their normalisation.
//
// What bounds it: the GELUs' vector instructions, 256 per point of some 18
// instructions and two transcendentals, 7200 of the 9300 cycles that a block
// takes of its SIMD when there are many (15.5 us per 4096 blocks); launching,
// staging and the first gather take 5 us more.  At 257^2 points, FP32, 23 us,
// where blocks of 64 points by four waves with the weights in registers, a
// barrier between the layers and three workgroups per compute unit took 32: two
// rounds of blocks where 1.3 were needed, each wave waiting for the slowest.
// BF16 23 us (was 32), FP64 32 (39); 12 instances of that size in one launch, FP32
// 196 us (263), BF16 197 (264), FP64 265 (327).
//
// BATCH: every running instance of a batch of closure solvers sharing one
// network; instance i (of the n_active still running) owns the blocks of CB
// points [bfirst[i], bfirst[i + 1]) and brings its own state and geometry
// (insts[i]); the arguments U0, decay0 and G0 are unused.
constexpr int CB = 64;               // evaluation points per block of the fused kernel and of batches' tables
constexpr int LDW = CLOSURE_IN + 8;  // LDS row of one point's activations or one unit's weights (bf16), padded
constexpr int NW = 16;               // waves per workgroup
constexpr int NPT = 16;              // points per wave
constexpr int NROWS = 2 * CLOSURE_HIDDEN + 16;  // weight rows: W1, W2, W3 (padded to 16)
constexpr size_t kNetLds = size_t(NROWS + NW * NPT) * LDW * 2 + size_t(2 * CLOSURE_HIDDEN + 16) * 4 + NW * 40 * 4;

// A pointer read from a table, as one to global memory.
template <typename T>
__device__ __forceinline__ T* in_global(T* p) {
  return (T*)(__attribute__((address_space(1))) T*)p;
}

template <typename T, bool BATCH>
__global__ void __launch_bounds__(64 * NW) closure_net_kernel(T* __restrict__ U0,
                                                              const typename ComputeOf<T>::type* __restrict__ decay0,
                                                              const ClosureGeo G0, const ClosureNet* __restrict__ net,
                                                              const ClosureInst* __restrict__ insts,
                                                              const int* __restrict__ bfirst, const int n_active) {
  using C = typename ComputeOf<T>::type;
  extern __shared__ __align__(16) unsigned char smem[];
  uint16_t* const Ws = reinterpret_cast<uint16_t*>(smem);  // [NROWS][LDW]
  float* const bias = reinterpret_cast<float*>(Ws + NROWS * LDW);  // b1, b2, b3
  const int tid = int(threadIdx.x), lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pt = lane & 15, grp = lane >> 4, fk = 8 * grp;
  uint16_t* const X = reinterpret_cast<uint16_t*>(bias + 2 * CLOSURE_HIDDEN + 16) + w * NPT * LDW;  // this wave's rows
  int* const otab =  // this wave's output geometry: plane, extents, nodal flags by output
      reinterpret_cast<int*>(reinterpret_cast<uint16_t*>(bias + 2 * CLOSURE_HIDDEN + 16) + NW * NPT * LDW) + w * 40;

  {
    const uint4* wv = reinterpret_cast<const uint4*>(net->w);  // rows of CLOSURE_IN / 8
    constexpr int Q = CLOSURE_IN / 8;
    for (int e = tid; e < NROWS * Q; e += 64 * NW)
      *reinterpret_cast<uint4*>(&Ws[(e / Q) * LDW + (e % Q) * 8]) = wv[e];
    for (int e = tid; e < 2 * CLOSURE_HIDDEN + 16; e += 64 * NW)
      bias[e] = e < CLOSURE_HIDDEN       ? net->b1[e]
                : e < 2 * CLOSURE_HIDDEN ? net->b2[e - CLOSURE_HIDDEN]
                                         : net->b3[e - 2 * CLOSURE_HIDDEN];
  }
  bool staged = false;

  // this workgroup's blocks of 16 points, round robin over its waves
  constexpr int SUB = CB / NPT;
  const int total0 = (G0.nx + 1) * (G0.ny + 1);
  const int nblk = BATCH ? SUB * bfirst[n_active] : (total0 + NPT - 1) / NPT;
  const int first = int(int64_t(nblk) * blockIdx.x / gridDim.x), last = int(int64_t(nblk) * (blockIdx.x + 1) / gridDim.x);
  int inst_now = -1;
  int kin[3], node[3];  // this lane's input moments: plane, nodal flags (1: x, 2: y)
  for (int gblk = first + w; gblk < last; gblk += NW) {
    int inst = 0;
    if constexpr (BATCH) {
      int lo = 0, hi = n_active - 1;  // last instance with bfirst[i] <= gblk / SUB
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (bfirst[mid] <= gblk / SUB) lo = mid; else hi = mid - 1;
      }
      inst = __builtin_amdgcn_readfirstlane(lo);
    }
    const int blk = BATCH ? gblk - SUB * bfirst[inst] : gblk;
    const ClosureGeo& G = BATCH ? insts[inst].G : G0;
    T* const U = BATCH ? in_global(static_cast<T*>(insts[inst].u)) : U0;
    const C* const decay = BATCH ? in_global(static_cast<const C*>(insts[inst].decay)) : decay0;
    if (inst != inst_now) {
      // (indexed per lane: dependent loads, once per instance).  Lane group g
      // has moments g, g + 4, g + 8; the twelfth does not exist: group 3 reads
      // the fourth again, uncounted.
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        const int p = grp + 4 * t < CLOSURE_PLANES ? grp + 4 * t : 3;
        kin[t] = G.k[p];
        node[t] = (G.nodex[p] ? 1 : 0) | (G.nodey[p] ? 2 : 0);
      }
      if (lane < 40) {
        const int f = lane >> 3, o = lane & 7;
        int v = 0;
        if (o < CLOSURE_OUT)
          v = f == 0 ? G.q[o] : f == 1 ? G.out_nx[o] : f == 2 ? G.out_ny[o] : f == 3 ? G.out_nodex[o] : G.out_nodey[o];
        otab[lane] = v;
      }
      inst_now = inst;
    }
    const int NXE = G.nx + 1, total = NXE * (G.ny + 1);
    // 1. inputs: lane group g gathers moments g, g + 4, g + 8 of point pt
    // (group 3: two moments and the material inputs)
    const int p0 = blk * NPT + pt;
    const bool live = p0 < total;
    const int i = live ? p0 % NXE : 0, j = live ? p0 / NXE : 0;
    // clamped (or wrapped) columns and rows of the stencil, per axis class:
    // [0] cell-centred, [1] nodal
    int colx[2][3], rowy[2][3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      colx[0][a] = min(max(i + a - 1, 0), G.nx - 1);
      const int xn = min(max(i + a - 1, 0), G.nx - G.px);
      colx[1][a] = G.px ? (xn + 1 == G.nx ? 0 : xn + 1) : xn;
      rowy[0][a] = min(max(j + a - 1, 0), G.ny - 1) * G.pitch;
      const int yn = min(max(j + a - 1, 0), G.ny - G.py);
      rowy[1][a] = (G.py ? (yn + 1 == G.ny ? 0 : yn + 1) : yn) * G.pitch;
    }
    C v[3][9];
    C ss = C(0);
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      const T* up = U + int64_t(kin[t]) * G.plane_stride;
      int cx[3], ry[3];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        cx[a] = node[t] & 1 ? colx[1][a] : colx[0][a];
        ry[a] = node[t] & 2 ? rowy[1][a] : rowy[0][a];
      }
#pragma unroll
      for (int q = 0; q < 9; ++q) v[t][q] = to_c(up[ry[q / 3] + cx[q % 3]]);
    }
    C sig_a = C(0), sig_t = C(0);
    if (grp == 3) {
      const int64_t o = int64_t(min(j, G.ny - 1)) * G.pitch + min(i, G.nx - 1);
      sig_a = decay[int64_t(G.dk_a) * G.plane_stride + o];
      sig_t = decay[int64_t(G.dk_t) * G.plane_stride + o];
    }
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int q = 0; q < 9; ++q)
        if (t < 2 || grp < 3) ss += v[t][q] * v[t][q];
    const C nu = sqrt(((__shfl(ss, pt) + __shfl(ss, 16 + pt)) + __shfl(ss, 32 + pt)) + __shfl(ss, 48 + pt)) + C(CLOSURE_EPS);
    const C rnu = C(1) / nu;
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int q = 0; q < 9; ++q)
        if (t < 2 || grp < 3) X[pt * LDW + 9 * (grp + 4 * t) + q] = uint16_t(bf16_in(v[t][q] * rnu));
    if (grp == 3) {
      const C fa = log10(sig_a + C(0.01)), fs = log10((sig_t - sig_a) + C(0.01));
      X[pt * LDW + 99] = uint16_t(bf16_bits(fa));
      X[pt * LDW + 100] = uint16_t(bf16_bits(fs));
      X[pt * LDW + 101] = 0;
#pragma unroll
      for (int q = 102; q < CLOSURE_IN; q += 2) *reinterpret_cast<uint32_t*>(&X[pt * LDW + q]) = 0;
    }
    if (!staged) {
      __syncthreads();  // the weights are in LDS
      staged = true;
    }
    // (a wave's LDS accesses keep their order; the fences keep the compiler's)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");

    // 2. hidden layers: H^T (units x points) = W X^T, in place in the wave's rows
#pragma unroll
    for (int layer = 0; layer < 2; ++layer) {
      uint4 xf[4];
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) xf[ks] = *reinterpret_cast<const uint4*>(&X[pt * LDW + 32 * ks + fk]);
#pragma unroll sizeof(C) == 8 ? 4 : 8
      for (int mi = 0; mi < CLOSURE_HIDDEN / 16; ++mi) {
        f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
          acc = mfma16(*reinterpret_cast<const uint4*>(&Ws[(layer * CLOSURE_HIDDEN + 16 * mi + pt) * LDW + 32 * ks + fk]),
                       xf[ks], acc);
        // rows: units 16 mi + 4 grp + r; column: point pt
        const int n = 16 * mi + 4 * grp;
        const float4 bv = *reinterpret_cast<const float4*>(&bias[layer * CLOSURE_HIDDEN + n]);
        *reinterpret_cast<uint2*>(&X[pt * LDW + n]) =
            make_uint2(bf16_hw2(gelu(acc[0] + bv.x), gelu(acc[1] + bv.y)),
                       bf16_hw2(gelu(acc[2] + bv.z), gelu(acc[3] + bv.w)));
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }

    // 3. output layer: Y^T (16 x points) = W3 X^T
    f32x4 y = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
      y = mfma16(*reinterpret_cast<const uint4*>(&Ws[(2 * CLOSURE_HIDDEN + pt) * LDW + 32 * ks + fk]),
                 *reinterpret_cast<const uint4*>(&X[pt * LDW + 32 * ks + fk]), y);
    if (live && grp < 2) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int o = 4 * grp + r;  // output of this lane
        if (o >= CLOSURE_OUT || i >= otab[8 + o] || j >= otab[16 + o]) continue;
        const int xo = internal_index(i, otab[24 + o], G.px, G.nx);
        const int yo = internal_index(j, otab[32 + o], G.py, G.ny);
        const C g = nu * C(y[r] + bias[2 * CLOSURE_HIDDEN + o]) / C(G.dx);
        U[int64_t(otab[o]) * G.plane_stride + int64_t(yo) * G.pitch + xo] = from_c<T>(g);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
  if (!staged) __syncthreads();
}

// ------------------------------------------------------------ fused closure
// The network and the odd sweep of P_5 in one kernel.  Every workgroup loops
// over blocks of 64 evaluation points: gather and normalise the inputs, three
// MFMA layers, then the odd update of the block's points.  The layers are
// computed transposed as in the kernel above, but the weights stay in registers
// (wave w owns hidden units [32 w, 32 w + 32)) and the activations go through
// LDS as [point][unit] rows.

// The odd update of one odd moment of P_5 at the internal point (X, Y) of its
// grid, with the couplings in the order of the sweep kernel (x terms, then y
// terms), the source, then the closure term g: u + tau (W - c u) E(-c tau).
template <typename T, typename C>
__device__ __forceinline__ C closure_odd_update(const T* __restrict__ U, const ClosureOddRow& r, const ClosureGeo& G,
                                                int X, int Y, C u, C g, C c, C E, C tau) {
  // plane bases are wave-uniform; the lane's offsets are 32-bit byte offsets
  // within a plane (planes stay below 2^31 bytes), so every load takes a
  // scalar base and one offset register
  const uint64_t ps = uint64_t(G.plane_stride);
  constexpr uint32_t TS = sizeof(T);
  const char* base = reinterpret_cast<const char*>(U);
  auto val = [&](int k, uint32_t off) {
    return to_c(*reinterpret_cast<const T*>(base + uint64_t(uint32_t(k)) * ps * TS + off));
  };
  const uint32_t row = uint32_t(Y) * uint32_t(G.pitch);
  C W = C(0);
  for (int t = 0; t < r.nx; ++t) {
    const int lo = r.xcell[t] ? map_axis(X - 1, G.nx, G.px, 1) : map_axis(X, G.nx, G.px, 0);
    const int hi = r.xcell[t] ? map_axis(X, G.nx, G.px, 1) : map_axis(X + 1, G.nx, G.px, 0);
    W = couple(W, C(r.xc[t]), val(r.xk[t], (row + uint32_t(hi)) * TS), val(r.xk[t], (row + uint32_t(lo)) * TS));
  }
  for (int t = 0; t < r.ny; ++t) {
    const int lo = r.ycell[t] ? map_axis(Y - 1, G.ny, G.py, 1) : map_axis(Y, G.ny, G.py, 0);
    const int hi = r.ycell[t] ? map_axis(Y, G.ny, G.py, 1) : map_axis(Y + 1, G.ny, G.py, 0);
    W = couple(W, C(r.yc[t]), val(r.yk[t], (uint32_t(hi) * uint32_t(G.pitch) + uint32_t(X)) * TS),
               val(r.yk[t], (uint32_t(lo) * uint32_t(G.pitch) + uint32_t(X)) * TS));
  }
  if (r.src >= 0) W += val(r.src, (row + uint32_t(X)) * TS);
  if (r.o >= 0) W += g;
  return sub_step(u, W, c, E, tau);
}

// The network, then the odd sweep at the block's points in the same workgroup
// (every odd moment at every evaluation point that lies on its grid), the
// order-5 moments read from in5 and written to out5 (out of place, so every
// workgroup's stencils see the state of the start of the sweep), orders 1 and 3
// in place (nothing else reads them).
//
// BATCH = true: odd sweep number j of a batched run of closure solvers
// sharing one network; instance i (of the n_active still running, sorted by
// their sweep counts) owns the evaluation blocks [bfirst[i], bfirst[i + 1])
// and brings its own state, geometry and odd rows (insts[i]); the arguments
// U0 .. odd0 are unused.
template <typename T, bool BATCH>
__global__ void __launch_bounds__(256, 3) closure_infer_kernel(T* __restrict__ U0, const T* __restrict__ in5_0,
                                                            T* __restrict__ out5_0,
                                                            const typename ComputeOf<T>::type* __restrict__ decay0,
                                                            const ClosureGeo G0, const ClosureNet* __restrict__ net,
                                                            const ClosureOdd odd0,
                                                            const ClosureInst* __restrict__ insts,
                                                            const int* __restrict__ bfirst, const int n_active,
                                                            const int jsweep) {
  using C = typename ComputeOf<T>::type;
  extern __shared__ __align__(16) unsigned char smem[];
  uint16_t* Xa = reinterpret_cast<uint16_t*>(smem);  // [64][LDW] inputs, then layer-2 activations
  uint16_t* Xb = Xa + CB * LDW;                      // [64][LDW] layer-1 activations
  uint16_t* W3 = Xb + CB * LDW;                      // [16][LDW] output layer, rows >= 6 zero
  C* nu_s = reinterpret_cast<C*>(W3 + 16 * LDW);     // [64]
  C* part = nu_s + CB;                                    // [4][64] partial sums of squares per wave
  C* gsh = part + 4 * CB;                                 // [6][64] closure terms of the block
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int fk = 8 * (lane >> 4);

  // this wave's weight fragments: rows 32 w + 16 mi + (lane % 16), k = 32 ks + fk
  const uint4* wv = reinterpret_cast<const uint4*>(net->w);  // rows of CLOSURE_IN / 8 uint4
  uint4 wf[2][2][4];
#pragma unroll
  for (int layer = 0; layer < 2; ++layer)
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const int row = layer * CLOSURE_HIDDEN + 32 * w + 16 * mi + (lane & 15);
        wf[layer][mi][ks] = wv[row * (CLOSURE_IN / 8) + (32 * ks + fk) / 8];
      }
  for (int e = tid; e < 16 * (CLOSURE_IN / 8); e += 256)
    *reinterpret_cast<uint4*>(&W3[(e / (CLOSURE_IN / 8)) * LDW + (e % (CLOSURE_IN / 8)) * 8]) =
        wv[2 * CLOSURE_HIDDEN * (CLOSURE_IN / 8) + e];
  float b3[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) b3[r] = net->b3[4 * (lane >> 4) + r];

  const int nblk = BATCH ? bfirst[n_active] : ((G0.nx + 1) * (G0.ny + 1) + CB - 1) / CB;
  for (int gblk = blockIdx.x; gblk < nblk; gblk += gridDim.x) {
    // this block's instance (batched runs) and its data
    int inst = 0;
    if constexpr (BATCH) {
      int lo = 0, hi = n_active - 1;  // last instance with bfirst[i] <= gblk
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (bfirst[mid] <= gblk) lo = mid; else hi = mid - 1;
      }
      inst = lo;
    }
    const int blk = BATCH ? gblk - bfirst[inst] : gblk;
    const ClosureGeo& G = BATCH ? insts[inst].G : G0;
    const ClosureOdd& odd = BATCH ? insts[inst].odd : odd0;
    T* const U = BATCH ? static_cast<T*>(insts[inst].u) : U0;
    const C* const decay = BATCH ? static_cast<const C*>(insts[inst].decay) : decay0;
    // the order-5 moments move between the state planes and the closure planes
    // at every odd sweep, and odd sweep j of a batched run reads them where
    // j / 2 earlier odd sweeps left them
    const bool flip = BATCH && ((jsweep >> 1) & 1);
    const T* const in5 = BATCH ? static_cast<const T*>(flip ? insts[inst].b5 : insts[inst].a5) : in5_0;
    T* const out5 = BATCH ? static_cast<T*>(flip ? insts[inst].a5 : insts[inst].b5) : out5_0;
    const C tau = BATCH ? C((jsweep == 0 || jsweep == insts[inst].nsweeps - 1) ? insts[inst].tau_half
                                                                             : insts[inst].tau_full)
                        : C(odd0.tau);
    const int NXE = G.nx + 1, total = NXE * (G.ny + 1);
    // 1. inputs: wave w gathers moments w, w + 4, w + 8 of point lane
    const int pt = blk * CB + lane;
    const bool live = pt < total;
    const int i = live ? pt % NXE : 0, j = live ? pt / NXE : 0;
    // clamped (or wrapped) columns and rows of the stencil, per axis class:
    // [0] cell-centred, [1] nodal
    int colx[2][3], rowy[2][3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      colx[0][a] = min(max(i + a - 1, 0), G.nx - 1);
      const int xn = min(max(i + a - 1, 0), G.nx - G.px);
      colx[1][a] = G.px ? (xn + 1 == G.nx ? 0 : xn + 1) : xn;
      rowy[0][a] = min(max(j + a - 1, 0), G.ny - 1) * G.pitch;
      const int yn = min(max(j + a - 1, 0), G.ny - G.py);
      rowy[1][a] = (G.py ? (yn + 1 == G.ny ? 0 : yn + 1) : yn) * G.pitch;
    }
    // the material inputs of this point (wave 3), loaded now so that they
    // arrive with the stencil
    C sig_a = C(0), sig_t = C(0);
    if (w == 3) {
      const int64_t o = int64_t(min(j, G.ny - 1)) * G.pitch + min(i, G.nx - 1);
      sig_a = decay[int64_t(G.dk_a) * G.plane_stride + o];
      sig_t = decay[int64_t(G.dk_t) * G.plane_stride + o];
    }
    // two passes over the stencil (the second re-reads cached values): the
    // sum of squares, then the normalised inputs
    C ss = C(0);
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      const int p = w + 4 * t;
      if (p < CLOSURE_PLANES) {
        const T* up = p < 5 ? U + int64_t(G.k[p]) * G.plane_stride : in5 + int64_t(p - 5) * G.plane_stride;
        const int cx = G.nodex[p], cy = G.nodey[p];
#pragma unroll
        for (int q = 0; q < 9; ++q) {
          const C v = to_c(up[rowy[cy][q / 3] + colx[cx][q % 3]]);
          ss += v * v;
        }
      }
    }
    // the second pass's first plane (every wave has one) is re-read while the
    // norm is reduced across the waves
    C v0[9];
    {
      const T* up = U + int64_t(G.k[w]) * G.plane_stride;  // w < 4: an order-4 plane
      const int cx = G.nodex[w], cy = G.nodey[w];
#pragma unroll
      for (int q = 0; q < 9; ++q) v0[q] = to_c(up[rowy[cy][q / 3] + colx[cx][q % 3]]);
    }
    __syncthreads();  // the previous block's reads of Xa, nu_s and part are done
    part[w * CB + lane] = ss;
    __syncthreads();
    const C nu = sqrt(((part[lane] + part[CB + lane]) + part[2 * CB + lane]) + part[3 * CB + lane]) + C(CLOSURE_EPS);
    const C rnu = C(1) / nu;
#pragma unroll
    for (int q = 0; q < 9; ++q) Xa[lane * LDW + 9 * w + q] = uint16_t(bf16_in(v0[q] * rnu));
#pragma unroll
    for (int t = 1; t < 3; ++t) {
      const int p = w + 4 * t;
      if (p < CLOSURE_PLANES) {
        const T* up = p < 5 ? U + int64_t(G.k[p]) * G.plane_stride : in5 + int64_t(p - 5) * G.plane_stride;
        const int cx = G.nodex[p], cy = G.nodey[p];
        // all nine loads first, so they are in flight together
        C v[9];
#pragma unroll
        for (int q = 0; q < 9; ++q) v[q] = to_c(up[rowy[cy][q / 3] + colx[cx][q % 3]]);
#pragma unroll
        for (int q = 0; q < 9; ++q) Xa[lane * LDW + 9 * p + q] = uint16_t(bf16_in(v[q] * rnu));
      }
    }
    if (w == 3) {
      const C fa = log10(sig_a + C(0.01)), fs = log10((sig_t - sig_a) + C(0.01));
      Xa[lane * LDW + 99] = uint16_t(bf16_bits(fa));
      Xa[lane * LDW + 100] = uint16_t(bf16_bits(fs));
      for (int q = 101; q < CLOSURE_IN; ++q) Xa[lane * LDW + q] = 0;
      nu_s[lane] = nu;
    }
    __syncthreads();

    // 2. hidden layers: H^T (units x points) = W X^T; wave w: 32 units x 64 points
#pragma unroll
    for (int layer = 0; layer < 2; ++layer) {
      const uint16_t* Xin = layer == 0 ? Xa : Xb;
      uint16_t* Xout = layer == 0 ? Xb : Xa;
      f32x4 acc[2][4];
#pragma unroll
      for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int nj = 0; nj < 4; ++nj) acc[mi][nj] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
        for (int nj = 0; nj < 4; ++nj) {
          const uint4 xf = *reinterpret_cast<const uint4*>(&Xin[(16 * nj + (lane & 15)) * LDW + 32 * ks + fk]);
#pragma unroll
          for (int mi = 0; mi < 2; ++mi) acc[mi][nj] = mfma16(wf[layer][mi][ks], xf, acc[mi][nj]);
        }
      }
#pragma unroll
      for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int nj = 0; nj < 4; ++nj) {
          // rows: units 32 w + 16 mi + 4 (lane / 16) + r; column: point 16 nj + lane % 16
          const float4 bv = *reinterpret_cast<const float4*>((layer == 0 ? net->b1 : net->b2) + 32 * w + 16 * mi +
                                                             4 * (lane >> 4));
          const uint32_t h01 = bf16_hw2(gelu(acc[mi][nj][0] + bv.x), gelu(acc[mi][nj][1] + bv.y));
          const uint32_t h23 = bf16_hw2(gelu(acc[mi][nj][2] + bv.z), gelu(acc[mi][nj][3] + bv.w));
          const int m = 16 * nj + (lane & 15);
          const int n = 32 * w + 16 * mi + 4 * (lane >> 4);
          *reinterpret_cast<uint2*>(&Xout[m * LDW + n]) = make_uint2(h01, h23);
        }
      __syncthreads();
    }

    // 3. output layer: Y^T (16 x points) = W3 X^T; wave w takes points [16 w, 16 w + 16)
    f32x4 y = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const uint4 af = *reinterpret_cast<const uint4*>(&W3[(lane & 15) * LDW + 32 * ks + fk]);
      const uint4 xf = *reinterpret_cast<const uint4*>(&Xa[(16 * w + (lane & 15)) * LDW + 32 * ks + fk]);
      y = mfma16(af, xf, y);
    }
    const int m = 16 * w + (lane & 15);  // point of this lane
    // 4. the closure terms of the block into LDS, then the odd update:
    // wave w takes odd rows w, w + 4, w + 8, lane = point of the block
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int o = 4 * (lane >> 4) + r;
      if (o < CLOSURE_OUT) gsh[o * CB + m] = nu_s[m] * C(y[r] + b3[r]) / C(G.dx);
    }
    __syncthreads();
    if (pt < total) {  // the point of this lane: (i, j) of the gather above
      // decay and E(-c tau) per output grid, reloaded when a row's decay plane differs
      int dk21 = -1, dk12 = -1;
      C c21 = C(0), e21 = C(0), c12 = C(0), e12 = C(0);
      const int w0 = __builtin_amdgcn_readfirstlane(w);
      for (int q = w0; q < CLOSURE_ODD_ROWS; q += 4) {
        const ClosureOddRow& r = odd.r[q];
        const int nd = r.node_x;
        // the row's grid: G21 has nx + 1 - px by ny points, G12 nx by ny + 1 - py
        if (nd ? (i >= G.nx + 1 - G.px || j >= G.ny) : (i >= G.nx || j >= G.ny + 1 - G.py)) continue;
        const int X = nd ? internal_index(i, 1, G.px, G.nx) : i;
        const int Y = nd ? j : internal_index(j, 1, G.py, G.ny);
        const int64_t off = int64_t(Y) * G.pitch + X;
        if (nd && r.dk != dk21) {
          c21 = decay[int64_t(r.dk) * G.plane_stride + off];
          e21 = expm1div(-c21 * tau);
          dk21 = r.dk;
        } else if (!nd && r.dk != dk12) {
          c12 = decay[int64_t(r.dk) * G.plane_stride + off];
          e12 = expm1div(-c12 * tau);
          dk12 = r.dk;
        }
        const T* src = r.o >= 0 ? in5 + int64_t(r.o) * G.plane_stride : U + int64_t(r.k) * G.plane_stride;
        const C u = to_c(src[off]);
        const C g = r.o >= 0 ? gsh[r.o * CB + lane] : C(0);
        const C v = closure_odd_update(U, r, G, X, Y, u, g, nd ? c21 : c12, nd ? e21 : e12, tau);
        T* dst = r.o >= 0 ? out5 + int64_t(r.o) * G.plane_stride : U + int64_t(r.k) * G.plane_stride;
        dst[off] = from_c<T>(v);
      }
    }
  }
}

// ------------------------------------------------------------ launches
namespace {
int device_cus() {
  static int cus = 0;
  if (!cus) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
      cus = 256;
  }
  return cus;
}
}  // namespace

int mlp_row_blocks(int B) { return std::min((B + TR - 1) / TR, 2 * device_cus()); }
int mlp_sum_chunks(int B) { return (B + CS_ROWS - 1) / CS_ROWS; }

hipError_t launch_mlp_rows(const MlpRows& g, bool train, hipStream_t stream) {
  if (g.B < 1) return hipErrorInvalidValue;
  const dim3 grid(mlp_row_blocks(g.B));
  if (train)
    hipLaunchKernelGGL(mlp_rows_kernel<true>, grid, dim3(256), 0, stream, g);
  else
    hipLaunchKernelGGL(mlp_rows_kernel<false>, grid, dim3(256), 0, stream, g);
  return hipGetLastError();
}

hipError_t launch_mlp_grad(const MlpGrad& g, hipStream_t stream) {
  if (g.B < 1 || g.splits < 1 || g.kchunk < KT || g.kchunk % KT) return hipErrorInvalidValue;
  const int64_t blocks = int64_t(g.splits) * GRAD_TILES + int64_t(mlp_sum_chunks(g.B)) * SUM_TILES;
  hipLaunchKernelGGL(mlp_grad_kernel, dim3(unsigned(blocks)), dim3(256), 0, stream, g);
  return hipGetLastError();
}

hipError_t launch_mlp_update(const MlpGrad& g, float* grads, const MlpAdam& a, const double* lpart, double* loss,
                             hipStream_t stream) {
  const int blocks = (CLOSURE_PARAMS + 255) / 256 + 1;
  hipLaunchKernelGGL(mlp_update_kernel, dim3(blocks), dim3(256), 0, stream, g, grads, a, lpart, mlp_row_blocks(g.B),
                     loss);
  return hipGetLastError();
}

hipError_t launch_adam(const MlpAdam& a, const float* grads, hipStream_t stream) {
  hipLaunchKernelGGL(adam_kernel, dim3((CLOSURE_PARAMS + 255) / 256), dim3(256), 0, stream, a, grads);
  return hipGetLastError();
}

hipError_t launch_closure_samples(int storage, const void* U, const void* decay, const ClosureGeo& G,
                                  const int* pts, int count, float* feat, float* targ, float* nu, hipStream_t stream) {
  const dim3 grid((unsigned(count) + 3) / 4);  // a wave per sample
  switch (storage) {
    case STORE_FP64:
      hipLaunchKernelGGL(closure_samples_kernel<double>, grid, dim3(256), 0, stream,
                         static_cast<const double*>(U), static_cast<const double*>(decay), G, pts, count, feat, targ, nu);
      break;
    case STORE_FP32:
      hipLaunchKernelGGL(closure_samples_kernel<float>, grid, dim3(256), 0, stream,
                         static_cast<const float*>(U), static_cast<const float*>(decay), G, pts, count, feat, targ, nu);
      break;
    case STORE_BF16:
      hipLaunchKernelGGL(closure_samples_kernel<bf16>, grid, dim3(256), 0, stream,
                         static_cast<const bf16*>(U), static_cast<const float*>(decay), G, pts, count, feat, targ, nu);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

size_t closure_infer_lds_bytes() {
  return size_t(2 * CB + 16) * LDW * 2 + size_t(5 * CB) * 8 + size_t(CLOSURE_OUT * CB) * 8;
}

namespace {
// Opts a kernel in to its LDS, once on every device (devices past 64: each time).
template <auto kernel>
hipError_t opt_in_lds(size_t lds) {
  static std::atomic<uint64_t> done{0};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = dev >= 0 && dev < 64 ? uint64_t(1) << dev : 0;
  if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
  e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
  if (e == hipSuccess) done.fetch_or(bit, std::memory_order_release);
  return e;
}

template <typename T, bool BATCH>
hipError_t launch_infer_t(void* U, const void* in5, void* out5, const void* decay, const ClosureGeo& G,
                          const ClosureNet* net, const ClosureOdd& odd, const ClosureInst* insts, const int* bfirst,
                          int n_active, int j, int nblk, hipStream_t stream) {
  using C = typename ComputeOf<T>::type;
  const size_t lds = closure_infer_lds_bytes();
  const hipError_t e = opt_in_lds<&closure_infer_kernel<T, BATCH>>(lds);
  if (e != hipSuccess) return e;
  // a few workgroups per compute unit, each looping over blocks of points with
  // the weights loaded once
  const int grid = std::min(nblk, 3 * device_cus());
  hipLaunchKernelGGL((closure_infer_kernel<T, BATCH>), dim3(grid), dim3(256), lds, stream, static_cast<T*>(U),
                     static_cast<const T*>(in5), static_cast<T*>(out5), static_cast<const C*>(decay), G, net, odd,
                     insts, bfirst, n_active, j);
  return hipGetLastError();
}

template <typename T, bool BATCH>
hipError_t launch_net_t(void* U, const void* decay, const ClosureGeo& G, const ClosureNet* net,
                        const ClosureInst* insts, const int* bfirst, int n_active, int nblk, hipStream_t stream) {
  using C = typename ComputeOf<T>::type;
  const hipError_t e = opt_in_lds<&closure_net_kernel<T, BATCH>>(kNetLds);
  if (e != hipSuccess) return e;
  const int grid = std::min(nblk, device_cus());  // one workgroup per compute unit
  hipLaunchKernelGGL((closure_net_kernel<T, BATCH>), dim3(grid), dim3(64 * NW), kNetLds, stream, static_cast<T*>(U),
                     static_cast<const C*>(decay), G, net, insts, bfirst, n_active);
  return hipGetLastError();
}

int points_of(const ClosureGeo& G) { return (G.nx + 1) * (G.ny + 1); }
}  // namespace

hipError_t launch_closure_infer(int storage, void* U, const void* decay, const ClosureGeo& G, const ClosureNet* net,
                                hipStream_t stream) {
  const int nblk = (points_of(G) + NPT - 1) / NPT;
  switch (storage) {
    case STORE_FP64: return launch_net_t<double, false>(U, decay, G, net, nullptr, nullptr, 0, nblk, stream);
    case STORE_FP32: return launch_net_t<float, false>(U, decay, G, net, nullptr, nullptr, 0, nblk, stream);
    case STORE_BF16: return launch_net_t<bf16, false>(U, decay, G, net, nullptr, nullptr, 0, nblk, stream);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_closure_sweep(int storage, void* U, const void* in5, void* out5, const void* decay,
                                const ClosureGeo& G, const ClosureNet* net, const ClosureOdd& odd,
                                hipStream_t stream) {
  const int nblk = (points_of(G) + CB - 1) / CB;
  switch (storage) {
    case STORE_FP64:
      return launch_infer_t<double, false>(U, in5, out5, decay, G, net, odd, nullptr, nullptr, 0, 0, nblk, stream);
    case STORE_FP32:
      return launch_infer_t<float, false>(U, in5, out5, decay, G, net, odd, nullptr, nullptr, 0, 0, nblk, stream);
    case STORE_BF16:
      return launch_infer_t<bf16, false>(U, in5, out5, decay, G, net, odd, nullptr, nullptr, 0, 0, nblk, stream);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_closure_batch_net(int storage, const ClosureInst* insts, const int* bfirst, int n_active, int blocks,
                                    const ClosureNet* net, hipStream_t stream) {
  if (n_active < 1 || blocks < 1) return hipErrorInvalidValue;
  const int nblk = int(std::min<int64_t>(int64_t(blocks) * (CB / NPT), 1 << 30));
  const ClosureGeo G{};
  switch (storage) {
    case STORE_FP64: return launch_net_t<double, true>(nullptr, nullptr, G, net, insts, bfirst, n_active, nblk, stream);
    case STORE_FP32: return launch_net_t<float, true>(nullptr, nullptr, G, net, insts, bfirst, n_active, nblk, stream);
    case STORE_BF16: return launch_net_t<bf16, true>(nullptr, nullptr, G, net, insts, bfirst, n_active, nblk, stream);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_closure_batch(int storage, const ClosureInst* insts, const int* bfirst, int n_active, int blocks,
                                int j, const ClosureNet* net, hipStream_t stream) {
  if (n_active < 1 || blocks < 1) return hipErrorInvalidValue;
  const ClosureGeo G{};
  const ClosureOdd odd{};
  switch (storage) {
    case STORE_FP64:
      return launch_infer_t<double, true>(nullptr, nullptr, nullptr, nullptr, G, net, odd, insts, bfirst, n_active, j,
                                          blocks, stream);
    case STORE_FP32:
      return launch_infer_t<float, true>(nullptr, nullptr, nullptr, nullptr, G, net, odd, insts, bfirst, n_active, j,
                                         blocks, stream);
    case STORE_BF16:
      return launch_infer_t<bf16, true>(nullptr, nullptr, nullptr, nullptr, G, net, odd, insts, bfirst, n_active, j,
                                        blocks, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace starmap
