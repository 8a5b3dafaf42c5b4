// Launch interface of the learned-closure kernels (mlp.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "kernels.hpp"

namespace starmap {

constexpr int CLOSURE_PLANES = 11;   // order-4 and order-5 moments of P_5
constexpr int CLOSURE_FEATURES = 101;  // 99 stencil values + 2 material inputs
constexpr int CLOSURE_IN = 128;       // padded input width
constexpr int CLOSURE_HIDDEN = 128;
constexpr int CLOSURE_OUT = 6;        // order-5 moments
constexpr double CLOSURE_EPS = 1e-20; // added to the stencil norm
// parameters of the FP32 blob: W1 (128 x 128), b1, W2 (128 x 128), b2, W3 (6 x 128), b3
constexpr int CLOSURE_PARAMS = CLOSURE_HIDDEN * CLOSURE_IN + CLOSURE_HIDDEN + CLOSURE_HIDDEN * CLOSURE_HIDDEN +
                               CLOSURE_HIDDEN + CLOSURE_OUT * CLOSURE_HIDDEN + CLOSURE_OUT;

// offsets of its parts
constexpr int OFF_W1 = 0;
constexpr int OFF_B1 = OFF_W1 + CLOSURE_HIDDEN * CLOSURE_IN;
constexpr int OFF_W2 = OFF_B1 + CLOSURE_HIDDEN;
constexpr int OFF_B2 = OFF_W2 + CLOSURE_HIDDEN * CLOSURE_HIDDEN;
constexpr int OFF_W3 = OFF_B2 + CLOSURE_HIDDEN;
constexpr int OFF_B3 = OFF_W3 + CLOSURE_OUT * CLOSURE_HIDDEN;
static_assert(OFF_B3 + CLOSURE_OUT == CLOSURE_PARAMS, "parameter blob layout");

// Network as the closure kernels read it: bfloat16 weight rows of W1, W2 and W3
// (padded to 16 rows of zeros), then FP32 biases (b3 padded to 16).
struct ClosureNet {
  uint16_t w[(2 * CLOSURE_HIDDEN + 16) * CLOSURE_IN];
  float b1[CLOSURE_HIDDEN];
  float b2[CLOSURE_HIDDEN];
  float b3[16];
};

// One order-6 coupling of an order-5 output: -m * D u_k along axis (0 x, 1 y);
// cell = 1 if plane k is cell-centred along that axis.
struct ClosureTerm {
  int k, axis, cell, pad;
  double m;
};

// Geometry of the closure inputs and outputs in a solver's state.
struct ClosureGeo {
  // input moments: plane, public extents, nodal flags per axis
  int k[CLOSURE_PLANES], pnx[CLOSURE_PLANES], pny[CLOSURE_PLANES], nodex[CLOSURE_PLANES], nodey[CLOSURE_PLANES];
  int nx, ny, px, py, pitch;
  int dk_a, dk_t;  // decay planes: sigma_a on G11, sigma_a + sigma_s on G11
  int64_t plane_stride;
  double dx, dy;
  // outputs: closure plane (inference), public extents, nodal flags
  int q[CLOSURE_OUT], out_nx[CLOSURE_OUT], out_ny[CLOSURE_OUT], out_nodex[CLOSURE_OUT], out_nodey[CLOSURE_OUT];
  // order-6 couplings of each output (training targets)
  int nterm[CLOSURE_OUT];
  ClosureTerm term[CLOSURE_OUT][4];
};

// The odd sweep of a P_5 closure solver fused with the closure network: one
// row per odd moment (orders 1, 3, 5), with its couplings to the even moments
// in the order of the rows of M_x, then M_y, and their coefficients
// -M(k, j) / dx, -M(k, j) / dy.
struct ClosureOddRow {
  int k;        // plane of the moment (orders 1 and 3: updated in place)
  int node_x;   // 1: grid G21 (nodal in x, cell-centred in y); 0: grid G12
  int dk;       // decay plane
  int src;      // source plane (absolute plane index) or -1
  int o;        // order-5 output index 0..5 (read and written through the order-5 buffers), or -1
  int nx, ny;   // couplings along x and y
  int xk[4], xcell[4], yk[4], ycell[4];  // input plane; 1 if the input is cell-centred along the axis
  double xc[4], yc[4];
};
constexpr int CLOSURE_ODD_ROWS = 12;
struct ClosureOdd {
  ClosureOddRow r[CLOSURE_ODD_ROWS];
  double tau;
};

// One instance of a batched run of closure solvers (device table): its state
// planes, the two homes of its order-5 moments (state planes a5, closure
// planes b5), decay planes, sub-step lengths, sweep count, geometry and odd
// rows.
struct ClosureInst {
  void* u;
  void* a5;
  void* b5;
  const void* decay;
  double tau_full, tau_half;
  int nsweeps, pad;
  ClosureGeo G;
  ClosureOdd odd;
};

// A batch's rows through the network.  Training also writes dY, dZ1 and dZ2
// (B x 6, B x 128, FP32), the operands of the weight gradients as transposed
// bfloat16 (blocks of 32 rows: [unit][row]; 128 units, dyt 8) and the loss's
// partial sums, one per workgroup.
struct MlpRows {
  const float* x;       // B x 128
  const float* t;       // B x 6 (training)
  const float* params;
  int B;
  float* y;             // B x 6 (forward only)
  float *dy, *dz1, *dz2;
  uint16_t *xt, *h1t, *h2t, *dz1t, *dz2t, *dyt;
  double* lpart;
};
int mlp_row_blocks(int B);  // workgroups of launch_mlp_rows
hipError_t launch_mlp_rows(const MlpRows& g, bool train, hipStream_t stream);

// The weight gradients' partials (splits of kchunk rows, a multiple of 32, each
// in the parameter blob's layout) and the column sums' (per 256 rows).
constexpr int SUM_COLS = 2 * CLOSURE_HIDDEN + CLOSURE_OUT;
struct MlpGrad {
  const float *dy, *dz1, *dz2;
  const uint16_t *xt, *h1t, *h2t, *dz1t, *dz2t, *dyt;
  float *part, *cpart;
  int B, splits, kchunk;
};
int mlp_sum_chunks(int B);
hipError_t launch_mlp_grad(const MlpGrad& g, hipStream_t stream);

// Adam state and constants; p = null: no update.
struct MlpAdam {
  float *p, *m, *v;
  float lr, b1, b2, eps, c1, c2;
};
// Sums of the partials into grads (in their order), the update, the loss.
hipError_t launch_mlp_update(const MlpGrad& g, float* grads, const MlpAdam& a, const double* lpart, double* loss,
                             hipStream_t stream);
hipError_t launch_adam(const MlpAdam& a, const float* grads, hipStream_t stream);
hipError_t launch_closure_samples(int storage, const void* U, const void* decay, const ClosureGeo& G,
                                  const int* pts, int count, float* feat, float* targ, float* nu,
                                  hipStream_t stream);
hipError_t launch_closure_infer(int storage, void* U, const void* decay, const ClosureGeo& G, const ClosureNet* net,
                                hipStream_t stream);
// The odd sweep of a P_5 closure solver with the network evaluated in the same
// kernel: reads the order-5 moments from in5 (plane r of output r at
// in5 + r * plane_stride) and writes their updates to out5; updates the
// orders 1 and 3 in place.
hipError_t launch_closure_sweep(int storage, void* U, const void* in5, void* out5, const void* decay,
                                const ClosureGeo& G, const ClosureNet* net, const ClosureOdd& odd,
                                hipStream_t stream);
// Odd sweep j of a batched run of closure solvers (one kernel, as launch_closure_sweep):
// the first n_active instances of insts, evaluation blocks numbered from
// bfirst[i]; one network for all.
hipError_t launch_closure_batch(int storage, const ClosureInst* insts, const int* bfirst, int n_active, int blocks,
                                int j, const ClosureNet* net, hipStream_t stream);
// The network alone over a batch of closure solvers (BATCH mode without the
// fused sweep): every running instance's closure planes, which its odd sweep
// then reads as sources.
hipError_t launch_closure_batch_net(int storage, const ClosureInst* insts, const int* bfirst, int n_active, int blocks,
                                    const ClosureNet* net, hipStream_t stream);
size_t closure_infer_lds_bytes();

}  // namespace starmap
