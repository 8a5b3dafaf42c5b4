// Parity sweep of the staggered-grid P_N scheme on gfx950 with the window of
// input orders staged in LDS: the sweep of FP64 states larger than the
// last-level cache, and of few orders on large grids (window.hip holds the sweep
// of the others and of FP32 and BF16 storage).
//
// One sweep applies the half-step operator S^p_tau of one parity p
// (Seibold & Frank, Sect. 4.3, eqs. solution_operator_even/_odd): for every
// component k of parity p and every point of its grid,
//   W_k = - sum_j Mx(k,j) D_x u_j - sum_j My(k,j) D_y u_j      (other parity j)
//   u_k <- u_k + tau (W_k + q_k - c_k u_k) E(-c_k tau),  E(z) = (e^z - 1)/z.
//
// Work decomposition: the outputs of a sweep are split into ranges of the
// azimuthal index m (an output (l, m) couples only to inputs (l -+ 1, m -+ 1),
// Lemma 2).  One workgroup of 256 threads handles one spatial tile of TX x TY
// points and one m range, walking the output orders from the top down.  For
// output order l it needs the input orders l + 1 and l - 1 inside the m range,
// staged in LDS as (TX+1) x (TY+1) tiles (one halo column and row, on the low
// side for cell-centred inputs and the high side for nodal ones); order l - 1
// stays staged for output order l - 2, and while one order is computed the
// next order's planes and output rows are already loading into registers.
// Every staged value feeds up to eight coupled outputs.  Boundary conditions
// enter only through the index mapping of the staging loads (wrap for
// periodic, clamp for extrapolation), so the stencil itself is uniform.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstddef>
#include <cstdint>

#include "device.hpp"
#include "kernels.hpp"

namespace starmap {

// Scalars of a sweep; the pointers travel as separate __restrict__ kernel
// arguments so the compiler may read the (uniform) program tables through the
// scalar cache while the state is written.
struct SweepScalars {
  uint32_t ps;  // plane stride in elements
  int pitch, nx, ny, px, py, ntx, nty, nchunks, zero_off, parity, strip;
  double tau;
};

// Output rows are read once per sweep, just before they are overwritten, and
// not read again before the next sweep: stream them past the caches.
__device__ __forceinline__ void store_stream(double* p, double v) { __builtin_nontemporal_store(v, p); }
__device__ __forceinline__ double load_stream(const double* p) { return __builtin_nontemporal_load(p); }

// Element at a 32-bit byte offset from a wave-uniform base: the address is
// base + zero-extended offset, which the compiler issues as a global access
// with a scalar base and one VGPR offset (no 64-bit address arithmetic).
__device__ __forceinline__ double* at(double* base, uint32_t byte_off) {
  return reinterpret_cast<double*>(reinterpret_cast<char*>(base) + byte_off);
}
__device__ __forceinline__ const double* at(const double* base, uint32_t byte_off) {
  return reinterpret_cast<const double*>(reinterpret_cast<const char*>(base) + byte_off);
}

// s_waitcnt immediate for vmcnt(0) with the other counters left alone
// (gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8).
constexpr int kWaitVm0 = 0x0F70;

// Tiles of 256 points, whose halo fits 128 threads: the window is staged by
// two halves of the workgroup, each half taking every other plane, each thread
// two x-adjacent points of it with one load of 16 bytes where they lie inside
// the grid: fewer vector memory instructions per staged plane than one point
// per thread.
template <int TX, int TY>
constexpr bool kWide = TX * TY == 256 && TX % 2 == 0 && TX + TY <= 128;

// Whether work item lb lies on a tile whose pairs all lie inside the grid
// along x (FAST = true below); uniform over the workgroup.
template <int TX, int TY>
__device__ __forceinline__ bool pair_fast(const SweepScalars& a, int lb) {
  const int2 txy = tile_xy(lb / a.nchunks, a.ntx, a.nty, a.strip);
  return txy.x * TX + TX <= a.nx;
}

// Body of one workgroup's work in a sweep: spatial tile and m range number lb
// (lb = tile * nchunks + range) of one instance.  FAST (wide tiles away from
// the grid's right edge) is a template argument, so the pair and the single
// accesses are separate code and no load sits under a branch on it.
template <int TX, int TY, int CAP, bool FAST>
__device__ __forceinline__ void sweep_tile(double* __restrict__ U, const double* __restrict__ decay,
                                           cptr<int> chunks, cptr<int> orders, cptr<int> loads, cptr<int> rows,
                                           cptr<double> rcoef, const SweepScalars& a, const int lb) {
  extern __shared__ __align__(16) unsigned char smem[];
  double* L = reinterpret_cast<double*>(smem);
  constexpr int LW = TX + 1;
  constexpr int P = (TX + 1) * (TY + 1);
  constexpr int NP = TX * TY;
  static_assert(NP == 256 || NP == 512, "tile must hold 256 or 512 points");
  static_assert(TX + TY <= 256, "halo points must fit one per thread");
  constexpr int PPT = NP / 256;  // output points per thread
  // Pipeline: while window o is computed, the planes of window o+1 (up to CAP)
  // and the first RB output rows of order o+1 are loaded into registers.
  constexpr int MAXP = CAP;
  constexpr int RB = CAP - 2;  // an m range of width w has w rows and w + 2 staged planes per order
  constexpr int LB = 8;        // planes per batch of the synchronous staging
  constexpr bool WIDE = kWide<TX, TY>;
  static_assert(WIDE || !FAST, "the fast path is for wide staging");
  constexpr int SE = WIDE ? NP / 128 : PPT;  // staged interior points per thread and plane
  constexpr int EPT = SE + 1;           // staged points per thread and plane: interior + halo
  constexpr int SP = WIDE ? 2 : 1;      // thread halves that take turns in the planes of a window
  static_assert(MAXP % SP == 0 && LB % SP == 0, "planes split evenly over the thread halves");
  const int tid = threadIdx.x;
  // staging thread index and half (WIDE: threads 0-127 stage planes 0, 2, ...
  // of a window, threads 128-255 planes 1, 3, ...)
  const int st = WIDE ? (tid & 127) : tid;
  const int half = WIDE ? __builtin_amdgcn_readfirstlane(tid >> 7) : 0;
  const int tile = lb / a.nchunks;
  const int4 chk = rec4(chunks, lb - tile * a.nchunks);
  if (chk.x >= chk.y) return;  // no output rows in this m range
  const int2 txy = tile_xy(tile, a.ntx, a.nty, a.strip);
  const int x0 = txy.x * TX;
  const int y0 = txy.y * TY;

  // Staging of one input plane into its (TX+1) x (TY+1) LDS tile.  The tile
  // holds global points (x0 - ox + lx, y0 - oy + ly), with ox (oy) = 1 for an
  // input cell-centred along x (y).  Staging thread t loads SE interior
  // points, x-adjacent on wide tiles (a wave reads whole aligned
  // row segments; they need not be the points t updates) and, for
  // t < TY + TX, one halo point: of the halo column read by x differences
  // (lx = 0 or TX) or of the halo row read by y differences (ly = 0 or TY);
  // the corners are never read.  Source and LDS offsets are affine in (ox, oy):
  // src = sb + ox * sx + oy * sy, dst = db + ox * ddx + oy * ddy.  ox and oy
  // are 0 or 1 and uniform, so they enter as masks (no integer multiplies);
  // source offsets are 32-bit byte offsets from the plane base (sums wrap
  // modulo 2^32 to the in-plane offset).
  uint32_t sb[EPT], sx[EPT], sy[EPT];
  int db[EPT], ddx[EPT], ddy[EPT];
  constexpr uint32_t TS = sizeof(double);
  bool sv[EPT];
#pragma unroll
  for (int p = 0; p < SE; ++p) {
    const int e = WIDE ? SE * st + p : tid + p * 256;
    const int tx = e % TX, ty = e / TX;
    const int xn = map_axis(x0 + tx, a.nx, a.px, 0), xc = map_axis(x0 + tx, a.nx, a.px, 1);
    const int yn = map_axis(y0 + ty, a.ny, a.py, 0), yc = map_axis(y0 + ty, a.ny, a.py, 1);
    sb[p] = uint32_t(yn * a.pitch + xn) * TS;
    sx[p] = uint32_t(xc - xn) * TS;
    sy[p] = uint32_t((yc - yn) * a.pitch) * TS;
    db[p] = ty * LW + tx;
    ddx[p] = 1;
    ddy[p] = LW;
    sv[p] = true;
  }
  {
    constexpr int h = SE;
    sv[h] = st < TY + TX;
    if (st < TY) {  // halo column, row i
      const int i = st;
      const int xn = map_axis(x0 + TX, a.nx, a.px, 0), xc = map_axis(x0 - 1, a.nx, a.px, 1);
      const int yn = map_axis(y0 + i, a.ny, a.py, 0), yc = map_axis(y0 + i, a.ny, a.py, 1);
      sb[h] = uint32_t(yn * a.pitch + xn) * TS;
      sx[h] = uint32_t(xc - xn) * TS;
      sy[h] = uint32_t((yc - yn) * a.pitch) * TS;
      db[h] = i * LW + TX;
      ddx[h] = -TX;
      ddy[h] = LW;
    } else {  // halo row, column j (lanes past the halo keep in-bounds values)
      const int j = st < TY + TX ? st - TY : 0;
      const int xn = map_axis(x0 + j, a.nx, a.px, 0), xc = map_axis(x0 + j, a.nx, a.px, 1);
      const int yn = map_axis(y0 + TY, a.ny, a.py, 0), yc = map_axis(y0 - 1, a.ny, a.py, 1);
      sb[h] = uint32_t(yn * a.pitch + xn) * TS;
      sx[h] = uint32_t(xc - xn) * TS;
      sy[h] = uint32_t((yc - yn) * a.pitch) * TS;
      db[h] = TY * LW + j;
      ddx[h] = 1;
      ddy[h] = -TY * LW;
    }
  }

  // my output points: LDS position, plane offset, and whether the point exists
  // on each of the sweep's two output grids
  int pos[PPT];
  uint32_t goff[PPT];  // element offset in a plane
  bool val0[PPT], val1[PPT];
  {
    // even sweep: slot 0 = G11 (cell, cell), slot 1 = G22 (node, node);
    // odd sweep:  slot 0 = G21 (node, cell), slot 1 = G12 (cell, node)
    const int nxc = a.nx, nxn = a.nx + 1 - a.px, nyc = a.ny, nyn = a.ny + 1 - a.py;
    const int vx0 = a.parity ? nxn : nxc, vy0 = a.parity ? nyc : nyc;
    const int vx1 = a.parity ? nxc : nxn, vy1 = a.parity ? nyn : nyn;
#pragma unroll
    for (int p = 0; p < PPT; ++p) {
      const int e = tid + p * 256;
      const int tx = e % TX, ty = e / TX;
      const int X = x0 + tx, Y = y0 + ty;
      pos[p] = ty * LW + tx;
      goff[p] = uint32_t(Y * a.pitch + X);
      val0[p] = X < vx0 && Y < vy0;
      val1[p] = X < vx1 && Y < vy1;
    }
  }

  // the staged points of one input plane (load record ld) into registers
  // Only the waves holding halo threads (t < TX + TY) load halo points: the
  // others skip that load instruction (a wave-uniform branch), its value
  // would never reach the LDS.
  const bool halo_wave = __builtin_amdgcn_readfirstlane(st >> 6) * 64 < TX + TY;
  auto load_window = [&](double (&v)[EPT], const int4 ld) {
    const double* src = plane_at(U, ld.x, a.ps);
    const uint32_t mx = 0u - uint32_t(ld.z), my = 0u - uint32_t(ld.w);
    if constexpr (FAST) {
      // the points are contiguous and aligned to their total size (x a
      // multiple of SE, pitch and plane stride multiples of 64 elements)
      const double2 w = *reinterpret_cast<const double2*>(at(src, sb[0] + (sx[0] & mx) + (sy[0] & my)));
      v[0] = w.x;
      v[1] = w.y;
    } else {
#pragma unroll
      for (int q = 0; q < SE; ++q) v[q] = *at(src, sb[q] + (sx[q] & mx) + (sy[q] & my));
    }
    if (halo_wave) v[EPT - 1] = *at(src, sb[EPT - 1] + (sx[EPT - 1] & mx) + (sy[EPT - 1] & my));
  };

  // synchronous staging of planes [b0, b1) of a load list into LDS
  auto stage_sync = [&](int first, int b0, int b1) {
    for (int bb = b0; bb < b1; bb += LB) {
      constexpr int LH = LB / SP;  // planes of the batch per thread half
      double v[LH][EPT];
      // the records first (clamped into the list: every scalar load is
      // unconditional, so they issue together), then the loads they describe
      int4 lr[LH];
#pragma unroll
      for (int b = 0; b < LH; ++b) lr[b] = rec4(loads, first + min(bb + SP * b + half, b1 - 1));
#pragma unroll
      for (int b = 0; b < LH; ++b)
        if (bb + SP * b + half < b1) load_window(v[b], lr[b]);
#pragma unroll
      for (int b = 0; b < LH; ++b) {
        if (bb + SP * b + half < b1) {
          // read again (a scalar cache hit) rather than kept live across the loads
          const int4 ld = rec4(loads, first + bb + SP * b + half);
#pragma unroll
          for (int q = 0; q < EPT; ++q)
            if (sv[q]) L[ld.y + db[q] + (ddx[q] & -ld.z) + (ddy[q] & -ld.w)] = v[b][q];
        }
      }
      // Every load of the batch has been consumed.  As at the end of the
      // order loop, the compiler cannot match the conditional loads with
      // their conditional stores: without this wait it takes the batch's
      // registers as possibly still loading at the next batch and waits for
      // all outstanding loads before each of its loads, one memory round
      // trip per plane.
      __builtin_amdgcn_s_waitcnt(kWaitVm0);
    }
  };

  // current values of the output rows r0, r0 + 1, ... (RB of them, < r1)
  auto load_rows = [&](double (&uv)[RB][PPT], int r0, int r1) {
    // plane and grid slot of every row first (row indices clamped into the
    // table: unconditional scalar loads that issue together), then the loads
    int rk[RB], rs[RB];
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      const int r = __builtin_amdgcn_readfirstlane(max(min(r0 + i, r1 - 1), 0));
      const cptr<int> rec = cat(rows, uint32_t(r) * 64u);
      rk[i] = rec[0];
      rs[i] = rec[1];
    }
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      const int r = __builtin_amdgcn_readfirstlane(r0 + i);
      if (r < r1) {
        const double* up = plane_at(U, rk[i], a.ps);
        const bool s1 = rs[i] != 0;
#pragma unroll
        for (int p = 0; p < PPT; ++p)
          uv[i][p] = (s1 ? val1[p] : val0[p]) ? load_stream(at(up, goff[p] * TS)) : 0.0;
      }
    }
  };

  // decay cache per output grid of the sweep: (plane id, c, E(-c tau))
  int cdk0 = -1, cdk1 = -1;
  double c0[PPT], e0[PPT], c1[PPT], e1[PPT];
  // The decay planes an order needs (one per output grid; they change with
  // the order when scattering or filtering is anisotropic) are loaded with
  // that order's window, so no load waits inside the compute.
  int ndk0 = -1, ndk1 = -1;
  double nc0[PPT], nc1[PPT];
  auto prefetch_decay = [&](const int4 od, double (&n0)[PPT], double (&n1)[PPT]) {
    // every row of an order shares the decay plane of its output grid
    ndk0 = -1;
    ndk1 = -1;
    for (int r = od.z; r < od.w && (ndk0 < 0 || ndk1 < 0); ++r) {
      const cptr<int> rr = cat(rows, uint32_t(r) * 64u);
      const int gs = rr[1], dk = rr[2];
      // value selects (a conditional store to one of two variables would be
      // merged into a store through a selected address, i.e. stack memory)
      ndk0 = (gs == 0 && ndk0 < 0) ? dk : ndk0;
      ndk1 = (gs != 0 && ndk1 < 0) ? dk : ndk1;
    }
    const bool l0 = ndk0 >= 0 && ndk0 != cdk0, l1 = ndk1 >= 0 && ndk1 != cdk1;
    const double* d0 = plane_at(decay, l0 ? ndk0 : 0, a.ps);
    const double* d1 = plane_at(decay, l1 ? ndk1 : 0, a.ps);
#pragma unroll
    for (int p = 0; p < PPT; ++p) {
      if (l0) n0[p] = val0[p] ? *at(d0, goff[p] * TS) : 0.0;
      if (l1) n1[p] = val1[p] ? *at(d1, goff[p] * TS) : 0.0;
    }
  };
  auto apply_decay = [&]() {
    if (ndk0 >= 0 && ndk0 != cdk0) {
#pragma unroll
      for (int p = 0; p < PPT; ++p) {
        c0[p] = nc0[p];
        e0[p] = expm1div(-nc0[p] * a.tau);
      }
      cdk0 = ndk0;
    }
    if (ndk1 >= 0 && ndk1 != cdk1) {
#pragma unroll
      for (int p = 0; p < PPT; ++p) {
        c1[p] = nc1[p];
        e1[p] = expm1div(-nc1[p] * a.tau);
      }
      cdk1 = ndk1;
    }
  };

  // the padding couplings read this plane of zeros
  for (int e = tid; e < P; e += 256) L[a.zero_off + e] = 0.0;
  // prologue: the first rows and decay values, then the first window, so
  // that all of them are in flight together (one memory round trip; the
  // window's LDS stores wait for the window loads, issued last)
  double ua[RB][PPT];
  {
    const int4 ord = rec4(orders, chk.x);
    load_rows(ua, ord.z, ord.w);
    prefetch_decay(ord, nc0, nc1);
    stage_sync(ord.x, 0, ord.y - ord.x);
  }
  __builtin_amdgcn_s_waitcnt(kWaitVm0);  // see the end of the order loop
  __syncthreads();

  for (int o = chk.x; o < chk.y; ++o) {
    const int4 ord = rec4(orders, o);
    apply_decay();
    const bool has_next = o + 1 < chk.y;
    const int4 nxt = has_next ? rec4(orders, o + 1) : make_int4(0, 0, 0, 0);
    const int nl = nxt.y - nxt.x;
    // 1. the next window into registers (every thread loads its own elements)
    constexpr int MH = MAXP / SP;  // planes of the window per thread half
    double stg[MH][EPT];
    {
      // the records first (clamped into the list: unconditional scalar loads
      // that issue together), then the loads they describe
      int4 nrec[MH];
#pragma unroll
      for (int b = 0; b < MH; ++b) nrec[b] = rec4(loads, nxt.x + max(min(SP * b + half, nl - 1), 0));
#pragma unroll
      for (int b = 0; b < MH; ++b)
        if (SP * b + half < nl) load_window(stg[b], nrec[b]);
    }
    // 2. the first output rows of the next order
    double ub[RB][PPT];
    if (has_next) {
      load_rows(ub, nxt.z, nxt.w);
      prefetch_decay(nxt, nc0, nc1);
    }
    // 3. update this order's rows from the current window
    for (int r0 = ord.z; r0 < ord.w; r0 += RB) {
      if (r0 != ord.z) {  // more rows than the registers hold: load the next batch now
        load_rows(ua, r0, ord.w);
        __builtin_amdgcn_s_waitcnt(kWaitVm0);
      }
#pragma unroll
      for (int i = 0; i < RB; ++i) {
        const int r = __builtin_amdgcn_readfirstlane(r0 + i);
        if (r < ord.w) {
          cptr<int> rec = cat(rows, uint32_t(r) * 64u);
          cptr<double> cf = cat(rcoef, uint32_t(r) * 64u);
          const int k = rec[0], gslot = rec[1], so = rec[3];
          double* up = plane_at(U, k, a.ps);
#pragma unroll
          for (int p = 0; p < PPT; ++p) {
            double W = 0.0;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              const double* lp = L + rec[4 + t] + pos[p];
              W = couple(W, cf[t], lp[1], lp[0]);
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              const double* lp = L + rec[8 + t] + pos[p];
              W = couple(W, cf[4 + t], lp[LW], lp[0]);
            }
            // the source, staged in LDS, joins the residual
            if (so >= 0) W += L[so + pos[p]];
            const double c = gslot ? c1[p] : c0[p];
            const double E = gslot ? e1[p] : e0[p];
            const double nv = sub_step(ua[i][p], W, c, E, a.tau);
            if (gslot ? val1[p] : val0[p]) store_stream(at(up, goff[p] * TS), nv);
          }
        }
      }
    }
    // 4. every read of the current window is done: install the next one
    __syncthreads();
#pragma unroll
    for (int b = 0; b < MH; ++b) {
      if (SP * b + half < nl) {
        const int4 ld = rec4(loads, nxt.x + SP * b + half);
#pragma unroll
        for (int q = 0; q < EPT; ++q)
          if (sv[q]) L[ld.y + db[q] + (ddx[q] & -ld.z) + (ddy[q] & -ld.w)] = stg[b][q];
      }
    }
    if (nl > MAXP) stage_sync(nxt.x, MAXP, nl);
    // Every load of this order has been consumed: wait for all of them here.
    // The compiler cannot match the conditional loads with their conditional
    // uses, so without this wait it assumes the window registers may still be
    // receiving and waits for every outstanding load at their first reuse,
    // which would stall the next order's prefetch right after it is issued.
    __builtin_amdgcn_s_waitcnt(kWaitVm0);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int p = 0; p < PPT; ++p) ua[i][p] = ub[i][p];
  }
}

template <int TX, int TY, int CAP>
__global__ void __launch_bounds__(256)
sweep_kernel(double* __restrict__ U, const double* __restrict__ decay, const int4* __restrict__ chunks,
             const int4* __restrict__ orders, const int4* __restrict__ loads, const int* __restrict__ rows,
             const double* __restrict__ rcoef, const SweepScalars a) {
  // logical block = tile * nchunks + chunk: the m ranges of one tile run on
  // the same XCD, one after another, and share its L2
  const int lb = xcd_tile(blockIdx.x, gridDim.x);
  if constexpr (kWide<TX, TY>) {
    if (pair_fast<TX, TY>(a, lb)) {
      sweep_tile<TX, TY, CAP, true>(U, decay, (cptr<int>)chunks, (cptr<int>)orders, (cptr<int>)loads, (cptr<int>)rows,
                                    (cptr<double>)rcoef, a, lb);
      return;
    }
  }
  sweep_tile<TX, TY, CAP, false>(U, decay, (cptr<int>)chunks, (cptr<int>)orders, (cptr<int>)loads, (cptr<int>)rows,
                                 (cptr<double>)rcoef, a, lb);
}

// Sweep number j of a batched run.  Instances are sorted by their number of
// sweeps (descending), so the instances still running at sweep j are the
// first n_active; their workgroups (tiles x m ranges) are numbered
// consecutively, instance i owning [first[i], first[i+1]).  Sweep j has odd
// parity for even j (the composition starts and ends with odd half-steps).
// BatchEntry as the device reads it: pointers read from memory carry no
// address space, so without this the compiler would use flat accesses (which
// share the LDS wait counter) and vector loads for the uniform tables.
template <typename P>
using gptr = __attribute__((address_space(1))) P*;
struct BatchEntryG {
  gptr<void> u;
  gptr<const void> decay;
  gptr<const int4> chunks[2];
  gptr<const int4> orders[2];
  gptr<const int4> loads[2];
  gptr<const int> rows[2];
  gptr<const void> rcoef[2];
  int64_t plane_stride;
  double tau_full, tau_half;
  int pitch, nx, ny, px, py, ntx, nty, nchunks;
  int zero_off[2];
  int nsweeps;
  int strip;
  int64_t even_b_delta;
};
static_assert(sizeof(BatchEntryG) == sizeof(BatchEntry), "device view of BatchEntry");
static_assert(offsetof(BatchEntryG, even_b_delta) == offsetof(BatchEntry, even_b_delta), "device view of BatchEntry");
static_assert(offsetof(BatchEntryG, plane_stride) == offsetof(BatchEntry, plane_stride), "device view of BatchEntry");
static_assert(offsetof(BatchEntryG, nsweeps) == offsetof(BatchEntry, nsweeps), "device view of BatchEntry");

template <int TX, int TY, int CAP>
__global__ void __launch_bounds__(256)
sweep_batch_kernel(const BatchEntry* __restrict__ table, const int* __restrict__ first, const int n_active,
                   const int j) {
  const int item = xcd_tile(blockIdx.x, gridDim.x);
  int lo = 0, hi = n_active - 1;  // last instance with first[i] <= item
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (first[mid] <= item) lo = mid; else hi = mid - 1;
  }
  const BatchEntryG& e = reinterpret_cast<const BatchEntryG*>(table)[lo];
  const int par = (j & 1) ? 0 : 1;
  // closure solvers: before even sweep j, (j + 1) / 2 odd sweeps have moved
  // the order-5 moments; an odd count leaves them in the closure planes
  const int64_t bd = (par == 0 && (((j + 1) >> 1) & 1)) ? e.even_b_delta : 0;
  SweepScalars a;
  a.ps = uint32_t(e.plane_stride);
  a.pitch = e.pitch;
  a.nx = e.nx;
  a.ny = e.ny;
  a.px = e.px;
  a.py = e.py;
  a.ntx = e.ntx;
  a.nty = e.nty;
  a.nchunks = e.nchunks;
  a.zero_off = e.zero_off[par];
  a.parity = par;
  a.strip = e.strip;
  a.tau = (j == 0 || j == e.nsweeps - 1) ? e.tau_half : e.tau_full;
  const int lb = item - first[lo];
  double* const u = (double*)(gptr<double>)e.u;
  const double* const dec = (const double*)(gptr<const double>)e.decay;
  const cptr<int> ch = (cptr<int>)((gptr<const char>)e.chunks[par] + bd);
  const cptr<int> od = (cptr<int>)((gptr<const char>)e.orders[par] + bd);
  const cptr<int> ldl = (cptr<int>)((gptr<const char>)e.loads[par] + bd);
  const cptr<int> rw = (cptr<int>)((gptr<const char>)e.rows[par] + bd);
  const cptr<double> rc = (cptr<double>)((gptr<const char>)e.rcoef[par] + bd);
  if constexpr (kWide<TX, TY>) {
    if (pair_fast<TX, TY>(a, lb)) {
      sweep_tile<TX, TY, CAP, true>(u, dec, ch, od, ldl, rw, rc, a, lb);
      return;
    }
  }
  sweep_tile<TX, TY, CAP, false>(u, dec, ch, od, ldl, rw, rc, a, lb);
}

// ------------------------------------------------------------ variants
namespace {
// FP64 (tx, ty, cap): cap 10 holds the widest m range's planes of one order in
// registers; cap 8 and 6 hold fewer (the rest is staged synchronously) but
// leave registers for a fourth (fifth) workgroup per CU, which pays at the
// narrower m ranges; cap 0 runs with the window in registers (window.hip).
constexpr TileShape kVariants64[] = {{64, 4, 10}, {128, 2, 10}, {32, 8, 10}, {32, 16, 10}, {64, 4, 0},
                                     {64, 8, 10}, {64, 8, 8},   {64, 8, 6},  {32, 8, 8},   {128, 2, 0},
                                     {64, 4, 8},  {32, 16, 8},  {64, 2, 0},  {64, 4, 6}};
// FP32 and BF16: all with the window in registers
constexpr TileShape kVariants32[] = {{64, 4, 0},  {128, 2, 0}, {32, 8, 0}, {32, 16, 0}, {128, 4, 0},
                                     {64, 8, 0},  {256, 2, 0}, {256, 1, 0}, {64, 2, 0},  {32, 4, 0},
                                     {128, 1, 0}, {16, 16, 0}, {512, 1, 0}, {16, 8, 0}};
constexpr int kNumVariants = sizeof(kVariants64) / sizeof(kVariants64[0]);
static_assert(kNumVariants == sizeof(kVariants32) / sizeof(kVariants32[0]), "one numbering for every storage type");

// Opt the kernels of one instantiation in to all of the device's LDS (once).
template <int TX, int TY, int CAP>
hipError_t prepare_t(size_t lds) {
  static size_t attr_bytes = 0;
  if (lds <= attr_bytes) return hipSuccess;
  int dev = 0, max_lds = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
  if (e != hipSuccess) return e;
  if (lds > size_t(max_lds)) return hipErrorInvalidValue;
  e = hipFuncSetAttribute(reinterpret_cast<const void*>(&sweep_kernel<TX, TY, CAP>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, max_lds);
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&sweep_batch_kernel<TX, TY, CAP>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, max_lds);
  if (e != hipSuccess) return e;
  attr_bytes = size_t(max_lds);
  return hipSuccess;
}

template <int TX, int TY>
size_t lds_t(int slots) {
  return size_t(slots) * (TX + 1) * (TY + 1) * sizeof(double);
}

template <int TX, int TY, int CAP>
hipError_t launch_t(const SweepArgs& a, int slots, hipStream_t stream) {
  const size_t lds = lds_t<TX, TY>(slots);
  hipError_t e = prepare_t<TX, TY, CAP>(lds);
  if (e != hipSuccess) return e;
  SweepScalars sc;
  sc.ps = uint32_t(a.plane_stride);
  sc.pitch = a.pitch;
  sc.nx = a.nx;
  sc.ny = a.ny;
  sc.px = a.px;
  sc.py = a.py;
  sc.ntx = a.ntx;
  sc.nty = a.nty;
  sc.nchunks = a.nchunks;
  sc.zero_off = a.zero_off;
  sc.parity = a.parity;
  sc.strip = a.strip;
  sc.tau = a.tau;
  const int blocks = a.ntx * a.nty * a.nchunks;
  hipLaunchKernelGGL((sweep_kernel<TX, TY, CAP>), dim3(blocks), dim3(256), lds, stream, a.u, a.decay, a.chunks,
                     a.orders, a.loads, a.rows, a.rcoef, sc);
  return hipGetLastError();
}

template <int TX, int TY, int CAP>
hipError_t launch_batch_t(const BatchEntry* table, const int* first, int n_active, int items, int j, int slots,
                          hipStream_t stream) {
  const size_t lds = lds_t<TX, TY>(slots);
  hipError_t e = prepare_t<TX, TY, CAP>(lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((sweep_batch_kernel<TX, TY, CAP>), dim3(items), dim3(256), lds, stream, table, first, n_active,
                     j);
  return hipGetLastError();
}

// the LDS variants, by their number in kVariants64
#define STARMAP_FOR_VARIANT(v, CALL)      \
  switch (v) {                            \
    case 0: return CALL(64, 4, 10);       \
    case 1: return CALL(128, 2, 10);      \
    case 2: return CALL(32, 8, 10);       \
    case 3: return CALL(32, 16, 10);      \
    case 5: return CALL(64, 8, 10);       \
    case 6: return CALL(64, 8, 8);        \
    case 7: return CALL(64, 8, 6);        \
    case 8: return CALL(32, 8, 8);        \
    case 10: return CALL(64, 4, 8);       \
    case 11: return CALL(32, 16, 8);      \
    case 13: return CALL(64, 4, 6);       \
  }                                       \
  return hipErrorInvalidValue;

}  // namespace

int sweep_variant_count() { return kNumVariants; }
TileShape sweep_variant(int storage, int v) {
  if (v < 0 || v >= kNumVariants) return TileShape{0, 0, 1};
  return storage == STORE_FP64 ? kVariants64[v] : kVariants32[v];
}

// The rules behind a solver that was given no tile, from timing every variant
// and width on 88 sizes (P_1 .. P_39, 48^2 .. 1400^2) and, in FP64, on 420 with
// and without decay planes by order and sources on more moments.  Where two are given,
// microseconds per sweep of the choice, then of the other.
//
// The last-level cache holds 256 MB: P_31 345^2 FP32 (253 MB) 77 us with the
// output rows kept in it, 82 past it; 360^2 (275 MB) 95 and 90.
constexpr double kCache = 2.56e8;
bool sweep_streams(double state_bytes) { return state_bytes > kCache; }

// FP64.  With the window in registers, 64 x 2 tiles (P_7 280^2 11.6, LDS 16;
// P_3 1000^2 34 and 36; P_5 400^2 14.3 and 15.3; P_9 550^2 44 and 58; P_15 447^2
// 62 and 77; P_31 150^2 36 and 59), but in LDS, above some 350^2 points,
//   - where one or two orders cannot hide the loads of a large grid: 64 x 8
//     (P_1 400^2 6.5, registers 6.9; 1000^2 17 and 24), for P_2 below 430^2 points
//     32 x 8 (380^2 9.1, 64 x 8 9.7; 440^2 10.1 and 9.4);
//   - where state and decay planes together leave the cache, and with them the y
//     neighbours' lines the L1 before they are asked for: 32 x 8, up to P_3 64 x 8
//     (P_39 500^2 557, registers 687; P_9 850^2 119 and 142; P_7 1000^2 89 and 132,
//     930^2 91 and 98; P_3 1500^2 67 and 84; P_5 1200^2 81 and 103; decay planes by
//     order: P_9 700^2 85 and 106, P_7 850^2 80 and 103, but P_13 500^2 92 and 83;
//     the state alone counts from P_7 on with sources on more moments, which the
//     LDS holds too: P_13 500^2 137 and 113), unless the LDS tiles are too few to
//     fill the chip (P_39 200^2 118, registers 108);
//   - up to P_6, whose few orders the general kernel's look-ups hold up most.  With
//     decay planes by order: 32 x 8 (P_4 1000^2 47 and 66, 350^2 11.4 and 14.2; P_6
//     700^2 41 and 50, but 350^2 21 and 20), P_3 from 800^2 on 64 x 8 (1000^2 34 and
//     44).  With sources on more moments: 32 x 8 for P_4 (500^2 18 and 23, 1000^2 56
//     and 86), P_5 from 800^2 on (850^2 64 and 74, but 700^2 46 and 44), P_3 and P_2
//     (500^2 14.1 and 16.5; 400^2 9.3, 64 x 8 10.1) where the tiles' last round on
//     the chip is nearly full (P_3 600^2 20.5 and 19.2), P_2 below 770^2 (850^2 24.4,
//     64 x 8 22.9).  But for P_4 with decay planes alone, not where a second round has
//     just begun (three steps of P_5 550^2 in changing media 351 and 323);
//   - for plain solvers of P_4 where the last round is nearly full (500^2 15.1 and
//     18.1, 850^2 36.1 and 37.1, but 600^2 23 and 21), of P_5 and P_6 where one round
//     is just full (500^2 18.5 and 20.2, 23.0 and 24.4).
// FP32, BF16.  Large states on wide tiles, which read the fewest lines twice,
// where the grid fills them (P_39 1000^2 FP32: 512 x 1 993, 128 x 2 1012; 500^2
// 236 and 247), else
// 64 wide (P_31 447^2, 448 columns: 64 x 8 114, 512 x 1 117, 128 x 2 121), P_8 ..
// P_15 64 x 4 (P_13 900 x 1000 112, 64 x 8 115).  FP32 states in the
// cache: 64 x 4 (P_9 317 x 203 7.0, 64 x 2 7.2; P_5 256^2 5.2 and 5.4; P_31
// 256^2 41 and 44), 64 x 2 where those are too few workgroups (P_3 150^2 3.7 and
// 3.9, P_9 150^2 5.6 and 6.0) and for few orders on large grids (P_3 1000^2 14.9
// and 15.6).  BF16: 128 x 4 (P_39 250^2 37, 64 x 2 40; P_7 512^2 13.0 and 13.6),
// small ones 64 x 2 (P_9 150^2 6.6, 128 x 4 7.2; P_21 300^2 19.8 and 20.4; P_31
// 256^2 29 and 31).
static int default_variant64(const SweepSizes& z) {
  const double points = double(z.cols) * z.rows;
  const double bytes = z.state_bytes + (z.N <= 6 || !z.sources ? z.decay_bytes : 0.0);
  const bool cached = !sweep_streams(z.state_bytes) && bytes <= (z.N <= 6 ? 2.5e8 : 2.7e8);
  if (points <= (cached ? 1.2e5 : 6.0e4)) return kNoLdsVariant;
  // rounds of 32 x 8 tiles, four on each of 256 compute units, and how full they are
  const double rounds = std::ceil(z.cols / 32.0) * std::ceil(z.rows / 8.0) / 1024.0, full = rounds / std::ceil(rounds);
  const bool general = z.by_order || z.sources;
  const bool spills = rounds > 1.0 && rounds < 1.3;  // into a nearly empty second round
  bool lds = !cached;
  switch (z.N) {
    case 1: return 7;
    case 2: return points < 1.8e5 || (z.sources && points < 6.0e5 && (rounds <= 1.0 || full > 0.85)) ? 8 : 7;
    case 3:
      if (!general) return cached ? kNoLdsVariant : 7;
      if (!z.sources && points > 6.4e5) return 7;
      lds = lds || (z.sources ? full > 0.85 : !spills);
      break;
    case 4: lds = lds || (z.sources ? !spills : z.by_order || full > 0.85); break;
    case 5:
      lds = lds || (z.sources ? points > 6.4e5 : z.by_order ? !spills : rounds <= 1.0 && full > 0.97);
      break;
    case 6:
      lds = lds || (!z.sources && (z.by_order ? !spills && points > 1.4e5 : rounds <= 1.0 && full > 0.97));
      break;
  }
  return lds ? 8 : kNoLdsVariant;
}

int sweep_default_variant(int storage, const SweepSizes& z) {
  if (storage == STORE_FP64) return default_variant64(z);
  const int N = z.N, cols = z.cols;
  const double points = double(cols) * z.rows, state_bytes = z.state_bytes;
  const bool cached = !sweep_streams(state_bytes);
  auto fills = [&](int wide) { return (cols + wide - 1) / wide * wide - cols <= cols / 20; };
  if (storage == STORE_BF16) return cached ? (points < 1.2e5 && state_bytes < 8.5e7 ? 8 : 4) : fills(256) ? 6 : 4;
  if (!cached) return N >= 8 && N < 16 ? 0 : N >= 16 && fills(512) ? 12 : fills(128) ? 1 : 5;
  return points < (N < 8 ? 5.0e4 : 3.0e4) || (N < 8 && points > 6.0e5) ? 8 : 0;
}

// m ranges.  LDS window: one range where it holds every index (P_5 400^2 15.3,
// at four 20.7; P_7 1000^2 89, at four 122), from P_13 on six (P_39 500^2 557,
// eight 618, four 580), else four, which from P_16 on is better for the general
// sweep, whose sources take LDS too (P_21 400^2 171, six 290; decay planes by order
// alone 130 and 165; P_16 500^2 170 and 198).  Registers: four, more workgroups,
// while the chip is not full (P_21 150^2 FP32 12, six 15; P_31 128^2 17 and 21.5;
// P_5 150^2 4.3 and 4.7; BF16 P_31 256^2 29 and 30), and no idle rows in P_15 (FP32
// 447^2 30.0, six 30.9); of grids that fill it six, which read fewer planes twice
// (FP32 P_21 300^2 27.6, four 28.2), which is one range of P_4 and P_5 (FP32 400^2
// 7.3 and 7.7, FP64 300^2 8.7 and 9.7); eight for P_8 .. P_15 (FP32 P_15 1000^2 155,
// six 160; P_9 1800^2 221 and 229) and in 512 x 1 tiles (P_39 1000^2 993, six 998).
int sweep_default_width(int storage, int variant, const SweepSizes& z) {
  const int N = z.N;
  const double points = double(z.cols) * z.rows;
  if (!sweep_in_registers(storage, variant)) {
    if (N >= 16 && (z.by_order || z.sources)) return 4;
    return N == 4 || N == 5 ? 6 : N == 6 || N == 7 ? 8 : N >= 13 ? 6 : 4;
  }
  if (storage == STORE_FP64) return (N == 4 || N == 5) && points > 4.0e4 ? 6 : 4;
  if (N == 4 || N == 5) return points > (storage == STORE_FP32 ? 1.2e5 : 2.0e5) ? 6 : 4;
  if (storage == STORE_BF16) return N >= 16 ? (variant == 8 ? 4 : 6) : N >= 8 && points > 5.0e5 ? 6 : 4;
  if (N >= 16) return variant == 12 ? 8 : points > 4.0e4 ? 6 : 4;
  return N >= 8 && points > 4.7e5 ? 8 : 4;
}

size_t sweep_lds_bytes(int v, int slots, int storage) {
  const TileShape t = sweep_variant(storage, v);
  if (t.cap == 0) return 0;
  return size_t(slots) * (t.tx + 1) * (t.ty + 1) * sizeof(double);
}

hipError_t prepare_sweep(int variant, int slots) {
#define STARMAP_CALL(X, Y, K) prepare_t<X, Y, K>(lds_t<X, Y>(slots))
  STARMAP_FOR_VARIANT(variant, STARMAP_CALL)
#undef STARMAP_CALL
}

hipError_t launch_sweep_batch(int variant, const BatchEntry* table, const int* first, int n_active, int items, int j,
                              int slots, hipStream_t stream) {
  if (n_active < 1 || items < 1) return hipErrorInvalidValue;
#define STARMAP_CALL(X, Y, K) launch_batch_t<X, Y, K>(table, first, n_active, items, j, slots, stream)
  STARMAP_FOR_VARIANT(variant, STARMAP_CALL)
#undef STARMAP_CALL
}

hipError_t launch_sweep(int variant, const SweepArgs& a, int slots, hipStream_t stream) {
#define STARMAP_CALL(X, Y, K) launch_t<X, Y, K>(a, slots, stream)
  STARMAP_FOR_VARIANT(variant, STARMAP_CALL)
#undef STARMAP_CALL
}
#undef STARMAP_FOR_VARIANT

// ------------------------------------------------------------ diagnostics
// Block partials in FP64, then one block sums them in a fixed order, so the
// result does not depend on scheduling.
template <typename T>
__global__ void __launch_bounds__(256) diag_partial_kernel(DiagArgs a) {
  __shared__ double s_sum[256], s_sq[256], s_max[256], s_bad[256];
  const int plane = blockIdx.x / a.blocks_per_plane;
  const int rb = blockIdx.x % a.blocks_per_plane;
  const int nxp = a.plane_nx[plane], nyp = a.plane_ny[plane];
  const int r0 = rb * a.rows_per_block;
  const int r1 = min(nyp, r0 + a.rows_per_block);
  const T* U = reinterpret_cast<const T*>(a.u) + int64_t(plane) * a.plane_stride;
  double sum = 0.0, sq = 0.0, mx = 0.0, bad = 0.0;
  for (int r = r0; r < r1; ++r) {
    for (int x = threadIdx.x; x < nxp; x += 256) {
      const double v = double(to_c(U[int64_t(r) * a.pitch + x]));
      if (!isfinite(v)) { bad += 1.0; continue; }
      sum += v;
      sq += v * v;
      mx = fmax(mx, fabs(v));
    }
  }
  s_sum[threadIdx.x] = sum;
  s_sq[threadIdx.x] = sq;
  s_max[threadIdx.x] = mx;
  s_bad[threadIdx.x] = bad;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) {
      s_sum[threadIdx.x] += s_sum[threadIdx.x + w];
      s_sq[threadIdx.x] += s_sq[threadIdx.x + w];
      s_max[threadIdx.x] = fmax(s_max[threadIdx.x], s_max[threadIdx.x + w]);
      s_bad[threadIdx.x] += s_bad[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    double* p = a.part + 4 * int64_t(blockIdx.x);
    p[0] = plane == 0 ? s_sum[0] : 0.0;
    p[1] = s_sq[0];
    p[2] = s_max[0];
    p[3] = s_bad[0];
  }
}

__global__ void __launch_bounds__(256) diag_final_kernel(const double* part, int nblocks, double* out) {
  __shared__ double s[4][256];
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
  for (int b = threadIdx.x; b < nblocks; b += 256) {
    a0 += part[4 * b + 0];
    a1 += part[4 * b + 1];
    a2 = fmax(a2, part[4 * b + 2]);
    a3 += part[4 * b + 3];
  }
  s[0][threadIdx.x] = a0;
  s[1][threadIdx.x] = a1;
  s[2][threadIdx.x] = a2;
  s[3][threadIdx.x] = a3;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) {
      s[0][threadIdx.x] += s[0][threadIdx.x + w];
      s[1][threadIdx.x] += s[1][threadIdx.x + w];
      s[2][threadIdx.x] = fmax(s[2][threadIdx.x], s[2][threadIdx.x + w]);
      s[3][threadIdx.x] += s[3][threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x < 4) out[threadIdx.x] = s[threadIdx.x][0];
}

int diag_blocks(int nplanes, int max_rows, int rows_per_block) {
  return nplanes * ((max_rows + rows_per_block - 1) / rows_per_block);
}

hipError_t launch_diagnostics(int storage, const DiagArgs& a, hipStream_t stream) {
  const int nb = a.nplanes * a.blocks_per_plane;
  switch (storage) {
    case STORE_FP64: hipLaunchKernelGGL(diag_partial_kernel<double>, dim3(nb), dim3(256), 0, stream, a); break;
    case STORE_FP32: hipLaunchKernelGGL(diag_partial_kernel<float>, dim3(nb), dim3(256), 0, stream, a); break;
    case STORE_BF16: hipLaunchKernelGGL(diag_partial_kernel<bf16>, dim3(nb), dim3(256), 0, stream, a); break;
    default: return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(diag_final_kernel, dim3(1), dim3(256), 0, stream, a.part, nb, a.out);
  return hipGetLastError();
}

}  // namespace starmap
