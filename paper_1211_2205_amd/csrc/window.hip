// Parity sweep of the staggered-grid P_N scheme on gfx950 with the window of
// input orders in registers: the sweep of FP32 and BF16 storage, and of most
// FP64 states that stay in the last-level cache (sweep.hip holds the FP64 kernel
// for the others, the rule, and what a sweep computes).
//
// Work decomposition: the outputs of a sweep are split into ranges of 2 NM
// azimuthal indices m (an output (l, m) couples only to inputs
// (l -+ 1, m -+ 1), Lemma 2).  One workgroup takes a spatial tile, one m range
// and a run of output orders; every thread owns V x-adjacent points of the
// tile and walks the output orders from the top down.  An order's rows need
// the x and y differences of the NM + 1 R and I planes of the input orders
// l + 1 and l - 1 in the range.  The differences of order l + 1 are in
// registers from the rows before; of each plane of order l - 1 the thread has
// loaded its own points and the y neighbour (the x neighbour is the next lane's
// value, but in small FP32 launches: kOverlap and by_edge below): it forms the
// plane's two differences, at once reloads the plane's registers with the order
// two below, and updates the row whose last input that plane was.
// Nothing is shared between threads: no LDS, no barrier, and every wave has a
// whole order's planes and rows in flight while it computes the order before.
//
// Why registers: staged through LDS, the same sweep spent two barriers and a
// load, an LDS store and eight LDS reads per plane and row on values that the
// L1 cache serves as well (the neighbour loads hit lines that the wave or its
// neighbours in the workgroup have just loaded).  Per sweep, LDS kernel with
// its best tile -> this kernel with its default one: P_39 1000^2 BF16 838 ->
// 518 us, FP32 1107 -> 1014 us; P_31 256^2 FP32 76 -> 40 us, BF16 71 -> 29 us;
// P_9 317 x 203 FP32 15.5 -> 7.9 us; P_7 280^2 FP64 16.2 -> 10.8 us; P_3 100^2
// FP64 7.4 -> 3.6 us.  P_39 1000^2 FP32 moves 4.9 GB per sweep at 4.8 TB/s; with
// every neighbour load left out it takes 1020 us, so the memory's rate for this
// mix of reads and writes bounds it.  FP64 states beyond the cache are slower
// here (P_39 500^2 687 against 557 us): eight-byte loads need twice the L1 lines
// in flight, so the y neighbours' lines are gone
// before they are asked for.
//
// Boundary conditions enter through the offsets of the neighbour loads (wrap
// for periodic axes, clamp for extrapolation).  A plane that does not exist
// (m < 0, m > l, order above N) is loaded through a buffer descriptor of no
// records, which gives zeros without touching memory, so the loads of an order
// are the same instructions everywhere and none sits under a branch (a load
// under a branch makes the compiler wait for all earlier ones).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "device.hpp"
#include "kernels.hpp"

namespace starmap {

namespace {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// Output rows are read once and written once per sweep.  With a state larger
// than the last-level cache they are accessed non-temporally (S; without it
// P_39 1000^2 FP32 takes 7% longer, P_31 447^2 14%), with a smaller one not, so
// that the next sweep finds them there (P_31 256^2 FP32 47 -> 40 us, P_39 150^2
// FP64 66 -> 52).
constexpr int kStream = 2;
// a byte offset past every pair of planes (planes stay below 2^31 bytes and are
// a multiple of 256)
constexpr uint32_t kOutside = 0xFFFFFF00u;

// x-adjacent points per thread: two BF16 values make one 32-bit access (one
// value per thread: half the bytes per instruction, four: 2% slower on P_39
// 1000^2, more on small grids); FP32 pairs were slower than single points
// (P_31 256^2: 83 against 53 us, fewer waves of eight-byte loads).
template <typename T>
constexpr int kPoints = sizeof(T) == 2 ? 2 : 1;

// Whether the x neighbours are the values of the lanes next to each lane, in
// tiles whose rows overlap by the lanes at their ends, or loads of their own.
// An eight-byte load holds the address unit for 16 cycles: with three per plane
// it was busy for 70% of a sweep (P_7 280^2 12.7 -> 10.8 us).  Four-byte loads
// take 6 cycles, less than two lane shifts and the overlap's idle lanes (P_9
// 317 x 203 FP32 7.2 -> 8.5).
template <typename T>
constexpr bool kOverlap = sizeof(T) == 8;
constexpr int kPiece = 62;  // points of a row that a wave of overlapping tiles owns

// With single points of four bytes and rows of whole waves (EDGE) the x neighbours
// are the values of the next lanes too, but the tiles do not overlap: one load
// per order brings the neighbours of the wave's row end, lane by lane a plane.

// A thread's V stored values of a row segment as one memory access.
template <typename T, int V>
using Word = std::conditional_t<sizeof(T) * V == 8, u32x2, std::conditional_t<sizeof(T) * V == 4, uint32_t, uint16_t>>;

template <typename W, int AUX = 0>
__device__ __forceinline__ W buf_load(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  if constexpr (sizeof(W) == 8)
    return __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, AUX);
  else if constexpr (sizeof(W) == 4)
    return __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, AUX);
  else
    return __builtin_amdgcn_raw_buffer_load_b16(r, off, 0, AUX);
}
template <typename W, int AUX>
__device__ __forceinline__ void buf_store(W v, __amdgpu_buffer_rsrc_t r, uint32_t off) {
  if constexpr (sizeof(W) == 8)
    __builtin_amdgcn_raw_buffer_store_b64(v, r, off, 0, AUX);
  else if constexpr (sizeof(W) == 4)
    __builtin_amdgcn_raw_buffer_store_b32(v, r, off, 0, AUX);
  else
    __builtin_amdgcn_raw_buffer_store_b16(v, r, off, 0, AUX);
}

// Value e of a thread's word.
template <typename T, int V>
__device__ __forceinline__ typename ComputeOf<T>::type value(Word<T, V> w, int e) {
  if constexpr (sizeof(T) == 8)
    return __builtin_bit_cast(double, w);
  else if constexpr (sizeof(T) == 4)
    return __uint_as_float(w);
  else if constexpr (V == 1)
    return __uint_as_float(uint32_t(w) << 16);
  else
    return __uint_as_float(e ? (w & 0xFFFF0000u) : (w << 16));
}
template <typename T, int V>
__device__ __forceinline__ Word<T, V> word(const typename ComputeOf<T>::type (&v)[V]) {
  if constexpr (sizeof(T) == 2)
    return uint32_t(from_c<bf16>(v[0]).bits) | (uint32_t(from_c<bf16>(v[V - 1]).bits) << 16);
  else
    return __builtin_bit_cast(Word<T, V>, v[0]);
}

// The value of the lane before (BEFORE) or after this one, in the wave's first
// or last lane `end`; every lane of the wave must take part.
template <bool BEFORE>
__device__ __forceinline__ float lane_near(float v, float end) {
  return __uint_as_float(uint32_t(__builtin_amdgcn_update_dpp(int(__float_as_uint(end)), int(__float_as_uint(v)),
                                                              BEFORE ? 0x138 : 0x130, 0xF, 0xF, false)));
}
template <bool BEFORE>
__device__ __forceinline__ double lane_near(double v, double end) {
  const u32x2 w = __builtin_bit_cast(u32x2, v), e = __builtin_bit_cast(u32x2, end);
  return __builtin_bit_cast(
      double, u32x2{__float_as_uint(lane_near<BEFORE>(__uint_as_float(w.x), __uint_as_float(e.x))),
                    __float_as_uint(lane_near<BEFORE>(__uint_as_float(w.y), __uint_as_float(e.y)))});
}

// Scalars of one sweep.
template <typename C>
struct WindowScalars {
  uint32_t ps;  // plane stride in elements
  int pitch, nx, ny, px, py;
  int lbw, ty;       // lanes per tile row (logarithm), tile rows
  int nseg;          // runs of output orders
  Divisor by_nseg;
  WindowOrder o;     // m ranges and tiles
  WindowPlanes planes;
  int N, top_shift;                  // order; planes from an order-N input to where it is read
  C tau;
};

template <typename T, int NM, int P, bool G, bool S, bool EDGE>
__device__ __forceinline__ void window_tile(T* __restrict__ U, const typename ComputeOf<T>::type* __restrict__ decay,
                                            cptr<typename ComputeOf<T>::type> coef, cptr<int> tab,
                                            const WindowScalars<typename ComputeOf<T>::type>& a, int grp, int chunk,
                                            int tl, int seg) {
  using C = typename ComputeOf<T>::type;
  constexpr int V = kPoints<T>;
  static_assert(V <= 2, "a pair at most");
  static_assert(!EDGE || (V == 1 && sizeof(T) == 4), "single points of four bytes");
  constexpr bool SHIFT = kOverlap<T> || EDGE;  // every x neighbour by lane shift
  using W = Word<T, V>;
  using W1 = Word<T, 1>;
  typedef C C8 __attribute__((ext_vector_type(8)));
  constexpr uint32_t TS = sizeof(T);
  constexpr int AUX = S ? kStream : 0;
  constexpr int NB = NM + 1;  // input planes of one order that the range needs, R and I each

  const int gtiles = group_tiles(a.o, grp);
  if (tl >= gtiles) return;
  const int tile = tile_number(a.o, grp, uint32_t(gtiles), uint32_t(tl));
  int m0 = chunk * 2 * NM;
  const int ltop = a.N - ((a.N - P) & 1), lbot = m0 + P;
  if (lbot > ltop) return;  // no output rows in this m range
  const int nord = ((ltop - lbot) >> 1) + 1;
  int o0 = 0, o1 = nord;
  if (a.nseg > 1) {
    o0 = divide(nord * seg, a.by_nseg);
    o1 = divide(nord * (seg + 1), a.by_nseg);
  }
  if (o0 >= o1) return;
  const int lfirst = ltop - 2 * o0, llast = ltop - 2 * (o1 - 1);

  // this thread's points (X .. X + V - 1, Y)
  const TileAt txy = tile_at(tile, a.o);
  const int bw = 1 << a.lbw;
  int Y = row_of(txy, a.ty, a.lbw, int(threadIdx.x));
  const int col = int(threadIdx.x) & (bw - 1);
  const int rows = a.ny + 1 - a.py, cols = a.nx + 1 - a.px;
  int X;
  bool in;
  if constexpr (kOverlap<T>) {
    // a piece of a row is a wave's, and its end lanes stand on the points next to
    // it; the first and the last point of an axis that does not wrap need none
    const int q = col & 63, x0 = ((txy.x << (a.lbw - 6)) + (col >> 6)) * kPiece;
    X = x0 + q - (a.px ? 1 : 0);
    in = Y < rows && X < cols && (q > 0 || (!a.px && X == 0)) && (q < 63 || (!a.px && X == a.nx)) &&
         (x0 == 0 || x0 < cols - (a.px ? 0 : 2));  // (a piece that is one too many)
    Y = min(Y, rows - 1);
  } else if constexpr (EDGE) {
    X = txy.x * bw + col;
    in = Y < rows && X < cols;
    Y = min(Y, rows - 1);
  } else {
    // lanes past the tile or the grid stand at the origin and store nothing
    X = (txy.x * bw + col) * V;
    in = Y < rows && X < cols;
    if (!in) X = Y = 0;
  }
  // points of the lane on the two output grids: R rows are cell-centred along
  // y (and along x in even sweeps), I rows nodal along y (and along x in even
  // sweeps); R inputs are cell-centred along y (and along x in odd sweeps),
  // I inputs nodal along y (and cell-centred along x in even sweeps)
  const int vxR = P ? cols : a.nx, vxI = P ? a.nx : cols;
  const bool okR = in && X < vxR && Y < a.ny, okI = in && X < vxI && Y < rows;
  // y: centre row of R inputs (the last cell again past the last one), and the
  // other end of the difference: the row below for cells, above for nodes
  const int ycR = min(Y, a.ny - 1);
  const int ynR = Y > 0 ? Y - 1 : (a.py ? a.ny - 1 : 0);
  const int ynI = a.py ? (Y + 1 == a.ny ? 0 : Y + 1) : min(Y + 1, a.ny);
  // x: for cells the point before the lane's first, for nodes the one after
  // its last one that a cell needs
  const int xlo = X > 0 ? X - 1 : (a.px ? a.nx - 1 : 0);
  const int nv = min(V, a.nx - X);
  const int xq = X + max(nv, 1);
  const int xhi = a.px ? (xq >= a.nx ? xq - a.nx : xq) : min(xq, a.nx);
  // columns that the lane loads of node and cell planes
  const int wrapped = X < 0 ? X + a.nx : X >= a.nx ? X - a.nx : X;
  const int xn = !SHIFT ? X : a.px ? min(wrapped, a.nx - 1) : max(min(X, a.nx), 0);
  const int xc = V > 1 ? X : min(xn, a.nx - 1);
  const int xcR = P ? xc : xn, xcI = P ? xn : xc;
  // The x neighbour is a value of the next lane (no load: P_39 1000^2 BF16 587
  // -> 532 us, the address unit had been the limit).  With two points per
  // thread the lanes at the ends of a wave, a tile row or the grid load it.
  const int lane = int(threadIdx.x) & 63;
  const bool endL = V == 1 || lane == 0 || col == 0 || !in || X == 0;
  const bool endH = V == 1 || lane == 63 || col == bw - 1 || !in || X + V >= cols;
  const uint32_t rowR = uint32_t(ycR * a.pitch), rowI = uint32_t(Y * a.pitch);
  const uint32_t cR = (rowR + xcR) * TS, bR = uint32_t(ynR * a.pitch + xcR) * TS;
  // (an I plane follows its R plane: one descriptor serves both)
  const uint32_t pbytes = a.ps * TS;
  const uint32_t cI = (rowI + xcI) * TS + pbytes, bI = uint32_t(ynI * a.pitch + xcI) * TS + pbytes;
  const uint32_t nR = (P ? endL : endH) ? (rowR + (P ? xlo : xhi)) * TS : kOutside;
  const uint32_t nI = (P ? endH : endL) ? (rowI + (P ? xhi : xlo)) * TS + pbytes : kOutside;
  const uint32_t go = uint32_t(Y * a.pitch + xn);
  const uint32_t sR = okR ? go * TS : kOutside, sI = okI ? go * TS + pbytes : kOutside;

  // EDGE: lane i < 2 NB reads the neighbour of the wave's row end in plane i & 1
  // (R or I) of pair i / 2: the cell before the first lane's, the node after the
  // last one's (offset from the order's first plane in memory, and index m)
  uint32_t eoff = kOutside;
  int em = 0;
  if constexpr (EDGE) {
    const int first = X - lane, after = first + 64, z = lane & 1, b = lane >> 1;
    const int lo = first > 0 ? first - 1 : (a.px ? a.nx - 1 : 0);
    const int hi = a.px ? min(after >= a.nx ? after - a.nx : after, a.nx - 1) : min(after, a.nx);
    em = m0 + P - 1 + 2 * b;
    if (b < NB && em >= z)
      eoff = uint32_t(2 * (NM - b) + z) * pbytes + ((z ? rowI : rowR) + (z == P ? hi : min(lo, a.nx - 1))) * TS;
  }

  // address of plane k, and the descriptor of a plane at an address
  auto plane_addr = [&](int k) { return uint64_t(U) + uint64_t(int64_t(k) * int64_t(pbytes)); };
  auto plane = [&](uint64_t p, uint32_t records) {
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(p), 0, int(records), 0x00020000);
  };
  // records of the pair of planes of index m in an order of highest index lm:
  // none past it (as bit operations: a comparison would travel as a 64-lane
  // mask).  The range of m = 0 has no planes of m < 0 and no I_0.
  const uint32_t pair = 2 * pbytes, pair0 = m0 > 0 ? pair : pbytes, none0 = m0 > 0 ? pair : 0;
  auto recs = [&](uint32_t of, int m, int lm) { return of & ~uint32_t((lm - m) >> 31); };

  // raw words of the input planes: centre, x neighbour, y neighbour
  struct In {
    W c, b;
    W1 n;
  };
  struct Diff {
    C x[V], y[V];
  };
  In rR[NB], rI[NB];
  // planes number b (m = m0 + P - 1 + 2 b) of an order, R at address p and I
  // after it, existing for m <= lm
  auto load_planes = [&](int b, uint64_t p, int lm) {
    const auto r = plane(p, recs(b ? pair : P ? pair0 : none0, m0 + P - 1 + 2 * b, lm));
    rR[b].c = buf_load<W>(r, cR);
    if constexpr (!SHIFT) rR[b].n = buf_load<W1>(r, nR);
    rR[b].b = buf_load<W>(r, bR);
    rI[b].c = buf_load<W>(r, cI);
    if constexpr (!SHIFT) rI[b].n = buf_load<W1>(r, nI);
    rI[b].b = buf_load<W>(r, bI);
  };
  // the row ends' neighbours in the planes of an order whose first one is at p
  auto load_edge = [&](uint64_t p, int lm) {
    return EDGE ? buf_load<uint32_t>(plane(p, uint32_t(NB) * pair), em <= lm ? eoff : kOutside) : 0u;
  };
  // differences of a plane: along x centre - lower (cells) or upper - centre
  // (nodes), along y likewise (R planes are cells, I planes nodes)
  auto diff = [&](const In& w, Diff& d, bool cell, bool isR, uint32_t edge, int b) {
    C v[V];
#pragma unroll
    for (int e = 0; e < V; ++e) v[e] = value<T, V>(w.c, e);
    C nb = value<T, 1>(w.n, 0);
    if constexpr (EDGE) {
      const C end = __uint_as_float(uint32_t(__builtin_amdgcn_readlane(int(edge), 2 * b + (isR ? 0 : 1))));
      nb = cell ? lane_near<true>(v[0], end) : lane_near<false>(v[0], end);
    } else if constexpr (kOverlap<T> || V > 1) {
      const C near = cell ? lane_near<true>(v[V - 1], v[V - 1]) : lane_near<false>(v[0], v[0]);
      nb = kOverlap<T> || !(cell ? endL : endH) ? near : nb;
    }
#pragma unroll
    for (int e = 0; e < V; ++e) {
      const C q = value<T, V>(w.b, e);
      d.y[e] = isR ? v[e] - q : q - v[e];
    }
    if constexpr (V == 1) {
      d.x[0] = cell ? v[0] - nb : nb - v[0];
    } else if (cell) {
      if constexpr (V > 1) {  // the point past the last cell repeats it
        v[V - 1] = !a.px && X + 1 == a.nx ? v[0] : v[V - 1];
        v[0] = !a.px && X == a.nx ? nb : v[0];
      }
#pragma unroll
      for (int e = 0; e < V; ++e) d.x[e] = v[e] - (e ? v[e ? e - 1 : 0] : nb);
    } else {
#pragma unroll
      for (int e = 0; e < V; ++e) d.x[e] = (e + 1 == V || e + 1 == nv ? nb : v[e + 1 < V ? e + 1 : e]) - v[e];
    }
  };

  // output rows: current values and, with G, source values (planes
  // tab[2 (N + 1) + k]; none: zeros)
  W uR[NM], uI[NM], qR[G ? NM : 1], qI[G ? NM : 1];
  auto load_row = [&](int q, uint64_t p, int lm, int k) {
    const uint32_t n = recs(P == 0 && q == 0 ? pair0 : pair, m0 + P + 2 * q, lm);
    const auto u = plane(p, n);
    uR[q] = buf_load<W, AUX>(u, sR);
    uI[q] = buf_load<W, AUX>(u, sI);
    if constexpr (G) {
      const int r = n ? tab[2 * (a.N + 1) + k] : -1, i = n > pbytes ? tab[2 * (a.N + 1) + k + 1] : -1;
      qR[q] = buf_load<W>(plane(plane_addr(r), r >= 0 ? pbytes : 0), sR);
      qI[q] = buf_load<W>(plane(plane_addr(i - 1), i >= 0 ? pair : 0), sI);
    }
  };

  // decay coefficients c and E(-c tau) of the two output grids.  Without G one
  // plane per grid serves every order but the zeroth, so E is formed once,
  // before the loop; with G order l's planes are tab[2 l] and tab[2 l + 1].
  C cR_[V], eR_[V], cI_[V], eI_[V], ldR[V], ldI[V];
  auto load_decay = [&](int l) {
    const C* d0 = plane_at(decay, G ? max(tab[2 * l], 0) : a.planes.r, a.ps);
    const C* d1 = plane_at(decay, G ? max(tab[2 * l + 1], 0) : a.planes.i, a.ps);
#pragma unroll
    for (int e = 0; e < V; ++e) {
      ldR[e] = d0[go + e];
      ldI[e] = d1[go + e];
    }
  };
  auto apply_decay = [&]() {
#pragma unroll
    for (int e = 0; e < V; ++e) {
      cR_[e] = ldR[e];
      eR_[e] = expm1div(-ldR[e] * a.tau);
      cI_[e] = ldI[e];
      eI_[e] = expm1div(-ldI[e] * a.tau);
    }
  };

  // prologue: the input planes of both neighbouring orders and the first rows,
  // all in flight together
  // planes and rows in memory order, from the highest m of the range down: of
  // this order the first row, number k0, at ps; of the next one the first row at
  // pn; the first plane loaded next at pl.  From one order to the next they move
  // by a distance that shrinks by four planes, so only the first ones take
  // multiplications (the scalar unit, which a compute unit's waves share, spends
  // as long on a small sweep as the address unit).
  int l = lfirst;
  int k0 = int(uint32_t(l * (l + 1)) >> 1) + l - (m0 + P) - 2 * (NM - 1);
  uint64_t ps = plane_addr(k0), pn = ps - uint64_t(uint32_t(2 * l + 1)) * pbytes,
           pl = pn - uint64_t(uint32_t(l)) * pbytes;
  int64_t dn = int64_t(2 * l - 3) * int64_t(pbytes);
  uint32_t rE = 0;      // EDGE: row ends of the planes in rR and rI
  Diff hR[NB], hI[NB];  // differences of input order l + 1
  {
    const int kh = k0 + l + 1 + (l + 1 == a.N ? a.top_shift : 0);
    load_decay(l);
    uint64_t p = plane_addr(kh);
    const uint32_t pE = load_edge(p, l < a.N ? l + 1 : -1);
#pragma unroll
    for (int b = NM; b >= 0; --b) {
      load_planes(b, p, l < a.N ? l + 1 : -1);
      p += pair;
    }
    In pR[NB], pI[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      pR[b] = rR[b];
      pI[b] = rI[b];
    }
    p = ps - uint64_t(uint32_t(l + 2)) * pbytes;
    rE = load_edge(p, l - 1);
#pragma unroll
    for (int b = NM; b >= 0; --b) {
      load_planes(b, p, l - 1);
      p += pair;
    }
    p = ps;
#pragma unroll
    for (int q = NM - 1; q >= 0; --q) {
      load_row(q, p, l, k0 + 2 * (NM - 1 - q));
      p += pair;
    }
    apply_decay();  // (while the planes arrive)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      diff(pR[b], hR[b], P == 1, true, pE, b);
      diff(pI[b], hI[b], P == 0, false, pE, b);
    }
  }
  // the zeroth moment, the last row of the even sweep's first range, has a
  // decay plane of its own (and, without G, the only source): updated last
  const bool zeroth = !G && P == 0 && m0 == 0 && llast == 0;
  C c0[V] = {};
  W q0{};
  if (zeroth) {
    const C* d = plane_at(decay, a.planes.zeroth, a.ps);
#pragma unroll
    for (int e = 0; e < V; ++e) c0[e] = d[go + e];
    const int src = a.planes.source;
    q0 = buf_load<W>(plane(plane_addr(src), src >= 0 ? pbytes : 0), sR);
  }

  const int lend = zeroth ? 2 : llast;
  for (; l >= lend; l -= 2) {
    // (keeps what derives from m0 out of the scalar registers between orders)
    asm volatile("" : "+s"(m0));
    const bool more = l - 2 >= llast;
    const int lm = more ? l - 3 : -1, ln = more ? l - 2 : -1;  // highest m of the planes and rows loaded next
    // with G: the next rows' decay planes, if they are other ones
    const bool redo = G && more && (tab[2 * l] != tab[2 * l - 4] || tab[2 * l + 1] != tab[2 * l - 3]);
    if (redo) load_decay(l - 2);
    const int kn = k0 - (2 * l + 1);
    uint64_t as = ps, an = pn, al = pl;
    const uint32_t nE = load_edge(al, lm);
    // the rows' coefficients (the table has eight rows of padding on both sides)
    const cptr<C8> cf = reinterpret_cast<cptr<C8>>(cat(coef, uint32_t(k0 + 8) * uint32_t(8 * sizeof(C))));
    C8 cr = cf[0], ci = cf[1];
    Diff lR, lI;  // differences of the plane before (index m + 1 of the next row)
#pragma unroll
    for (int b = NM; b >= 0; --b) {
      Diff dR, dI;
      diff(rR[b], dR, P == 1, true, rE, b);
      diff(rI[b], dI, P == 0, false, rE, b);
      // (the differences before the loads that overwrite their sources)
#pragma unroll
      for (int e = 0; e < V; ++e) asm volatile("" : "+v"(dR.x[e]), "+v"(dR.y[e]), "+v"(dI.x[e]), "+v"(dI.y[e]));
      load_planes(b, al, lm);
      al += pair;
      if (b < NM) {  // the rows of index m0 + P + 2 b
        const int j = 2 * (NM - 1 - b);
        C8 crn{}, cin{};
        if (b > 0) {  // the next rows' coefficients, read ahead
          crn = cf[j + 2];
          cin = cf[j + 3];
        }
        const auto out = plane(as, recs(P == 0 && b == 0 ? pair0 : pair, m0 + P + 2 * b, l));
        as += pair;
#pragma unroll
        for (int z = 0; z < 2; ++z) {
          // an R row takes the x differences of R planes and the y differences
          // of I planes, an I row the others
          const Diff &xl1 = z ? lI : lR, &xl0 = z ? dI : dR, &xh1 = z ? hI[b + 1] : hR[b + 1], &xh0 = z ? hI[b] : hR[b];
          const Diff &yl1 = z ? lR : lI, &yl0 = z ? dR : dI, &yh1 = z ? hR[b + 1] : hI[b + 1], &yh0 = z ? hR[b] : hI[b];
          const C8& c8 = z ? ci : cr;
          C nv_[V];
#pragma unroll
          for (int e = 0; e < V; ++e) {
            C w = fma(c8[0], xl1.x[e], C(0));
            w = fma(c8[1], xl0.x[e], w);
            w = fma(c8[2], xh1.x[e], w);
            w = fma(c8[3], xh0.x[e], w);
            w = fma(c8[4], yl1.y[e], w);
            w = fma(c8[5], yl0.y[e], w);
            w = fma(c8[6], yh1.y[e], w);
            w = fma(c8[7], yh0.y[e], w);
            if constexpr (G) w += value<T, V>(z ? qI[b] : qR[b], e);
            const C u = value<T, V>(z ? uI[b] : uR[b], e);
            const C r = sub_step(u, w, z ? cI_[e] : cR_[e], z ? eI_[e] : eR_[e], a.tau);
            // (a lane's second point past the grid keeps the padding's value)
            nv_[e] = e == 0 || X + e < (z ? vxI : vxR) ? r : u;
          }
          buf_store<W, AUX>(word<T, V>(nv_), out, z ? sI : sR);
        }
        load_row(b, an, ln, kn + j);
        an += pair;
        hR[b + 1] = lR;
        hI[b + 1] = lI;
        cr = crn;
        ci = cin;
      }
      lR = dR;
      lI = dI;
      __builtin_amdgcn_sched_barrier(0);
    }
    hR[0] = lR;
    hI[0] = lI;
    rE = nE;
    k0 = kn;
    ps = pn;
    pn -= uint64_t(dn);
    pl -= uint64_t(dn) - pair;
    dn -= 4 * int64_t(pbytes);
    if (redo) apply_decay();
  }
  if (zeroth) {  // R_0^0 couples to R_1^1 and I_1^1 alone
    const cptr<C> cf = cat(coef, uint32_t(8) * uint32_t(8 * sizeof(C)));
    C nv_[V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
      C w = fma(cf[2], hR[1].x[e], C(0));
      w = fma(cf[6], hI[1].y[e], w) + value<T, V>(q0, e);
      const C u = value<T, V>(uR[0], e);
      const C r = sub_step(u, w, c0[e], expm1div(-c0[e] * a.tau), a.tau);
      nv_[e] = e == 0 || X + e < vxR ? r : u;
    }
    buf_store<W, AUX>(word<T, V>(nv_), plane(plane_addr(0), pbytes), sR);
  }
}

// Threads per workgroup at most (a tile of 512 points of FP32).
template <typename T>
constexpr int kMaxThreads = sizeof(T) == 8 ? 256 : 512;

template <typename T, int NM, int P, bool G, bool S, bool EDGE>
__global__ void __launch_bounds__(kMaxThreads<T>)
window_kernel(T* __restrict__ U, const typename ComputeOf<T>::type* __restrict__ decay,
              const typename ComputeOf<T>::type* __restrict__ coef, const int* __restrict__ tab,
              const WindowScalars<typename ComputeOf<T>::type> a) {
  using C = typename ComputeOf<T>::type;
  // (a launch of several runs of orders has one group)
  window_tile<T, NM, P, G, S, EDGE>(U, decay, (cptr<C>)coef, (cptr<int>)tab, a, a.nseg > 1 ? 0 : int(blockIdx.z),
                                    int(blockIdx.y), int(blockIdx.x), int(blockIdx.z));
}

// WindowEntry as the device reads it (pointers with their address space, as
// for the LDS kernel's table).
template <typename Q>
using gptr = __attribute__((address_space(1))) Q*;
struct WindowEntryG {
  gptr<void> u;
  gptr<const void> decay;
  gptr<const void> coef;
  gptr<const int> tab;
  int64_t plane_stride;
  double tau_full, tau_half;
  WindowOrder order;
  WindowPlanes planes[2];
  int pitch, nx, ny, px, py, N, nm, nsweeps, top_shift, pad;
};
static_assert(sizeof(WindowEntryG) == sizeof(WindowEntry), "device view of WindowEntry");

// Sweep number j of a batched run (instances and workgroup prefix as for the
// LDS kernel); each instance brings its own width of m ranges, up to NMAX: a
// batch of narrow ones needs fewer registers (with the shorter way to the first
// load, 24 media of P_3 .. P_9 on 64^2 .. 256^2 cells, FP32: 3.63 -> 3.43 ms).
template <typename T, int NMAX, int P, bool G, bool S, bool EDGE>
__global__ void __launch_bounds__(kMaxThreads<T>)
window_batch_kernel(const WindowEntry* __restrict__ table, const int* __restrict__ first, const int n_active,
                    const int j, const int lbw) {
  using C = typename ComputeOf<T>::type;
  const int item = int(blockIdx.x);
  // the last instance with first[i] <= item, 64 at a time: a bisection's reads
  // wait for one another
  int lo = -1;
  for (int i = 0; i < n_active; i += 64) {
    const int k = i + (int(threadIdx.x) & 63);
    lo += __popcll(__ballot(k < n_active && first[min(k, n_active - 1)] <= item));
  }
  lo = __builtin_amdgcn_readfirstlane(lo);
  const WindowEntryG& e = reinterpret_cast<const WindowEntryG*>(table)[lo];
  WindowScalars<C> a;
  a.ps = uint32_t(e.plane_stride);
  a.pitch = e.pitch;
  a.nx = e.nx;
  a.ny = e.ny;
  a.px = e.px;
  a.py = e.py;
  a.lbw = lbw;
  a.ty = int(blockDim.x) >> lbw;
  a.o = e.order;
  a.planes = e.planes[P];
  a.nseg = 1;
  a.N = e.N;
  // closure solvers: before even sweep j, (j + 1) / 2 odd sweeps have moved
  // the order-5 moments; an odd count leaves them in the closure planes
  a.top_shift = (P == 0 && (((j + 1) >> 1) & 1)) ? e.top_shift : 0;
  a.tau = C((j == 0 || j == e.nsweeps - 1) ? e.tau_half : e.tau_full);
  T* const u = (T*)(gptr<T>)e.u;
  const C* const dec = (const C*)(gptr<const C>)e.decay;
  const cptr<C> cf = (cptr<C>)(gptr<const C>)e.coef;
  const cptr<int> tab = (cptr<int>)e.tab;
  const int nm = e.nm, it = item - ((cptr<int>)first)[lo];
  const int grp = divide(it, a.o.per), within = it - grp * (a.o.gsize * a.o.nchunks);
  const int chunk = divide(within, a.o.by_gsize), tl = within - chunk * a.o.gsize;
  if (NMAX == 2 || nm == 2)
    window_tile<T, 2, P, G, S, EDGE>(u, dec, cf, tab, a, grp, chunk, tl, 0);
  else if (NMAX == 3 || nm == 3)
    window_tile<T, NMAX < 3 ? 2 : 3, P, G, S, EDGE>(u, dec, cf, tab, a, grp, chunk, tl, 0);
  else
    window_tile<T, NMAX < 4 ? 2 : 4, P, G, S, EDGE>(u, dec, cf, tab, a, grp, chunk, tl, 0);
}

// Runs of orders of a launch: one of few waves is a chain of memory round trips,
// one per order, so its orders are split into runs that start their own chains
// (one more window to load each) while the chip has room for them: up to 2048
// waves, with the many orders of P_16 and up 2400, and two runs where that makes
// 3300.  Microseconds per sweep without -> with: FP32 P_9 64^2 4.8 -> 4.0, P_7
// 128^2 4.65 -> 4.46, P_13 100^2 6.2 -> 5.45, P_31 64^2 10.9 -> 8.3, P_31 100^2
// 14.6 -> 11.7; BF16 P_9 64^2 6.0 -> 4.4, P_31 100^2 15.5 -> 11.8.  Beyond it
// costs (FP32 P_7 128^2 in three 4.67, P_31 64^2 in three 9.0).  FP64, whose waves
// load twice the bytes, gains with fewer: P_9 64^2 5.6 -> 5.1, P_39 64^2 19.7 ->
// 16.5 in two (more, and smaller grids of P_16 and up, were not timed), but P_3
// 150^2 4.3 -> 4.55, P_7 128^2 5.6 -> 6.4; an order of the general
// kernel, with decay planes and sources to look up, takes longer (beam P_7 100^2
// 7.4 -> 6.3, P_13 100^2 11.4 -> 9.5, P_7 128^2 7.7 -> 7.25; P_9 150^2 9.65 -> 9.9).
int window_runs(int value_bytes, bool general, const WindowOrder& o, int waves_per_tile, int N) {
  const int waves = o.ntx * o.nty * o.nchunks * waves_per_tile;
  if (waves < 1 || o.groups > 1) return 1;  // (a launch of several runs has one group)
  int n;
  if (value_bytes == 8)
    n = N >= 16                   ? (waves <= 1400 ? 2 : 1)
        : waves <= 400            ? 1200 / waves
        : general && waves <= 1000 ? 2
                                  : 1;
  else
    n = N >= 16 ? std::max(2400 / waves, waves <= 1650 ? 2 : 1) : 2048 / waves;
  return std::min(std::max(n, 1), N / 2 + 1);
}

// The logarithm of a power of two, -1 of another number.
int log2_of(int n) {
  int l = 0;
  while ((1 << l) < n) ++l;
  return n >= 1 && (1 << l) == n ? l : -1;
}

// Whether a sweep's x neighbours at row ends come by one load per order: rows of
// whole waves, an order's planes of a range within a descriptor's reach, and two
// waves for each of the chip's 1024 SIMDs, so that the address unit is what they
// wait for (24 media of P_3 .. P_9 34.7 -> 33.1 us per sweep, P_9 317 x 203 7.16
// -> 7.0, P_31 256^2 40.6 -> 40.0; the 780 waves of a P_7 128^2 run with changing
// media, which wait for their loads, 28.7 -> 29.5 per step).
template <typename T>
bool by_edge(int tx, int nm, int64_t plane_stride, int64_t threads) {
  return sizeof(T) == 4 && tx >= 64 && threads >= 2048 * 64 &&
         uint64_t(nm + 1) * 2 * uint64_t(plane_stride) * sizeof(T) < kOutside;
}

// f with the parity and the flags as types (edge: with four-byte values only).
template <typename T, typename F>
hipError_t by_flags(bool parity, bool general, bool streaming, bool edge, F f) {
  using No = std::integral_constant<int, 0>;
  using Yes = std::integral_constant<int, 1>;
  auto at = [&](auto p, auto g, auto s) {
    if constexpr (sizeof(T) == 4)
      if (edge) return f(p, g, s, Yes{});
    return f(p, g, s, No{});
  };
  auto with = [&](auto p, auto g) { return streaming ? at(p, g, Yes{}) : at(p, g, No{}); };
  if (parity) return general ? with(Yes{}, Yes{}) : with(Yes{}, No{});
  return general ? with(No{}, Yes{}) : with(No{}, No{});
}

template <typename T, int NM>
hipError_t launch_t(int storage, const WindowArgs& w, hipStream_t stream) {
  using C = typename ComputeOf<T>::type;
  WindowScalars<C> a;
  a.ps = uint32_t(w.plane_stride);
  a.pitch = w.pitch;
  a.nx = w.nx;
  a.ny = w.ny;
  a.px = w.px;
  a.py = w.py;
  const int bw = w.tx / kPoints<T>;
  a.lbw = log2_of(bw);
  a.ty = w.ty;
  const int threads = bw * w.ty;
  const WindowGrid g = window_grid(storage, w.nx, w.ny, w.px, w.py, w.tx, w.ty, w.N, w.nm);
  a.o = window_order(g, w.strip);
  const int blocks1 = g.ntx * g.nty * g.nchunks;
  a.nseg = window_runs(int(sizeof(T)), w.general != 0, a.o, threads / 64, w.N);
  a.by_nseg = divisor(a.nseg);
  a.planes = w.planes;
  a.N = w.N;
  a.top_shift = w.top_shift;
  a.tau = C(w.tau);
  if (a.lbw < (kOverlap<T> ? 6 : 0) || threads < 64 || threads > kMaxThreads<T>) return hipErrorInvalidValue;
  if (blocks1 < 1 || g.nchunks > 65535 || a.o.groups > 65535) return hipErrorInvalidValue;
  const dim3 blocks(unsigned(a.o.gsize), unsigned(g.nchunks), unsigned(a.nseg > 1 ? a.nseg : a.o.groups));
  T* u = static_cast<T*>(w.u);
  const C *d = static_cast<const C*>(w.decay), *cf = static_cast<const C*>(w.coef);
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, blocks, dim3(threads), 0, stream, u, d, cf, w.tab, a);
    return hipGetLastError();
  };
  const bool edge = by_edge<T>(w.tx, NM, w.plane_stride, int64_t(blocks1) * threads);
  return by_flags<T>(w.parity, w.general, w.streaming, edge,
                     [&](auto p, auto g, auto s, auto e) {
                       return launch(&window_kernel<T, NM, decltype(p)::value, decltype(g)::value, decltype(s)::value,
                                                    decltype(e)::value>);
                     });
}

template <typename T>
hipError_t launch_nm(int storage, const WindowArgs& w, hipStream_t stream) {
  switch (w.nm) {
    case 2: return launch_t<T, 2>(storage, w, stream);
    case 3: return launch_t<T, 3>(storage, w, stream);
    case 4: return launch_t<T, 4>(storage, w, stream);
  }
  return hipErrorInvalidValue;
}

template <typename T, int NMAX>
hipError_t launch_batch_t(const WindowEntry* table, const int* first, int n_active, int items, int j, int tx, int ty,
                          int64_t max_stride, bool general, bool streaming, hipStream_t stream) {
  const int lbw = log2_of(tx / kPoints<T>), threads = tx / kPoints<T> * ty;
  if (lbw < (kOverlap<T> ? 6 : 0) || threads < 64 || threads > kMaxThreads<T>) return hipErrorInvalidValue;
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(items), dim3(threads), 0, stream, table, first, n_active, j, lbw);
    return hipGetLastError();
  };
  return by_flags<T>(!(j & 1), general, streaming, by_edge<T>(tx, NMAX, max_stride, int64_t(items) * threads),
                     [&](auto p, auto g, auto s, auto e) {
                       return launch(&window_batch_kernel<T, NMAX, decltype(p)::value, decltype(g)::value,
                                                          decltype(s)::value, decltype(e)::value>);
                     });
}

template <typename T, typename... A>
hipError_t launch_batch_nm(int nm, A... args) {
  switch (nm) {
    case 2: return launch_batch_t<T, 2>(args...);
    case 3: return launch_batch_t<T, 3>(args...);
    case 4: return launch_batch_t<T, 4>(args...);
  }
  return hipErrorInvalidValue;
}

}  // namespace

int window_nm(int N, int width) {
  // as many ranges as the width asks for, of equal (even) widths
  const int w = width < 4 ? 4 : width > 8 ? 8 : width;
  const int chunks = (N + 1 + w - 1) / w;
  const int nm = (N + 1 + 2 * chunks - 1) / (2 * chunks);
  return nm < 2 ? 2 : nm > 4 ? 4 : nm;
}

WindowGrid window_grid(int storage, int nx, int ny, int px, int py, int tx, int ty, int N, int nm) {
  // tiles over every point that lies on one of the grids.  With FP64 the end lanes
  // of a row's pieces stand on the points next to the piece, except at an end of the
  // grid (window_tile).
  WindowGrid g;
  const int cols = nx + 1 - px;
  if (storage == STORE_FP64) {
    const int pieces = std::max(1, (cols - (px ? 0 : 2) + kPiece - 1) / kPiece), across = std::max(1, tx / 64);
    g.ntx = (pieces + across - 1) / across;
  } else {
    g.ntx = (cols + tx - 1) / tx;
  }
  g.nty = (ny + 1 - py + ty - 1) / ty;
  g.nchunks = (N + 1 + 2 * nm - 1) / (2 * nm);
  return g;
}

hipError_t launch_window(int storage, const WindowArgs& w, hipStream_t stream) {
  switch (storage) {
    case STORE_FP64: return launch_nm<double>(storage, w, stream);
    case STORE_FP32: return launch_nm<float>(storage, w, stream);
    case STORE_BF16: return launch_nm<bf16>(storage, w, stream);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_window_batch(int storage, const WindowEntry* table, const int* first, int n_active, int items, int j,
                               int tx, int ty, int nm, int64_t max_stride, bool general, bool streaming,
                               hipStream_t stream) {
  if (n_active < 1 || items < 1) return hipErrorInvalidValue;
  switch (storage) {
    case STORE_FP64:
      return launch_batch_nm<double>(nm, table, first, n_active, items, j, tx, ty, max_stride, general, streaming,
                                     stream);
    case STORE_FP32:
      return launch_batch_nm<float>(nm, table, first, n_active, items, j, tx, ty, max_stride, general, streaming,
                                    stream);
    case STORE_BF16:
      return launch_batch_nm<bf16>(nm, table, first, n_active, items, j, tx, ty, max_stride, general, streaming,
                                   stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace starmap
