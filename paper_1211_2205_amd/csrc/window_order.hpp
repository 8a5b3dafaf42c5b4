// How a register-window sweep's workgroups are numbered: the tiles and m ranges
// of a sweep, and the order in which a workgroup's number walks them.  Plain C++
// shared by the launch code, the kernel (constexpr functions run on the device
// too) and the test that enumerates it on the host.
#pragma once

#include <algorithm>
#include <cstdint>

namespace starmap {

struct WindowGrid {
  int ntx, nty, nchunks;  // tiles per axis, m ranges
};

// Division of 0 <= n < 2^31 by a constant: n / d = n m >> s.
struct Divisor {
  uint32_t m = 0, s = 0;
};
// 2^s / d rounded up, with s so large (2^31 d at least) that the error, below
// one part in 2^31, changes no quotient of a number below 2^31.
constexpr Divisor divisor(int d) {
  Divisor r;
  d = d < 1 ? 1 : d;
  r.s = 31;
  while ((int64_t(1) << (r.s - 31)) < d) ++r.s;
  r.m = uint32_t((uint64_t(1) << r.s) / uint32_t(d) + 1);
  return r;
}
// Quotients by constants of a launch as multiplications: the six divisions
// between a workgroup's number and its first load, each some 28 dependent
// instructions, had been a tenth of a small sweep (P_3 100^2 FP64 4.14 -> 3.78
// us, P_9 317 x 203 FP32 8.1 -> 7.5; with the plane numbers as arguments, not
// read from a table first, 3.63 and 7.2).
constexpr int divide(int n, const Divisor& d) { return int((uint64_t(uint32_t(n)) * d.m) >> d.s); }

// How a workgroup's number becomes an m range and a tile: groups of gsize tiles
// (the last may be smaller), a group's ranges one after another, a range's tiles.
struct WindowOrder {
  Divisor per, by_gsize;     // numbers per group and per range of a group
  Divisor band, rows, last;  // tiles per strip; a strip's width, the last strip's
  int ntx, nty, nchunks, strip, gsize, groups;
};
// Numbers in all.
constexpr int window_items(const WindowOrder& o) { return o.groups * o.gsize * o.nchunks; }

// Tiles of one group, about: the workgroups of a group are numbered range by
// range, and the ranges of low m, which have the most orders, come first.
// Ranges as the inner index, as the LDS kernel takes them (its ranges share
// staged lines), leave the long ranges to the end of a launch: P_39 1000^2 FP32
// 1100 against 1026 us, P_31 256^2 53 against 48 us.  One group over the whole
// of a large grid loses the overlap of the ranges' shared planes: 1040 us.
constexpr int kWindowGroup = 512;
constexpr int kXcds = 8;

constexpr WindowOrder window_order(const WindowGrid& g, int strip) {
  WindowOrder o{};
  o.ntx = g.ntx;
  o.nty = g.nty;
  o.nchunks = g.nchunks;
  o.strip = strip;
  // groups of equal size, in whole turns of the XCDs (rounded up so, many groups
  // hold more than all tiles: as many as it takes, and none is empty)
  const int ntiles = g.ntx * g.nty;
  o.groups = std::max(1, (ntiles + kWindowGroup / 2) / kWindowGroup);
  const int per = (ntiles + o.groups - 1) / o.groups;
  o.gsize = o.groups > 1 ? (per + kXcds - 1) / kXcds * kXcds : ntiles;
  o.groups = (ntiles + o.gsize - 1) / std::max(o.gsize, 1);
  o.per = divisor(o.gsize * g.nchunks);
  o.by_gsize = divisor(o.gsize);
  const int w = strip >= 2 ? strip : strip <= -2 ? -strip : 1;
  const int across = strip <= -2 ? g.nty : g.ntx, along = strip <= -2 ? g.ntx : g.nty;
  o.band = divisor(int(std::min<int64_t>(int64_t(w) * across, 0x7FFFFFFF)));
  o.rows = divisor(w);
  o.last = divisor(along % w);
  return o;
}

// Tiles of a group (the last one may be smaller).
constexpr int group_tiles(const WindowOrder& o, int grp) { return std::min(o.gsize, o.ntx * o.nty - grp * o.gsize); }
// Tile number of member tl < n of a group of n tiles.  Consecutive workgroups run on the chip's XCDs in turn: each takes a run of
// neighbouring tiles, whose shared rows its L2 then holds (P_9 317 x 203 FP32
// 8.2 -> 7.5 us, P_7 280^2 FP64 14.6 -> 14.0, P_39 1000^2 BF16 528 -> 517).
constexpr int tile_number(const WindowOrder& o, int grp, uint32_t n, uint32_t tl) {
  const uint32_t xcd = tl % kXcds;
  return grp * o.gsize + int(xcd * (n / kXcds) + std::min(xcd, n % kXcds) + tl / kXcds);
}

// Tile number t of the order (tile_xy of device.hpp with its divisors).
struct TileAt {
  int x, y;
};
constexpr TileAt tile_at(int t, const WindowOrder& o) {
  const int band = divide(t, o.band);
  if (o.strip >= 2) {
    const int row0 = band * o.strip, rows = std::min(o.strip, o.nty - row0);
    const int r = t - band * (o.strip * o.ntx), q = divide(r, rows == o.strip ? o.rows : o.last);
    return {q, row0 + (r - q * rows)};
  }
  if (o.strip <= -2) {
    const int w = -o.strip, col0 = band * w, cols = std::min(w, o.ntx - col0);
    const int r = t - band * (w * o.nty), q = divide(r, cols == w ? o.rows : o.last);
    return {col0 + (r - q * cols), q};
  }
  return {t - band * o.ntx, band};
}

// Row of the grid that a thread of a tile of ty rows stands on: 2^lbw lanes per
// row.  (Rows times lanes may exceed an int.)
constexpr int row_of(const TileAt& tile, int ty, int lbw, int thread) { return tile.y * ty + (thread >> lbw); }

}  // namespace starmap
