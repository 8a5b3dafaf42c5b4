// Enumerates the workgroup numbering of register-window sweeps on the host.
//   groups MAX            for every number of tiles up to MAX: groups of gsize
//                         tiles, none of them empty, hold each tile once
//   rows                  tiles of every shape on the last rows that planes of 2^31
//                         bytes leave room for: each row once, in order
//   tiles NTX NTY STRIP   prints "x y" of every tile in the order of the numbers
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "window_order.hpp"

using namespace starmap;

int main(int argc, char** argv) {
  if (argc == 3 && !std::strcmp(argv[1], "groups")) {
    for (int n = 1; n <= std::atoi(argv[2]); ++n) {
      const WindowOrder o = window_order({n, 1, 3}, 1);
      if (window_items(o) != o.groups * o.gsize * 3 || (o.groups - 1) * o.gsize >= n || o.groups * o.gsize < n) {
        std::printf("%d tiles: %d groups of %d\n", n, o.groups, o.gsize);
        return 1;
      }
    }
    return 0;
  }
  if (argc == 2 && !std::strcmp(argv[1], "rows")) {
    const int last = int((int64_t(1) << 31) / (64 * 4));  // rows of 64 values, the shortest, of four bytes
    for (int threads = 64; threads <= 512; threads *= 2)
      for (int lbw = 3; (1 << lbw) <= threads; ++lbw) {
        const int ty = threads >> lbw;
        for (int y = last / ty - 2; y <= last / ty; ++y)
          for (int t = 0; t < threads; ++t)
            if (row_of({0, y}, ty, lbw, t) != y * ty + t / (1 << lbw)) {
              std::printf("%d threads, %d per row, tile row %d: %d\n", threads, 1 << lbw, y,
                          row_of({0, y}, ty, lbw, t));
              return 1;
            }
      }
    return 0;
  }
  if (argc == 5 && !std::strcmp(argv[1], "tiles")) {
    const WindowOrder o = window_order({std::atoi(argv[2]), std::atoi(argv[3]), 2}, std::atoi(argv[4]));
    for (int item = 0; item < window_items(o); ++item) {  // as the batched kernel takes them apart
      const int grp = divide(item, o.per), within = item - grp * (o.gsize * o.nchunks);
      const int chunk = divide(within, o.by_gsize), tl = within - chunk * o.gsize, n = group_tiles(o, grp);
      if (tl >= n) continue;
      const TileAt at = tile_at(tile_number(o, grp, n, tl), o);
      std::printf("%d %d %d\n", chunk, at.x, at.y);
    }
    return 0;
  }
  return 2;
}
