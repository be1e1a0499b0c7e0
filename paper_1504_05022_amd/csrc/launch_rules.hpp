// Rules that size launches.  Host code only, without the HIP headers.
#pragma once

#include <stdint.h>

namespace spg {

// HIP takes fewer than 2^32 threads in a dimension of a launch.
constexpr int64_t kLaunchThreads = (int64_t(1) << 32) - 1;

constexpr int CP_NT = 256;   // threads per work-group of the copies into C
constexpr int CP_ROWS = 32;  // short rows per wavefront, at most

// Threads of a copy of `rows` rows, r per wavefront.
inline int64_t copy_threads(int64_t rows, int r) {
  const int64_t per = int64_t(CP_NT / 64) * r;  // rows per work-group
  return (rows + per - 1) / per * CP_NT;
}

// Rows per wavefront for `rows` rows of `products` products: about 320 of
// them, so that a wavefront's passes can all be in flight (32 rows each,
// whatever their length, before: 20 banded products 453 us, now 370; the
// short rows of a power-law square 83 and 68; C of 300000 narrow rows 231 and
// 184), more rows where they are tiny (9 products: 32 rows 22 us, two 53), and
// four wavefronts per SIMD or more; no fewer rows than a launch can hold.
inline int copy_rows(int64_t rows, int64_t products) {
  int r = CP_ROWS;
  while (r > 2 &&
         (static_cast<int64_t>(r) * products > 320 * rows || rows < 4096 * static_cast<int64_t>(r)) &&
         copy_threads(rows, r / 2) <= kLaunchThreads)
    r /= 2;
  return r;
}

// The batch's copy: work-groups per row tile (a problem's rows in tiles of
// tile_rows, the last or only one of each in part).  As many as the tiles'
// rows fill on average, r per wavefront: one for every r rows a tile could hold
// launches up to 32 for a problem of one row (10000 problems of five rows: 828
// us, now 52).  A work-group takes the tile's further rows in turn.
inline int copy_parts(int64_t tiles, int64_t rows, int r, int tile_rows) {
  const int64_t per = int64_t(CP_NT / 64) * r;
  int64_t parts = (rows + tiles * per - 1) / (tiles * per);
  const int64_t most = kLaunchThreads / (CP_NT * tiles);
  if (parts > tile_rows / per) parts = tile_rows / per;
  if (parts > most) parts = most;
  return parts > 1 ? static_cast<int>(parts) : 1;
}

// The short rows' launches: one per capacity class with rows, but that a class
// of at most kFewRows joins the next one with rows, of at most eight times its
// capacity, and a class joined by others, with at most kFewRows in all, joins
// the next one in turn.  Their rows then sort with idle lanes, up to a row of one
// product in a kernel for 512, but there are few of them and a launch costs more:
// 100 rows at each of 37 sizes from 1 to 500 take 42 us and 105 in a one-shot
// batch, 45 and 113 where no row is taken beyond eight times its capacity;
// the replay of one banded problem of 60000 rows 38 and 46.
constexpr int64_t kFewRows = 2048;

// rows[c], cap[c] (ascending): rows and capacity of class c; to[c]: the class
// whose kernel takes them.
template <int N> void join_classes(int n, const int64_t (&rows)[N], const int (&cap)[N], int (&to)[N]) {
  int64_t held[N];
  for (int c = 0; c < n; ++c) held[c] = rows[c];
  for (int c = 0; c < n; ++c) {
    to[c] = c;
    if (held[c] == 0 || held[c] > kFewRows) continue;
    int d = c + 1;
    while (d < n && held[d] == 0) ++d;
    if (d == n || cap[d] > 8 * cap[c]) continue;
    held[d] += held[c];
    to[c] = d;
  }
  for (int c = n; c-- > 0;) to[c] = to[to[c]];
}

// Entries of A per wavefront of the gradient kernel: `full`, or as few as give
// 2048 wavefronts (eight per CU), with at least 384 products (the loads that
// one has in flight) on average.  One row of 100 entries, 100 products each:
// dA 84 us in one wavefront, 11 in 25.
inline int grad_chunk(int full, int64_t nnz, int64_t products) {
  int ch = full;
  while (ch > 1 && nnz < int64_t(2048) * ch &&
         static_cast<double>(products) * (ch / 2) >= 384.0 * static_cast<double>(nnz))
    ch /= 2;
  return ch;
}

}  // namespace spg
