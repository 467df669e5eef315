// The shape of a matrix's row tiles, from samples of its rows (host code).
#pragma once

#include <algorithm>
#include <vector>

#include "row_tiles.h"

namespace ld {

// A set of column indices below n.
class ColumnSet {
 public:
  explicit ColumnSet(int64_t n) : bits_((size_t)(n + 63) / 64, 0) {}
  // true where c was not in it
  bool add(int32_t c) {
    uint64_t& w = bits_[(size_t)c >> 6];
    const uint64_t m = uint64_t(1) << (c & 63), old = w;
    w |= m;
    return !(old & m);
  }
  // true where c was in it
  bool remove(int32_t c) {
    uint64_t& w = bits_[(size_t)c >> 6];
    const uint64_t m = uint64_t(1) << (c & 63), old = w;
    w &= ~m;
    return (old & m) != 0;
  }

 private:
  std::vector<uint64_t> bits_;
};

// Calls f with the column of every entry of a tile's rows.
template <typename F>
inline void for_tile_columns(int64_t n, const int32_t* rp, const int32_t* ci, const TileShape& s,
                             int64_t tile, F f) {
  const int64_t ng = (n + kRowGroup - 1) / kRowGroup;
  for (int k = 0; k < kTileGroups; ++k) {
    const int64_t g = tile_group(s, ng, tile, k);
    if (g < 0) continue;
    const int64_t r0 = g * kRowGroup, r1 = std::min(n, r0 + kRowGroup);
    for (int32_t q = rp[r0]; q < rp[r1]; ++q) f(ci[q]);
  }
}

// Distinct columns of 8 sampled tiles of the given shape, per tile, and the part
// of them that the next tile has too (`shared`, may be null).  `set` is empty
// before and after.
inline double sample_tiles(int64_t n, const int32_t* rp, const int32_t* ci, const TileShape& s,
                           ColumnSet& set, double* shared = nullptr) {
  const int ns = (int)std::min<int64_t>(s.ntile, 8);
  int64_t total = 0, common = 0;
  for (int i = 0; i < ns; ++i) {
    const int64_t tile = (2 * i + 1) * s.ntile / (2 * ns);
    for_tile_columns(n, rp, ci, s, tile, [&](int32_t c) { total += set.add(c); });
    if (shared && tile + 1 < s.ntile)
      for_tile_columns(n, rp, ci, s, tile + 1, [&](int32_t c) { common += set.remove(c); });
    for_tile_columns(n, rp, ci, s, tile, [&](int32_t c) { set.remove(c); });
  }
  if (shared) *shared = total > 0 ? (double)common / (double)total : 0.0;
  return ns > 0 ? (double)total / ns : 0.0;
}

// The tile shape: consecutive groups, or (a grid's rows in natural order) 4
// groups on each of 4 lines where a sample of tiles then has a smaller union.
// The line stride is the offset from a middle row to the centre of its next
// run of consecutive columns (every row holds its diagonal entry).  The sample
// takes one step per entry of its 8 (16) tiles: sorting their columns instead
// made the creation of a grid covariance of 100 x 120 rows 0.6 ms longer and,
// with 419 entries per row, of 200 x 300 rows 5 ms.
inline TileShape choose_tile_shape(int64_t n, const int32_t* rp, const int32_t* ci) {
  TileShape best = make_tile_shape(n, 0, 0);
  const int64_t row = n / 2;
  int32_t k = rp[row];
  const int32_t end = rp[row + 1];
  while (k < end && ci[k] <= row) ++k;
  while (k < end && ci[k] == ci[k - 1] + 1) ++k;  // the diagonal's run
  if (k < end) {
    int32_t q = k;
    while (q + 1 < end && ci[q + 1] == ci[q] + 1) ++q;
    const int64_t stride = ((int64_t)ci[k] + ci[q]) / 2 - row;
    const int64_t sg = (stride + kRowGroup / 2) / kRowGroup;
    if (sg >= 4) {
      const TileShape s = make_tile_shape(n, sg, 4);
      ColumnSet set(n);
      if (s.sg > 0 && sample_tiles(n, rp, ci, s, set) < sample_tiles(n, rp, ci, best, set))
        best = s;
    }
  }
  return best;
}

}  // namespace ld
