// Host driver for the tile shapes of the row-tile product: reads n, the line
// stride in groups and the groups per line; prints gx, sg and, tile by tile,
// the groups of each tile (-1 where a tile has fewer).
#include <cstdio>

#include "row_tiles.h"

int main() {
  long long n, sg;
  int gx;
  while (std::scanf("%lld %lld %d", &n, &sg, &gx) == 3) {
    const ld::TileShape s = ld::make_tile_shape(n, sg, gx);
    const long long ng = (n + ld::kRowGroup - 1) / ld::kRowGroup;
    std::printf("%d %d %lld", s.gx, s.sg, (long long)s.ntile);
    for (long long t = 0; t < s.ntile; ++t)
      for (int k = 0; k < ld::kTileGroups; ++k)
        std::printf(" %lld", (long long)ld::tile_group(s, ng, t, k));
    std::printf("\n");
  }
  return 0;
}
