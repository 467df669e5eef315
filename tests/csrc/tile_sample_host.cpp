// Host driver for the choice of the tile shape: reads n, nnz, the row pointers
// and the columns; prints gx, sg and, for consecutive groups and for 4 groups
// on each of 4 lines of every given stride (in groups), the sampled columns.
#include <cstdio>

#include "tile_sample.h"

int main() {
  long long n, nnz;
  int ns;
  while (std::scanf("%lld %lld %d", &n, &nnz, &ns) == 3) {
    std::vector<int> sg((size_t)ns), rp((size_t)n + 1), ci((size_t)nnz);
    for (int& v : sg)
      if (std::scanf("%d", &v) != 1) return 1;
    for (int& v : rp)
      if (std::scanf("%d", &v) != 1) return 1;
    for (int& v : ci)
      if (std::scanf("%d", &v) != 1) return 1;
    const ld::TileShape s = ld::choose_tile_shape(n, rp.data(), ci.data());
    std::printf("%d %d", s.gx, s.sg);
    ld::ColumnSet set(n);
    for (int v : sg) {
      const ld::TileShape t = ld::make_tile_shape(n, v, 4);
      // twice: the set is empty again
      ld::sample_tiles(n, rp.data(), ci.data(), t, set);
      std::printf(" %.17g", ld::sample_tiles(n, rp.data(), ci.data(), t, set));
    }
    std::printf("\n");
  }
  return 0;
}
