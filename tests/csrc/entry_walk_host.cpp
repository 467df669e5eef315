// Host driver for the walk over a row's entries: reads the row's ends and the
// lanes; prints, lane by lane, the entries that the lane takes, each lane's
// list ended by -1 (-2: more entries than the row has).
#include <cstdio>
#include <cstdlib>

#include "entry_walk.h"

int main() {
  int kb, ke, L;
  while (std::scanf("%d %d %d", &kb, &ke, &L) == 3) {
    for (int l = 0; l < L; ++l) {
      long long left = (long long)ke - kb + 1;
      auto put = [&](long long k) {
        if (left-- > 0) std::printf("%lld ", k);
        if (left < 0) {
          std::printf("-2\n");
          std::exit(0);
        }
      };
      ld::lane_entries(
          kb, ke, l, L,
          [&](auto k) {
            for (int u = 0; u < 4; ++u) put((long long)k + u * L);
          },
          [&](auto k) { put((long long)k); });
      std::printf("-1 ");
    }
    std::printf("\n");
  }
  return 0;
}
