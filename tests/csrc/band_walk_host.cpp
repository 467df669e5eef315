// Host driver for the band walk of the product: reads n rows, the stride, the
// rows per chunk and the blocks; prints the chunks per band and, block by
// block, the chunks that the block takes, each block's list ended by -1.
#include <cstdio>

#include "band_walk.h"

int main() {
  long long n, stride;
  int rpc, nbk;
  while (std::scanf("%lld %lld %d %d", &n, &stride, &rpc, &nbk) == 4) {
    const ld::BandMap b = ld::make_band_map(stride, rpc);
    const int nchunk = (int)((n + rpc - 1) / rpc);
    std::printf("%d", b.c);
    for (int bk = 0; bk < nbk; ++bk) {
      ld::BandWalk w(b, bk, nbk);
      for (int ch = w.next(nchunk); ch < nchunk; ch = w.next(nchunk)) std::printf(" %d", ch);
      std::printf(" -1");
    }
    std::printf("\n");
  }
  return 0;
}
