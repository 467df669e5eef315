// Chunks of rows in bands, one eighth of a stride per XCD (host and device
// code; the tests compile this header for the host alone).
#pragma once

#include "row_tiles.h"  // LD_HOST_DEVICE

namespace ld {

// On a 3-D grid the rows P = N^2 apart are neighbours, and a product that
// sweeps the rows in order over all XCDs gathers them in another XCD than the
// one that has them: every plane then enters three L2s.  Here the chunks of
// each run of P rows are cut into 8 bands, band k = 8 p + x of the matrix
// belongs to XCD x, and its blocks walk their bands p = 0, 1, ...: rows P
// apart meet in one L2, and only the band's edges are gathered twice.
// Band k is chunks [e(k), e(k + 1)), e(k) = floor(k * m / 2^kBandShift): any
// P will do, bands differ by at most one chunk, and `c` is the largest.
constexpr int kBandShift = 20;
struct BandMap {
  uint64_t m = 0;  // chunks per band times 2^kBandShift
  int c = 0;       // 0: no bands
};
inline BandMap make_band_map(int64_t stride, int rows_per_chunk) {
  BandMap b;
  b.m = ((uint64_t)stride << kBandShift) / (uint64_t)(8 * rows_per_chunk);
  b.c = (int)((b.m + (1u << kBandShift) - 1) >> kBandShift);
  return b;
}

// One block's walk: block bk of nbk (a multiple of 8; block b runs on XCD
// b % 8) takes every (nbk / 8)-th slot of its XCD's bands, c slots per band.
struct BandWalk {
  uint64_t m;
  int c, off = 0, band = 0, doff = 0, dband = 0;
  LD_HOST_DEVICE inline BandWalk(const BandMap& b, int bk, int nbk) : m(b.m), c(b.c) {
    if (c == 0) return;
    const int w = bk >> 3, nw = nbk >> 3;
    const int p = w / c;
    off = w - p * c;
    band = 8 * p + (bk & 7);
    dband = nw / c;
    doff = nw - dband * c;
    dband *= 8;
  }
  // the next chunk, or nchunk at the end (slots past a band's last chunk are
  // passed over)
  LD_HOST_DEVICE inline int next(int nchunk) {
    for (;;) {
      const int ch = (int)((uint64_t)band * m >> kBandShift) + off;
      const int hi = (int)((uint64_t)(band + 1) * m >> kBandShift);
      if (ch - off >= nchunk) return nchunk;
      band += dband;
      off += doff;
      if (off >= c) {
        off -= c;
        band += 8;
      }
      if (ch < hi && ch < nchunk) return ch;
    }
  }
};

}  // namespace ld
