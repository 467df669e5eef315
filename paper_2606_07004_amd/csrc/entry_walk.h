// Walks over a CSR row's entries by several lanes (host and device code; the
// tests compile this header for the host alone).
#pragma once

#include "row_tiles.h"  // LD_HOST_DEVICE

namespace ld {

// Entries kb + l, kb + l + L, ... of the row [kb, ke), four at a time by
// four(k) (k, k + L, k + 2 L, k + 3 L), the remaining ones by one(k).  A row
// may end at 2^31 - 1, the largest entry count of a matrix, and the index one
// step past an entry is then no int: positions are unsigned.
template <typename F4, typename F1>
LD_HOST_DEVICE inline void lane_entries(int kb, int ke, int l, int L, F4 four, F1 one) {
  const unsigned e = (unsigned)ke, d = (unsigned)L;
  unsigned k = (unsigned)kb + (unsigned)l;
  for (; k + 3 * d < e; k += 4 * d) four(k);
  for (; k < e; k += d) one(k);
}

}  // namespace ld
