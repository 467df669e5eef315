// Row groups of a CSR matrix and the tiles they form (host and device code;
// the tests compile this header for the host alone).
#pragma once

#include <limits.h>
#include <stdint.h>

#if defined(__HIPCC__)
#define LD_HOST_DEVICE __host__ __device__
#else
#define LD_HOST_DEVICE
#endif

namespace ld {

constexpr int kRowGroup = 4;  // consecutive rows of a group

// Tiles of kTileGroups row groups (k_rowtile.hip): the groups of a tile are
// gx consecutive ones on kTileGroups / gx consecutive lines of sg groups
// (band_tiles tiles, tpb per band of lines), the groups from rest0 on (all of
// them with sg = 0) kTileGroups consecutive ones.
constexpr int kTileGroups = 16;
constexpr int kTileMaxUnion = 1248;  // union columns of a tile (160 KB of LDS at 128 bytes each)
constexpr int kTileLoadRows = 64;    // ust is a multiple: union rows a block loads at a time (most)
// unused entries past the last group's in val, val64 and lidx: a wave reads
// its four groups' entries up to the longest one's, in rounds of 16
constexpr int kTilePad = kTileMaxUnion + 32;
struct TileShape {
  int gx = kTileGroups, sg = 0, tpb = 1;
  int64_t band_tiles = 0, rest0 = 0, ntile = 0;
};
// Group k of a tile, or -1.  With sg > 0 the groups form lines of sg (the
// matrix's line stride over kRowGroup): a tile is gx consecutive groups of
// kTileGroups / gx consecutive lines; groups past the last whole band of
// lines, and all of them with sg = 0, are taken kTileGroups at a time.
LD_HOST_DEVICE inline int64_t tile_group(const TileShape& s, int64_t ng, int64_t tile, int k) {
  const int ly = kTileGroups / s.gx;
  if (tile < s.band_tiles) {
    // ng < 2^29: 32-bit arithmetic
    const int band = (int)tile / s.tpb, q = (int)tile - band * s.tpb;
    const int line = k / s.gx, x = q * s.gx + (k - line * s.gx);
    return x < s.sg ? (band * ly + line) * s.sg + x : -1;
  }
  const int64_t g = s.rest0 + (tile - s.band_tiles) * kTileGroups + k;
  return g < ng ? g : -1;
}

// The tile shape with lines of line_groups groups, gx of them per tile and
// line (0: consecutive groups).
inline TileShape make_tile_shape(int64_t n, int64_t line_groups, int gx) {
  const int64_t ng = (n + kRowGroup - 1) / kRowGroup;
  TileShape s{};
  s.gx = kTileGroups;
  s.tpb = 1;
  if (line_groups > 0 && line_groups <= INT_MAX && gx >= 1 && gx < kTileGroups &&
      kTileGroups % gx == 0) {
    const int ly = kTileGroups / gx;
    const int64_t bands = ng / (ly * line_groups);
    if (bands > 0) {
      s.gx = gx;
      s.sg = (int)line_groups;
      s.tpb = (int)((line_groups + gx - 1) / gx);
      s.band_tiles = bands * s.tpb;
      s.rest0 = bands * ly * line_groups;
    }
  }
  s.ntile = s.band_tiles + (ng - s.rest0 + kTileGroups - 1) / kTileGroups;
  return s;
}

}  // namespace ld
