// The order in which the workgroups of a product take its tiles.
#pragma once

#include <hip/hip_runtime.h>

namespace oz2 {

constexpr int kXcds = 8;
constexpr int kCus = 256;   // compute units that the launch rules count with

// Workgroup -> place in the walk over tiles: the hardware deals workgroups
// round-robin to the XCDs; each XCD gets a contiguous range of the walk.
__host__ __device__ __forceinline__ int xcd_place(int bid, int launched) {
  const int xcd = bid % kXcds, loc = bid / kXcds;
  const int per = launched / kXcds, extra = launched % kXcds;
  return xcd * per + (xcd < extra ? xcd : extra) + loc;
}

// The same for launches of one workgroup per CU: every kCus of the walk in a
// round over all XCDs, in which an XCD takes 8 x 4 of 16 x 16 places, so that a
// round reads 32 panels of the operands from memory and not 12 for each XCD.
__host__ __device__ __forceinline__ int round_place(int bid, int launched) {
  const int first = bid & ~(kCus - 1);
  if (first + kCus > launched) return first + xcd_place(bid - first, launched - first);
  const int xcd = bid % kXcds, loc = (bid - first) / kXcds;
  return first + 16 * (4 * (xcd >> 1) + (loc >> 3)) + 8 * (xcd & 1) + (loc & 7);
}

// Place -> (slice z, tile tx, ty): slice by slice, and in a slice groups of
// `group` tile rows (the 32 workgroups of an XCD share their panels in its L2).
struct TilePos {
  int z, tx, ty;
};
__host__ __device__ __forceinline__ TilePos tile_at(int place, int tiles_x, int tiles_y,
                                                    int group = 8) {
  const int per_slice = tiles_x * tiles_y;
  const int z = place / per_slice;
  int t = place % per_slice;
  const int g = t / (group * tiles_y);
  const int gx0 = g * group;
  const int gsz = group < tiles_x - gx0 ? group : tiles_x - gx0;
  t -= g * group * tiles_y;
  return {z, gx0 + t % gsz, t / gsz};
}

// Parts of each tile of the last round (0: none) for `tiles` 256x256 tiles: the
// last round's tiles are cut when there are at most half a round of them (in
// two) or a quarter (in four); with more, the parts make a second round of
// their own.  14 products of 2048^3 (896 tiles, 128 in the last round): 120.5
// us whole, 113 in parts.
inline int tail_parts(long tiles) {
  const long rem = tiles % kCus;
  if (tiles < kCus || rem == 0 || 2 * rem > kCus) return 0;
  return 4 * rem <= kCus ? 4 : 2;
}

}  // namespace oz2
