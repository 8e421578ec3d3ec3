// launch_rules.h -- which kernels a call launches for the block sizes the host
// knows of.  Plain C++ (no HIP), so that the rules can be checked by themselves.
#pragma once

#include <algorithm>

namespace clair {

// Instances of k_tile, each for blocks of up to 12, 16, 20, 24, 28 or 32 points.
inline int tile_bound(int points) { return std::max(12, (std::min(points, 32) + 3) / 4 * 4); }

// The instances a call launches for rows of up to `points` points.
struct TilePick {
  int first;   // its bound
  int second;  // the bound of a further one, which runs instead where the batch's largest block is above `first`
               // (0: none)
};

// points: the largest block last read back.  sized: it is this batch's own.
// Otherwise (asynchronous calls) larger blocks may come, and rows above the
// instance's bound go to k_rows_wg one workgroup each (40,000 rows of 14 points:
// 6.6 ms, 0.13 here), so a second instance reaches as far as `reach`: the device
// knows the largest block and runs one of the two (the other one's empty launch:
// 4 us).
inline TilePick tile_pick(int points, int reach, bool sized) {
  const int first = tile_bound(points);
  const int wide = tile_bound(reach);
  if (sized || first >= wide) return {first, 0};
  return {first, wide};
}

// how far an unsized call's bin B reaches: the block bounds 16, 20, 24 and 32
inline int bin_b_reach(int points) { return points <= 16 ? 16 : points <= 24 ? tile_bound(points) : 32; }

}  // namespace clair
