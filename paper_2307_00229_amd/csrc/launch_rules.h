// launch_rules.h -- which kernels a call launches for the block sizes the host
// knows of.  Plain C++ (no HIP), so that the rules can be checked by themselves.
#pragma once

#include <stdint.h>

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

// Fine points per workgroup of the chunk-wise passes (symbolic search,
// projection): the tuning's, halved while the batch has fewer workgroups than
// CUs, though not below 64.  The passes then fill the chip on small inputs too;
// the results do not depend on the chunk.  150^2 at distance 5: its two
// 22-workgroup passes took 254 us with 1024 points (search 124, projection 130)
// and the projection takes 39 with 64; from about 262,000 points on the chunk is
// the tuning's own.  (Two workgroups a CU were tried: more of them meet at the
// matrix's counters and rows take more steps to find their chunk: 330^2
// five-point, distance 1, numeric pass 31 and projection 14 us against 25 and 12;
// 40^3 seven-point, projection 19 against 13.)
inline int shrunk_chunk(int chunk, int64_t n_total, int cus) {
  while (chunk / 2 >= 64 && n_total < (int64_t)chunk * cus) chunk /= 2;
  return chunk;
}

// What a call's launches were sized for, or what it found: the largest block
// and whether there were rows of bin A, of bin B, for the workgroup solvers, and
// unfinished chunks for the two further searches.
struct CallSizes {
  int points = 0;
  bool rows_a = false, rows_b = false, rows_wg = false, mid = false, big = false;
};

// Whether launches sized for `had` also serve a call that found `got`: no pass
// was left out that has work, its rows of up to 32 points fit the tile, and the
// FP64 scratch (scratch_doubles a slot, 0: none) takes its rows above 64 points,
// which do not fit in LDS.
inline bool launches_hold(const CallSizes& had, const CallSizes& got, int64_t scratch_doubles) {
  if ((got.mid && !had.mid) || (got.big && !had.big)) return false;
  if ((got.rows_a && !had.rows_a) || (got.rows_b && !had.rows_b) || (got.rows_wg && !had.rows_wg)) return false;
  if (tile_bound(got.points) > tile_bound(had.points)) return false;
  return got.points <= 64 || (int64_t)got.points * got.points <= scratch_doubles;
}

// how far an unsized call's bin B reaches: the block bounds 16, 20, 24 and 32
inline int bin_b_reach(int points) { return points <= 16 ? 16 : points <= 24 ? tile_bound(points) : 32; }

}  // namespace clair
