// search_device.h -- the neighbourhood search of a row by a group of lanes.
//
// N(i) = the F-points reachable from C-point i by a walk of at most ell edges
// (u -> v with u != v, a stored nonzero a_uv and strong_edge) whose interior
// vertices are F-points.  The points met are kept in an open-addressing hash
// table in LDS and listed in the order found, so the points first reached at
// one distance form a run [lo, hi) that the next level expands.  The order
// depends on timing, the set does not; the caller writes every point at its
// rank among the row's points, so N(i) comes out sorted.
//
// Base patterns: classical (the first level is row i's), aggregates (mrp / mem
// replace the first level), or the literal reading of S^{ell-1} T with
// T = [S_fc, I] (the second level also expands i; C-points may be interior
// vertices from the second level on and are left out of the result; i never
// enters).
//
// Why a hash table: the search before this one held the set in one thread's
// registers (32 compares per candidate, about 190 VGPRs); a nine-point row at
// distance 2 has 72 candidates for 24 points.  The set of a group in LDS costs
// one compare-and-swap per candidate whatever the size, and any number of
// lanes can feed it.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "clair_device.h"

namespace clair {

namespace {

// LDS of a group: up to CAP points, H hash slots (a power of two)
template <int CAP, int H>
struct SearchBuf {
  static_assert((H & (H - 1)) == 0 && H >= 2 * CAP && CAP % 4 == 0, "table size");
  alignas(16) int tab[H];     // -1: free
  alignas(16) int list[CAP];  // the points in the order found, INT32_MAX beyond
  int cnt;        // points found (above CAP: more than the list holds)
};

constexpr int kSearchIn = 4;

// lanes of a group of G: a part of a wavefront, a wavefront, or (G = 256) the
// workgroup
template <int G>
__device__ __forceinline__ void group_sync() {
  if constexpr (G <= 64) wave_sync(); else __syncthreads();
}

template <int CAP, int H>
__device__ __forceinline__ bool search_over(const SearchBuf<CAP, H>& b) {
  return __hip_atomic_load(&b.cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > CAP;
}

// v into the set (over its bound the row is left to a larger search and the
// set's contents do not matter; the probes are bounded by the table)
template <int CAP, int H>
__device__ __forceinline__ void search_insert(SearchBuf<CAP, H>& b, int v) {
  int h = (int)(((uint32_t)v * 2654435761u) >> 16) & (H - 1);
  for (int probe = 0; probe < H; ++probe) {
    const int prev = atomicCAS(&b.tab[h], -1, v);
    if (prev == v) return;
    if (prev == -1) {
      const int pos = atomicAdd(&b.cnt, 1);
      if (pos < CAP) b.list[pos] = v;
      return;
    }
    h = (h + 1) & (H - 1);
  }
  b.cnt = CAP + 1;  // every slot was taken: over the bound
}

// the points one step from u, read from the graph's row by `stride` lanes
// (this one is number sub)
template <int CAP, int H>
__device__ __forceinline__ void search_row(SearchBuf<CAP, H>& b, const GDesc& d, int u, int i, bool allow_c, int sub,
                                           int stride) {
  const int e1 = d.grp[u + 1];
  for (int e = d.grp[u] + sub; e < e1 && !search_over(b); e += stride) {
    const int k = d.gci[e];
    const double x = d.gva[e];
    if ((unsigned)k >= (unsigned)d.n || k == u || k == i || x == 0.0) continue;
    if ((d.cf[k] == 0 || allow_c) && strong_edge(x, k, d.theta, d.cmax)) search_insert(b, k);
  }
}

// The search; every lane of the group calls (lane = 0..G-1).  lw = log2 of the
// compact adjacency's width, or 0 to read the graph's rows.  Returns the
// number of points listed in b.list (C-points included in the literal
// reading), or -1 when there are more than CAP.
template <int G, int CAP, int H>
__device__ __forceinline__ int group_search(SearchBuf<CAP, H>& b, const GDesc& d, int i, int lw, int lane) {
  static_assert(G >= 8, "a compact adjacency row is read by up to eight lanes of one group");
  for (int t = lane; t < H; t += G) b.tab[t] = -1;
  for (int t = lane; t < CAP; t += G) b.list[t] = INT32_MAX;
  if (lane == 0) b.cnt = 0;
  group_sync<G>();
  const bool literal = d.literal != 0 && d.ell >= 3;  // (the readings agree up to distance 2)
  // level 1
  if (d.agg_rp) {
    for (int e = d.agg_rp[i] + lane; e < d.agg_rp[i + 1]; e += G) search_insert(b, d.agg_list[e]);
  } else if (lw && d.fadj) {
    if (lane < (1 << lw)) {
      const int v = d.fadj[((int64_t)i << lw) + lane];
      const int first = __shfl(v, (threadIdx.x & 63) & ~((1 << lw) - 1), 64);
      if (first == kAdjOverflow) search_row(b, d, i, i, false, lane, 1 << lw);
      else if (v >= 0) search_insert(b, v);
    }
  } else {
    search_row(b, d, i, i, false, lane, G);
  }
  group_sync<G>();
  int lo = 0;
  for (int L = 2; L <= d.ell; ++L) {
    const int hi = b.cnt;
    if (hi > CAP) return -1;  // group-uniform
    const bool allow_c = literal && L < d.ell;
    const bool with_i = literal && L == 2;
    if (lo == hi && !with_i) break;
    group_sync<G>();  // every lane has read the count
    if (with_i) search_row(b, d, i, i, allow_c, lane, G);
    if (lw && d.fadj && !literal) {
      const int m = (hi - lo) << lw;
      // kSearchIn slots per lane in flight at once (one at a time, a level
      // waits for memory once per G slots)
      const int sub = lane & ((1 << lw) - 1);
      for (int t0 = lane; t0 < m; t0 += G * kSearchIn) {
        int u[kSearchIn], v[kSearchIn];
#pragma unroll
        for (int r = 0; r < kSearchIn; ++r) {
          const int t = t0 + G * r;
          u[r] = t < m ? b.list[lo + (t >> lw)] : -1;
        }
#pragma unroll
        for (int r = 0; r < kSearchIn; ++r) v[r] = u[r] >= 0 ? d.fadj[((int64_t)u[r] << lw) + sub] : -1;
#pragma unroll
        for (int r = 0; r < kSearchIn; ++r) {
          const int first = __shfl(v[r], (threadIdx.x & 63) & ~((1 << lw) - 1), 64);
          if (first == kAdjOverflow) search_row(b, d, u[r], i, false, sub, 1 << lw);
          else if (v[r] >= 0 && !search_over(b)) search_insert(b, v[r]);
        }
      }
    } else {
      for (int t = lane / 8; lo + t < hi; t += G / 8)
        search_row(b, d, b.list[lo + t], i, allow_c, lane % 8, 8);
    }
    group_sync<G>();
    lo = hi;
  }
  const int n = b.cnt;
  return n > CAP ? -1 : n;
}

// The result of a literal search holds the C-points walked through: they are
// taken out of the list (which keeps gaps, INT32_MAX), the F-points counted.
template <int G, int CAP, int H>
__device__ __forceinline__ int drop_c_points(SearchBuf<CAP, H>& b, const GDesc& d, int n, int lane) {
  if (lane == 0) b.cnt = 0;
  group_sync<G>();
  for (int t = lane; t < n; t += G) {
    if (d.cf[b.list[t]] != 0) b.list[t] = INT32_MAX;
    else atomicAdd(&b.cnt, 1);
  }
  group_sync<G>();
  return b.cnt;
}

// rank of v among the listed points (its place in the sorted N(i))
template <int CAP, int H>
__device__ __forceinline__ int search_rank(const SearchBuf<CAP, H>& b, int n, int v) {
  const int4* l = reinterpret_cast<const int4*>(b.list);
  int r = 0;
#pragma unroll 4
  for (int t = 0; t < (n + 3) / 4; ++t) {
    const int4 q = l[t];
    r += (q.x < v ? 1 : 0) + (q.y < v ? 1 : 0) + (q.z < v ? 1 : 0) + (q.w < v ? 1 : 0);
  }
  return r;
}

}  // namespace

}  // namespace clair
