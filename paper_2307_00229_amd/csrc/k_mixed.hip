// k_mixed.hip -- the batched, mixed-precision restriction setup.
//
// Stages (one launch each, over all matrices of a batch):
//   k_adj        the compact adjacency of the search graph (ell >= 2, sparse
//                graphs): for every point, the F-points one step reaches.
//   k_count      symbolic pass per chunk of fine points: the C-points of the
//                chunk; rows at ell = 1 (up to 8 entries) and at ell = 2 over
//                the adjacency sized from a sorted candidate list, by one thread
//                each (up to four edges a point) or by a quad (up to eight), and
//                written to their slot; a chunk with every
//                row sized gets its chunk-local prefix of |N(i)|+1 here;
//                clears the projection's column lists of the chunk.
//   k_count_mid  the other rows of unfinished chunks at distance 1 and 2: one
//                thread per row, up to 32 points in registers (over the
//                adjacency when built), then the chunk's prefix.  Larger rows
//                are queued, unsized.
//   k_count_wide the same at distance 3 and more: sixteen lanes per row up to
//                32 points, a wavefront up to 128, in LDS.
//   k_count_big  one workgroup per queued row: a workgroup-wide search sizes
//                it (queued for the workgroup solver); the last row of a chunk
//                to be sized redoes the chunk's prefix.
//   k_scan       one workgroup: chunk bases -> global row numbers, R offsets,
//                n_c and nnz(R) per matrix, bin sizes, the largest block,
//                capacity check, R.row_ptr[n_c].
//   k_quad8      (k_quad.hip) persistent over the rows, four lanes per row with
//                |N| <= 8: see there.
//   k_tile       (k_tile.hip) sixteen lanes per row with up to 32 points: FP32
//                inverse (Gauss-Jordan) and FP64 iterative refinement of
//                (A[N,N])^T z = -A[i,N]^T, R row write, column lists of the
//                projection.  Rows whose FP32 factorisation is not trusted are
//                queued for k_rows_wg.
//   k_rows8      the one-thread-per-row bin-A solver (group 1).
//   k_rows_gj    (k_block.hip) a workgroup per queued row of 33 to 128 points.
//   k_rows_wg    persistent, one workgroup per queued row: for 33..128 points
//                an FP32 blocked LU with matrix-core trailing updates and FP64
//                refinement; otherwise, or when that does not converge, FP64 LU
//                with partial pivoting (block in LDS, or in global scratch when
//                large).
//   k_colproj    one workgroup per chunk of fine points, one thread per F-point,
//                over the column lists:
//                z_ij -= B_i (sum_k z_kj B_k - B_j) / sum_k B_k^2 per F-entry;
//                counts F-points no row reaches.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <utility>

#include "clair_device.h"
#include "clair_launch.h"
#include "mixed_device.h"
#include "search_device.h"

namespace clair {

namespace {

constexpr int kNT = 256;  // threads per workgroup of the symbolic pass
// workgroup-wide search caps
constexpr int kWN = kMaxBlock;
constexpr int kWC = 4096;

// Workgroup-wide neighbourhood search for rows of any size up to kWN points:
// the same set as group_search (F-points reachable from C-point i by at most ell
// edges with F-points inside the walk).  The entries of a level's frontier
// rows are taken in windows of kWC: each window is sorted (bitonic, in LDS),
// reduced to points that are new (first of their run, not yet in N, not yet
// in this level) and merged into the level.  No bound on the number of
// candidates, so dense coarse-level rows work too.
struct WideBuf {
  int nb0[kWN], nb1[kWN];  // neighbourhood, double buffered, sorted
  int fr[kWN];             // frontier: the previous level's new points, sorted
  int nl[kWN];             // this level's new points so far, sorted
  int dp[kWN + 1];         // prefix of the frontier's row lengths
  int cand[kWC];           // window candidates (sorted in place)
  int kb[kWC];             // kept candidates of the window, sorted
  int sh[kNT];             // scan scratch
};

// Returns |N(i)| with the sorted list in *out, or -1 when it exceeds kWN
// (block-uniform).  Must be called by all kNT threads of the workgroup.
__device__ int block_bfs(int n, int i, int ell, gptr<const int32_t> __restrict__ rp, gptr<const int32_t> __restrict__ ci,
                         gptr<const double> __restrict__ va, gptr<const int8_t> __restrict__ cf, double theta,
                         gptr<const double> __restrict__ cmax, gptr<const int32_t> __restrict__ mrp,
                         gptr<const int32_t> __restrict__ mem, WideBuf& b, int** out, bool literal = false) {
  const int tid = threadIdx.x;
  constexpr int nt = kNT;
  int* cur = b.nb0;
  int* nxt = b.nb1;
  int s = 0;
  int fsz = 1;  // level-0 frontier is {i}
  int d0 = 1;
  if (mrp) {
    // aggregation-based: level 1 is the aggregate's F-points (sorted)
    const int a0 = mrp[i], na = mrp[i + 1] - a0;
    if (na > kWN) return -1;
    for (int t = tid; t < na; t += nt) {
      cur[t] = mem[a0 + t];
      b.fr[t] = mem[a0 + t];
    }
    __syncthreads();
    s = na;
    fsz = na;
    d0 = 2;
  }
  // literal reading (S^{ell-1} T taken as written): the second step also
  // expands i itself, C-points may be interior vertices until the last step
  // (and are dropped at the end), and i never enters
  for (int depth = d0; depth <= ell && (fsz > 0 || (literal && depth == 2)); ++depth) {
    const bool with_i = literal && depth == 2;  // frontier slot fsz is i
    const int fn = fsz + (with_i ? 1 : 0);
    const bool allow_c = literal && depth >= 2 && depth < ell;
    auto fu = [&](int t) { return (depth == 1 || (with_i && t == fsz)) ? i : b.fr[t]; };
    // row lengths of the frontier, prefix
    const int per = (fn + nt - 1) / nt;
    const int t0 = tid * per, t1 = min(t0 + per, fn);
    int sum = 0;
    for (int t = t0; t < t1; ++t) {
      const int u = fu(t);
      sum += rp[u + 1] - rp[u];
    }
    int E;
    int pre = block_exclusive_scan(sum, b.sh, &E);
    for (int t = t0; t < t1; ++t) {
      const int u = fu(t);
      b.dp[t] = pre;
      pre += rp[u + 1] - rp[u];
    }
    if (tid == 0) b.dp[fn] = E;
    __syncthreads();
    int nnl = 0;
    for (int w0 = 0; w0 < E; w0 += kWC) {
      const int wn = min(kWC, E - w0);
      int P = 1;
      while (P < wn) P <<= 1;
      for (int t = tid; t < P; t += nt) {
        int k = INT32_MAX;
        if (t < wn) {
          const int ef = w0 + t;
          int lo = 0, hi = fn - 1;  // last frontier vertex with dp <= ef
          while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (b.dp[mid] <= ef) lo = mid; else hi = mid - 1;
          }
          const int u = fu(lo);
          const int e = rp[u] + (ef - b.dp[lo]);
          const int kk = ci[e];
          if (kk != u && kk != i && (unsigned)kk < (unsigned)n && va[e] != 0.0 && (cf[kk] == 0 || allow_c) &&
              strong_edge(va[e], kk, theta, cmax))
            k = kk;
        }
        b.cand[t] = k;
      }
      __syncthreads();
      for (int kk = 2; kk <= P; kk <<= 1) {
        for (int j = kk >> 1; j > 0; j >>= 1) {
          for (int t = tid; t < P; t += nt) {
            const int x = t ^ j;
            if (x > t) {
              const int a = b.cand[t], c2 = b.cand[x];
              if ((a > c2) == ((t & kk) == 0)) { b.cand[t] = c2; b.cand[x] = a; }
            }
          }
          __syncthreads();
        }
      }
      const int per2 = (P + nt - 1) / nt;
      const int q0 = tid * per2, q1 = min(q0 + per2, P);
      int kept = 0;
      for (int t = q0; t < q1; ++t) {
        const int x = b.cand[t];
        kept += (x != INT32_MAX && (t == 0 || b.cand[t - 1] != x) && find_sorted(cur, s, x) < 0 &&
                 find_sorted(b.nl, nnl, x) < 0) ? 1 : 0;
      }
      int kn;
      int kp = block_exclusive_scan(kept, b.sh, &kn);
      for (int t = q0; t < q1; ++t) {
        const int x = b.cand[t];
        if (x != INT32_MAX && (t == 0 || b.cand[t - 1] != x) && find_sorted(cur, s, x) < 0 &&
            find_sorted(b.nl, nnl, x) < 0)
          b.kb[kp++] = x;
      }
      __syncthreads();
      if (s + nnl + kn > kWN) return -1;
      for (int t = tid; t < nnl; t += nt) nxt[t + lower_bound_i32(b.kb, kn, b.nl[t])] = b.nl[t];
      for (int t = tid; t < kn; t += nt) nxt[t + lower_bound_i32(b.nl, nnl, b.kb[t])] = b.kb[t];
      __syncthreads();
      nnl += kn;
      for (int t = tid; t < nnl; t += nt) b.nl[t] = nxt[t];
      __syncthreads();
    }
    for (int t = tid; t < s; t += nt) nxt[t + lower_bound_i32(b.nl, nnl, cur[t])] = cur[t];
    for (int t = tid; t < nnl; t += nt) {
      nxt[t + lower_bound_i32(cur, s, b.nl[t])] = b.nl[t];
      b.fr[t] = b.nl[t];
    }
    __syncthreads();
    int* tmp = cur;
    cur = nxt;
    nxt = tmp;
    s += nnl;
    fsz = nnl;
  }
  if (literal) {  // the C-points were interior vertices only: keep the F-points, in order
    const int per = (s + nt - 1) / nt;
    const int t0 = tid * per, t1 = min(t0 + per, s);
    int kf = 0;
    for (int t = t0; t < t1; ++t) kf += cf[cur[t]] == 0 ? 1 : 0;
    int f;
    int pos = block_exclusive_scan(kf, b.sh, &f);
    for (int t = t0; t < t1; ++t)
      if (cf[cur[t]] == 0) nxt[pos++] = cur[t];
    __syncthreads();
    *out = nxt;
    return f;
  }
  *out = cur;
  return s;
}

// ---------------------------------------------------------------------------
// validation: CSR sorted, in range; cf is not checked (any nonzero is C)
// ---------------------------------------------------------------------------
__global__ void k_validate(Work w) {
  for (int m = 0; m < w.nmat; ++m) {
    const GDesc d = gview(w.desc[m]);
    for (int r = blockIdx.x * blockDim.x + threadIdx.x; r < d.n; r += gridDim.x * blockDim.x) {
      const int e0 = d.rp[r], e1 = d.rp[r + 1];
      bool bad = (e1 < e0) || e0 < 0 || e1 > d.nnz || (r == 0 && e0 != 0) || (r == d.n - 1 && e1 != d.nnz);
      for (int e = e0; e < e1 && !bad; ++e) {
        const int k = d.ci[e];
        bad = (k < 0 || k >= d.n || (e > e0 && k <= d.ci[e - 1]));
      }
      if (d.grp != d.rp) {  // a strength matrix: sorted rows, indices in range
        const int g0 = d.grp[r], g1 = d.grp[r + 1];
        bad = bad || g1 < g0 || g0 < 0 || (r == 0 && g0 != 0);
        for (int e = g0; e < g1 && !bad; ++e) {
          const int k = d.gci[e];
          bad = (k < 0 || k >= d.n || (e > g0 && k <= d.gci[e - 1]));
        }
      }
      if (bad) flag_row(&w.st[m], ST_INVALID, r);
    }
  }
}

// ---------------------------------------------------------------------------
// symbolic pass
// ---------------------------------------------------------------------------

// The compact adjacency of the matrices whose descriptor carries one: the
// workgroup of logical block b takes 256 points of chunk b / ceil(chunk / 256)
// (the chunk's XCD is the one k_count gives it).  The points' entries are
// consecutive, so the workgroup reads them in tiles of kAdjTile, a thread at a
// time the entries 256 apart (their loads in flight together), and leaves in
// LDS the column of each entry that is an edge to an F-point, -1 for the
// others; then each thread collects its own point's.
//
// Bound: the entries' bytes.  With one thread reading its own row, the lanes of
// a load were 20 and 40 bytes apart and the address unit was the limit
// (64 five-point matrices of 64^2 to 768^2: 221 us, now 196; 2048^2 nine-point
// rows: 190, now 141; 128^3 seven-point rows: 65, now 62).  A tile of 256 times
// five entries: a larger one issues its empty loads (2048: 199, 151 and 63 us;
// 2560: 234, 159 and 74), a smaller one takes two turns for five-point rows
// (1024: 211, 147 and 62).
constexpr int kAdjTile = 1280;

template <int W>
__global__ __launch_bounds__(256) void k_adj(Work w) {
  __shared__ int s_k[kAdjTile];
  const int per = (w.chunk + 255) / 256;
  const int b = xcd_logical_block();
  const int c = b / per;
  const int m = chunk_matrix(w.desc, w.nmat, c);
  const GDesc d = gview(w.desc[m]);
  if (!d.fadj) return;
  const int f0 = (c - d.chunk0) * w.chunk;
  const int f1 = min(f0 + w.chunk, d.n);
  const int u0 = f0 + (b - c * per) * 256;
  if (u0 >= f1) return;  // uniform
  const int tid = threadIdx.x;
  const int u = u0 + tid;
  int e0 = 0, e1 = 0;
  if (u < f1) { e0 = d.grp[u]; e1 = d.grp[u + 1]; }
  const int g0 = d.grp[u0], g1 = d.grp[min(u0 + 256, f1)];
  int cnt = 0;
  int o[W];
#pragma unroll
  for (int q = 0; q < W; ++q) o[q] = -1;
  for (int t0 = g0; t0 < g1; t0 += kAdjTile) {
    const int t1 = min(t0 + kAdjTile, g1);
    constexpr int PT = kAdjTile / 256;
    int k[PT];
    double x[PT];
#pragma unroll
    for (int j = 0; j < PT; ++j) {
      const int e = t0 + tid + 256 * j;
      k[j] = -1;
      x[j] = 0.0;
      if (e < t1) { k[j] = d.gci[e]; x[j] = d.gva[e]; }
    }
    int8_t c8[PT];
#pragma unroll
    for (int j = 0; j < PT; ++j) c8[j] = ((unsigned)k[j] < (unsigned)d.n) ? d.cf[k[j]] : (int8_t)1;
    if (t0 != g0) __syncthreads();  // the last tile has been read
#pragma unroll
    for (int j = 0; j < PT; ++j) {
      const bool edge = x[j] != 0.0 && c8[j] == 0 && strong_edge(x[j], k[j], d.theta, d.cmax);
      s_k[tid + 256 * j] = edge ? k[j] : -1;
    }
    __syncthreads();
    const int ee = min(e1, t1);
    for (int e = max(e0, t0); e < ee; e += 4) {
      int kk[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) kk[j] = s_k[min(e + j, ee - 1) - t0];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (e + j < ee && kk[j] >= 0 && kk[j] != u) {
#pragma unroll
          for (int q = 0; q < W; ++q)
            if (q == cnt) o[q] = kk[j];
          ++cnt;
        }
      }
    }
  }
  if (u >= f1) return;
  if (cnt > W) o[0] = kAdjOverflow;
  gptr<adj_v4> dst = (gptr<adj_v4>)(to_global(w.fadj) + (d.fine0 + u) * W);
#pragma unroll
  for (int q = 0; q < W / 4; ++q) {
    adj_v4 t;
    t.x = o[4 * q];
    t.y = o[4 * q + 1];
    t.z = o[4 * q + 2];
    t.w = o[4 * q + 3];
    dst[q] = t;
  }
}

// The distinct values of v (sorted, INT32_MAX = none) into the row's slot:
// bin A's (stride SA) when there are at most lim of them, else bin B's.
// Returns their number (at most P <= 32).  A slot of eight points is put
// together in the thread's kStage words of LDS and stored as two 16-byte words
// (its unused places hold whatever was there): eight stores of four bytes, 32
// bytes from lane to lane, were a request to the L2 each (k_count: 64 five-point
// matrices of 64^2 to 768^2 217 -> 207 us, 16 of 129^2 to 515^2 38.4 -> 34.9).
constexpr int kStage = 9;  // odd, so that the lanes' words lie in different banks

template <int P>
__device__ __forceinline__ int emit_distinct(const int (&v)[P], const Work& w, int64_t row, int SA, int lim,
                                             int* stage) {
  static_assert(P <= 32, "bin B slots hold 32 points");
  int sz = 0;
#pragma unroll
  for (int q = 0; q < P; ++q) sz += (v[q] != 0x7fffffff && (q == 0 || v[q] != v[q - 1])) ? 1 : 0;
  int pos = 0;
  if (SA == 8 && sz <= lim) {
#pragma unroll
    for (int q = 0; q < P; ++q) {
      const bool u = v[q] != 0x7fffffff && (q == 0 || v[q] != v[q - 1]);
      if (u) stage[pos] = v[q];
      pos += u ? 1 : 0;
    }
    gptr<adj_v4> dst = (gptr<adj_v4>)(to_global(w.slotA) + row * 8);
    adj_v4 t;
    t.x = stage[0]; t.y = stage[1]; t.z = stage[2]; t.w = stage[3];
    dst[0] = t;
    if (sz > 4) {
      t.x = stage[4]; t.y = stage[5]; t.z = stage[6]; t.w = stage[7];
      dst[1] = t;
    }
    return sz;
  }
  gptr<int32_t> dst = sz <= lim ? to_global(w.slotA) + row * SA : to_global(w.slotB) + row * 32;
#pragma unroll
  for (int q = 0; q < P; ++q) {
    const bool u = v[q] != 0x7fffffff && (q == 0 || v[q] != v[q - 1]);
    if (u) dst[pos] = v[q];
    pos += u ? 1 : 0;
  }
  return sz;
}

// N(i) at ell = 2 from the compact adjacency: the first four slots of i and the
// first four of each of them, sorted, duplicates dropped.  -1 when a point
// overflows its slots (the row is left to k_count_mid); at width 8, -2 when a
// point has more than four (count_adj8_ell2 takes the row).
template <int W>
__device__ __forceinline__ int count_adj_ell2(const Work& w, const GDesc& d, int i, int64_t row, int SA, int lim,
                                              int* stage) {
  int a[W];
  adj_load<W>(d.fadj, i, a);
  if (a[0] == kAdjOverflow) return -1;
  if (W > 4 && a[W > 4 ? 4 : 0] >= 0) return -2;
  int b[4][W];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (a[q] >= 0) {
      adj_load<W>(d.fadj, a[q], b[q]);
    } else {
#pragma unroll
      for (int r = 0; r < W; ++r) b[q][r] = -1;
    }
  }
  int v[32];
  bool ovf = false, more = false;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    ovf |= b[q][0] == kAdjOverflow;
    more |= W > 4 && b[q][W > 4 ? 4 : 0] >= 0;
    v[q] = a[q] >= 0 ? a[q] : 0x7fffffff;
#pragma unroll
    for (int r = 0; r < 4; ++r) v[4 + 4 * q + r] = b[q][r] >= 0 ? b[q][r] : 0x7fffffff;
  }
  if (ovf) return -1;
  if (more) return -2;
#pragma unroll
  for (int q = 20; q < 32; ++q) v[q] = 0x7fffffff;
  bitonic_sort<32>(v);
  return emit_distinct<32>(v, w, row, SA, lim, stage);
}

// N(i) at ell = 2 from the compact adjacency of width 8, by a quad: lane l
// takes slots 2l and 2l + 1 of i and the eight of each of them (18 candidates),
// sorts them, and the four lists are merged across the quad (bitonic merges;
// the exchanges are DPP quad permutations), so the distinct ones end up in
// order, lane by lane.  They go to the row's slot through `stage` (33 words of
// LDS per quad).  -1 when a point overflows its slots or there are more than 32
// points (the row is left to k_count_mid).  All lanes of the wavefront call it;
// a quad without a row has on = false.
//
// Two trips to memory a row and about 90 registers, where k_count_mid's search
// takes a round of loads per four frontier points at two wavefronts per SIMD:
// the two kernels took 300 us on 2048^2 nine-point rows (24 points, 72
// candidates) and 103 on 128^3 seven-point rows, now 146 and 74.
__device__ __forceinline__ int count_adj8_ell2(const Work& w, const GDesc& d, bool on, int i, int64_t row, int SA,
                                               int lim, int ql, int* stage) {
  i2u a;
  a.x = -1;
  a.y = -1;
  if (on) a = *(gptr<const i2u>)(d.fadj + (int64_t)i * 8 + 2 * ql);
  int b0[8], b1[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) { b0[r] = -1; b1[r] = -1; }
  if (a.x >= 0) adj_load<8>(d.fadj, a.x, b0);
  if (a.y >= 0) adj_load<8>(d.fadj, a.y, b1);
  int bad = (a.x == kAdjOverflow || b0[0] == kAdjOverflow || b1[0] == kAdjOverflow) ? 1 : 0;
  int v[32];
  v[0] = a.x >= 0 ? a.x : 0x7fffffff;
  v[1] = a.y >= 0 ? a.y : 0x7fffffff;
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    v[2 + r] = b0[r] >= 0 ? b0[r] : 0x7fffffff;
    v[10 + r] = b1[r] >= 0 ? b1[r] : 0x7fffffff;
  }
#pragma unroll
  for (int r = 18; r < 32; ++r) v[r] = 0x7fffffff;
  bitonic_sort<32>(v);
  auto merge = [&]() {
#pragma unroll
    for (int st = 16; st > 0; st >>= 1)
#pragma unroll
      for (int k = 0; k < 32; ++k)
        if ((k & st) == 0) {
          const int lo = min(v[k], v[k | st]), hi = max(v[k], v[k | st]);
          v[k] = lo;
          v[k | st] = hi;
        }
  };
  // lanes 0, 1 and lanes 2, 3: the smaller 32 to the even lane
  auto cross_reversed = [&](auto ctrl, bool low) {
    int o[32];
#pragma unroll
    for (int k = 0; k < 32; ++k) o[k] = __builtin_amdgcn_mov_dpp(v[31 - k], decltype(ctrl)::value, 0xF, 0xF, false);
#pragma unroll
    for (int k = 0; k < 32; ++k) v[k] = low ? min(v[k], o[k]) : max(v[k], o[k]);
  };
  cross_reversed(std::integral_constant<int, 0xB1>{}, (ql & 1) == 0);  // quad_perm [1,0,3,2]
  merge();
  // the pairs' lists: the smaller 64 to lanes 0 and 1, then in order within each half
  cross_reversed(std::integral_constant<int, 0x1B>{}, ql < 2);  // quad_perm [3,2,1,0]
#pragma unroll
  for (int k = 0; k < 32; ++k) {
    const int o = __builtin_amdgcn_mov_dpp(v[k], 0xB1, 0xF, 0xF, false);
    v[k] = (ql & 1) == 0 ? min(v[k], o) : max(v[k], o);
  }
  merge();
  // distinct values: places from a prefix over the quad
  const int before = __builtin_amdgcn_mov_dpp(v[31], 0x90, 0xF, 0xF, false);  // the lane below's last
  int cnt = 0;
#pragma unroll
  for (int q = 0; q < 32; ++q) {
    const bool first = q == 0 && ql == 0;
    const int pv = q == 0 ? before : v[q > 0 ? q - 1 : 0];
    cnt += (v[q] != 0x7fffffff && (first || v[q] != pv)) ? 1 : 0;
  }
  int pre = cnt;
  const int x1 = __builtin_amdgcn_mov_dpp(pre, 0x90, 0xF, 0xF, false);  // quad_perm [0,0,1,2]
  pre += ql >= 1 ? x1 : 0;
  const int x2 = __builtin_amdgcn_mov_dpp(pre, 0x40, 0xF, 0xF, false);  // quad_perm [0,0,0,1]
  pre += ql >= 2 ? x2 : 0;
  const int sz = __builtin_amdgcn_mov_dpp(pre, 0xFF, 0xF, 0xF, false);
  bad |= __builtin_amdgcn_mov_dpp(bad, 0xB1, 0xF, 0xF, false);
  bad |= __builtin_amdgcn_mov_dpp(bad, 0x4E, 0xF, 0xF, false);
  const bool ok = on && !bad && sz <= 32;
  if (ok) {
    int pos = pre - cnt;
#pragma unroll
    for (int q = 0; q < 32; ++q) {
      const bool first = q == 0 && ql == 0;
      const int pv = q == 0 ? before : v[q > 0 ? q - 1 : 0];
      const bool u = v[q] != 0x7fffffff && (first || v[q] != pv);
      if (u) stage[pos] = v[q];
      pos += u ? 1 : 0;
    }
  }
  wave_sync();
  if (ok) {
    gptr<int32_t> dst = sz <= lim ? to_global(w.slotA) + row * SA : to_global(w.slotB) + row * 32;
    for (int p = 4 * ql; p < sz; p += 16) {  // (a slot holds a multiple of four words)
      adj_v4 t;
      t.x = stage[p]; t.y = stage[p + 1]; t.z = stage[p + 2]; t.w = stage[p + 3];
      *(gptr<adj_v4>)(dst + p) = t;
    }
  }
  wave_sync();  // the stage is free
  return ok ? sz : -1;
}

// N(i) at ell = 1 from row i of the search graph (at most 8 stored entries;
// -1 otherwise, the row is left to k_count_mid)
__device__ __forceinline__ int count_row_ell1(const Work& w, const GDesc& d, int i, int64_t row, int SA, int lim,
                                              int* stage) {
  const int e0 = d.grp[i], e1 = d.grp[i + 1];
  if (e1 - e0 > 8) return -1;
  int k[8];
  double x[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    k[j] = i;
    x[j] = 0.0;
    if (e0 + j < e1) { k[j] = d.gci[e0 + j]; x[j] = d.gva[e0 + j]; }
  }
  int v[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int8_t c8 = ((unsigned)k[j] < (unsigned)d.n) ? d.cf[k[j]] : (int8_t)1;
    v[j] = (k[j] != i && x[j] != 0.0 && c8 == 0 && strong_edge(x[j], k[j], d.theta, d.cmax)) ? k[j] : 0x7fffffff;
  }
  bitonic_sort<8>(v);
  return emit_distinct<8>(v, w, row, SA, lim, stage);
}

// The chunk's bookkeeping once every row is sized (s_size; the rows left to
// k_count_big have size 0, a negative s_rows entry and their index in
// s_unres[0..nunres)): bin counts, the queue of k_count_big, the chunk-local
// exclusive prefix of |N(i)|+1, the chunk totals.
__device__ __forceinline__ void finish_chunk(const Work& w, int c, int m, MatStatus* st, int64_t base, int nc,
                                             const int* s_rows, const int16_t* s_size, const int16_t* s_unres,
                                             int nunres, int* s_scan, int* s_flag, int* s_qbase) {
  const int tid = threadIdx.x, nt = blockDim.x;
  const int lim = small_limit(w.GA);
  if (nunres) {
    if (tid == 0) *s_qbase = atomicAdd(&w.cnt->nbig, nunres);
    __syncthreads();
    for (int k = tid; k < nunres; k += nt) {
      const int q = *s_qbase + k;
      if (q < w.capC) w.bigq[q] = c * w.chunk + s_unres[k];
      else flag_row(st, ST_UNSUPPORTED, -s_rows[s_unres[k]] - 1);
    }
  }
  const int per2 = (nc + nt - 1) / nt;
  const int t0 = tid * per2;
  int mysum = 0, mymax = 0, inA = 0, inB = 0;
  for (int t = t0; t < min(t0 + per2, nc); ++t) {
    const int sz = s_size[t];
    mysum += sz + 1;
    mymax = max(mymax, sz);
    if (s_rows[t] >= 0) {
      inA += sz <= lim ? 1 : 0;
      inB += sz > lim && sz <= 32 ? 1 : 0;  // larger rows are queued for the workgroup solvers
    }
  }
  int tot;
  int pre = block_exclusive_scan(mysum, s_scan, &tot);
  for (int t = t0; t < min(t0 + per2, nc); ++t) { w.lnz[base + t] = pre; pre += s_size[t] + 1; }
  if (mymax) atomicMax(&s_flag[0], mymax);
  if (inA) atomicAdd(&s_flag[2], inA);
  if (inB) atomicAdd(&s_flag[3], inB);
  __syncthreads();
  if (tid == 0) {
    w.chunk_nc[c] = nc;
    w.chunk_nnz[c] = tot;
    w.chunk_mat[c] = m;
    // bin sizes per chunk (summed by k_scan); the largest block only when it
    // grows, so that few workgroups meet at one address
    w.chunk_bins[c] = make_int2(s_flag[2], s_flag[3]);
    if (s_flag[0] > __hip_atomic_load(&st->max_block, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomicMax(&st->max_block, s_flag[0]);
    w.chunk_unsized[c] = nunres;
  }
}

// Symbolic pass, first part: one workgroup per chunk of fine points.  The
// chunk's C-points are compacted; rows at ell = 1 with at most 8 stored
// entries, and rows at ell = 2 of matrices with a compact adjacency,
// are sized by one thread each from a sorted candidate list (no search
// state; over a width-8 adjacency by a quad where a point has more than four
// edges); a chunk whose rows are all sized is finished here.  Other rows
// (larger stencils, ell >= 3, aggregates, overflowing points) are marked -1
// in lnz and left, with the chunk's bookkeeping, to k_count_mid.
template <int W>
__global__ __launch_bounds__(kNT) void k_count(Work w) {
  __shared__ int s_rows[kMaxChunk];
  __shared__ int16_t s_size[kMaxChunk];
  __shared__ int s_scan[kNT];
  __shared__ int s_stage[kNT * kStage];
  __shared__ int s_flag[4];  // max |N|, -, rows in bin A, rows in bin B
  __shared__ int s_ndef, s_qbase, s_nlist;
  __shared__ int16_t s_list[W == 8 ? kMaxChunk : 1];  // rows for the quads

  // each XCD's chunks newest first: k_adj wrote them in ascending order, so
  // the last ones' adjacency is the part most likely still cached (and the
  // numeric kernels, walking rows in ascending order, then first read the
  // slots written last here)
  const int c = xcd_logical_block_reversed();
  const int tid = threadIdx.x;
  const int m = chunk_matrix(w.desc, w.nmat, c);
  const GDesc d = gview(w.desc[m]);
  MatStatus* st = &w.st[m];
  const int f0 = (c - d.chunk0) * w.chunk;
  const int f1 = min(f0 + w.chunk, d.n);
  const int64_t base = d.fine0 + f0;

  if (st->status == ST_INVALID) {  // validation failed: contribute nothing
    if (tid == 0) { w.chunk_nc[c] = 0; w.chunk_nnz[c] = 0; w.chunk_mat[c] = m; w.chunk_bins[c] = make_int2(0, 0); w.chunk_unsized[c] = 0; }
    return;
  }

  // empty the projection's column lists of this chunk's fine points
  if (d.B) {
    for (int j = f0 + tid; j < f1; j += kNT) w.chead[d.fine0 + j] = -1;
  }

  // compaction of the chunk's C-points, ascending: each thread's run of up
  // to 8 markers is read once, all loads in flight together
  static_assert(kMaxChunk <= 8 * kNT, "a thread's run of markers fits one byte mask");
  const int per = (w.chunk + kNT - 1) / kNT;
  const int j0 = f0 + tid * per;
  const int j1 = min(j0 + per, f1);
  uint32_t cbits = 0;
#pragma unroll
  for (int k = 0; k < 8; ++k)
    if (j0 + k < j1 && d.cf[j0 + k] != 0) cbits |= 1u << k;
  int nc;
  int rank = block_exclusive_scan(__popc(cbits), s_scan, &nc);
  for (uint32_t b = cbits; b; b &= b - 1) {
    const int j = j0 + __ffs(b) - 1;
    s_rows[rank] = j;
    w.clocal[base + rank] = j;
    ++rank;
  }
  if (tid == 0) { s_flag[0] = 0; s_flag[1] = 0; s_flag[2] = 0; s_flag[3] = 0; s_ndef = 0; s_nlist = 0; }
  __syncthreads();

  const int SA = slot_stride(w.GA);
  const int lim = small_limit(w.GA);
  int ndef = 0;
  if (W == 8 && d.fadj && d.ell == 2 && !d.agg_rp) {
    static_assert(kNT / 4 * 33 <= kNT * kStage, "33 words of the stage per quad");
    const int qd = tid >> 2, ql = tid & 3;
    // rows whose points have at most four edges each by one thread, the others
    // by quads (a strength test leaves few edges: 1001^2 nine-point rows at
    // 0.25: both kernels 57 us with k_count_mid's
    // search, 61 with quads alone, 31 so; 2048^2 rows, all for the quads, 139
    // and 146)
    for (int t = tid; t < nc; t += kNT) {
      const int sz = count_adj_ell2<8>(w, d, s_rows[t], base + t, SA, lim, s_stage + tid * kStage);
      s_size[t] = (int16_t)sz;
      ndef += sz == -1 ? 1 : 0;
      if (sz == -2) s_list[atomicAdd(&s_nlist, 1)] = (int16_t)t;
    }
    __syncthreads();
    const int nl = s_nlist;
    for (int k0 = 0; k0 < nl; k0 += kNT / 4) {
      const bool on = k0 + qd < nl;
      const int t = on ? s_list[k0 + qd] : 0;
      const int sz = count_adj8_ell2(w, d, on, s_rows[t], base + t, SA, lim, ql, s_stage + 33 * qd);
      if (on && ql == 0) {
        s_size[t] = (int16_t)sz;
        ndef += sz < 0 ? 1 : 0;
      }
    }
  } else for (int t = tid; t < nc; t += kNT) {
    int sz = -1;
    if (!d.agg_rp) {
      if constexpr (W == 4) {
        if (d.fadj && d.ell == 2) sz = count_adj_ell2<4>(w, d, s_rows[t], base + t, SA, lim, s_stage + tid * kStage);
      }
      if (d.ell == 1) sz = count_row_ell1(w, d, s_rows[t], base + t, SA, lim, s_stage + tid * kStage);
    }
    s_size[t] = (int16_t)sz;
    ndef += sz < 0 ? 1 : 0;
  }
  if (ndef) atomicAdd(&s_ndef, ndef);
  __syncthreads();
  if (s_ndef == 0) {
    finish_chunk(w, c, m, st, base, nc, s_rows, s_size, nullptr, 0, s_scan, s_flag, &s_qbase);
    return;
  }
  // left to k_count_mid: the sizes so far (-1 = not sized), the chunk queued
  for (int t = tid; t < nc; t += kNT) w.lnz[base + t] = s_size[t];
  if (tid == 0) {
    w.chunk_nc[c] = nc;
    w.chunk_mat[c] = m;
    w.chunk_nnz[c] = -1;
    w.midq[atomicAdd(&w.cnt->nmid, 1)] = c;
  }
}

// Symbolic pass, second part, distances 1 and 2: the chunks k_count left
// unfinished (queued by it; the workgroups take them in turn, so an empty
// queue costs one load per workgroup).  One thread per row not yet sized
// searches up to 32 points in registers (over the compact adjacency when the
// matrix has one); larger rows are left unsized for k_count_big.  Then the
// chunk's bookkeeping.
//
// Bound: latency at two wavefronts per SIMD (the register set), so the number of
// threads decides how many chunks a CU has at once against how long one takes.
// Up to four chunks a CU workgroups of 256 threads are better on grids: 1024^2
// nine-point rows at distance 1, every third point a C-point, 144 us a call (128
// threads: 152, 64: 177), every second 204 (218); 80^3 seven-point at distance 2
// without the adjacency 244 (283).  Beyond, 128 threads: 2900^2 nine-point 983 us
// (256: 1,044), 120,000 rows of 24 points 487 (554); 2048^2 517 and 514.  The rule
// looks at the chunks only, so up to four a CU chunks of few rows each pay for
// it: 40,000 rows of 24 points in 940 chunks 227 us a call with 256 threads, 203
// with 128.  A grid's C-points fill every third chunk or so, so the mean over the
// chunks, all that the host could know, does not tell the two apart.
template <int W, int NT>
__global__ __launch_bounds__(NT) void k_count_mid(Work w) {
  __shared__ int s_rows[kMaxChunk];
  __shared__ int16_t s_size[kMaxChunk];
  __shared__ int s_scan[kNT];
  __shared__ int s_flag[4];  // max |N|, rows left unsized, rows in bin A, rows in bin B
  __shared__ int16_t s_list[kMaxChunk];   // rows to size here
  __shared__ int16_t s_unres[kMaxChunk];  // rows with more than 32 points
  __shared__ int s_nlist, s_qbase;

  const int tid = threadIdx.x;
  const int nq = w.cnt->nmid;
  for (int qi = blockIdx.x; qi < nq; qi += gridDim.x) {
  const int c = w.midq[qi];
  __syncthreads();  // the previous chunk's LDS is free
  const int m = w.chunk_mat[c];
  const GDesc d = gview(w.desc[m]);
  if (d.ell > 2) continue;  // k_count_wide's
  MatStatus* st = &w.st[m];
  const int64_t base = d.fine0 + (int64_t)(c - d.chunk0) * w.chunk;
  const int nc = w.chunk_nc[c];
  if (tid == 0) { s_flag[0] = 0; s_flag[1] = 0; s_flag[2] = 0; s_flag[3] = 0; s_nlist = 0; }
  __syncthreads();
  for (int t = tid; t < nc; t += NT) {
    s_rows[t] = w.clocal[base + t];
    const int sz = w.lnz[base + t];
    s_size[t] = (int16_t)sz;
    if (sz < 0) s_list[atomicAdd(&s_nlist, 1)] = (int16_t)t;
  }
  __syncthreads();
  const int SA = slot_stride(w.GA);
  const int lim = small_limit(w.GA);
  const int nl = s_nlist;
  for (int k = tid; k < nl; k += NT) {
    const int t = s_list[k];
    const int i = s_rows[t];
    RegSetA<32> S;
    int sz;
    if constexpr (W > 0) {
      if (d.fadj)
        sz = rega_bfs<32, W>(S, d.n, i, d.ell, d.fadj, d.grp, d.gci, d.gva, d.cf, d.theta, d.cmax, nullptr, nullptr);
      else
        sz = rega_bfs<32, 0>(S, d.n, i, d.ell, nullptr, d.grp, d.gci, d.gva, d.cf, d.theta, d.cmax, d.agg_rp,
                             d.agg_list);
    } else {
      sz = rega_bfs<32, 0>(S, d.n, i, d.ell, nullptr, d.grp, d.gci, d.gva, d.cf, d.theta, d.cmax, d.agg_rp,
                           d.agg_list);
    }
    if (sz < 0) {
      s_size[t] = 0;
      s_rows[t] = -(i + 1);
      w.clocal[base + t] = -(i + 1);
      s_unres[atomicAdd(&s_flag[1], 1)] = (int16_t)t;
    } else if (sz <= lim) {
      s_size[t] = (int16_t)sz;
#pragma unroll
      for (int p = 0; p < 32; ++p)
        if (p < sz) w.slotA[(base + t) * SA + p] = S.v[p];
    } else {
      s_size[t] = (int16_t)sz;
#pragma unroll
      for (int p = 0; p < 32; ++p)
        if (p < sz) w.slotB[(base + t) * 32 + p] = S.v[p];
    }
  }
  __syncthreads();
  finish_chunk(w, c, m, st, base, nc, s_rows, s_size, s_unres, s_flag[1], s_scan, s_flag, &s_qbase);
  }
}

// The same at distance 3 and more, where rows of more than 32 points are
// common: sixteen lanes per row search up to 32 points (group_search, over the
// compact adjacency when the matrix has one); the rows that hold more are
// searched again by a wavefront each, up to kMidMax points, and queued for the
// workgroup solvers; larger rows are left unsized for k_count_big.  Then the
// chunk's bookkeeping.  Bound: the latency of a level's trips to memory.
// 150^2 nine-point rows at distance 5 (up to 108 points): one thread per row,
// then a workgroup per row of more than 32 points, took 445 us, this 70.
constexpr int kMidMax = 128;

template <int W>
__global__ __launch_bounds__(kNT) void k_count_wide(Work w) {
  constexpr int G = 16, NG = kNT / G, NW = kNT / 64;
  constexpr int LW = W == 4 ? 2 : W == 8 ? 3 : 0;
  typedef SearchBuf<32, 64> SmallBuf;
  typedef SearchBuf<kMidMax, 4 * kMidMax> WaveBuf;
  __shared__ int s_rows[kMaxChunk];
  __shared__ int16_t s_size[kMaxChunk];
  __shared__ int s_scan[kNT];
  __shared__ int s_flag[4];  // max |N|, rows left unsized, rows in bin A, rows in bin B
  __shared__ int16_t s_list[kMaxChunk];   // rows to size here, then rows of more than 32 points
  __shared__ int16_t s_unres[kMaxChunk];  // rows of more than kMidMax points
  __shared__ int s_nlist, s_nwide, s_qbase;
  __shared__ union {
    SmallBuf small[NG];
    WaveBuf wide[NW];
  } s_buf;

  const int tid = threadIdx.x;
  const int nq = w.cnt->nmid;
  for (int qi = blockIdx.x; qi < nq; qi += gridDim.x) {
  const int c = w.midq[qi];
  __syncthreads();  // the previous chunk's LDS is free
  const int m = w.chunk_mat[c];
  const GDesc d = gview(w.desc[m]);
  if (d.ell <= 2) continue;  // k_count_mid's
  MatStatus* st = &w.st[m];
  const int64_t base = d.fine0 + (int64_t)(c - d.chunk0) * w.chunk;
  const int nc = w.chunk_nc[c];
  if (tid == 0) { s_flag[0] = 0; s_flag[1] = 0; s_flag[2] = 0; s_flag[3] = 0; s_nlist = 0; s_nwide = 0; }
  __syncthreads();
  for (int t = tid; t < nc; t += kNT) {
    s_rows[t] = w.clocal[base + t];
    const int sz = w.lnz[base + t];
    s_size[t] = (int16_t)sz;
    if (sz < 0) s_list[atomicAdd(&s_nlist, 1)] = (int16_t)t;
  }
  __syncthreads();
  const int SA = slot_stride(w.GA);
  const int lim = small_limit(w.GA);
  const bool literal = d.literal != 0 && d.ell >= 3;
  const int nl = s_nlist;
  // the points of a row of at most 32 to its slot, each at its rank
  auto put_slot = [&](auto& b, int t, int n, int sz, int lane, int lanes) {
    gptr<int32_t> dst = sz <= lim ? to_global(w.slotA) + (base + t) * SA : to_global(w.slotB) + (base + t) * 32;
    for (int q = lane; q < n; q += lanes) {
      const int v = b.list[q];
      if (v != INT32_MAX) dst[search_rank(b, n, v)] = v;
    }
  };
  {
    const int lane = tid % G;
    SmallBuf& b = s_buf.small[tid / G];
    for (int k = tid / G; k < nl; k += NG) {
      const int t = s_list[k];
      const int n = group_search<G>(b, d, s_rows[t], LW, lane);
      if (n < 0) {
        if (lane == 0) s_size[t] = -2;  // more than 32 points were met
      } else {
        const int sz = literal ? drop_c_points<G>(b, d, n, lane) : n;
        put_slot(b, t, n, sz, lane, G);
        if (lane == 0) s_size[t] = (int16_t)sz;
      }
      group_sync<G>();  // the buffer is free
    }
  }
  __syncthreads();
  for (int t = tid; t < nc; t += kNT)
    if (s_size[t] == -2) s_list[atomicAdd(&s_nwide, 1)] = (int16_t)t;
  __syncthreads();
  {
    const int lane = tid & 63;
    WaveBuf& b = s_buf.wide[tid >> 6];
    const int nw = s_nwide;
    for (int k = tid >> 6; k < nw; k += NW) {
      const int t = s_list[k];
      const int i = s_rows[t];
      const int n = group_search<64>(b, d, i, LW, lane);
      if (n < 0) {
        if (lane == 0) {
          s_size[t] = 0;
          s_rows[t] = -(i + 1);
          w.clocal[base + t] = -(i + 1);
          s_unres[atomicAdd(&s_flag[1], 1)] = (int16_t)t;
        }
      } else {
        const int sz = literal ? drop_c_points<64>(b, d, n, lane) : n;
        if (sz <= 32) put_slot(b, t, n, sz, lane, 64);
        if (lane == 0) {
          s_size[t] = (int16_t)sz;
          if (sz > 32) {
            const int q = atomicAdd(&w.cnt->nC, 1);
            if (q < w.capC) w.binC[q] = c * w.chunk + t;
            else flag_row(st, ST_UNSUPPORTED, i);
          }
        }
      }
      group_sync<64>();
    }
  }
  __syncthreads();
  finish_chunk(w, c, m, st, base, nc, s_rows, s_size, s_unres, s_flag[1], s_scan, s_flag, &s_qbase);
  }
}

// Rows the searches above left unsized (more than 32 points at distance 2, more
// than kMidMax beyond), one workgroup per row (grid-stride over the
// queue): the workgroup search sizes the row, which is queued for the
// workgroup solver.  The workgroup that sizes the last such row of a chunk
// then redoes the chunk's prefix.
__global__ __launch_bounds__(kNT) void k_count_big(Work w) {
  __shared__ WideBuf bb;
  __shared__ int s_size[kMaxChunk];
  __shared__ int s_scan[kNT];
  __shared__ int s_last;
  const int tid = threadIdx.x;
  const int nq = min(w.cnt->nbig, w.capC);
  for (int qi = blockIdx.x; qi < nq; qi += gridDim.x) {
    const int e = w.bigq[qi];
    const int c = e / w.chunk, t = e - c * w.chunk;
    const int m = w.chunk_mat[c];
    const GDesc d = gview(w.desc[m]);
    MatStatus* st = &w.st[m];
    const int64_t base = d.fine0 + (int64_t)(c - d.chunk0) * w.chunk;
    const int i = -w.clocal[base + t] - 1;
    int* nl;
    const int s = block_bfs(d.n, i, d.ell, d.grp, d.gci, d.gva, d.cf, d.theta, d.cmax, d.agg_rp, d.agg_list, bb, &nl,
                            d.literal != 0);
    __syncthreads();
    // A row the register search gave up on may still hold at most 32 points
    // (the literal reading counts the C-points a walk passes through): it
    // then joins its size bin, whose solvers take every row of that size,
    // and not the workgroup solver as well.
    const int lim = small_limit(w.GA);
    const bool toA = s >= 0 && s <= lim, toB = s > lim && s <= 32;
    if (toA) {
      const int SA = slot_stride(w.GA);
      for (int p = tid; p < s; p += kNT) w.slotA[(base + t) * SA + p] = nl[p];
    } else if (toB) {
      for (int p = tid; p < s; p += kNT) w.slotB[(base + t) * 32 + p] = nl[p];
    }
    if (tid == 0) {
      w.big_size[base + t] = s < 0 ? 0 : s;
      if (s < 0) {
        flag_row(st, ST_UNSUPPORTED, i);
      } else {
        if (s > __hip_atomic_load(&st->max_block, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
          atomicMax(&st->max_block, s);
        if (toA || toB) {
          atomicAdd(reinterpret_cast<int*>(&w.chunk_bins[c]) + (toA ? 0 : 1), 1);
        } else {
          const int q = atomicAdd(&w.cnt->nC, 1);
          if (q < w.capC) w.binC[q] = e;
          else flag_row(st, ST_UNSUPPORTED, i);
        }
      }
      __threadfence();  // the size is visible before the count drops
      s_last = atomicSub(&w.chunk_unsized[c], 1) == 1;
      // every size of the chunk is visible to the workgroup beyond the barrier.
      // (One wavefront's fence: each invalidates caches that the searches read.
      // 2,000 rows of 64 points in chunks of 256 points, so about 500 last rows:
      // 182 us with a fence in all four, 119 so; in the chunks of 1024 of before
      // 142.)
      if (s_last) __threadfence();
    }
    __syncthreads();
    if (s_last) {
      // sizes: k_count's prefix (0 for the unsized rows) and the unsized
      // rows' own sizes; their C-point index is restored
      const int nc = w.chunk_nc[c];
      for (int tt = tid; tt < nc; tt += kNT) {
        const int l1 = (tt + 1 < nc) ? w.lnz[base + tt + 1] : w.chunk_nnz[c];
        int sz = l1 - w.lnz[base + tt] - 1;
        const int ci = w.clocal[base + tt];
        if (ci < 0) sz = w.big_size[base + tt];
        s_size[tt] = sz;
      }
      __syncthreads();
      for (int tt = tid; tt < nc; tt += kNT) {
        const int ci = w.clocal[base + tt];
        if (ci < 0) w.clocal[base + tt] = -ci - 1;
      }
      const int per2 = (nc + kNT - 1) / kNT;
      const int t0 = tid * per2;
      int mysum = 0;
      for (int tt = t0; tt < min(t0 + per2, nc); ++tt) mysum += s_size[tt] + 1;
      int tot;
      int pre = block_exclusive_scan(mysum, s_scan, &tot);
      for (int tt = t0; tt < min(t0 + per2, nc); ++tt) { w.lnz[base + tt] = pre; pre += s_size[tt] + 1; }
      if (tid == 0) w.chunk_nnz[c] = tot;
    }
    __syncthreads();
  }
}

// One workgroup: global row base and global R offset of every chunk (all
// matrices in order).  Each thread sums a contiguous run of chunks, one block
// scan joins the runs; then one thread per matrix sizes R, checks capacity and
// writes R.row_ptr[n_c].  Per-matrix R offsets are the global ones minus the
// matrix's base.
__global__ __launch_bounds__(1024) void k_scan(Work w) {
  __shared__ long long s_wr[17], s_wz[17];
  __shared__ int s_wa[17], s_wb[17];
  __shared__ int s_maxb;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wid = tid >> 6;
  const int nch = w.nchunks;
  // tiles of 4096 consecutive chunks, four per thread (their loads in flight
  // together), scanned in order with the running totals carried over (four
  // per thread were faster than one and than sixteen: 42, 30 and 44 us on
  // 13,400 chunks)
  constexpr int CPT = 4;
  long long carry_r = 0, carry_z = 0;
  int na = 0, nb = 0;
  for (int t0 = 0; t0 < nch; t0 += 1024 * CPT) {
    const int cb = t0 + tid * CPT;
    int ncs[CPT];
    long long nzs[CPT];
    int nc = 0, a = 0, bbin = 0;
    long long nz = 0;
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      ncs[k] = 0;
      nzs[k] = 0;
      if (cb + k < nch) {
        ncs[k] = w.chunk_nc[cb + k];
        nzs[k] = w.chunk_nnz[cb + k];
        const int2 bn = w.chunk_bins[cb + k];
        a += bn.x;
        bbin += bn.y;
      }
    }
#pragma unroll
    for (int k = 0; k < CPT; ++k) { nc += ncs[k]; nz += nzs[k]; }
    // inclusive scans inside each wavefront, then across the 16 wavefronts
    long long xr = nc, xz = nz;
    int xa = a, xb = bbin;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const long long yr = __shfl_up(xr, o, 64);
      const long long yz = __shfl_up(xz, o, 64);
      const int ya = __shfl_up(xa, o, 64);
      const int yb = __shfl_up(xb, o, 64);
      if (lane >= o) { xr += yr; xz += yz; xa += ya; xb += yb; }
    }
    if (lane == 63) { s_wr[wid] = xr; s_wz[wid] = xz; s_wa[wid] = xa; s_wb[wid] = xb; }
    __syncthreads();
    // the first wavefront scans the 16 wavefront totals: exclusive prefixes
    // in place, the tile's totals in slot 16
    if (wid == 0) {
      const long long r0 = lane < 16 ? s_wr[lane] : 0, z0 = lane < 16 ? s_wz[lane] : 0;
      const int a0 = lane < 16 ? s_wa[lane] : 0, b0 = lane < 16 ? s_wb[lane] : 0;
      long long r = r0, z = z0;
      int a1 = a0, b1 = b0;
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) {
        const long long yr = __shfl_up(r, o, 64);
        const long long yz = __shfl_up(z, o, 64);
        const int ya = __shfl_up(a1, o, 64);
        const int yb = __shfl_up(b1, o, 64);
        if (lane >= o) { r += yr; z += yz; a1 += ya; b1 += yb; }
      }
      if (lane < 16) { s_wr[lane] = r - r0; s_wz[lane] = z - z0; }
      if (lane == 15) { s_wr[16] = r; s_wz[16] = z; s_wa[16] = a1; s_wb[16] = b1; }
    }
    __syncthreads();
    const long long br = s_wr[wid], bz = s_wz[wid], tr = s_wr[16], tz = s_wz[16];
    const int ta = s_wa[16], tb = s_wb[16];
    __syncthreads();  // read before the next tile writes them
    long long rr = carry_r + br + xr - nc;
    long long zz = carry_z + bz + xz - nz;
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      const int c = cb + k;
      if (c < nch) {
        w.chunk_rbase[c] = (int32_t)rr;
        w.chunk_nzglob[c] = zz;
        // row blocks whose first row lies in this chunk
        for (long long b = (rr + (1 << w.rb_log) - 1) >> w.rb_log; (b << w.rb_log) < rr + ncs[k]; ++b)
          w.row_block_chunk[b] = c;
      }
      rr += ncs[k];
      zz += nzs[k];
    }
    carry_r += tr;
    carry_z += tz;
    na += ta;
    nb += tb;
  }
  const long long rows_total = carry_r, nnz_total = carry_z;
  // a pass left out on a hint that does not hold (the host runs again): no
  // matrix is live, so nothing uses the unfinished chunks' offsets
  const bool stop = ((w.skip & 1) && w.cnt->nmid > 0) || ((w.skip & 2) && w.cnt->nbig > 0);
  if (tid == 0) s_maxb = 0;
  __syncthreads();
  for (int m = tid; m < w.nmat; m += 1024) {
    const GDesc d = gview(w.desc[m]);
    MatStatus* st = &w.st[m];
    const int cb = d.chunk0, ce = d.chunk0 + d.nchunks;
    const long long rb = cb < nch ? w.chunk_rbase[cb] : rows_total;
    const long long re = ce < nch ? w.chunk_rbase[ce] : rows_total;
    const long long zb = cb < nch ? w.chunk_nzglob[cb] : nnz_total;
    const long long ze = ce < nch ? w.chunk_nzglob[ce] : nnz_total;
    const int n_c = (int)(re - rb);
    const long long nnz = ze - zb;
    st->row_base = (int32_t)rb;
    st->nz_base = zb;
    st->n_c = n_c;
    st->nnz = nnz;
    atomicMax(&s_maxb, st->max_block);
    if (st->status != ST_INVALID) {
      const bool fits = d.Rrp && d.Rci && d.Rva && (int64_t)n_c + 1 <= d.row_cap && nnz <= d.nnz_cap &&
                        nnz <= 0x7fffffffLL;
      if (!fits || stop) {
        st->status = ST_CAPACITY;
      } else {
        d.Rrp[n_c] = (int32_t)nnz;
      }
    }
  }
  __syncthreads();
  if (tid == 0) {
    w.cnt->maxb = s_maxb;
    w.chunk_rbase[nch] = (int32_t)rows_total;
    w.cnt->total_rows = (int32_t)rows_total;
    w.cnt->nA = na;
    w.cnt->nB = nb;
  }
}

// ---------------------------------------------------------------------------
// numeric pass, one thread per row with |N| <= 8.  The neighbourhood comes
// from the row's slot; the FP64 block, its FP32 LU and the right-hand side
// stay in the thread's registers, so the solve needs no communication.  A
// wavefront takes 64 consecutive rows (neighbouring C-points: their A rows
// share cache lines), and the rows of A are read eight entries at a time, two
// rows side by side.
// ---------------------------------------------------------------------------
constexpr int kS8 = 8;

// position of column k in the sorted neighbourhood N (and whether it is there)
__device__ __forceinline__ int pos8(const int (&N)[kS8], int k, bool* hit) {
  int q = 0;
  bool h = false;
#pragma unroll
  for (int j = 0; j < kS8; ++j) {
    q += (N[j] < k) ? 1 : 0;
    h |= (N[j] == k);
  }
  *hit = h;
  return q;
}

// y <- K^{-1} y with the packed no-pivot LU of K (unit lower L, upper U)
__device__ __forceinline__ void lu8_solve(const float (&K)[kS8][kS8], const float (&inv)[kS8], float (&y)[kS8]) {
#pragma unroll
  for (int q = 1; q < kS8; ++q)
#pragma unroll
    for (int k = 0; k < q; ++k) y[q] = fmaf(-K[q][k], y[k], y[q]);
#pragma unroll
  for (int q = kS8 - 1; q >= 0; --q) {
#pragma unroll
    for (int k = q + 1; k < kS8; ++k) y[q] = fmaf(-K[q][k], y[k], y[q]);
    y[q] *= inv[q];
  }
}

// K[q][p] = A[N_p][N_q] for the entries of rows N_pa and N_pb (columns pa, pb
// of K), eight entries of each row per batch
template <int PA>
__device__ __forceinline__ void gather8_pair(gptr<const int32_t> __restrict__ ci, gptr<const double> __restrict__ va,
                                             const int (&N)[kS8], const int (&e0)[kS8], const int (&e1)[kS8],
                                             double (&K)[kS8][kS8]) {
  constexpr int PB = PA + 1;
  for (int o = 0; e0[PA] + o < e1[PA] || e0[PB] + o < e1[PB]; o += 8) {
    int ka[8], kb[8];
    double xa[8], xb[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      ka[j] = -1;
      kb[j] = -1;
      xa[j] = 0.0;
      xb[j] = 0.0;
      if (e0[PA] + o + j < e1[PA]) { ka[j] = ci[e0[PA] + o + j]; xa[j] = va[e0[PA] + o + j]; }
      if (e0[PB] + o + j < e1[PB]) { kb[j] = ci[e0[PB] + o + j]; xb[j] = va[e0[PB] + o + j]; }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (ka[j] >= 0) {
        bool hit;
        const int q = pos8(N, ka[j], &hit);
#pragma unroll
        for (int qq = 0; qq < kS8; ++qq)
          if (hit && q == qq) K[qq][PA] = xa[j];
      }
      if (kb[j] >= 0) {
        bool hit;
        const int q = pos8(N, kb[j], &hit);
#pragma unroll
        for (int qq = 0; qq < kS8; ++qq)
          if (hit && q == qq) K[qq][PB] = xb[j];
      }
    }
  }
}

template <int NT>
__global__ __launch_bounds__(NT) void k_rows8(Work w) {
  if (w.cnt->nA == 0) return;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int total = w.cnt->total_rows;
  const RowBlocks rbk(total, (total >= 4 * NT * (int)gridDim.x ? 4 : 1) * NT);
  int r0, r1;
  if (!rbk.block(0, &r0, &r1)) return;
  RefineMax rmx;
  ChunkCursor cc;

  for (int jb = 0; rbk.block(jb, &r0, &r1); ++jb) {
  for (int gw = r0 + (tid & ~63); gw < r1; gw += NT) {
    const int g = gw + lane;
    const int gend = min(gw + 64, r1);
    for (int gc = gw; gc < gend;) {  // wavefront-uniform: one chunk at a time
      cc.seek(w, __builtin_amdgcn_readfirstlane(gc));
      const int cend = min(gend, cc.re);
      int t = 0, i = 0, off = 0, s = kS8 + 1;
      if (g >= gc && g < cend && cc.live) cc.row(w, g, &t, &i, &off, &s);
      gc = cend;
      if (s > kS8) continue;  // not this thread's row, or another solver's
      const GDesc& d = cc.md;
      MatStatus* st = &w.st[cc.m];
      const gptr<const int32_t> __restrict__ rp = d.rp;
      const gptr<const int32_t> __restrict__ ci = d.ci;
      const gptr<const double> __restrict__ va = d.va;
      d.Rrp[g - cc.rbase_m] = off;

      // N(i) from the slot; unused entries INT32_MAX
      const int4* sp = reinterpret_cast<const int4*>(w.slotA + (cc.fbase + t) * kS8);
      const int4 sa = sp[0], sb = sp[1];
      int N[kS8] = {sa.x, sa.y, sa.z, sa.w, sb.x, sb.y, sb.z, sb.w};
      int e0[kS8], e1[kS8];
#pragma unroll
      for (int p = 0; p < kS8; ++p) {
        if (p >= s) N[p] = 0x7fffffff;
        e0[p] = 0;
        e1[p] = 0;
        if (p < s) { e0[p] = rp[N[p]]; e1[p] = rp[N[p] + 1]; }
      }
      const int fi0 = rp[i], fi1 = rp[i + 1];

      // f = -A[i,N]
      double f[kS8];
#pragma unroll
      for (int q = 0; q < kS8; ++q) f[q] = 0.0;
      for (int e = fi0; e < fi1; e += 8) {
        int kk[8];
        double xx[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          kk[j] = -1;
          xx[j] = 0.0;
          if (e + j < fi1) { kk[j] = ci[e + j]; xx[j] = va[e + j]; }
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          if (kk[j] >= 0) {
            bool hit;
            const int q = pos8(N, kk[j], &hit);
#pragma unroll
            for (int qq = 0; qq < kS8; ++qq)
              if (hit && q == qq) f[qq] = -xx[j];
          }
        }
      }

      // K = (A[N,N])^T in FP64, identity on the padding
      double K[kS8][kS8];
#pragma unroll
      for (int q = 0; q < kS8; ++q)
#pragma unroll
        for (int p = 0; p < kS8; ++p) K[q][p] = (q == p && q >= s) ? 1.0 : 0.0;
      gather8_pair<0>(ci, va, N, e0, e1, K);
      gather8_pair<2>(ci, va, N, e0, e1, K);
      gather8_pair<4>(ci, va, N, e0, e1, K);
      gather8_pair<6>(ci, va, N, e0, e1, K);

      // scale by a power of two, FP32 LU without pivoting; a small or
      // non-finite pivot hands the row to the FP64 solver with pivoting
      double amax = 0.0, knorm = 0.0, fnorm = 0.0;
#pragma unroll
      for (int q = 0; q < kS8; ++q) {
        double rs = 0.0;
#pragma unroll
        for (int p = 0; p < kS8; ++p) {
          amax = fmax(amax, fabs(K[q][p]));
          rs += fabs(K[q][p]);
        }
        knorm = fmax(knorm, rs);
        fnorm = fmax(fnorm, fabs(f[q]));
      }
      int ex = 0;
      frexp(amax > 0.0 ? amax : 1.0, &ex);
      const double scale = ldexp(1.0, -ex);
      float L[kS8][kS8];
#pragma unroll
      for (int q = 0; q < kS8; ++q)
#pragma unroll
        for (int p = 0; p < kS8; ++p) L[q][p] = (float)(K[q][p] * scale);
      float inv[kS8];
      bool bad = !(amax > 0.0) || !(amax * scale < 1e30);
#pragma unroll
      for (int k = 0; k < kS8; ++k) {
        const float piv = L[k][k];
        bad |= !(fabsf(piv) >= 0x1p-24f);
        inv[k] = __builtin_amdgcn_rcpf(piv);
#pragma unroll
        for (int q = k + 1; q < kS8; ++q) {
          const float l = L[q][k] * inv[k];
          L[q][k] = l;
#pragma unroll
          for (int p = k + 1; p < kS8; ++p) L[q][p] = fmaf(-l, L[k][p], L[q][p]);
        }
      }

      double z[kS8];
      int it = 0;
      bool conv = false;
      if (!bad) {
        float y[kS8];
#pragma unroll
        for (int q = 0; q < kS8; ++q) y[q] = (float)(f[q] * scale);
        lu8_solve(L, inv, y);
#pragma unroll
        for (int q = 0; q < kS8; ++q) z[q] = (double)y[q];
        for (it = 1; it <= kRefineMax; ++it) {
          double rn = 0.0, zn = 0.0;
#pragma unroll
          for (int q = 0; q < kS8; ++q) {
            double r = f[q];
#pragma unroll
            for (int p = 0; p < kS8; ++p) r = fma(-K[q][p], z[p], r);
            y[q] = (float)(r * scale);
            rn = fmax(rn, fabs(r));
            zn = fmax(zn, fabs(z[q]));
          }
          if (rn <= 0x1p-47 * (knorm * zn + fnorm)) { conv = true; break; }
          lu8_solve(L, inv, y);
#pragma unroll
          for (int q = 0; q < kS8; ++q) z[q] += (double)y[q];
        }
#pragma unroll
        for (int q = 0; q < kS8; ++q) conv &= (z[q] == z[q]);
      }
      if (!conv) {
        // FP32 factorisation not trusted: the workgroup solver redoes the row in FP64
        const int qc = atomicAdd(&w.cnt->nC, 1);
        if (qc < w.capC) w.binC[qc] = cc.c * w.chunk + t;
        else flag_row(st, ST_UNSUPPORTED, i);
        continue;
      }
      rmx.add(w, cc.m, it);

      // R row: the F-entries of N(i) around the injected C-point
      int dpos = 0;
#pragma unroll
      for (int p = 0; p < kS8; ++p) dpos += (N[p] < i) ? 1 : 0;
#pragma unroll
      for (int p = 0; p < kS8; ++p)
        if (p < s) put_f_entry(w, d, cc.fine0, off + p + (p >= dpos ? 1 : 0), N[p], i, z[p]);
      d.Rci[off + dpos] = i;
      d.Rva[off + dpos] = 1.0;
    }
  }
  }
  rmx.flush(w);
}

// ---------------------------------------------------------------------------
// workgroup-per-row FP64 solver (bin C)
// ---------------------------------------------------------------------------
constexpr int kWT = 256;
static_assert(kWT == kNT, "block_bfs runs on kNT threads");

__device__ __forceinline__ void block_argmax(double v, int idx, double* shv, int* shi, double* outv, int* outi) {
  const int tid = threadIdx.x;
  shv[tid] = v;
  shi[tid] = idx;
  __syncthreads();
  for (int o = kWT / 2; o > 0; o >>= 1) {
    if (tid < o) {
      const double a = shv[tid], b = shv[tid + o];
      const int ia = shi[tid], ib = shi[tid + o];
      if (b > a || (b == a && ib < ia)) { shv[tid] = b; shi[tid] = ib; }
    }
    __syncthreads();
  }
  *outv = shv[0];
  *outi = shi[0];
  __syncthreads();
}

// ---------------------------------------------------------------------------
// blocks of 32 < |N| <= 128 in the workgroup solver: FP32 LU of the scaled
// block in LDS, blocked by panels of 32 columns, the trailing updates on the
// matrix cores (v_mfma_f32_32x32x2f32, one 32x32 tile per wavefront and
// step), FP32 triangular solves, FP64 residuals from A's CSR rows and
// iterative refinement.  No pivoting: a tiny pivot or no convergence hands
// the row to the FP64 solver with partial pivoting.
// ---------------------------------------------------------------------------
constexpr int kMfmaMax = 128;
constexpr int kRefineMaxBf16 = 10;  // refinement steps of the BF16-update factorisation
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef short bf16x4 __attribute__((ext_vector_type(4)));

// x rounded to bfloat16 (nearest, ties to even), as its 16 bits; x finite
__device__ __forceinline__ short to_bf16(float x) {
  uint32_t u = __float_as_uint(x);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (short)(u >> 16);
}

// max of v over the workgroup (all threads call; result to all)
__device__ __forceinline__ double block_maxd(double v, double* shv) {
  const int tid = threadIdx.x;
  shv[tid] = v;
  __syncthreads();
  for (int o = kWT / 2; o > 0; o >>= 1) {
    if (tid < o) shv[tid] = fmax(shv[tid], shv[tid + o]);
    __syncthreads();
  }
  const double r = shv[0];
  __syncthreads();
  return r;
}

// y <- K^{-1} y for the packed LU (unit lower L below the diagonal, U on and
// above it) of the S x S block in LDS (stride lda, S a multiple of 32); y in
// LDS.  All threads call.  Blocked by 32: wavefront 0 solves a diagonal block
// (unrolled, the solved entry of each step to all lanes by v_readlane), then
// every thread updates the remaining entries with that block's column strip,
// one mat-vec row per thread.
__device__ __forceinline__ void mf_lu_solve(const float* K, int lda, int S, float* y) {
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  for (int o = 0; o < S; o += 32) {  // forward, unit lower
    if (tid < 64) {
      float v = (lane < 32) ? y[o + lane] : 0.f;
#pragma unroll
      for (int k = 0; k < 32; ++k) {
        const float yk = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k));
        if (lane > k && lane < 32) v = fmaf(-K[(o + lane) * lda + o + k], yk, v);
      }
      if (lane < 32) y[o + lane] = v;
    }
    __syncthreads();
    for (int q = o + 32 + tid; q < S; q += kWT) {
      float acc = y[q];
#pragma unroll 8
      for (int k = 0; k < 32; ++k) acc = fmaf(-K[q * lda + o + k], y[o + k], acc);
      y[q] = acc;
    }
    __syncthreads();
  }
  for (int o = S - 32; o >= 0; o -= 32) {  // backward, upper
    if (tid < 64) {
      float v = (lane < 32) ? y[o + lane] : 0.f;
#pragma unroll
      for (int k = 31; k >= 0; --k) {
        if (lane == k) v = v / K[(o + k) * lda + o + k];
        const float yk = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k));
        if (lane < k) v = fmaf(-K[(o + lane) * lda + o + k], yk, v);
      }
      if (lane < 32) y[o + lane] = v;
    }
    __syncthreads();
    for (int q = tid; q < o; q += kWT) {
      float acc = y[q];
#pragma unroll 8
      for (int k = 0; k < 32; ++k) acc = fmaf(-K[q * lda + o + k], y[o + k], acc);
      y[q] = acc;
    }
    __syncthreads();
  }
}

// Returns true with the solution in z[0..s) when the row converged.
// N: sorted neighbourhood (LDS); K: LDS buffer of (kMfmaMax+1)*kMfmaMax
// floats; f, z, r: LDS FP64 vectors of kMfmaMax; y: LDS FP32 vector of
// kMfmaMax.  bf16: the trailing updates take their L21 and U12 tiles
// rounded to bfloat16 (v_mfma_f32_32x32x8bf16_1k, FP32 accumulation), and
// the refinement may take up to kRefineMaxBf16 steps.
// LDS scratch of the residual's column lists (see below)
struct ResidLists {
  int* cnt;  // [kMfmaMax + 1]
  int* off;  // [kMfmaMax + 1]
  int* pp;   // [cap] block row p of each entry
  int* pe;   // [cap] its entry in A
  int* bnd;  // [2 kMfmaMax] row bounds, for rows whose lists exceed cap
  int cap;
};

__device__ __forceinline__ bool mixed_big_row(const GDesc& d, int i, const int* N, int s, float* K, double* f, double* z,
                              double* r, float* y, double* shv, int* s_flag, int* it_out, const ResidLists& rl,
                              bool bf16) {
  const int tid = threadIdx.x;
  const int lane = tid & 63, wv = tid >> 6;
  const int S = (s + 31) & ~31;
  const int lda = S + 1;
  // scale: a power of two from the largest entry of the rows of N; norms
  double amax = 0.0, rsum = 0.0;
  for (int p = tid; p < s; p += kWT) {
    const int u = N[p];
    double rs = 0.0;
    for (int ee = d.rp[u]; ee < d.rp[u + 1]; ++ee) {
      const double v = fabs(d.va[ee]);
      amax = fmax(amax, v);
      rs += v;
    }
    rsum = fmax(rsum, rs);
  }
  amax = block_maxd(amax, shv);
  const double knorm = block_maxd(rsum, shv);
  if (!(amax > 0.0) || !(amax < 1e300)) return false;
  int ex = 0;
  frexp(amax, &ex);
  const double scale = ldexp(1.0, -ex);
  // the scaled block in FP32, identity on the padding; f = -A[i,N] in FP64
  for (int t = tid; t < S * lda; t += kWT) {
    const int q = t / lda, p = t - q * lda;
    K[t] = (q == p && q >= s) ? 1.f : 0.f;
  }
  for (int t = tid; t < kMfmaMax; t += kWT) { f[t] = 0.0; z[t] = 0.0; }
  __syncthreads();
  for (int p = tid; p < s; p += kWT) {
    const int u = N[p];
    for (int ee = d.rp[u]; ee < d.rp[u + 1]; ++ee) {
      const int q = find_sorted(N, s, d.ci[ee]);
      if (q >= 0) K[q * lda + p] = (float)(d.va[ee] * scale);
    }
  }
  for (int ee = d.rp[i] + tid; ee < d.rp[i + 1]; ee += kWT) {
    const int q = find_sorted(N, s, d.ci[ee]);
    if (q >= 0) f[q] = -d.va[ee];
  }
  if (tid == 0) s_flag[0] = 0;
  __syncthreads();

  // ---- blocked LU, panels of 32 columns ----
  for (int P0 = 0; P0 < S; P0 += 32) {
    const int Pe = P0 + 32;
    for (int k = P0; k < Pe; ++k) {
      const float piv = K[k * lda + k];
      if (tid == 0 && !(fabsf(piv) >= 0x1p-24f)) s_flag[0] = 1;
      const float pinv = __builtin_amdgcn_rcpf(piv);
      for (int q = k + 1 + tid; q < S; q += kWT) K[q * lda + k] *= pinv;
      __syncthreads();
      // rows of this block row: every column to the right (they become U);
      // rows below: the panel's columns only
      const int nr1 = Pe - k - 1, nc1 = S - k - 1;  // block-row part
      const int nr2 = S - Pe, nc2 = Pe - k - 1;     // panel part below
      const int n1 = nr1 * nc1, n2 = nr2 * nc2;
      for (int t = tid; t < n1 + n2; t += kWT) {
        int q, c;
        if (t < n1) { q = k + 1 + t / nc1; c = k + 1 + t % nc1; }
        else { const int u = t - n1; q = Pe + u / nc2; c = k + 1 + u % nc2; }
        K[q * lda + c] = fmaf(-K[q * lda + k], K[k * lda + c], K[q * lda + c]);
      }
      __syncthreads();
    }
    // trailing update K22 -= L21 U12 on the matrix cores
    const int T = (S - Pe) / 32;
    for (int tile = wv; tile < T * T; tile += kWT / 64) {
      const int i0 = Pe + 32 * (tile / T), j0 = Pe + 32 * (tile % T);
      floatx16 acc;
#pragma unroll
      for (int rr = 0; rr < 16; ++rr) {
        const int row = i0 + 8 * (rr / 4) + 4 * (lane / 32) + (rr % 4);
        acc[rr] = K[row * lda + j0 + (lane % 32)];
      }
      if (bf16) {
        // lane l supplies A[l % 32][4 (l / 32) + j] and B[4 (l / 32) + j][l % 32], j < 4
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          const int kc = P0 + 8 * kk + 4 * (lane / 32);
          bf16x4 a, b;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            a[j] = to_bf16(-K[(i0 + lane % 32) * lda + kc + j]);
            b[j] = to_bf16(K[(kc + j) * lda + j0 + lane % 32]);
          }
          acc = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(a, b, acc, 0, 0, 0);
        }
      } else {
#pragma unroll
        for (int kk = 0; kk < 16; ++kk) {
          const int kc = P0 + 2 * kk + lane / 32;
          const float a = -K[(i0 + lane % 32) * lda + kc];
          const float b = K[kc * lda + j0 + lane % 32];
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc, 0, 0, 0);
        }
      }
#pragma unroll
      for (int rr = 0; rr < 16; ++rr) {
        const int row = i0 + 8 * (rr / 4) + 4 * (lane / 32) + (rr % 4);
        K[row * lda + j0 + (lane % 32)] = acc[rr];
      }
    }
    __syncthreads();
  }
  if (s_flag[0]) return false;

  // ---- solve and refine ----
  const double fnorm = [&] {
    double m = 0.0;
    for (int t = tid; t < s; t += kWT) m = fmax(m, fabs(f[t]));
    return block_maxd(m, shv);
  }();
  for (int t = tid; t < S; t += kWT) y[t] = (t < s) ? (float)(f[t] * scale) : 0.f;
  __syncthreads();
  mf_lu_solve(K, lda, S, y);
  for (int t = tid; t < s; t += kWT) z[t] = y[t];
  __syncthreads();
  // The residual r_q = f_q - sum_p a_{N_p, N_q} z_p reads, for each q, the
  // entries of column N_q in the rows N_p: lists built once per row (counted,
  // placed, then each ordered by p), so every residual sums in ascending p
  // (the same bits on every run) with independent loads.  Rows whose lists
  // exceed the scratch search each row N_p by bisection instead.
  int* cnt = rl.cnt;
  int* off = rl.off;
  for (int q = tid; q <= s; q += kWT) cnt[q] = 0;
  __syncthreads();
  for (int p = tid; p < s; p += kWT) {
    const int u = N[p];
    const int e1 = d.rp[u + 1];
    for (int e = d.rp[u]; e < e1; ++e) {
      const int q = find_sorted(N, s, d.ci[e]);
      if (q >= 0) atomicAdd(&cnt[q], 1);
    }
  }
  __syncthreads();
  if (tid == 0) {
    int o = 0;
    for (int q = 0; q < s; ++q) {
      off[q] = o;
      o += cnt[q];
      cnt[q] = 0;
    }
    off[s] = o;
  }
  __syncthreads();
  const bool lists = off[s] <= rl.cap;  // workgroup-uniform
  if (lists) {
    for (int p = tid; p < s; p += kWT) {
      const int u = N[p];
      const int e1 = d.rp[u + 1];
      for (int e = d.rp[u]; e < e1; ++e) {
        const int q = find_sorted(N, s, d.ci[e]);
        if (q >= 0) {
          const int k = off[q] + atomicAdd(&cnt[q], 1);
          rl.pp[k] = p;
          rl.pe[k] = e;
        }
      }
    }
    __syncthreads();
    for (int q = tid; q < s; q += kWT) {  // insertion sort of list q by p
      for (int k = off[q] + 1; k < off[q + 1]; ++k) {
        const int kp = rl.pp[k], ke = rl.pe[k];
        int m = k - 1;
        while (m >= off[q] && rl.pp[m] > kp) {
          rl.pp[m + 1] = rl.pp[m];
          rl.pe[m + 1] = rl.pe[m];
          --m;
        }
        rl.pp[m + 1] = kp;
        rl.pe[m + 1] = ke;
      }
    }
  } else {
    for (int p = tid; p < s; p += kWT) { rl.bnd[2 * p] = d.rp[N[p]]; rl.bnd[2 * p + 1] = d.rp[N[p] + 1]; }
  }
  __syncthreads();
  const int itmax = bf16 ? kRefineMaxBf16 : kRefineMax;
  for (int it = 1; it <= itmax; ++it) {
    // r = f - K z with the FP64 entries of A, summed in ascending p
    for (int q = tid; q < s; q += kWT) {
      double acc = f[q];
      if (lists) {
        const int k1 = off[q + 1];
        for (int k = off[q]; k < k1; ++k) acc = fma(-d.va[rl.pe[k]], z[rl.pp[k]], acc);
      } else {
        const int col = N[q];
        for (int p = 0; p < s; ++p) {
          int lo = rl.bnd[2 * p];
          const int e1 = rl.bnd[2 * p + 1];
          int hi = e1;
          while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (d.ci[mid] < col) lo = mid + 1; else hi = mid;
          }
          if (lo < e1 && d.ci[lo] == col) acc = fma(-d.va[lo], z[p], acc);
        }
      }
      r[q] = acc;
    }
    __syncthreads();
    if (it > 1) {
      double rn = 0.0, zn = 0.0;
      for (int t = tid; t < s; t += kWT) { rn = fmax(rn, fabs(r[t])); zn = fmax(zn, fabs(z[t])); }
      rn = block_maxd(rn, shv);
      zn = block_maxd(zn, shv);
      if (rn <= 0x1p-47 * (knorm * zn + fnorm)) {
        *it_out = it;
        bool finite = true;
        for (int t = 0; t < s; ++t) finite &= (z[t] == z[t]);
        return finite;
      }
    }
    for (int t = tid; t < S; t += kWT) y[t] = (t < s) ? (float)(r[t] * scale) : 0.f;
    __syncthreads();
    mf_lu_solve(K, lda, S, y);
    for (int t = tid; t < s; t += kWT) z[t] += (double)y[t];
    __syncthreads();
  }
  return false;
}

__global__ __launch_bounds__(kWT) void k_rows_wg(Work w) {
  __shared__ WideBuf bb;
  // the FP64 block of the pivoting solver and the FP32 block of the mixed
  // solver share this buffer (one row at a time)
  constexpr int kBlkBytes = (int)std::max(sizeof(double) * kLdsBlockMax * (kLdsBlockMax + 1),
                                          sizeof(float) * kMfmaMax * (kMfmaMax + 1));
  __shared__ __align__(16) char s_blk[kBlkBytes];
  double* sK = reinterpret_cast<double*>(s_blk);
  float* sK32 = reinterpret_cast<float*>(s_blk);
  __shared__ double sf[kMaxBlock];
  __shared__ double s_z[kMfmaMax], s_r[kMfmaMax];
  __shared__ float s_y[kMfmaMax];
  __shared__ double shv[kWT];
  __shared__ int shi[kWT];
  __shared__ int s_bad, s_mflag;

  const int tid = threadIdx.x;
  const int qlen = min(w.cnt->nC, w.capC);
  // FP64 rows solved by this workgroup, per run of rows of one matrix
  int run_m = -1, run_n = 0;
  for (int pass = 0; pass < 2; ++pass) {
    // pass 0: blocks that fit in LDS, all workgroups; pass 1: larger blocks,
    // one global scratch slot per workgroup
    if (pass == 1 && (int64_t)blockIdx.x >= w.scratch_slots) {
      if (w.scratch_slots == 0) {
        // no scratch: report oversized rows instead of solving them
        for (int qi = blockIdx.x; qi < qlen; qi += gridDim.x) {
          const int e = w.binC[qi];
          if (w.gj && w.bigq[qi]) continue;  // solved by k_rows_gj
          const int c = e / w.chunk;
          const RowInfo ri = row_info(w, c, e - c * w.chunk);
          if (ri.s > kLdsBlockMax && tid == 0) flag_row(&w.st[ri.m], ST_UNSUPPORTED, ri.i);
        }
      }
      continue;
    }
    const int stride = (pass == 0) ? gridDim.x : (int)min<int64_t>(gridDim.x, w.scratch_slots);
    for (int qi = blockIdx.x; qi < qlen; qi += stride) {
      const int e = w.binC[qi];
      if (w.gj && w.bigq[qi]) continue;  // solved by k_rows_gj
      const int c = e / w.chunk;
      const RowInfo ri = row_info(w, c, e - c * w.chunk);
      const bool big = ri.s > kLdsBlockMax;
      if (big != (pass == 1)) continue;
      MatStatus* st = &w.st[ri.m];
      if (!matrix_live(*st)) continue;
      const GDesc d = gview(w.desc[ri.m]);
      const int i = ri.i;
      if (tid == 0) d.Rrp[ri.r] = ri.off;
      int* N;
      const int s = block_bfs(d.n, i, d.ell, d.grp, d.gci, d.gva, d.cf, d.theta, d.cmax, d.agg_rp, d.agg_list, bb,
                              &N, d.literal != 0);
      __syncthreads();
      if (s != ri.s) {
        if (tid == 0) flag_row(st, s < 0 ? ST_UNSUPPORTED : ST_INVALID, i);
        __syncthreads();
        continue;
      }
      // blocks above 32 points: the mixed solver first
      int itm = 0;
      bool mixed_ok = false;
      if (s > 32 && s <= kMfmaMax) {
        static_assert(kWN >= kMfmaMax + 1 && kWN + 1 >= 2 * kMfmaMax, "the residual's lists fit the search's buffers");
        const ResidLists rl{bb.fr, bb.nl, bb.cand, bb.kb, bb.dp, kWC};
        mixed_ok = mixed_big_row(d, i, N, s, sK32, sf, s_z, s_r, s_y, shv, &s_mflag, &itm, rl, w.bf16 != 0);
        if (!mixed_ok && w.bf16) {
          // the BF16-update factorisation did not converge: FP32 updates next
          if (tid == 0) atomicAdd(&st->n_retry, 1);
          mixed_ok = mixed_big_row(d, i, N, s, sK32, sf, s_z, s_r, s_y, shv, &s_mflag, &itm, rl, false);
        }
      }
      if (mixed_ok) {
        for (int t = tid; t < s; t += kWT) sf[t] = s_z[t];
        if (tid == 0 && itm > __hip_atomic_load(&st->refine_max, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
          atomicMax(&st->refine_max, itm);
        __syncthreads();
      } else {
      if (big && (int64_t)s * s > w.scratch_stride) {
        // the scratch was sized for smaller blocks (an asynchronous call
        // after a smaller batch): report the row instead of solving it
        if (tid == 0) flag_row(st, ST_UNSUPPORTED, i);
        __syncthreads();
        continue;
      }
      const int ld = big ? s : (kLdsBlockMax + 1);
      double* K = big ? (w.scratch + (int64_t)blockIdx.x * w.scratch_stride) : sK;
      for (int t = tid; t < s * ld; t += kWT) K[t] = 0.0;
      for (int t = tid; t < s; t += kWT) sf[t] = 0.0;
      __syncthreads();
      // K[q][p] = a_{N_p, N_q}: thread p walks row N_p
      for (int p = tid; p < s; p += kWT) {
        const int u = N[p];
        const int e1 = d.rp[u + 1];
        for (int ee = d.rp[u]; ee < e1; ++ee) {
          const int q = find_sorted(N, s, d.ci[ee]);
          if (q >= 0) K[(int64_t)q * ld + p] = d.va[ee];
        }
      }
      for (int ee = d.rp[i] + tid; ee < d.rp[i + 1]; ee += kWT) {
        const int q = find_sorted(N, s, d.ci[ee]);
        if (q >= 0) sf[q] = -d.va[ee];
      }
      __syncthreads();
      // max |K| for the singularity threshold
      double amax = 0.0;
      for (int t = tid; t < s * s; t += kWT) amax = fmax(amax, fabs(K[(int64_t)(t / s) * ld + (t % s)]));
      int dummy;
      block_argmax(amax, 0, shv, shi, &amax, &dummy);
      const double tiny = 1e-14 * amax;
      if (tid == 0) s_bad = 0;
      __syncthreads();
      for (int k = 0; k < s; ++k) {
        double best = -1.0;
        int bi = k;
        for (int q = k + tid; q < s; q += kWT) {
          const double v = fabs(K[(int64_t)q * ld + k]);
          if (v > best) { best = v; bi = q; }
        }
        int p;
        block_argmax(best, bi, shv, shi, &best, &p);
        if (!(best > tiny)) { if (tid == 0) s_bad = 1; __syncthreads(); break; }
        if (p != k) {
          for (int cc = tid; cc < s; cc += kWT) {
            const double t0 = K[(int64_t)k * ld + cc];
            K[(int64_t)k * ld + cc] = K[(int64_t)p * ld + cc];
            K[(int64_t)p * ld + cc] = t0;
          }
          if (tid == 0) { const double t0 = sf[k]; sf[k] = sf[p]; sf[p] = t0; }
          __syncthreads();
        }
        const double piv = K[(int64_t)k * ld + k];
        const int rem = s - k - 1;
        for (int t = tid; t < rem * (rem + 1); t += kWT) {
          const int q = k + 1 + t / (rem + 1);
          const int cc = k + t % (rem + 1);  // cc == k handles the right-hand side
          const double l = K[(int64_t)q * ld + k] / piv;
          if (cc == k) sf[q] -= l * sf[k];
          else K[(int64_t)q * ld + cc] -= l * K[(int64_t)k * ld + cc];
        }
        __syncthreads();
      }
      if (s_bad) {
        if (tid == 0) flag_row(st, ST_SINGULAR, i);
        for (int t = tid; t < s; t += kWT) sf[t] = 0.0;
        __syncthreads();
      } else {
        for (int k = s - 1; k >= 0; --k) {
          if (tid == 0) sf[k] /= K[(int64_t)k * ld + k];
          __syncthreads();
          for (int q = tid; q < k; q += kWT) sf[q] -= K[(int64_t)q * ld + k] * sf[k];
          __syncthreads();
        }
      }
      if (tid == 0) {
        if (ri.m != run_m) {
          if (run_n) atomicAdd(&w.st[run_m].n_fp64, run_n);
          run_m = ri.m;
          run_n = 0;
        }
        ++run_n;
      }
      }  // FP64 solver
      // R row
      int dpos = 0;
      {
        int cntb = 0;
        for (int p = tid; p < s; p += kWT) cntb += N[p] < i;
        shi[tid] = cntb;
        __syncthreads();
        for (int o = kWT / 2; o > 0; o >>= 1) { if (tid < o) shi[tid] += shi[tid + o]; __syncthreads(); }
        dpos = shi[0];
        __syncthreads();
      }
      for (int p = tid; p < s; p += kWT) put_f_entry(w, d, ri.fine0, ri.off + p + (p >= dpos ? 1 : 0), N[p], i, sf[p]);
      if (tid == 0) {
        d.Rci[ri.off + dpos] = i;
        d.Rva[ri.off + dpos] = 1.0;
      }
      __syncthreads();
    }
  }
  if (tid == 0 && run_n) atomicAdd(&w.st[run_m].n_fp64, run_n);
}

// ---------------------------------------------------------------------------
// projection
// ---------------------------------------------------------------------------
// Constraint projection, one workgroup per chunk of fine points, one thread
// per F-point j (the survey's exchange step: Algorithm 1's projection applied
// per F-column, QQ^T being diagonal): the entries of column j are those
// linked into its list by the solvers; the thread orders them by R position
// (ascending row, so the sums are the same on every run), forms
// d_j = sum B_i^2 and r_j = sum z_ij B_i - B_j in that order and sets
// z_ij -= B_i r_j / d_j.  A column with d_j = 0 is left alone and counted as
// uncovered.  Lists of up to kPL entries are ordered in registers; a longer
// list is taken kPL entries at a time, each pass keeping the smallest
// positions above the last one summed.
constexpr int kPL = 4;

struct ColEntry {
  int e[kPL];     // batch-wide R entry, INT32_MAX when empty
  int ci[kPL];    // the row's C-point
  double z[kPL];  // the entry's value before the projection
  int n;

  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int k = 0; k < kPL; ++k) { e[k] = INT32_MAX; ci[k] = 0; z[k] = 0.0; }
    n = 0;
  }
  // keep the kPL smallest positions (sorted); returns false when an entry
  // had to be dropped
  __device__ __forceinline__ bool insert(int ee, int ii, double zz) {
    int pos = 0;
#pragma unroll
    for (int k = 0; k < kPL; ++k) pos += (e[k] < ee) ? 1 : 0;
    const bool full = n == kPL;
    if (pos >= kPL) return false;
#pragma unroll
    for (int k = kPL - 1; k > 0; --k)
      if (k > pos) { e[k] = e[k - 1]; ci[k] = ci[k - 1]; z[k] = z[k - 1]; }
#pragma unroll
    for (int k = 0; k < kPL; ++k)
      if (k == pos) { e[k] = ee; ci[k] = ii; z[k] = zz; }
    n = full ? kPL : n + 1;
    return !full;
  }
};

// One F-column of any length (the general path of k_colproj): returns true
// when the column is uncovered (d_j = 0)
__device__ bool project_column(const Work& w, const GDesc& d, int64_t nzb, int j, int head) {
  // A list holds at most one record per row, so a walk of more than n steps
  // means a record linked twice (a cycle): the column is then left as
  // written and counted as uncovered rather than walked for ever.
  // first pass: the kPL smallest positions of the list
  ColEntry L;
  L.clear();
  bool more = false;
  int steps = 0;
  for (int e = head; e >= 0;) {
    const int2 lk = w.clink[e];
    const double zv = d.Rva[e - nzb];
    more |= !L.insert(e, lk.y, zv);
    e = lk.x;
    if (++steps > d.n) return true;
  }
  double dsum = 0.0, rsum = 0.0;
#pragma unroll
  for (int k = 0; k < kPL; ++k) {
    if (k < L.n) {
      const double bi = d.B[L.ci[k]];
      dsum = fma(bi, bi, dsum);
      rsum = fma(L.z[k], bi, rsum);
    }
  }
  // longer lists: further passes, each over the positions above the last
  // one taken
  int last = L.e[kPL - 1];
  while (more) {
    ColEntry M;
    M.clear();
    more = false;
    for (int e = head; e >= 0;) {
      const int2 lk = w.clink[e];
      if (e > last) more |= !M.insert(e, lk.y, d.Rva[e - nzb]);
      e = lk.x;
    }  // (the first walk ended, so this one does)
#pragma unroll
    for (int k = 0; k < kPL; ++k) {
      if (k < M.n) {
        const double bi = d.B[M.ci[k]];
        dsum = fma(bi, bi, dsum);
        rsum = fma(M.z[k], bi, rsum);
      }
    }
    last = M.e[kPL - 1];
  }
  if (!(dsum > 0.0)) return true;
  const double q = (rsum - d.B[j]) / dsum;
  if (L.n < kPL || L.e[kPL - 1] == last) {
    // the whole list is in registers
#pragma unroll
    for (int k = 0; k < kPL; ++k)
      if (k < L.n) d.Rva[L.e[k] - nzb] = L.z[k] - d.B[L.ci[k]] * q;
  } else {
    for (int e = head; e >= 0;) {  // the walk ended above, so no cycle here
      const int2 lk = w.clink[e];
      d.Rva[e - nzb] -= d.B[lk.y] * q;
      e = lk.x;
    }
  }
  return false;
}

// Constraint projection kernel: IC F-points per thread walked together (their
// list loads in flight at once), each list of up to kPI records in
// registers; a longer list takes the general path.
constexpr int kIC = 4, kPI = 4;

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_colproj(Work w) {
  __shared__ int s_unc;
  // chunks newest first: the numeric kernels walked each XCD's rows in
  // ascending order, so the last chunks' records and values are the ones
  // most likely still in the caches
  const int c = xcd_logical_block_reversed();
  const int tid = threadIdx.x;
  const int m = w.chunk_mat[c];
  const GDesc d = gview(w.desc[m]);
  if (!d.B || !matrix_live(w.st[m])) return;
  const int64_t nzb = d.link_base;  // list entry of R position p: nzb + p
  const int f0 = (c - d.chunk0) * w.chunk;
  const int f1 = min(f0 + w.chunk, d.n);
  if (tid == 0) s_unc = 0;
  __syncthreads();
  int unc = 0;
  for (int jb = f0 + tid; jb < f1; jb += blockDim.x * kIC) {
    int j[kIC], e[kIC], head[kIC], n[kIC];
    int re[kIC][kPI], ri[kIC][kPI];
    double rz[kIC][kPI];
#pragma unroll
    for (int q = 0; q < kIC; ++q) {
      j[q] = jb + q * (int)blockDim.x;
      head[q] = -1;
      n[q] = 0;
      if (j[q] < f1) {
        const int8_t cj = d.cf[j[q]];
        const int h = w.chead[d.fine0 + j[q]];
        if (cj == 0) {
          head[q] = h;
          if (h < 0) ++unc;
        }
      }
      e[q] = head[q];
    }
    // walk the lists together, kPI steps
#pragma unroll
    for (int k = 0; k < kPI; ++k) {
#pragma unroll
      for (int q = 0; q < kIC; ++q) {
        re[q][k] = INT32_MAX;
        ri[q][k] = 0;
        rz[q][k] = 0.0;
        if (e[q] >= 0) {
          const int2 lk = w.clink[e[q]];
          re[q][k] = e[q];
          ri[q][k] = lk.y;
          rz[q][k] = d.Rva[e[q] - nzb];
          e[q] = lk.x;
          ++n[q];
        }
      }
    }
#pragma unroll
    for (int q = 0; q < kIC; ++q) {
      if (head[q] < 0) continue;
      if (e[q] >= 0) {  // more than kPI records
        unc += project_column(w, d, nzb, j[q], head[q]) ? 1 : 0;
        continue;
      }
      // order the records by R position (a sorting network on kPI = 4)
#define CLAIR_CS(A, B)                                                   \
  if (re[q][B] < re[q][A]) {                                            \
    const int te = re[q][A]; re[q][A] = re[q][B]; re[q][B] = te;         \
    const int ti = ri[q][A]; ri[q][A] = ri[q][B]; ri[q][B] = ti;         \
    const double tz = rz[q][A]; rz[q][A] = rz[q][B]; rz[q][B] = tz;      \
  }
      CLAIR_CS(0, 1) CLAIR_CS(2, 3) CLAIR_CS(0, 2) CLAIR_CS(1, 3) CLAIR_CS(1, 2)
#undef CLAIR_CS
      double bi[kPI];
#pragma unroll
      for (int k = 0; k < kPI; ++k) bi[k] = (k < n[q]) ? d.B[ri[q][k]] : 0.0;
      const double bj = d.B[j[q]];
      double dsum = 0.0, rsum = 0.0;
#pragma unroll
      for (int k = 0; k < kPI; ++k) {
        if (k < n[q]) {
          dsum = fma(bi[k], bi[k], dsum);
          rsum = fma(rz[q][k], bi[k], rsum);
        }
      }
      if (!(dsum > 0.0)) { ++unc; continue; }
      const double qq = (rsum - bj) / dsum;
#pragma unroll
      for (int k = 0; k < kPI; ++k)
        if (k < n[q]) d.Rva[re[q][k] - nzb] = rz[q][k] - bi[k] * qq;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) unc += __shfl_xor(unc, o, 64);
  if ((tid & 63) == 0 && unc) atomicAdd(&s_unc, unc);
  __syncthreads();
  if (tid == 0 && s_unc) atomicAdd((unsigned long long*)&w.st[m].n_uncovered, (unsigned long long)s_unc);
}

// Column maxima for the strength test: cmax[v] = max over w != v of |a_wv|,
// for every matrix of the batch (batch-wide fine numbering).  Non-negative
// doubles order like their bit patterns, so an unsigned 64-bit atomic max
// takes the maximum.
//
// Bound: the rate of atomics in memory (about 130 a ns), so a workgroup gathers
// the maxima of its own run of points in LDS and sends one atomic for each;
// only entries that leave the run go to memory one by one.  1001^2 nine-point
// rows: 69 us with an atomic per entry (also with eight entries a thread in
// flight), now 52 (two rows a thread: 55).
__global__ void k_colmax_clear(Work w, int64_t n_total) {
  for (int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; g < n_total; g += (int64_t)gridDim.x * blockDim.x)
    w.cmax[g] = 0.0;
}

constexpr int kCMT = 1024, kCMRows = 4;  // threads of a workgroup; rows a thread takes, at most

__global__ __launch_bounds__(kCMT) void k_colmax(Work w, int64_t n_total, int rows) {
  __shared__ unsigned long long s_max[kCMT * kCMRows];
  const int tid = threadIdx.x;
  const int np = kCMT * rows;
  const int64_t g0 = (int64_t)blockIdx.x * np;
  for (int t = tid; t < np; t += kCMT) s_max[t] = 0;
  __syncthreads();
  for (int r = 0; r < rows; ++r) {
    const int64_t g = g0 + r * kCMT + tid;
    if (g >= n_total) break;
    int lo = 0, hi = w.nmat - 1;  // the matrix holding fine point g
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (w.desc[mid].fine0 <= g) lo = mid; else hi = mid - 1;
    }
    const GDesc d = gview(w.desc[lo]);
    if (d.theta == 0.0 || !matrix_live(w.st[lo])) continue;
    const int u = (int)(g - d.fine0);
    const int64_t at = d.fine0 - g0;  // column v's place in s_max: at + v
    const int e1 = d.grp[u + 1];
    for (int e = d.grp[u]; e < e1; e += 8) {  // column maxima of the search graph
      int v[8];
      double x[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        v[k] = e + k < e1 ? d.gci[e + k] : u;
        x[k] = e + k < e1 ? d.gva[e + k] : 0.0;
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        if (v[k] == u || (unsigned)v[k] >= (unsigned)d.n) continue;
        const unsigned long long b = (unsigned long long)__double_as_longlong(fabs(x[k]));
        const int64_t q = at + v[k];
        if ((uint64_t)q < (uint64_t)np) atomicMax(&s_max[q], b);
        else atomicMax(reinterpret_cast<unsigned long long*>(w.cmax + d.fine0 + v[k]), b);
      }
    }
  }
  __syncthreads();
  for (int t = tid; t < np; t += kCMT)
    if (s_max[t]) atomicMax(reinterpret_cast<unsigned long long*>(w.cmax + g0 + t), s_max[t]);
}

// Member lists of the aggregates (matrices given with aggregates only):
// count per root, scan (host), scatter through cursors, sort per root.  An
// F-point j joins root r = agg[j] when r is a C-point index in range.
__device__ __forceinline__ int fine_matrix(const Work& w, int64_t g) {
  int lo = 0, hi = w.nmat - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (w.desc[mid].fine0 <= g) lo = mid; else hi = mid - 1;
  }
  return lo;
}

__device__ __forceinline__ int agg_root(const GDesc& d, int j) {
  if (!d.agg || d.cf[j] != 0) return -1;
  const int r = d.agg[j];
  return ((unsigned)r < (unsigned)d.n && d.cf[r] != 0) ? r : -1;
}

__global__ void k_agg_count(Work w, int64_t n_total) {
  for (int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; g < n_total; g += (int64_t)gridDim.x * blockDim.x) {
    const int m = fine_matrix(w, g);
    const GDesc d = gview(w.desc[m]);
    const int r = agg_root(d, (int)(g - d.fine0));
    if (r >= 0) atomicAdd(&w.agg_cnt[d.fine0 + r], 1);
  }
}

__global__ void k_agg_fill(Work w, int64_t n_total) {
  for (int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; g < n_total; g += (int64_t)gridDim.x * blockDim.x) {
    const int m = fine_matrix(w, g);
    const GDesc d = gview(w.desc[m]);
    const int j = (int)(g - d.fine0);
    const int r = agg_root(d, j);
    if (r >= 0) w.agg_list[w.agg_rp[d.fine0 + r] + atomicAdd(&w.agg_cnt[d.fine0 + r], 1)] = j;
  }
}

__global__ void k_agg_sort(Work w, int64_t n_total) {
  for (int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; g < n_total; g += (int64_t)gridDim.x * blockDim.x) {
    const int e0 = w.agg_rp[g], e1 = w.agg_rp[g + 1];
    for (int a = e0 + 1; a < e1; ++a) {
      const int k = w.agg_list[a];
      int b = a - 1;
      while (b >= e0 && w.agg_list[b] > k) {
        w.agg_list[b + 1] = w.agg_list[b];
        --b;
      }
      w.agg_list[b + 1] = k;
    }
  }
}

__global__ void k_fill_i32(int32_t* a, int64_t n, int32_t v) {
  for (int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; g < n; g += (int64_t)gridDim.x * blockDim.x) a[g] = v;
}

// A numeric pass without the symbolic pass before it (a plan's execute): the
// projection's column lists of all fine points emptied, and R.row_ptr[n_c] of
// every matrix.
__global__ void k_clear_sums(Work w, int64_t n) {
  for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x)
    w.chead[j] = -1;
  if (blockIdx.x == 0) {
    for (int m = threadIdx.x; m < w.nmat; m += blockDim.x) {
      const MatStatus& st = w.st[m];
      if (matrix_live(st) && w.desc[m].Rrp) w.desc[m].Rrp[st.n_c] = (int32_t)st.nnz;
    }
  }
}

}  // namespace

// a kernel, not a memset: the call may be captured into a graph
hipError_t launch_clear_sums(const Work& w, int64_t n_total, int blocks, hipStream_t s) {
  hipLaunchKernelGGL(k_clear_sums, dim3(blocks), dim3(256), 0, s, w, n_total);
  return hipGetLastError();
}

hipError_t launch_colmax(const Work& w, int64_t n_total, int cus, hipStream_t s) {
  if (n_total <= 0) return hipSuccess;
  const int64_t cb = std::min<int64_t>((n_total + 255) / 256, (int64_t)cus * 8);
  hipLaunchKernelGGL(k_colmax_clear, dim3((unsigned)cb), dim3(256), 0, s, w, n_total);
  // four rows a thread where that leaves most CUs a workgroup, else one
  const int rows = n_total >= (int64_t)kCMT * kCMRows * cus / 2 ? kCMRows : 1;
  const int64_t per = (int64_t)kCMT * rows;
  hipLaunchKernelGGL(k_colmax, dim3((unsigned)((n_total + per - 1) / per)), dim3(kCMT), 0, s, w, n_total, rows);
  return hipGetLastError();
}

hipError_t launch_agg_lists(const Work& w, int64_t n_total, int blocks, int cus, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_i32, dim3(blocks), dim3(256), 0, s, w.agg_cnt, n_total, 0);
  hipLaunchKernelGGL(k_agg_count, dim3(blocks), dim3(256), 0, s, w, n_total);
  hipError_t e = launch_exclusive_scan(w.agg_cnt, (int)n_total, w.agg_rp, w.agg_sums, cus, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_fill_i32, dim3(blocks), dim3(256), 0, s, w.agg_cnt, n_total, 0);
  hipLaunchKernelGGL(k_agg_fill, dim3(blocks), dim3(256), 0, s, w, n_total);
  hipLaunchKernelGGL(k_agg_sort, dim3(blocks), dim3(256), 0, s, w, n_total);
  return hipGetLastError();
}

hipError_t launch_validate(const Work& w, int blocks, hipStream_t s) {
  hipLaunchKernelGGL(k_validate, dim3(blocks), dim3(256), 0, s, w);
  return hipGetLastError();
}

hipError_t launch_adj(const Work& w, hipStream_t s) {
  if (w.nchunks == 0 || w.adj_w == 0) return hipSuccess;
  const int per = (w.chunk + 255) / 256;
  const dim3 grid((unsigned)w.nchunks * (unsigned)per);
  if (w.adj_w == 4) hipLaunchKernelGGL(k_adj<4>, grid, dim3(256), 0, s, w);
  else if (w.adj_w == 8) hipLaunchKernelGGL(k_adj<8>, grid, dim3(256), 0, s, w);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_count(const Work& w, hipStream_t s) {
  if (w.nchunks == 0) return hipSuccess;
  const dim3 grid(w.nchunks), block(kNT);
  if (w.adj_w == 4) hipLaunchKernelGGL(k_count<4>, grid, block, 0, s, w);
  else if (w.adj_w == 8) hipLaunchKernelGGL(k_count<8>, grid, block, 0, s, w);
  else if (w.adj_w == 0) hipLaunchKernelGGL(k_count<0>, grid, block, 0, s, w);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_count_mid(const Work& w, int cus, hipStream_t s) {
  if (w.nchunks == 0) return hipSuccess;
  const dim3 grid(std::min(w.nchunks, std::max(8, cus * 8)));
#define CLAIR_MID(WW, NTT)                                                             \
  if (w.adj_w == WW && (NTT == 256) == (w.nchunks <= 4 * cus)) {                       \
    hipLaunchKernelGGL((k_count_mid<WW, NTT>), grid, dim3(NTT), 0, s, w);              \
    return hipGetLastError();                                                          \
  }
  CLAIR_MID(0, 256)
  CLAIR_MID(4, 256)
  CLAIR_MID(8, 256)
  CLAIR_MID(0, 128)
  CLAIR_MID(4, 128)
  CLAIR_MID(8, 128)
#undef CLAIR_MID
  return hipErrorInvalidValue;
}

hipError_t launch_count_wide(const Work& w, int blocks, hipStream_t s) {
  if (w.nchunks == 0) return hipSuccess;
  const dim3 grid(std::min(w.nchunks, std::max(1, blocks))), block(kNT);
  if (w.adj_w == 0) hipLaunchKernelGGL(k_count_wide<0>, grid, block, 0, s, w);
  else if (w.adj_w == 4) hipLaunchKernelGGL(k_count_wide<4>, grid, block, 0, s, w);
  else if (w.adj_w == 8) hipLaunchKernelGGL(k_count_wide<8>, grid, block, 0, s, w);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_count_big(const Work& w, int blocks, hipStream_t s) {
  if (w.nchunks == 0) return hipSuccess;
  hipLaunchKernelGGL(k_count_big, dim3(blocks), dim3(kNT), 0, s, w);
  return hipGetLastError();
}

hipError_t launch_scan(const Work& w, hipStream_t s) {
  hipLaunchKernelGGL(k_scan, dim3(1), dim3(1024), 0, s, w);
  return hipGetLastError();
}

hipError_t launch_rows8(const Work& w, int wg_threads, int cus, hipStream_t s) {
#define CLAIR_R8(NTT)                                                                       \
  if (wg_threads == NTT) {                                                                  \
    int per = 0;                                                                            \
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_rows8<NTT>, NTT, 0); \
    if (e != hipSuccess) return e;                                                          \
    const int blocks = (std::max(1, per) * cus + 7) / 8 * 8;                               \
    hipLaunchKernelGGL((k_rows8<NTT>), dim3(blocks), dim3(NTT), 0, s, w);                   \
    return hipGetLastError();                                                               \
  }
  CLAIR_R8(256)
  CLAIR_R8(128)
  CLAIR_R8(64)
#undef CLAIR_R8
  return hipErrorInvalidValue;
}

hipError_t launch_rows_wg(const Work& w, int blocks, hipStream_t s) {
  hipLaunchKernelGGL(k_rows_wg, dim3(blocks), dim3(kWT), 0, s, w);
  return hipGetLastError();
}

hipError_t launch_project(const Work& w, hipStream_t s) {
  hipLaunchKernelGGL(k_colproj, dim3(w.nchunks), dim3(256), 0, s, w);
  return hipGetLastError();
}

}  // namespace clair
