// mixed_device.h -- device code shared by the kernels of the mixed form
// (k_mixed, k_quad, k_tile and k_block.hip): row bookkeeping, work distribution, lane-group
// communication.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <stdint.h>

#include "clair_device.h"

namespace clair {

namespace {

// chunk index of global row g (0 <= g < total rows): between the chunks that
// hold the first rows of g's block of rows and of the next one, by bisection
// (one chunk where chunks are large; a few small ones otherwise)
__device__ __forceinline__ int row_chunk_fast(const Work& w, int g) {
  const int b = g >> w.rb_log;
  int lo = w.row_block_chunk[b];
  int hi = (int64_t)(b + 1) << w.rb_log < w.cnt->total_rows ? w.row_block_chunk[b + 1] : w.nchunks - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (w.chunk_rbase[mid] <= g) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// workgroups of NT threads of a kernel that fit on a CU at once (a property of
// the kernel and the architecture, asked for once per kernel: the query costs a
// few microseconds), -1 on failure
template <auto F, int NT>
inline int resident_blocks() {
  static std::atomic<int> known{0};
  int per = known.load(std::memory_order_relaxed);
  if (per > 0) return per;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, F, NT, 0) != hipSuccess) return -1;
  known.store(per, std::memory_order_relaxed);
  return per;
}

struct RowInfo {
  int m;     // matrix
  int i;     // fine index of the C-point
  int r;     // matrix-local row of R
  int off;   // first R entry of the row
  int s;     // |N(i)|
  int64_t fine0;
};

// row t of chunk c
__device__ __forceinline__ RowInfo row_info(const Work& w, int c, int t) {
  RowInfo ri;
  ri.m = w.chunk_mat[c];
  const GDesc d = gview(w.desc[ri.m]);
  const int64_t base = d.fine0 + (int64_t)(c - d.chunk0) * w.chunk;
  ri.i = w.clocal[base + t];
  const int l0 = w.lnz[base + t];
  const int l1 = (t + 1 < w.chunk_nc[c]) ? w.lnz[base + t + 1] : w.chunk_nnz[c];
  ri.off = (int)(w.chunk_nzglob[c] - w.st[ri.m].nz_base) + l0;
  ri.s = l1 - l0 - 1;
  ri.r = w.chunk_rbase[c] + t - w.st[ri.m].row_base;
  ri.fine0 = d.fine0;
  return ri;
}

__device__ __forceinline__ bool matrix_live(const MatStatus& st) {
  return st.status != ST_CAPACITY && st.status != ST_INVALID;
}

// F-entry (i, j) of R at position pos of its matrix: the value, and with a
// constraint vector the entry joins the list of column j for the projection
// (list entry link_base + pos, below the matrix's R capacity; one atomic
// exchange on the list head; the projection orders each list itself, so the
// exchange order does not matter)
__device__ __forceinline__ void put_f_entry(const Work& w, const GDesc& d, int64_t fine0, int pos, int j, int i,
                                            double z) {
  d.Rci[pos] = j;
  d.Rva[pos] = z;
  if (d.B) {
    const int64_t eg = d.link_base + pos;
    const int prev = atomicExch(&w.chead[fine0 + j], (int32_t)eg);
    w.clink[eg] = make_int2(prev, i);
  }
}

// Per-lane cache of the chunk a run of consecutive rows lies in: reloaded only
// when the row index crosses into another chunk, so a row costs one level of
// (coalesced) per-row loads instead of the chunk -> matrix -> descriptor chain.
// The matrix's pointers are not part of it: held per lane through a solve they
// cost up to 40 VGPRs, so the solvers read the few they need from the
// descriptor (row_desc) before the gather and again before the row's stores.
struct RowCursor {
  int c = -1;
  int rb = 0, re = 0;   // global rows [rb, re) of chunk c
  int m = 0;
  int nc = 0;           // C-rows in the chunk
  int tot = 0;          // nnz(R) of the chunk
  int2 bins = {0, 0};   // rows of the chunk in bin A and bin B
  int zoff = 0;         // R offset of the chunk inside its matrix
  int rbase_m = 0;      // first global row of the matrix
  int64_t fbase = 0;    // fine offset of the chunk's first point (batch-wide)
  bool live = false;

  __device__ __forceinline__ void seek(const Work& w, int g) {
    if (c >= 0 && g >= rb && g < re) return;
    c = row_chunk_fast(w, g);
    rb = w.chunk_rbase[c];
    re = w.chunk_rbase[c + 1];
    m = w.chunk_mat[c];
    const MatStatus& st = w.st[m];
    nc = w.chunk_nc[c];
    tot = w.chunk_nnz[c];
    bins = w.chunk_bins[c];
    zoff = (int)(w.chunk_nzglob[c] - st.nz_base);
    rbase_m = st.row_base;
    fbase = w.desc[m].fine0 + (int64_t)(c - w.desc[m].chunk0) * w.chunk;
    live = matrix_live(st);
  }
  // row g (inside the chunk): fine index, R offset and |N|
  __device__ __forceinline__ void row(const Work& w, int g, int* t, int* i, int* off, int* sz) const {
    const int tt = g - rb;
    *t = tt;
    *i = w.clocal[fbase + tt];
    const int l0 = w.lnz[fbase + tt];
    const int l1 = (tt + 1 < nc) ? w.lnz[fbase + tt + 1] : tot;
    *off = zoff + l0;
    *sz = l1 - l0 - 1;
  }
};

// matrix m's descriptor, read here and not kept from an earlier read
__device__ __forceinline__ GDesc row_desc(const Work& w, int m) {
  asm volatile("" ::: "memory");
  return gview(w.desc[m]);
}

// RowCursor with the matrix's pointers kept (md), for the solvers of few
// registers or short rows: the four-lane solver took 671 us with them kept and
// 824 with them read again per row (three wavefronts per SIMD either way).
struct ChunkCursor {
  int c = -1;
  int rb = 0, re = 0;   // global rows [rb, re) of chunk c
  int m = 0;
  int nc = 0;           // C-rows in the chunk
  int tot = 0;          // nnz(R) of the chunk
  int2 bins = {0, 0};   // rows of the chunk in bin A and bin B
  int zoff = 0;         // R offset of the chunk inside its matrix
  int rbase_m = 0;      // first global row of the matrix
  int64_t fbase = 0;    // fine offset of the chunk's first point (batch-wide)
  int64_t fine0 = 0;    // fine offset of the matrix (batch-wide)
  bool live = false;
  GDesc md;             // the matrix's pointers and geometry

  __device__ __forceinline__ void seek(const Work& w, int g) {
    if (c >= 0 && g >= rb && g < re) return;
    c = row_chunk_fast(w, g);
    rb = w.chunk_rbase[c];
    re = w.chunk_rbase[c + 1];
    m = w.chunk_mat[c];
    md = gview(w.desc[m]);
    const MatStatus& st = w.st[m];
    nc = w.chunk_nc[c];
    tot = w.chunk_nnz[c];
    bins = w.chunk_bins[c];
    zoff = (int)(w.chunk_nzglob[c] - st.nz_base);
    rbase_m = st.row_base;
    fine0 = md.fine0;
    fbase = md.fine0 + (int64_t)(c - md.chunk0) * w.chunk;
    live = matrix_live(st);
  }
  // row g (inside the chunk): fine index, R offset and |N|
  __device__ __forceinline__ void row(const Work& w, int g, int* t, int* i, int* off, int* sz) const {
    const int tt = g - rb;
    *t = tt;
    *i = w.clocal[fbase + tt];
    const int l0 = w.lnz[fbase + tt];
    const int l1 = (tt + 1 < nc) ? w.lnz[fbase + tt + 1] : tot;
    *off = zoff + l0;
    *sz = l1 - l0 - 1;
  }
};


// Logical workgroup index: the hardware deals workgroups to the 8 XCDs
// round-robin (block b runs on XCD b % 8).  Give each XCD a contiguous range
// of logical indices, so the rows one XCD works on are neighbours in the grid
// and share its L2.
__device__ __forceinline__ int xcd_logical_block(int nb) {
  const int b = blockIdx.x;
  const int x = b % 8, q = nb / 8, r = nb % 8;
  return x * q + min(x, r) + b / 8;
}
__device__ __forceinline__ int xcd_logical_block() { return xcd_logical_block(gridDim.x); }
// The same ranges, each walked from its end: the first workgroups of an XCD
// take the last blocks of its range.
__device__ __forceinline__ int xcd_logical_block_reversed() {
  const int nb = gridDim.x;
  const int b = blockIdx.x;
  const int x = b % 8, q = nb / 8, r = nb % 8;
  return x * q + min(x, r) + (q + (x < r ? 1 : 0)) - 1 - b / 8;
}

// Rows of the persistent numeric kernels: XCD x (= blockIdx.x % 8, the
// hardware deals workgroups round-robin) owns a contiguous eighth of all
// rows, and its workgroups take blocks of nb rows from it in turn.  The rows
// in flight on one XCD at any time are then neighbours, whose blocks share A
// rows in that XCD's L2 (with a contiguous range per workgroup they would be
// as many separate streams through A as there are workgroups).
struct RowBlocks {
  int xb, xe, k, nx, nb;
  __device__ __forceinline__ RowBlocks(int total, int nb_) {
    const int x = blockIdx.x % 8;
    const int per = (total + 7) / 8;
    xb = min(total, x * per);
    xe = min(total, xb + per);
    nx = (int)gridDim.x / 8 + ((int)(gridDim.x % 8) > x ? 1 : 0);
    k = blockIdx.x / 8;
    nb = nb_;
  }
  // the j-th block of this workgroup: rows [*b, *e); false past the end
  __device__ __forceinline__ bool block(int j, int* b, int* e) const {
    const int64_t s0 = xb + ((int64_t)k + (int64_t)j * nx) * nb;
    if (s0 >= xe) return false;
    *b = (int)s0;
    *e = min(xe, (int)s0 + nb);
    return true;
  }
};

// Most refinement steps of the rows a thread (lane 0 of a group) finished,
// per matrix: gathered in registers and sent with one global atomic when the
// thread moves on to another matrix or ends (one atomic per row would meet
// at a handful of addresses in a batch of many matrices).
struct RefineMax {
  int m = -1, v = 0;
  __device__ __forceinline__ void flush(const Work& w) {
    if (m >= 0 && v > __hip_atomic_load(&w.st[m].refine_max, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomicMax(&w.st[m].refine_max, v);
  }
  __device__ __forceinline__ void add(const Work& w, int mm, int it) {
    if (mm != m) {
      flush(w);
      m = mm;
      v = 0;
    }
    v = max(v, it);
  }
  // the last flush, by the whole wavefront (lanes without rows too): one atomic
  // per wavefront and matrix.  One per row group, where each has a row only, met
  // at one address: 330^2 five-point rows, distance 1, numeric pass 25 -> 16 us.
  __device__ __forceinline__ void flush_wave(const Work& w) {
    uint64_t left = __ballot(m >= 0);
    while (left) {
      const int lead = __ffsll((unsigned long long)left) - 1;
      const int mm = __builtin_amdgcn_readlane(m, lead);
      int mx = m == mm ? v : 0;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) mx = max(mx, __shfl_xor(mx, o, 64));
      if ((int)(threadIdx.x & 63) == lead &&
          mx > __hip_atomic_load(&w.st[mm].refine_max, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMax(&w.st[mm].refine_max, mx);
      left &= ~__ballot(m == mm);
    }
  }
};

// rows bin A takes: |N| <= 8 (GA = 1, 4 or 8), else |N| <= GA
__device__ __forceinline__ int small_limit(int GA) { return GA <= 4 ? 8 : GA; }
// stride of a row's slot in slotA
__device__ __forceinline__ int slot_stride(int GA) { return GA <= 4 ? 8 : GA; }

// Communication inside a group of G lanes (G = 8 or 16; groups are
// aligned runs of G lanes of a wavefront).
//
// gpart: the value of a partner lane for a butterfly-like reduction.  Steps 1
// and 2 pair lanes inside a quad (DPP quad_perm [1,0,3,2] and [2,3,0,1]), step
// 4 mirrors the halves of 8 lanes (DPP row_half_mirror), step 8 mirrors the
// halves of 16 (DPP row_mirror).  After the steps up to G/2 every lane holds the
// group's reduction.
template <int STEP>
__device__ __forceinline__ int gpart(int v) {
  if constexpr (STEP == 1) return __builtin_amdgcn_update_dpp(v, v, 0xB1, 0xF, 0xF, false);
  else if constexpr (STEP == 2) return __builtin_amdgcn_update_dpp(v, v, 0x4E, 0xF, 0xF, false);
  else if constexpr (STEP == 4) return __builtin_amdgcn_update_dpp(v, v, 0x141, 0xF, 0xF, false);
  else {
    static_assert(STEP == 8, "within sixteen lanes");
    return __builtin_amdgcn_update_dpp(v, v, 0x140, 0xF, 0xF, false);
  }
}
template <int STEP>
__device__ __forceinline__ double gpartd(double v) {
  return __hiloint2double(gpart<STEP>(__double2hiint(v)), gpart<STEP>(__double2loint(v)));
}

template <int G>
__device__ __forceinline__ int group_ori(int v) {
  v |= gpart<1>(v);
  if constexpr (G >= 4) v |= gpart<2>(v);
  if constexpr (G >= 8) v |= gpart<4>(v);
  if constexpr (G >= 16) v |= gpart<8>(v);
  return v;
}

// Position of key in the G sorted entries nb[0..G) (padded with INT32_MAX),
// or -1: a branch-free lower bound of fixed depth log2(G).  Several searches
// in a row have no loop between them, so their LDS reads overlap.
template <int G>
__device__ __forceinline__ int find_pos(const int* nb, int key) {
  int pos = 0;
#pragma unroll
  for (int step = G / 2; step >= 1; step >>= 1) pos += (nb[pos + step - 1] < key) ? step : 0;
  return (pos < G && nb[pos] == key) ? pos : -1;
}

constexpr int kRefineMax = 5;

}  // namespace

}  // namespace clair
