// k_block.hip -- rows of 33 to 128 points of the mixed form, one workgroup per
// row, the block's FP32 inverse in registers.
//
// The workgroup is a 16 x 16 grid of threads; thread (tr, tc) holds the block's
// rows tr, tr + 16, ... and columns tc, tc + 16, ... (a T x T tile, T =
// ceil(s / 16)).  Gauss-Jordan in place without pivoting: step k sends the pivot
// row and the pivot column through LDS (two buffers in turn, one barrier per
// step) and every thread updates its tile; the pivots are the LU's, so the
// tiny-pivot test is the LU's.  Each correction of the FP64 refinement is then
// one mat-vec with the inverse (partial sums over the tile, a sum over 16
// lanes), and the FP64 residual reads the block's entries, kept as column lists
// in LDS in ascending row order (the same bits on every run).  A tiny pivot, no
// convergence, more entries than the lists hold or a search of more than 128
// points leaves the row to k_rows_wg.
//
// Bound: the latency of s steps with one barrier each, hidden by four workgroups
// per CU (128 VGPRs, 53 more spilled to 216 bytes of scratch a lane, and 34.9 KB
// of LDS: one kernel serves T = 3 to 8).  The blocked LU of k_rows_wg holds
// its block in LDS (one workgroup per CU), takes two barriers and a pass over
// LDS per column and solves triangles in every correction: 2,500 rows of up to
// 108 points (150^2 nine-point at distance 5) take 3,385 us there, 295 here.  A
// block of more entries than the lists hold pays for the search and the count in
// vain: 300 rows of 128 points with about 100 entries a row, 57 us of 2,020.
// The matrix cores have nothing to add at this size: the whole elimination is
// 4 MFLOP a row, and a 32-column panel would still be 32 dependent steps.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "clair_device.h"
#include "clair_launch.h"
#include "mixed_device.h"
#include "search_device.h"

namespace clair {

namespace {

constexpr int kGT = 256;         // threads
constexpr int kGMax = 128;       // points
constexpr int kGEntries = 2048;  // entries of the residual's lists

struct BlockBuf {
  union {
    SearchBuf<kGMax, 4 * kGMax> search;
    float band[16 * 9 * 16];                     // sixteen rows of the block while the tiles are filled
    struct { float u[2][16 * 8], l[2][16 * 8]; } step;  // pivot row and column, by turns
  };
  double val[kGEntries];   // the lists: entries a_{N_p, N_q} of column q of A (row q of the block) ...
  uint16_t row[kGEntries]; // ... and their p
  int N[kGMax];
  int off[kGMax + 1], cnt[kGMax];
  double f[kGMax], z[kGMax], r[kGMax];
  float y[16 * 8];  // a correction's right-hand side, entry 16 b + tc at [tc * 8 + b]
  double red[8];
  int bad;
};

// max of two values over the workgroup, to every thread
__device__ __forceinline__ void block_max2(double& a, double& b, double* red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    a = fmax(a, __shfl_xor(a, o, 64));
    b = fmax(b, __shfl_xor(b, o, 64));
  }
  const int wv = threadIdx.x >> 6;
  __syncthreads();  // the previous use has been read
  if ((threadIdx.x & 63) == 0) { red[wv] = a; red[4 + wv] = b; }
  __syncthreads();
  a = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
  b = fmax(fmax(red[4], red[5]), fmax(red[6], red[7]));
}

// v summed over the 16 lanes of a DPP row, to all of them
__device__ __forceinline__ float row16_sum(float v) {
  v += __int_as_float(gpart<1>(__float_as_int(v)));
  v += __int_as_float(gpart<2>(__float_as_int(v)));
  v += __int_as_float(gpart<4>(__float_as_int(v)));
  v += __int_as_float(gpart<8>(__float_as_int(v)));
  return v;
}

// Solves the row whose lists, N, f are in B (s points, T = ceil(s / 16)): true
// with the solution in B.z.  All threads call.
template <int T>
__device__ __forceinline__ bool block_solve(BlockBuf& B, int s, double scale, double knorm, int* it_out) {
  constexpr int TP = 8, LDB = 16 * (T | 1);
  const int tid = threadIdx.x;
  const int tc = tid & 15, tr = tid >> 4;
  float kf[T][T];
  // the scaled block, sixteen rows at a time through LDS
#pragma unroll
  for (int a = 0; a < T; ++a) {
    for (int t = tid; t < 16 * LDB; t += kGT) B.band[t] = 0.f;
    __syncthreads();
    const int q = 16 * a + tr;
    if (q < s)
      for (int k = B.off[q] + tc; k < B.off[q + 1]; k += 16) B.band[tr * LDB + B.row[k]] = (float)(B.val[k] * scale);
    __syncthreads();
#pragma unroll
    for (int b = 0; b < T; ++b) kf[a][b] = B.band[tr * LDB + 16 * b + tc];
    __syncthreads();
  }
  int bad = 0;
#pragma unroll
  for (int ak = 0; ak < T; ++ak) {
    const int kn = min(16, s - 16 * ak);
#pragma unroll 1
    for (int kk = 0; kk < kn; ++kk) {
      float* U = B.step.u[kk & 1];
      float* L = B.step.l[kk & 1];
      if (tr == kk) {
#pragma unroll
        for (int b = 0; b < T; ++b) U[tc * TP + b] = kf[ak][b];
      }
      if (tc == kk) {
#pragma unroll
        for (int a = 0; a < T; ++a) L[tr * TP + a] = kf[a][ak];
      }
      __syncthreads();
      float u[T], l[T];
#pragma unroll
      for (int b = 0; b < T; ++b) u[b] = U[tc * TP + b];
#pragma unroll
      for (int a = 0; a < T; ++a) l[a] = L[tr * TP + a];
      const float piv = U[kk * TP + ak];
      bad |= !(fabsf(piv) >= 0x1p-24f);
      const float pinv = __builtin_amdgcn_rcpf(piv);
      const bool pr = tr == kk, pc = tc == kk;
#pragma unroll
      for (int a = 0; a < T; ++a) {
        const float lk = l[a] * pinv;
        // the pivot row subtracts (1 - 1/pivot) of itself
        const float la = (a == ak && pr) ? 1.f - pinv : lk;
#pragma unroll
        for (int b = 0; b < T; ++b) {
          const float x = fmaf(-la, u[b], kf[a][b]);
          kf[a][b] = (b == ak && pc) ? ((a == ak && pr) ? pinv : -lk) : x;
        }
      }
    }
  }
  if (bad) B.bad = 1;  // (the same on every thread)
  __syncthreads();
  if (B.bad) return false;
  double fn = 0.0, none = 0.0;
  if (tid < s) fn = fabs(B.f[tid]);
  block_max2(fn, none, B.red);
  // z += Kinv (scale x) for the FP64 vector x
  auto correct = [&](const double* x, bool first) {
    if (tid < 16 * T) B.y[(tid & 15) * TP + (tid >> 4)] = tid < s ? (float)(x[tid] * scale) : 0.f;
    __syncthreads();
    float v[T];
#pragma unroll
    for (int b = 0; b < T; ++b) v[b] = B.y[tc * TP + b];
#pragma unroll
    for (int a = 0; a < T; ++a) {
      float p = 0.f;
#pragma unroll
      for (int b = 0; b < T; ++b) p = fmaf(kf[a][b], v[b], p);
      p = row16_sum(p);
      const int q = 16 * a + tr;
      if (tc == a && q < s) B.z[q] = first ? (double)p : B.z[q] + (double)p;
    }
    __syncthreads();
  };
  correct(B.f, true);
#pragma unroll 1
  for (int it = 1; it <= kRefineMax; ++it) {
    // r = f - K z with the FP64 entries, in ascending p
    double rn = 0.0, zn = 0.0;
    if (tid < s) {
      double acc = B.f[tid];
      const int k1 = B.off[tid + 1];
      for (int k = B.off[tid]; k < k1; ++k) acc = fma(-B.val[k], B.z[B.row[k]], acc);
      B.r[tid] = acc;
      rn = fabs(acc);
      zn = fabs(B.z[tid]);
      if (!(acc == acc)) rn = __builtin_huge_val();  // (fmax drops a NaN)
    }
    block_max2(rn, zn, B.red);
    // the FP32 solution is never accurate to FP64 rounding: the first
    // correction is applied unchecked
    if (it > 1 && zn < __builtin_huge_val() && rn <= 0x1p-47 * (knorm * zn + fn)) {
      *it_out = it;
      return true;
    }
    correct(B.r, false);
  }
  return false;
}

__global__ __launch_bounds__(kGT) __attribute__((amdgpu_waves_per_eu(4))) void k_rows_gj(Work w) {
  __shared__ BlockBuf B;
  const int tid = threadIdx.x;
  const int qlen = min(w.cnt->nC, w.capC);
  const int lw = w.adj_live ? (w.adj_w == 4 ? 2 : w.adj_w == 8 ? 3 : 0) : 0;
  for (int qi = blockIdx.x; qi < qlen; qi += gridDim.x) {
    const int e = w.binC[qi];
    if (tid == 0) w.bigq[qi] = 0;
    const int c = e / w.chunk;
    const RowInfo ri = row_info(w, c, e - c * w.chunk);
    const int s = ri.s;
    if (s <= 32 || s > kGMax) continue;
    // without an FP64 scratch (which a row that does not converge here would need)
    // rows above kLdsBlockMax points are reported by k_rows_wg, not solved
    if (s > kLdsBlockMax && w.scratch_slots == 0) continue;
    MatStatus* st = &w.st[ri.m];
    if (!matrix_live(*st)) continue;
    const GDesc d = gview(w.desc[ri.m]);
    const int i = ri.i;
    __syncthreads();  // the previous row's buffers are free
    {
      int n = group_search<kGT>(B.search, d, i, lw, tid);
      __syncthreads();
      if (n < 0) continue;  // more points met than the table holds: k_rows_wg
      int f = n;
      if (d.literal != 0 && d.ell >= 3) f = drop_c_points<kGT>(B.search, d, n, tid);
      if (f != s) continue;  // a pattern other than the symbolic pass's: k_rows_wg reports it
      for (int q = tid; q < n; q += kGT) {
        const int v = B.search.list[q];
        if (v != INT32_MAX) B.N[search_rank(B.search, n, v)] = v;
      }
      if (tid < kGMax) { B.cnt[tid] = 0; B.f[tid] = 0.0; B.z[tid] = 0.0; }
      if (tid == 0) B.bad = 0;
    }
    __syncthreads();
    // column lists of the block, counted and placed (two threads per row of A)
    const int p = tid >> 1, sub = tid & 1;
    int e0 = 0, e1 = 0;
    if (p < s) {
      const i2u v = *(gptr<const i2u>)(d.rp + B.N[p]);
      e0 = v.x;
      e1 = v.y;
    }
    double amax = 0.0, rsum = 0.0;
    for (int k = e0 + sub; k < e1; k += 2) {
      const double a = fabs(d.va[k]);
      amax = fmax(amax, a);
      rsum += a;
      const int q = find_sorted(B.N, s, d.ci[k]);
      if (q >= 0) atomicAdd(&B.cnt[q], 1);
    }
    rsum += __shfl_xor(rsum, 1, 64);
    for (int k = d.rp[i] + tid; k < d.rp[i + 1]; k += kGT) {
      const int q = find_sorted(B.N, s, d.ci[k]);
      if (q >= 0) B.f[q] = -d.va[k];
    }
    block_max2(amax, rsum, B.red);
    if (!(amax > 0.0) || !(amax < 1e300)) continue;
    if (tid < 64) {  // offsets: two lists per lane
      const int c0 = B.cnt[2 * tid], c1 = B.cnt[2 * tid + 1];
      int x = c0 + c1;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o, 64);
        if (tid >= o) x += y;
      }
      B.off[2 * tid] = x - c0 - c1;
      B.off[2 * tid + 1] = x - c1;
      if (tid == 63) B.off[kGMax] = x;
      B.cnt[2 * tid] = x - c0 - c1;
      B.cnt[2 * tid + 1] = x - c1;
    }
    __syncthreads();
    if (B.off[kGMax] > kGEntries) continue;  // workgroup-uniform
    for (int k = e0 + sub; k < e1; k += 2) {
      const int q = find_sorted(B.N, s, d.ci[k]);
      if (q >= 0) {
        const int at = atomicAdd(&B.cnt[q], 1);
        B.row[at] = (uint16_t)p;
        B.val[at] = d.va[k];
      }
    }
    __syncthreads();
    if (tid < s) {  // list tid in ascending p
      const int k0 = B.off[tid], k1 = B.off[tid + 1];
      for (int k = k0 + 1; k < k1; ++k) {
        const uint16_t rp = B.row[k];
        const double rv = B.val[k];
        int m = k - 1;
        while (m >= k0 && B.row[m] > rp) {
          B.row[m + 1] = B.row[m];
          B.val[m + 1] = B.val[m];
          --m;
        }
        B.row[m + 1] = rp;
        B.val[m + 1] = rv;
      }
    }
    __syncthreads();
    int ex = 0;
    frexp(amax, &ex);
    const double scale = ldexp(1.0, -ex);
    int it = 0;
    bool ok;
    switch ((s + 15) / 16) {  // 33 points and more: T >= 3
      case 3: ok = block_solve<3>(B, s, scale, rsum, &it); break;
      case 4: ok = block_solve<4>(B, s, scale, rsum, &it); break;
      case 5: ok = block_solve<5>(B, s, scale, rsum, &it); break;
      case 6: ok = block_solve<6>(B, s, scale, rsum, &it); break;
      case 7: ok = block_solve<7>(B, s, scale, rsum, &it); break;
      default: ok = block_solve<8>(B, s, scale, rsum, &it); break;
    }
    if (!ok) continue;
    if (tid == 0) {
      w.bigq[qi] = 1;  // solved
      d.Rrp[ri.r] = ri.off;
      if (it > __hip_atomic_load(&st->refine_max, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMax(&st->refine_max, it);
    }
    // R row: N is sorted, so the C-point stands after the points below it
    const int dpos = lower_bound_i32(B.N, s, i);
    if (tid < s) put_f_entry(w, d, ri.fine0, ri.off + tid + (tid >= dpos ? 1 : 0), B.N[tid], i, B.z[tid]);
    if (tid == 0) {
      d.Rci[ri.off + dpos] = i;
      d.Rva[ri.off + dpos] = 1.0;
    }
  }
}

}  // namespace

// persistent grid over the queue, as many workgroups as fit on the device
hipError_t launch_rows_gj(const Work& w, int cus, hipStream_t s) {
  const int per = resident_blocks<k_rows_gj, kGT>();
  if (per < 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_rows_gj, dim3(std::max(1, per) * cus), dim3(kGT), 0, s, w);
  return hipGetLastError();
}

}  // namespace clair
