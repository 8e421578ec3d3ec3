// k_transpose.hip -- CSR transpose on the device.
//
// Used to form P = (R built on A^T)^T: the input A^T of the restriction
// setup, and the transpose of its result.  Rows of the output are sorted by
// column like every CSR array of the library.  Stages: column counts
// (integer atomics) -> exclusive scan (per-block scans, then every block adds
// the totals before it, scanned themselves where there are many) -> scatter (the counts, counted down) -> sort of each
// output row (the scatter order within a column is arbitrary).  Values are
// copied, so the transpose is exact.
//
// Bound: launches and the latency of the dependent steps of an entry (index,
// cursor, store).  Every thread has kTB entries of its row in flight and
// output rows of up to kTS entries are sorted in registers: on a 511 x 511
// five-point matrix the eight kernels of one entry at a time took 73 us, these
// six take 45.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "clair_device.h"
#include "clair_launch.h"

namespace clair {

namespace {

constexpr int kTT = 256;            // threads per workgroup
constexpr int kTPer = 4;            // scan entries per thread
constexpr int kTBlk = kTT * kTPer;  // scan entries per workgroup

__global__ void k_t_zero(int32_t* a, int n) {
  for (int j = blockIdx.x * kTT + threadIdx.x; j < n; j += gridDim.x * kTT) a[j] = 0;
}

// Up to so many blocks each sums the totals before its own (k_t_scan_add); above,
// the totals are scanned in turn, as the former's reads grow with their square.  A
// transpose of a diagonal of 2^21 entries 69 us so and 79 with the totals scanned,
// 2^23: 164 and 163, 2^24: 320 and 284, 2^27: 4,430 and 2,243.
constexpr int kTFlat = 8192;
constexpr int kTB = 8;  // entries of a row a thread has in flight
constexpr int kTS = 8;  // output rows of up to kTS entries are sorted in registers

// cnt[j] = entries of column j (indices outside [0, ncol) are skipped and
// flagged in *bad)
__global__ __launch_bounds__(kTT) void k_t_count(int m, int ncol, int64_t nnz, const int32_t* __restrict__ rp,
                                                 const int32_t* __restrict__ ci, int32_t* cnt, int32_t* bad) {
  if (rp[0] != 0 || rp[m] != nnz) {  // the arrays that follow are sized from nnz: no row is walked
    if (blockIdx.x == 0 && threadIdx.x == 0) *bad = 1;
    return;
  }
  for (int i = blockIdx.x * kTT + threadIdx.x; i < m; i += gridDim.x * kTT) {
    const int e1 = rp[i + 1];
    for (int e = rp[i]; e < e1; e += kTB) {
      int j[kTB];
#pragma unroll
      for (int k = 0; k < kTB; ++k) j[k] = e + k < e1 ? ci[e + k] : 0;
#pragma unroll
      for (int k = 0; k < kTB; ++k) {
        if (e + k >= e1) continue;
        if ((unsigned)j[k] < (unsigned)ncol) atomicAdd(&cnt[j[k]], 1);
        else atomicExch(bad, 1);
      }
    }
  }
}

// exclusive scan of cnt[0..n) into out[0..n), per block of kTBlk entries;
// block totals to sums[b].  (stop: nothing is written when it is given and set)
__global__ __launch_bounds__(kTT) void k_t_scan_blocks(const int32_t* cnt, int n, int32_t* out, int32_t* sums,
                                                       const int32_t* stop) {
  if (stop && *stop) return;
  __shared__ int sh[kTT / 64];
  const int base = blockIdx.x * kTBlk + threadIdx.x * kTPer;
  int v[kTPer];
  int my = 0;
#pragma unroll
  for (int k = 0; k < kTPer; ++k) {
    v[k] = (base + k < n) ? cnt[base + k] : 0;
    my += v[k];
  }
  int tot;
  int pre = block_exclusive_scan(my, sh, &tot);
#pragma unroll
  for (int k = 0; k < kTPer; ++k) {
    if (base + k < n) out[base + k] = pre;
    pre += v[k];
  }
  if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// out[j] += the totals of the blocks before j's; out[n] = the sum of all
// nb blocks (one workgroup per block; each sums the totals it needs, so no
// kernel of one workgroup stands between the two)
__global__ __launch_bounds__(kTT) void k_t_scan_add(int32_t* out, int n, const int32_t* sums, int nb,
                                                    const int32_t* stop) {
  if (stop && *stop) return;
  __shared__ int sh[kTT / 64];
  const int b = blockIdx.x;
  int my = 0;
  for (int k = threadIdx.x; k < b; k += kTT) my += sums[k];
  int base;
  (void)block_exclusive_scan(my, sh, &base);
  const int j0 = b * kTBlk + threadIdx.x;
#pragma unroll
  for (int k = 0; k < kTPer; ++k)
    if (j0 + k * kTT < n) out[j0 + k * kTT] += base;
  if (b == nb - 1 && threadIdx.x == 0) out[n] = base + sums[b];
}

// the same with the totals already scanned (sums[nb] the sum of all)
__global__ __launch_bounds__(kTT) void k_t_scan_shift(int32_t* out, int n, const int32_t* sums, int nb,
                                                      const int32_t* stop) {
  if (stop && *stop) return;
  const int b = blockIdx.x;
  const int base = sums[b];
  const int j0 = b * kTBlk + threadIdx.x;
#pragma unroll
  for (int k = 0; k < kTPer; ++k)
    if (j0 + k * kTT < n) out[j0 + k * kTT] += base;
  if (b == nb - 1 && threadIdx.x == 0) out[n] = sums[nb];
}

__global__ void k_t_scan_none(int32_t* out, const int32_t* stop) {
  if (!stop || !*stop) out[0] = 0;
}

// scatter: entry (i, j) to out row j at trp[j] + the column's count, counted
// down (a skipped index was never counted)
__global__ __launch_bounds__(kTT) void k_t_fill(int m, int ncol, int64_t nnz, const int32_t* __restrict__ rp,
                                                const int32_t* __restrict__ ci, const double* __restrict__ va,
                                                const int32_t* __restrict__ trp, int32_t* left, int32_t* tci,
                                                double* tva, const int32_t* stop) {
  if (rp[0] != 0 || rp[m] != nnz || (stop && *stop)) return;
  for (int i = blockIdx.x * kTT + threadIdx.x; i < m; i += gridDim.x * kTT) {
    const int e1 = rp[i + 1];
    for (int e = rp[i]; e < e1; e += kTB) {
      int j[kTB], pos[kTB];
      double x[kTB];
#pragma unroll
      for (int k = 0; k < kTB; ++k) {
        j[k] = e + k < e1 ? ci[e + k] : -1;
        x[k] = e + k < e1 ? va[e + k] : 0.0;
      }
#pragma unroll
      for (int k = 0; k < kTB; ++k)
        if ((unsigned)j[k] < (unsigned)ncol) pos[k] = trp[j[k]] + atomicSub(&left[j[k]], 1) - 1;
#pragma unroll
      for (int k = 0; k < kTB; ++k)
        if ((unsigned)j[k] < (unsigned)ncol) { tci[pos[k]] = i; tva[pos[k]] = x[k]; }
    }
  }
}

// sort every output row by column: rows of up to kTS entries in registers
// (every entry goes to its rank; equal columns keep their order), longer rows
// by insertion in place
__global__ __launch_bounds__(kTT) void k_t_sort(int ncol, const int32_t* __restrict__ trp, int32_t* tci, double* tva,
                                                const int32_t* stop) {
  if (stop && *stop) return;
  for (int j = blockIdx.x * kTT + threadIdx.x; j < ncol; j += gridDim.x * kTT) {
    const int e0 = trp[j], e1 = trp[j + 1];
    if (e1 - e0 <= 1) continue;
    if (e1 - e0 <= kTS) {
      int c[kTS];
      double x[kTS];
#pragma unroll
      for (int k = 0; k < kTS; ++k) {
        c[k] = e0 + k < e1 ? tci[e0 + k] : INT32_MAX;
        x[k] = e0 + k < e1 ? tva[e0 + k] : 0.0;
      }
#pragma unroll
      for (int k = 0; k < kTS; ++k) {
        int r = 0;
#pragma unroll
        for (int t = 0; t < kTS; ++t) r += (c[t] < c[k] || (t < k && c[t] == c[k])) ? 1 : 0;
        if (e0 + k < e1) { tci[e0 + r] = c[k]; tva[e0 + r] = x[k]; }
      }
      continue;
    }
    for (int a = e0 + 1; a < e1; ++a) {
      const int k = tci[a];
      const double x = tva[a];
      int b = a - 1;
      while (b >= e0 && tci[b] > k) {
        tci[b + 1] = tci[b];
        tva[b + 1] = tva[b];
        --b;
      }
      tci[b + 1] = k;
      tva[b + 1] = x;
    }
  }
}

int grid_for(int n, int cus) { return std::max(1, std::min((n + kTT - 1) / kTT, cus * 8)); }

}  // namespace

size_t transpose_scratch_ints(int ncol) { return (size_t)ncol + 1 + scan_scratch_ints(ncol); }

// block totals and their sum; the totals of blocks of those
size_t scan_scratch_ints(int n) {
  const size_t nb = (size_t)n / kTBlk + 1;
  return nb + 1 + nb / kTBlk + 1;
}

hipError_t launch_exclusive_scan(const int32_t* cnt, int n, int32_t* out, int32_t* sums, int cus, hipStream_t s,
                                 const int32_t* stop) {
  (void)cus;
  const int nb = (n + kTBlk - 1) / kTBlk;
  if (nb == 0) {
    hipLaunchKernelGGL(k_t_scan_none, dim3(1), dim3(1), 0, s, out, stop);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_t_scan_blocks, dim3(nb), dim3(kTT), 0, s, cnt, n, out, sums, stop);
  if (nb > kTFlat) {  // (once: 2^31 entries are 2^21 blocks, 2^11 blocks of those)
    hipError_t e = launch_exclusive_scan(sums, nb, sums, sums + nb + 1, cus, s, stop);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_t_scan_shift, dim3(nb), dim3(kTT), 0, s, out, n, sums, nb, stop);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_t_scan_add, dim3(nb), dim3(kTT), 0, s, out, n, sums, nb, stop);
  return hipGetLastError();
}

hipError_t launch_transpose(int m, int ncol, int64_t nnz, const int32_t* rp, const int32_t* ci, const double* va,
                            int32_t* trp, int32_t* tci, double* tva, int32_t* scratch, int cus, hipStream_t s,
                            bool keep) {
  int32_t* left = scratch;
  int32_t* bad = scratch + ncol;
  const int32_t* stop = keep ? bad : nullptr;
  int32_t* sums = scratch + ncol + 1;
  hipLaunchKernelGGL(k_t_zero, dim3(grid_for(ncol + 1, cus)), dim3(kTT), 0, s, left, ncol + 1);
  if (m > 0) hipLaunchKernelGGL(k_t_count, dim3(grid_for(m, cus)), dim3(kTT), 0, s, m, ncol, nnz, rp, ci, left, bad);
  hipError_t e = launch_exclusive_scan(left, ncol, trp, sums, cus, s, stop);
  if (e != hipSuccess) return e;
  if (m > 0)
    hipLaunchKernelGGL(k_t_fill, dim3(grid_for(m, cus)), dim3(kTT), 0, s, m, ncol, nnz, rp, ci, va, trp, left, tci, tva, stop);
  if (ncol > 0) hipLaunchKernelGGL(k_t_sort, dim3(grid_for(ncol, cus)), dim3(kTT), 0, s, ncol, trp, tci, tva, stop);
  return hipGetLastError();
}

}  // namespace clair
