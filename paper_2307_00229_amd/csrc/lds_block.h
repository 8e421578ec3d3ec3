// lds_block.h -- a row's FP64 block in LDS, sixteen lanes per row: what the
// per-row FP64 solver and the ILU(0) inverse share.
//
// Why sixteen lanes and LDS: a thread per row with its block in global memory
// spends every step of the elimination on dependent scattered accesses (163 us
// for 16,641 rows of 8 points, 21 so); here a step is one pass of the lanes over the
// rows below the pivot.  Above 40 points a block takes a workgroup of sixteen
// threads by itself; calls on 5,000 rows of 41, 48 and 64 points: FP64 form 17.8, 26
// and 59 ms with a thread per row, 0.62, 0.97 and 2.6 so (50,000 rows of 64: 82 and 23),
// three ILU(0) iterations 4.5, 6.0 and 9.6 ms, now 1.3, 1.7 and 3.7.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "clair_device.h"
#include "mixed_device.h"

namespace clair {

namespace {

constexpr int kLB = 16;  // lanes per row

// rows per workgroup of kLB lanes each, so that the blocks fit 64 KB
__host__ __device__ inline int lds_rows(int smax) { return smax <= 40 ? 4 : 1; }
__host__ __device__ inline int lds_ld(int smax) { return smax | 1; }  // stride of a block row
// doubles of LDS per row: the block, a vector, the points (int32)
__host__ __device__ inline size_t lds_row_doubles(int smax) {
  return (size_t)smax * lds_ld(smax) + smax + (smax + 1) / 2;
}

struct LdsBlock {
  double* K;  // K[a][b] = a_{N_b, N_a} at a * ld + b
  double* f;
  int* nb;    // N, sorted
  int ld;
};

__device__ __forceinline__ LdsBlock lds_block(double* base, int grp, int smax) {
  LdsBlock b;
  b.K = base + (size_t)grp * lds_row_doubles(smax);
  b.f = b.K + (size_t)smax * lds_ld(smax);
  b.nb = reinterpret_cast<int*>(b.f + smax);
  b.ld = lds_ld(smax);
  return b;
}

// The points of row [e0, e0 + s] of R (N and the C-point i itself) to b.nb; the
// block K = A[N,N]^T (entries of one position summed).  All lanes of the group.
__device__ __forceinline__ void lds_gather(const LdsBlock& b, int s, int i, const int32_t* __restrict__ Rci, int e0,
                                           const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                                           const double* __restrict__ va, int lane) {
  for (int t = lane; t <= s; t += kLB) {
    const int v = Rci[e0 + t];
    if (v < i) b.nb[t] = v;
    else if (v > i) b.nb[t - 1] = v;
  }
  for (int t = lane; t < s * b.ld; t += kLB) b.K[t] = 0.0;
  wave_sync();
  for (int p = lane / 8; p < s; p += kLB / 8) {  // eight lanes per row of A
    const int u = b.nb[p];
    const int e1 = rp[u + 1];
    for (int e = rp[u] + lane % 8; e < e1; e += 8) {
      const int q = find_sorted(b.nb, s, ci[e]);
      if (q >= 0) unsafeAtomicAdd(&b.K[q * b.ld + p], va[e]);
    }
  }
  wave_sync();
}

}  // namespace

}  // namespace clair
