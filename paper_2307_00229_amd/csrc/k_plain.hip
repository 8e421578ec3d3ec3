// k_plain.hip -- the plain FP64 per-row form of the restriction setup.
//
// The straightforward GPU formulation, kept as the baseline the mixed,
// batched path is measured against: one matrix at a time, sixteen lanes per
// C-row, one kernel per stage, FP64 everywhere, local blocks in LDS, Gaussian
// elimination with partial pivoting.  Stages:
//   C-point count per block -> scan -> C list -> |N(i)| per row -> scan ->
//   column indices -> gather + solve -> projection sums -> projection.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "clair_device.h"
#include "clair_launch.h"
#include "lds_block.h"
#include "search_device.h"

namespace clair {

namespace {

constexpr int kPT = 256;
constexpr int kPlainCap = 64;  // neighbourhood capacity of a row

enum { PF_STATUS = 0, PF_FIRST_BAD = 1, PF_MAX_BLOCK = 2, PF_UNCOVERED = 3 };

__device__ void pflag(int32_t* flags, int code, int row) {
  atomicCAS(&flags[PF_STATUS], 0, code);
  atomicMin(&flags[PF_FIRST_BAD], row);
}

// The search of a row by sixteen lanes (group_search), up to kPlainCap points
// (C-points walked through in the literal reading included).  A thread per row
// with its points in a private array took 28 us a pass on 16,641 rows, this
// 12 (sizes) and 8 (fill).
constexpr int kPG = 16;
typedef SearchBuf<kPlainCap, 2 * kPlainCap> PlainBuf;

__device__ __forceinline__ GDesc plain_desc(const PlainWork& p) {
  GDesc d{};
  d.n = p.n;
  d.ell = p.ell;
  d.theta = p.theta;
  d.literal = p.literal;
  d.cf = to_global(p.cf);
  d.cmax = to_global((const double*)p.cmax);
  d.grp = to_global(p.grp);
  d.gci = to_global(p.gci);
  d.gva = to_global(p.gva);
  d.agg_rp = nullptr;
  d.fadj = nullptr;
  return d;
}

// points listed (gaps, INT32_MAX, where C-points were dropped) into *n; returns
// |N(i)| or -1
__device__ __forceinline__ int plain_search(const GDesc& d, int i, PlainBuf& b, int lane, int* n) {
  *n = group_search<kPG>(b, d, i, 0, lane);
  if (*n < 0) return -1;
  return d.literal != 0 && d.ell >= 3 ? drop_c_points<kPG>(b, d, *n, lane) : *n;
}

// cmax[v] = max over w != v of |a_wv| (bit patterns of non-negative doubles
// order like their values)
__global__ void k_p_colmax_clear(PlainWork p) {
  const int j = blockIdx.x * kPT + threadIdx.x;
  if (j < p.n) p.cmax[j] = 0.0;
}

__global__ void k_p_colmax(PlainWork p) {
  const int u = blockIdx.x * kPT + threadIdx.x;
  if (u >= p.n) return;
  for (int e = p.grp[u]; e < p.grp[u + 1]; ++e) {
    const int v = p.gci[e];
    if (v != u && (unsigned)v < (unsigned)p.n)
      atomicMax(reinterpret_cast<unsigned long long*>(p.cmax + v),
                          (unsigned long long)__double_as_longlong(fabs(p.gva[e])));
  }
}

__global__ void k_p_count_c(PlainWork p) {
  __shared__ int sh[kPT];
  const int j = blockIdx.x * kPT + threadIdx.x;
  sh[threadIdx.x] = (j < p.n && p.cf[j] != 0) ? 1 : 0;
  __syncthreads();
  for (int o = kPT / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) p.blk_cnt[blockIdx.x] = sh[0];
}

// single-workgroup exclusive scan of a[0..n), a[n] = total
__global__ __launch_bounds__(1024) void k_p_scan_single(int32_t* a, int n) {
  __shared__ int sh[1024];
  __shared__ int carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int b = 0; b < n; b += 1024) {
    const int j = b + threadIdx.x;
    const int v = (j < n) ? a[j] : 0;
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
      const int t = ((int)threadIdx.x >= o) ? sh[threadIdx.x - o] : 0;
      __syncthreads();
      sh[threadIdx.x] += t;
      __syncthreads();
    }
    if (j < n) a[j] = carry + sh[threadIdx.x] - v;
    __syncthreads();
    if (threadIdx.x == 0) carry += sh[1023];
    __syncthreads();
  }
  if (threadIdx.x == 0) a[n] = carry;
}

__global__ void k_p_clist(PlainWork p) {
  __shared__ int sh[kPT];
  const int j = blockIdx.x * kPT + threadIdx.x;
  const int isc = (j < p.n && p.cf[j] != 0) ? 1 : 0;
  sh[threadIdx.x] = isc;
  __syncthreads();
  for (int o = 1; o < kPT; o <<= 1) {
    const int t = ((int)threadIdx.x >= o) ? sh[threadIdx.x - o] : 0;
    __syncthreads();
    sh[threadIdx.x] += t;
    __syncthreads();
  }
  if (isc) p.clist[p.blk_cnt[blockIdx.x] + sh[threadIdx.x] - 1] = j;
}

__global__ __launch_bounds__(kPT) void k_p_sizes(PlainWork p, int n_c) {
  __shared__ PlainBuf sb[kPT / kPG];
  __shared__ int smax;
  const int lane = threadIdx.x % kPG, grp = threadIdx.x / kPG;
  if (threadIdx.x == 0) smax = 0;
  __syncthreads();
  const int r = blockIdx.x * (kPT / kPG) + grp;
  if (r < n_c) {
    const GDesc d = plain_desc(p);
    const int i = p.clist[r];
    int n;
    int s = plain_search(d, i, sb[grp], lane, &n);
    if (lane == 0) {
      if (s < 0) {
        pflag(p.flags, ST_UNSUPPORTED, i);
        s = 0;
      }
      p.sizes[r] = s + 1;
      atomicMax(&smax, s);
    }
  }
  // largest block: one atomic per workgroup, when it grows
  __syncthreads();
  if (threadIdx.x == 0 &&
      smax > __hip_atomic_load(&p.flags[PF_MAX_BLOCK], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    atomicMax(&p.flags[PF_MAX_BLOCK], smax);
}

// three-phase scan of sizes[0..n) into R.row_ptr
__global__ void k_p_blocksum(const int32_t* a, int n, int32_t* sums) {
  __shared__ int sh[kPT];
  const int j = blockIdx.x * kPT + threadIdx.x;
  sh[threadIdx.x] = (j < n) ? a[j] : 0;
  __syncthreads();
  for (int o = kPT / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) sums[blockIdx.x] = sh[0];
}

__global__ void k_p_apply(const int32_t* a, int n, const int32_t* sums, int nblk, int32_t* out) {
  __shared__ int sh[kPT];
  const int j = blockIdx.x * kPT + threadIdx.x;
  const int v = (j < n) ? a[j] : 0;
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int o = 1; o < kPT; o <<= 1) {
    const int t = ((int)threadIdx.x >= o) ? sh[threadIdx.x - o] : 0;
    __syncthreads();
    sh[threadIdx.x] += t;
    __syncthreads();
  }
  if (j < n) out[j] = sums[blockIdx.x] + sh[threadIdx.x] - v;
  if (blockIdx.x == 0 && threadIdx.x == 0) out[n] = sums[nblk];
}

__global__ __launch_bounds__(kPT) void k_p_fill(PlainWork p, int n_c) {
  __shared__ PlainBuf sb[kPT / kPG];
  const int lane = threadIdx.x % kPG, grp = threadIdx.x / kPG;
  const int r = blockIdx.x * (kPT / kPG) + grp;
  if (r >= n_c) return;
  const GDesc d = plain_desc(p);
  const int i = p.clist[r];
  int n;
  const int s = plain_search(d, i, sb[grp], lane, &n);
  const int pos = p.Rrp[r];
  if (s < 0 || s + 1 != p.Rrp[r + 1] - pos) return;
  for (int q = lane; q < n; q += kPG) {
    const int v = sb[grp].list[q];
    if (v != INT32_MAX) p.Rci[pos + search_rank(sb[grp], n, v) + (v > i ? 1 : 0)] = v;
  }
  if (lane == 0) p.Rci[pos + search_rank(sb[grp], n, i)] = i;
}

// sixteen lanes per row: FP64 block in LDS, elimination with partial pivoting
// (the largest magnitude, the first of equal ones), each lane taking the rows
// below the pivot in turn
__global__ void k_p_solve(PlainWork p, int n_c, int smax) {
  extern __shared__ double s_base[];
  const int lane = threadIdx.x % kLB, grp = threadIdx.x / kLB;
  const int r = blockIdx.x * (blockDim.x / kLB) + grp;
  if (r >= n_c) return;
  const int i = p.clist[r];
  const int e0 = p.Rrp[r], s = p.Rrp[r + 1] - e0 - 1;
  if (s <= 0) {
    if (s == 0 && lane == 0) p.Rva[e0] = 1.0;
    return;
  }
  const LdsBlock b = lds_block(s_base, grp, smax);
  double* K = b.K;
  double* f = b.f;
  const int ld = b.ld;
  for (int t = lane; t < s; t += kLB) f[t] = 0.0;
  lds_gather(b, s, i, p.Rci, e0, p.rp, p.ci, p.va, lane);
  for (int e = p.rp[i] + lane; e < p.rp[i + 1]; e += kLB) {
    const int q = find_sorted(b.nb, s, p.ci[e]);
    if (q >= 0) f[q] = -p.va[e];
  }
  double amax = 0.0;
  for (int t = lane; t < s * ld; t += kLB)
    if (t % ld < s) amax = fmax(amax, fabs(K[t]));
  amax = fmax(amax, gpartd<1>(amax));
  amax = fmax(amax, gpartd<2>(amax));
  amax = fmax(amax, gpartd<4>(amax));
  amax = fmax(amax, gpartd<8>(amax));
  const double tiny = 1e-14 * amax;
  wave_sync();
  bool sing = false;
  for (int k = 0; k < s; ++k) {
    const double dk = fabs(K[k * ld + k]);
    double best = -1.0;
    int piv = k;
    for (int q = k + lane; q < s; q += kLB) {
      const double v = fabs(K[q * ld + k]);
      if (v > best) { best = v; piv = q; }
    }
#define CLAIR_PIV(STEP)                                                        \
  {                                                                            \
    const double ob = gpartd<STEP>(best);                                      \
    const int op = gpart<STEP>(piv);                                           \
    if (ob > best || (ob == best && op < piv)) { best = ob; piv = op; }        \
  }
    CLAIR_PIV(1) CLAIR_PIV(2) CLAIR_PIV(4) CLAIR_PIV(8)
#undef CLAIR_PIV
    // (a NaN on the diagonal is no pivot and hides the others, as when the
    // column is searched from the diagonal down)
    if (!(dk == dk) || !(best > tiny)) { sing = true; break; }
    if (piv != k) {
      for (int c = lane; c < s; c += kLB) {
        const double t = K[k * ld + c];
        K[k * ld + c] = K[piv * ld + c];
        K[piv * ld + c] = t;
      }
      if (lane == 0) { const double t = f[k]; f[k] = f[piv]; f[piv] = t; }
      wave_sync();
    }
    const double pv = K[k * ld + k];
    const double fk = f[k];
    for (int q = k + 1 + lane; q < s; q += kLB) {
      const double l = K[q * ld + k] / pv;
      for (int c = k + 1; c < s; ++c) K[q * ld + c] -= l * K[k * ld + c];
      f[q] -= l * fk;
    }
    wave_sync();
  }
  if (sing) {
    if (lane == 0) pflag(p.flags, ST_SINGULAR, i);
    for (int q = lane; q < s; q += kLB) f[q] = 0.0;
  } else {
    for (int k = s - 1; k >= 0; --k) {
      const double x = f[k] / K[k * ld + k];
      wave_sync();
      if (lane == 0) f[k] = x;
      for (int q = lane; q < k; q += kLB) f[q] -= K[q * ld + k] * x;
      wave_sync();
    }
  }
  wave_sync();
  for (int q = lane; q < s; q += kLB) p.Rva[e0 + q + (b.nb[q] > i ? 1 : 0)] = f[q];
  if (lane == 0) p.Rva[e0 + lower_bound_i32(b.nb, s, i)] = 1.0;
}

__global__ void k_p_colsum(PlainWork p, int n_c) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n_c) return;
  const int i = p.clist[r];
  const double bi = p.B[i];
  for (int e = p.Rrp[r]; e < p.Rrp[r + 1]; ++e) {
    const int j = p.Rci[e];
    if (j == i) continue;
    unsafeAtomicAdd(&p.dsum[j], bi * bi);
    unsafeAtomicAdd(&p.rsum[j], p.Rva[e] * bi);
  }
}

__global__ void k_p_project(PlainWork p, int n_c) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r < n_c) {
    const int i = p.clist[r];
    const double bi = p.B[i];
    for (int e = p.Rrp[r]; e < p.Rrp[r + 1]; ++e) {
      const int j = p.Rci[e];
      if (j == i) continue;
      const double dj = p.dsum[j];
      if (dj > 0.0) p.Rva[e] -= bi * (p.rsum[j] - p.B[j]) / dj;
    }
  }
}

__global__ void k_p_uncovered(PlainWork p) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  int u = (j < p.n && p.cf[j] == 0 && !(p.dsum[j] > 0.0)) ? 1 : 0;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) u += __shfl_xor(u, o, 64);
  if ((threadIdx.x & 63) == 0 && u) atomicAdd(&p.flags[PF_UNCOVERED], u);
}

inline int nblk(int n) { return (n + kPT - 1) / kPT; }

}  // namespace

hipError_t plain_colmax(const PlainWork& p, hipStream_t s) {
  if (p.n > 0 && p.theta != 0.0) {
    hipLaunchKernelGGL(k_p_colmax_clear, dim3(nblk(p.n)), dim3(kPT), 0, s, p);
    hipLaunchKernelGGL(k_p_colmax, dim3(nblk(p.n)), dim3(kPT), 0, s, p);
  }
  return hipGetLastError();
}
hipError_t plain_count_c(const PlainWork& p, hipStream_t s) {
  if (p.n > 0) hipLaunchKernelGGL(k_p_count_c, dim3(nblk(p.n)), dim3(kPT), 0, s, p);
  return hipGetLastError();
}
hipError_t plain_scan_blocks(int32_t* a, int n, hipStream_t s) {
  hipLaunchKernelGGL(k_p_scan_single, dim3(1), dim3(1024), 0, s, a, n);
  return hipGetLastError();
}
hipError_t plain_clist(const PlainWork& p, hipStream_t s) {
  if (p.n > 0) hipLaunchKernelGGL(k_p_clist, dim3(nblk(p.n)), dim3(kPT), 0, s, p);
  return hipGetLastError();
}
hipError_t plain_sizes(const PlainWork& p, int n_c, hipStream_t s) {
  if (n_c > 0) hipLaunchKernelGGL(k_p_sizes, dim3((n_c + kPT / kPG - 1) / (kPT / kPG)), dim3(kPT), 0, s, p, n_c);
  return hipGetLastError();
}
hipError_t plain_scan(const PlainWork& p, int n_c, hipStream_t s) {
  const int nb = nblk(n_c);
  if (n_c > 0) hipLaunchKernelGGL(k_p_blocksum, dim3(nb), dim3(kPT), 0, s, p.sizes, n_c, p.scan_tmp);
  hipLaunchKernelGGL(k_p_scan_single, dim3(1), dim3(1024), 0, s, p.scan_tmp, nb);
  hipLaunchKernelGGL(k_p_apply, dim3(nb > 0 ? nb : 1), dim3(kPT), 0, s, p.sizes, n_c, p.scan_tmp, nb, p.Rrp);
  return hipGetLastError();
}
hipError_t plain_fill(const PlainWork& p, int n_c, hipStream_t s) {
  if (n_c > 0) hipLaunchKernelGGL(k_p_fill, dim3((n_c + kPT / kPG - 1) / (kPT / kPG)), dim3(kPT), 0, s, p, n_c);
  return hipGetLastError();
}
hipError_t plain_solve(const PlainWork& p, int n_c, int smax, hipStream_t s) {
  if (n_c > 0) {
    const int R = lds_rows(smax);
    hipLaunchKernelGGL(k_p_solve, dim3((n_c + R - 1) / R), dim3(kLB * R), sizeof(double) * R * lds_row_doubles(smax), s,
                       p, n_c, smax);
  }
  return hipGetLastError();
}
hipError_t plain_colsum(const PlainWork& p, int n_c, hipStream_t s) {
  if (n_c > 0) hipLaunchKernelGGL(k_p_colsum, dim3(nblk(n_c)), dim3(kPT), 0, s, p, n_c);
  return hipGetLastError();
}
hipError_t plain_project(const PlainWork& p, int n_c, hipStream_t s) {
  if (n_c > 0) hipLaunchKernelGGL(k_p_project, dim3(nblk(n_c)), dim3(kPT), 0, s, p, n_c);
  if (p.n > 0) hipLaunchKernelGGL(k_p_uncovered, dim3(nblk(p.n)), dim3(kPT), 0, s, p);
  return hipGetLastError();
}

}  // namespace clair
