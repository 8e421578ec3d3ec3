// k_tile.hip -- the lane-group solver of the mixed form for rows of up to 32
// points (bin B: |N| above the bin-A bound; bin A when its bound is 16 or 32).
//
// Sixteen lanes per row, as a 4 x 4 grid: lane (r, c) = (l / 4, l % 4) holds
// rows r, r + 4, ... and columns c, c + 4, ... of K = (A[N,N])^T, a T x T tile
// (blocks of up to 4 T points), in FP64 and in FP32, both in registers.  A
// Gauss-Jordan step then needs the pivot column from within the quad (DPP), T
// entries of the pivot row from another quad (ds_swizzle) and T^2 FMAs for four
// rows a wavefront, none of them idle.  (One lane per block row, the solver
// before, broadcast 4 T entries through LDS per step for two rows and left the
// lanes beyond 4 T idle: 409 LDS and 898 VALU instructions a 24-point row.)
//
// Gather: eight lanes read a row of A together (its ninth entry by one lane per
// row), every load in flight at once; each entry is located in N and the block
// goes through LDS in two halves, so that LDS (3.5 KB a row at 24 points) does not
// allow fewer wavefronts than the registers do: two per SIMD above 20 points
// (three spill: 922 against 1,495 us at 24), three up to 20 (at 20 points with
// four VGPRs spilled), four at 12 (128 VGPRs).
//
// Bound: VALU issue (about 70% busy).  466,489 rows of 24 points (2048^2
// nine-point): 1,260 us with one lane per block row, 927 here; 262,144 rows of
// up to 18 points (128^3 seven-point): 467 and 334.  Whole calls on 120,000 rows
// of 32 points, distance 1: 1,026 and 895 us (976 with one lane per block row in
// bin A of 32); dense blocks of 32 points, 40 entries a row of A, gain nothing
// (408 and 403).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "clair_device.h"
#include "clair_launch.h"
#include "mixed_device.h"

namespace clair {

namespace {

// lane k of the quad to all four (a DPP quad permutation; k is a constant once
// the calling loops are unrolled)
template <int K>
__device__ __forceinline__ int quad_bcast(int v) {
  constexpr int ctrl = K | (K << 2) | (K << 4) | (K << 6);
  return __builtin_amdgcn_mov_dpp(v, ctrl, 0xF, 0xF, false);
}
template <int K>
__device__ __forceinline__ float quad_bcastf(float v) {
  return __int_as_float(quad_bcast<K>(__float_as_int(v)));
}
// quad K of the sixteen lanes to all four quads, lane by lane (ds_swizzle keeps
// the lane's place in its quad and the half of 32 it lies in)
template <int K>
__device__ __forceinline__ float row_bcastf(float v) {
  return __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), 0x13 | ((K << 2) << 5)));
}
__device__ __forceinline__ float quad_sum(float v) {
  v += __int_as_float(gpart<1>(__float_as_int(v)));
  v += __int_as_float(gpart<2>(__float_as_int(v)));
  return v;
}
__device__ __forceinline__ double quad_sum(double v) {
  v += gpartd<1>(v);
  v += gpartd<2>(v);
  return v;
}
// max over the four quads of values equal within each quad
__device__ __forceinline__ double quads_maxd(double v) {
  v = fmax(v, gpartd<4>(v));
  v = fmax(v, gpartd<8>(v));
  return v;
}

template <int T>
struct TileBuf {
  static constexpr int SM = 4 * T, HA = (T + 1) / 2, LD = SM + 1;
  alignas(16) double half[4 * HA * LD + 16];  // 4 HA rows of the block at a time, a place per lane for entries outside
  // vectors by column group: entry 4 b + c at [c * 8 + b]
  alignas(16) double z[4 * 8];
  alignas(16) double f[4 * 8];
  alignas(16) float y[4 * 8];
  int nb[32];      // sorted N(i), INT32_MAX beyond |N|
  alignas(8) i2u eb[32];  // bounds of the rows of A
};

// place of entry q in the vectors above
__device__ __forceinline__ int by_group(int q) { return (q & 3) * 8 + (q >> 2); }

// One Gauss-Jordan step, pivot 4 AK + RK.  One update serves every lane: the
// pivot row subtracts (1 - 1/pivot) of itself, which scales it; the pivot
// column's lanes take u = pivot + 1, so that a column entry x becomes
// x - x / pivot (pivot + 1) = -x / pivot and the pivot itself 1 / pivot (the
// block is scaled to at most 1, so this costs a rounding or two of FP32).
//
// What that leaves in a row: the FP64 refinement stops at a residual of
// 2^-47 (|K| |z| + |f|), as in the solver of one lane per block row before, and
// which residual first passes depends on how the inverse is rounded.  The same
// largest error of a row on both sides, 2 to 5e-14, and either is the better
// one: root mean squares before and here 4.8e-15 and 6.3e-15 (dominant random
// blocks of 24 points), 3.8e-16 and 1.2e-15 (40^3 seven-point, eps = 0.1),
// 1.2e-14 and 3.2e-15 (the same, eps = 1e-4), 1.7e-14 and 2.6e-15 (200^2
// nine-point, eps = 1e-4).
template <int T, int AK, int RK>
__device__ __forceinline__ void tile_step(float (&kf)[T][T], int r, int c, int& bad) {
  float u[T];
#pragma unroll
  for (int b = 0; b < T; ++b) u[b] = row_bcastf<RK>(kf[AK][b]);
  const float piv = quad_bcastf<RK>(u[AK]);
  bad |= !(fabsf(piv) >= 0x1p-24f);
  // FP32 factors only precondition the FP64 refinement: the hardware
  // reciprocal (1 ulp) is accurate enough
  const float pinv = __builtin_amdgcn_rcpf(piv);
  float la[T];
#pragma unroll
  for (int a = 0; a < T; ++a) la[a] = quad_bcastf<RK>(kf[a][AK]) * pinv;
  la[AK] = r == RK ? 1.f - pinv : la[AK];
  u[AK] = c == RK ? piv + 1.f : u[AK];
#pragma unroll
  for (int a = 0; a < T; ++a)
#pragma unroll
    for (int b = 0; b < T; ++b) kf[a][b] = fmaf(-la[a], u[b], kf[a][b]);
  // keep the scheduler from interleaving steps (that multiplies live rows)
  __builtin_amdgcn_sched_barrier(0);
}

template <int T, int AK>
__device__ __forceinline__ void tile_steps(float (&kf)[T][T], int r, int c, int s, int& bad) {
  // a step is left out when no row of the wavefront has that many points
  // (wavefront-uniform: every active lane takes the same steps)
  if constexpr (AK < T) {
    if (__ballot(4 * AK < s)) tile_step<T, AK, 0>(kf, r, c, bad);
    if (__ballot(4 * AK + 1 < s)) tile_step<T, AK, 1>(kf, r, c, bad);
    if (__ballot(4 * AK + 2 < s)) tile_step<T, AK, 2>(kf, r, c, bad);
    if (__ballot(4 * AK + 3 < s)) tile_step<T, AK, 3>(kf, r, c, bad);
    tile_steps<T, AK + 1>(kf, r, c, s, bad);
  }
}

// which = 0: bin A (|N| <= GA, GA = 16 or 32); which = 1: bin B (the bin-A bound
// < |N| <= 32).  It runs for batches whose largest block lies in (above, upto].  A row
// of more than 4 T points goes to the workgroup solvers.
template <int T>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(T <= 5 ? 3 : 2))) void k_tile(Work w, int which, int above, int upto) {
  typedef TileBuf<T> Buf;
  constexpr int SM = Buf::SM, HA = Buf::HA, LD = Buf::LD, HALF = 4 * HA * LD;
  constexpr int NG = 4;               // rows of a wavefront
  constexpr int NR = (SM + 1) / 2;    // gather rounds: two rows of A each
  constexpr int NL = SM > 16 ? 2 : 1; // points per lane (l, l + 16)
  __shared__ Buf sb[NG];
  const int tid = threadIdx.x;
  const int grp = tid >> 4, l = tid & 15, r = l >> 2, c = l & 3;
  Buf& gb = sb[grp];
  if ((which ? w.cnt->nB : w.cnt->nA) == 0 || w.cnt->maxb <= above || w.cnt->maxb > upto) return;
  const int smin = which ? small_limit(w.GA) + 1 : 0;
  const int32_t* slots = which ? w.slotB : w.slotA;
  const int sstride = which ? 32 : w.GA;
  // runs of eight rows a group where there are plenty (the row ahead is loaded
  // within a run), of two on small batches, so that every wavefront has some
  const int total = w.cnt->total_rows;
  const RowBlocks rbk(total, (total >= 64 * (int)gridDim.x ? 8 : 2) * NG);
  int r0, r1;
  if (!rbk.block(0, &r0, &r1)) return;
  RefineMax rmx;
  RowCursor cc;

  // one row ahead: chunk-local data and slot entries of the group's next row
  int nx_t = 0, nx_i = 0, nx_off = 0, nx_s = 0, nx_n[2] = {0, 0};
  for (int jb = 0; rbk.block(jb, &r0, &r1); ++jb) {
  bool ahead = false;
  for (int g = r0 + grp; g < r1; g += NG) {  // uniform over the sixteen lanes
    int t, i, off, s, n[2];
    if (ahead) {
      t = nx_t; i = nx_i; off = nx_off; s = nx_s; n[0] = nx_n[0]; n[1] = nx_n[1];
    } else {
      cc.seek(w, g);
      if ((which ? cc.bins.y : cc.bins.x) == 0) {  // no row of this chunk is ours: on to the next one
        g += (cc.re - g + NG - 1) / NG * NG - NG;
        continue;
      }
      cc.row(w, g, &t, &i, &off, &s);
      const int32_t* sl = slots + (cc.fbase + t) * sstride;
      n[0] = sl[l];
      n[1] = NL > 1 && sstride > 16 ? sl[l + 16] : 0;
    }
    ahead = g + NG < r1 && g + NG < cc.re;
    if (ahead) {
      cc.row(w, g + NG, &nx_t, &nx_i, &nx_off, &nx_s);
      const int32_t* sl = slots + (cc.fbase + nx_t) * sstride;
      nx_n[0] = sl[l];
      nx_n[1] = NL > 1 && sstride > 16 ? sl[l + 16] : 0;
    }
    if (s < smin || s > SM || !cc.live) {
      if (s > SM && s >= smin && s <= (which ? 32 : w.GA) && cc.live && l == 0) {
        // a row larger than this kernel's blocks: the workgroup solvers
        const int qc = atomicAdd(&w.cnt->nC, 1);
        if (qc < w.capC) w.binC[qc] = cc.c * w.chunk + t;
        else flag_row(&w.st[cc.m], ST_UNSUPPORTED, i);
      }
      continue;
    }
    const GDesc d = row_desc(w, cc.m);
    // the rows' bounds (a lane without a point reads row i's and drops them)
    int nv[2];
    i2u eb[2];
#pragma unroll
    for (int h = 0; h < NL; ++h) {
      nv[h] = l + 16 * h < s ? n[h] : INT32_MAX;
      eb[h] = *(gptr<const i2u>)(d.rp + (l + 16 * h < s ? n[h] : i));
    }
    const i2u ib = *(gptr<const i2u>)(d.rp + i);
    wave_sync();  // the previous row's buffers are free
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      gb.nb[l + 16 * h] = h < NL ? nv[h] : INT32_MAX;
      gb.f[l + 16 * h] = 0.0;
    }
    for (int q = l; q < HALF; q += 16) gb.half[q] = 0.0;
    int over = 0;  // entries beyond the ninth of the longest row
#pragma unroll
    for (int h = 0; h < NL; ++h) {
      if (l + 16 * h >= s) eb[h].y = eb[h].x;
      gb.eb[l + 16 * h] = eb[h];
      over = max(over, eb[h].y - eb[h].x - 9);
    }
    wave_sync();
    // position of column k in N: two levels from registers, the rest from LDS
    const int n7 = gb.nb[7], n15 = gb.nb[15], n23 = gb.nb[23];
    auto find = [&](int k) {
      int pos = 0;
      if constexpr (SM > 16) {
        const bool up = k > n15;
        pos = up ? 16 : 0;
        pos += k > (up ? n23 : n7) ? 8 : 0;
      } else {
        pos = k > n7 ? 8 : 0;
      }
      pos += gb.nb[pos + 3] < k ? 4 : 0;
      pos += gb.nb[pos + 1] < k ? 2 : 0;
      pos += gb.nb[pos] < k ? 1 : 0;
      return gb.nb[pos] == k ? pos : -1;
    };
    // ---- gather: entry (q, p) of the block at q LD + p, -1 for an entry of A
    // outside it; f = -A[i,N]
    int at[NR + NL];
    double av[NR + NL];
    if (d.nnz > 0) {
      int k[NR + NL], kf_ = -1;
      double vf = 0.0;
      const int l8 = l & 7, hi = l >> 3;
#pragma unroll
      for (int j = 0; j < NR; ++j) {  // round j: rows 2 j and 2 j + 1
        const i2u v = gb.eb[2 * j + hi];
        const int e = v.x + l8;
        const int ec = max(min(e, v.y - 1), 0);
        const int kk = d.ci[ec];
        av[j] = d.va[ec];
        k[j] = e < v.y ? kk : -1;
      }
#pragma unroll
      for (int h = 0; h < NL; ++h) {  // the ninth entries
        const int e = eb[h].x + 8;
        const int ec = max(min(e, eb[h].y - 1), 0);
        const int kk = d.ci[ec];
        av[NR + h] = d.va[ec];
        k[NR + h] = e < eb[h].y ? kk : -1;
      }
      if (ib.x + l < ib.y) { kf_ = d.ci[ib.x + l]; vf = d.va[ib.x + l]; }
#pragma unroll
      for (int j = 0; j < NR; ++j) {
        const int q = find(k[j]);
        at[j] = q >= 0 ? q * LD + 2 * j + hi : -1;
      }
#pragma unroll
      for (int h = 0; h < NL; ++h) {
        const int q = find(k[NR + h]);
        at[NR + h] = q >= 0 ? q * LD + l + 16 * h : -1;
      }
      const int q = find(kf_);
      if (q >= 0) gb.f[by_group(q)] = -vf;
      for (int e = ib.x + l + 16; e < ib.y; e += 16) {
        const int q2 = find(d.ci[e]);
        if (q2 >= 0) gb.f[by_group(q2)] = -d.va[e];
      }
    } else {
#pragma unroll
      for (int j = 0; j < NR + NL; ++j) { at[j] = -1; av[j] = 0.0; }
    }
    // entries beyond the ninth, a row of A per lane and four in flight: the first
    // pass takes those of the first half and marks those of the second in a word
    // per row (where z will stand), so that the second pass reads no others again;
    // beyond 64 of them it reads all.  40,000 rows of 24 points whose rows of A
    // have about 45 entries: 676 us a call with every entry read and located in
    // both passes, one at a time, 450 here (one lane per block row: 560), all with
    // 128 threads a workgroup in the symbolic pass; 475 with its 256 of today.
    uint64_t* later = reinterpret_cast<uint64_t*>(gb.z);
    auto rest1 = [&]() {
      uint64_t m[NL] = {};
#pragma unroll 1
      for (int o = 0; o < over; o += 4) {
        int k[NL][4];
#pragma unroll
        for (int h = 0; h < NL; ++h)
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const int e = eb[h].x + 9 + o + t;
            k[h][t] = e < eb[h].y ? d.ci[e] : -1;
          }
#pragma unroll
        for (int h = 0; h < NL; ++h)
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const int q = find(k[h][t]);
            if (q >= 4 * HA) { if (o + t < 64) m[h] |= 1ull << (o + t); }
            else if (q >= 0) gb.half[q * LD + l + 16 * h] = d.va[eb[h].x + 9 + o + t];
          }
      }
#pragma unroll
      for (int h = 0; h < NL; ++h) later[l + 16 * h] = m[h];
    };
    auto rest2 = [&]() {
#pragma unroll
      for (int h = 0; h < NL; ++h) {
        const int e0 = eb[h].x + 9;
        const bool all = eb[h].y - e0 > 64;
        for (uint64_t m = later[l + 16 * h]; m;) {
          int k[2];
          double x[2];
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            k[t] = -1;
            x[t] = 0.0;
            if (m) {
              const int e = e0 + __ffsll((unsigned long long)m) - 1;
              k[t] = d.ci[e];
              x[t] = d.va[e];
            }
            m &= m - 1;
          }
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            const int q = find(k[t]);
            if (q >= 0) gb.half[q * LD + l + 16 * h - HALF] = x[t];
          }
        }
        for (int e = all ? e0 + 64 : eb[h].y; e < eb[h].y; ++e) {
          const int q = find(d.ci[e]);
          if (q >= 4 * HA) gb.half[q * LD + l + 16 * h - HALF] = d.va[e];
        }
      }
    };
    double K[T][T];
#pragma unroll
    for (int j = 0; j < NR + NL; ++j)
      gb.half[(unsigned)at[j] < (unsigned)HALF ? at[j] : HALF + l] = av[j];
    if (over > 0) rest1();
    wave_sync();
#pragma unroll
    for (int a = 0; a < HA; ++a)
#pragma unroll
      for (int b = 0; b < T; ++b) K[a][b] = gb.half[(4 * a + r) * LD + 4 * b + c];
    wave_sync();
    for (int q = l; q < HALF; q += 16) gb.half[q] = 0.0;
    wave_sync();
#pragma unroll
    for (int j = 0; j < NR + NL; ++j)
      gb.half[at[j] >= HALF ? at[j] - HALF : HALF + l] = av[j];
    if (over > 0) rest2();
    wave_sync();
#pragma unroll
    for (int a = HA; a < T; ++a)
#pragma unroll
      for (int b = 0; b < T; ++b) K[a][b] = gb.half[(4 * (a - HA) + r) * LD + 4 * b + c];

    // ---- FP32 inverse of the scaled block ----
    double amax = 0.0;
#pragma unroll
    for (int a = 0; a < T; ++a)
#pragma unroll
      for (int b = 0; b < T; ++b) amax = fmax(amax, fabs(K[a][b]));
    amax = fmax(amax, gpartd<1>(amax));
    amax = fmax(amax, gpartd<2>(amax));
    amax = quads_maxd(amax);
    int bad = s > 0 && (!(amax > 1e-300) || !(amax < 1e300));  // (no block: nothing to solve)
    int ex = 0;
    frexp(bad || s == 0 ? 1.0 : amax, &ex);
    const double scale = ldexp(1.0, -ex);
    float kf[T][T];
    double knorm = 0.0;  // largest row sum of the block, for the stopping test: in FP64
#pragma unroll
    for (int a = 0; a < T; ++a) {
      double rs = 0.0;
#pragma unroll
      for (int b = 0; b < T; ++b) {
        kf[a][b] = (float)(K[a][b] * scale);
        rs += fabs(K[a][b]);
      }
      knorm = fmax(knorm, quad_sum(rs));
    }
    knorm = quads_maxd(knorm);
    // identity on the padding (its rows of the FP64 block stay zero)
#pragma unroll
    for (int a = 0; a < T; ++a)
      if (r == c && 4 * a + r >= s) kf[a][a] = 1.f;
    tile_steps<T, 0>(kf, r, c, s, bad);
    bad = group_ori<16>(bad);

    // The block's entries again: in LDS its second half still stands as the gather
    // left it, and the largest tile reads it there (held in registers through the
    // elimination its 64 VGPRs made 63 spills).
    auto block = [&](int a, int b) {
      if (T == 8 && a >= HA) return gb.half[(4 * (a - HA) + r) * LD + 4 * b + c];
      return K[a][b];
    };

    // ---- solve and refine in FP64 (z stays in LDS) ----
    // z += Kinv v for the right-hand side v of this lane's rows
    auto correct = [&](const float (&x)[T], bool first) {
      if (c == 0) {
#pragma unroll
        for (int a = 0; a < T; ++a) gb.y[r * 8 + a] = x[a];
      }
      wave_sync();
      float v[T];
#pragma unroll
      for (int b = 0; b < T; ++b) v[b] = gb.y[c * 8 + b];
      wave_sync();
#pragma unroll
      for (int a = 0; a < T; ++a) {
        float p = 0.f;
#pragma unroll
        for (int b = 0; b < T; ++b) p = fmaf(kf[a][b], v[b], p);
        p = quad_sum(p);
        if (c == 0) gb.z[r * 8 + a] = first ? (double)p : gb.z[r * 8 + a] + (double)p;
      }
      wave_sync();
    };
    int it = 0;
    bool conv = false;
    if (!bad) {
      float x[T];
      double fnorm = 0.0;
#pragma unroll
      for (int a = 0; a < T; ++a) {
        const double fa = gb.f[r * 8 + a];
        fnorm = fmax(fnorm, fabs(fa));
        x[a] = (float)(fa * scale);
      }
      fnorm = quads_maxd(fnorm);
      correct(x, true);
#pragma unroll 1
      for (it = 1; it <= kRefineMax; ++it) {
        double rn = 0.0, zn = 0.0;
        {
          double zc[T];
#pragma unroll
          for (int b = 0; b < T; ++b) {
            zc[b] = gb.z[c * 8 + b];
            zn = fmax(zn, fabs(zc[b]));
          }
#pragma unroll
          for (int a = 0; a < T; ++a) {
            double p = 0.0;
#pragma unroll
            for (int b = 0; b < T; ++b) p = fma(-block(a, b), zc[b], p);
            p = gb.f[r * 8 + a] + quad_sum(p);
            rn = fmax(rn, fabs(p));
            if (!(p == p)) rn = __builtin_huge_val();  // (fmax drops a NaN)
            x[a] = (float)(p * scale);
          }
        }
        // the FP32 solution itself is never accurate to FP64 rounding: the
        // first correction is applied unchecked
        if (it > 1) {
          rn = quads_maxd(rn);
          zn = fmax(zn, gpartd<1>(zn));
          zn = fmax(zn, gpartd<2>(zn));
          if (zn < __builtin_huge_val() && rn <= 0x1p-47 * (knorm * zn + fnorm)) { conv = true; break; }
        }
        correct(x, false);
      }
    }
    if (!conv) {
      // FP32 factorisation not trusted: the workgroup solver redoes the row in FP64
      if (l == 0) {
        const int qc = atomicAdd(&w.cnt->nC, 1);
        if (qc < w.capC) w.binC[qc] = cc.c * w.chunk + t;
        else flag_row(&w.st[cc.m], ST_UNSUPPORTED, i);
      }
      continue;
    }
    if (l == 0) rmx.add(w, cc.m, it);

    const GDesc o = row_desc(w, cc.m);
    // ---- R row: F-entries of N(i) around the injected C-point (the last
    // residual left z in LDS) ----
    int below = 0;
#pragma unroll
    for (int h = 0; h < NL; ++h) below += nv[h] < i ? 1 : 0;
    below += gpart<1>(below);
    below += gpart<2>(below);
    below += gpart<4>(below);
    below += gpart<8>(below);
    if (l == 0) {
      o.Rrp[g - cc.rbase_m] = off;
      o.Rci[off + below] = i;
      o.Rva[off + below] = 1.0;
    }
#pragma unroll
    for (int h = 0; h < NL; ++h) {
      const int q = l + 16 * h;
      if (q < s) put_f_entry(w, o, o.fine0, off + q + (q >= below ? 1 : 0), nv[h], i, gb.z[by_group(q)]);
    }
  }
  }
  rmx.flush_wave(w);
}

}  // namespace

// persistent grid: as many workgroups as fit on the device at once.  sm: the
// largest block to take (at most 32); above, upto as in k_tile.
hipError_t launch_tile(const Work& w, int which, int sm, int above, int upto, int cus, hipStream_t s) {
#define CLAIR_TILE(TT)                                                                     \
  if (sm <= 4 * TT) {                                                                      \
    const int per = resident_blocks<k_tile<TT>, 64>();                                     \
    if (per < 0) return hipErrorInvalidValue;                                              \
    const int blocks = (std::max(1, per) * cus + 7) / 8 * 8;                              \
    hipLaunchKernelGGL((k_tile<TT>), dim3(blocks), dim3(64), 0, s, w, which, above, upto);              \
    return hipGetLastError();                                                              \
  }
  CLAIR_TILE(3)
  CLAIR_TILE(4)
  CLAIR_TILE(5)
  CLAIR_TILE(6)
  CLAIR_TILE(7)
  CLAIR_TILE(8)
#undef CLAIR_TILE
  return hipErrorInvalidValue;
}

}  // namespace clair
