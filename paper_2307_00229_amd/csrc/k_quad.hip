// k_quad.hip -- the bin-A solver of the mixed form: four lanes (a quad) per row
// with |N| <= 8.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "clair_device.h"
#include "clair_launch.h"
#include "mixed_device.h"

namespace clair {

namespace {

// ---------------------------------------------------------------------------
// numeric pass, four lanes (a quad) per row with |N| <= 8.  Lane l of the quad
// owns rows l and l + 4 of K = (A[N,N])^T, so the elimination's first rows and
// the substitutions' first half drop out of the second half of the steps.  The
// block is transposed once through LDS by the gather; the LU, both triangular
// solves and the FP64 residual then broadcast within the quad with DPP quad
// permutations (register moves, no LDS round trip).  A row of at most four
// points takes the 4 x 4 corner only, one block row per lane.
//
// Bound: the memory system's latency under scattered reads (two dependent
// trips a row, about 2.8 TB/s of lines moved), at three wavefronts per SIMD
// (the registers' limit; four spill).  So everything is about trips and lines:
// the quad reads each row of A together, all of a row's entries are in flight
// at once, the next row's bookkeeping is loaded one row ahead, and the column
// lists' exchanges are collected one row later.  64 five-point matrices of
// 64^2 to 768^2 (3.65 M rows): 730 us with one lane per row of A and waited
// exchanges, 717 with the shared gather, 667 with the two latency steps; 16
// matrices of 129^2 to 515^2 (484,487 rows): 107 us, where eight lanes per row
// took 134.  Rows of A of six entries and more take a second trip: nine-point
// rows at distance 1 are as fast as with eight lanes per row, no faster
// (1024^2, every second point a C-point: 84 and 87 us, every third: 54 and 51).
// ---------------------------------------------------------------------------
// lane src of the quad, to all four (src is a constant once the calling loops
// are unrolled, so the switch folds to one DPP move)
__device__ __forceinline__ int qbi(int v, int src) {
  switch (src) {
    case 0: return __builtin_amdgcn_mov_dpp(v, 0x00, 0xF, 0xF, false);
    case 1: return __builtin_amdgcn_mov_dpp(v, 0x55, 0xF, 0xF, false);
    case 2: return __builtin_amdgcn_mov_dpp(v, 0xAA, 0xF, 0xF, false);
    default: return __builtin_amdgcn_mov_dpp(v, 0xFF, 0xF, 0xF, false);
  }
}
__device__ __forceinline__ float qb(float v, int src) { return __int_as_float(qbi(__float_as_int(v), src)); }
__device__ __forceinline__ double qbd(double v, int src) {
  return __hiloint2double(qbi(__double2hiint(v), src), qbi(__double2loint(v), src));
}
// quad reductions: partners lane^1 and lane^2 (quad_perm [1,0,3,2] and [2,3,0,1])
__device__ __forceinline__ float qmaxf(float v) {
  v = fmaxf(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, false)));
  v = fmaxf(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xF, 0xF, false)));
  return v;
}
__device__ __forceinline__ double qxd(double v, int ctrl_is_b1) {
  const int lo = ctrl_is_b1 ? __builtin_amdgcn_mov_dpp(__double2loint(v), 0xB1, 0xF, 0xF, false)
                            : __builtin_amdgcn_mov_dpp(__double2loint(v), 0x4E, 0xF, 0xF, false);
  const int hi = ctrl_is_b1 ? __builtin_amdgcn_mov_dpp(__double2hiint(v), 0xB1, 0xF, 0xF, false)
                            : __builtin_amdgcn_mov_dpp(__double2hiint(v), 0x4E, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double qmaxd(double v) {
  v = fmax(v, qxd(v, 1));
  v = fmax(v, qxd(v, 0));
  return v;
}
__device__ __forceinline__ int qori(int v) {
  v |= __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, false);
  v |= __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, false);
  return v;
}

struct QuadBuf {
  double K[8 * 8];  // gathered block, row q of K at stride 8
  double f[8];
  int nb[8];
};

// row k of the block: register slot k / 4 of lane k % 4, broadcast in the quad
#define QB_ROW(arr0, arr1, k, p) ((k) < 4 ? qb(arr0[p], (k)) : qb(arr1[p], (k) - 4))

// The column-list records of a lane's last row: the list heads' exchange is
// under way, its results are stored once the next row's loads are out (or at
// the end), so that a row does not wait for its exchanges.
struct PendingLinks {
  int64_t e0 = -1, e1 = -1;  // batch-wide R entries, -1: none
  int prev0 = 0, prev1 = 0;
  int i = 0;
  __device__ __forceinline__ void flush(const Work& w) {
    if (e0 >= 0) w.clink[e0] = make_int2(prev0, i);
    if (e1 >= 0) w.clink[e1] = make_int2(prev1, i);
    e0 = -1;
    e1 = -1;
  }
};

// R's row (at most eight F-entries, lane l's points l and l + 4, around the
// C-point's own) and the F-entries' column lists (see put_f_entry)
__device__ __forceinline__ void emit_quad(const Work& w, const GDesc& d, PendingLinks& pend, int64_t fine0, int off,
                                          int s, int ql, int i, int dpos, int n0, int n1, double z0, double z1) {
  pend.flush(w);  // (a row without a gather)
  const bool h0 = ql < s, h1 = ql + 4 < s;
  const int p0 = off + ql + (ql >= dpos ? 1 : 0), p1 = off + ql + 4 + (ql + 4 >= dpos ? 1 : 0);
  if (d.B) {
    if (h0) { pend.e0 = d.link_base + p0; pend.prev0 = atomicExch(&w.chead[fine0 + n0], (int32_t)pend.e0); }
    if (h1) { pend.e1 = d.link_base + p1; pend.prev1 = atomicExch(&w.chead[fine0 + n1], (int32_t)pend.e1); }
    pend.i = i;
  }
  if (h0) { d.Rci[p0] = n0; d.Rva[p0] = z0; }
  if (h1) { d.Rci[p1] = n1; d.Rva[p1] = z1; }
  if (ql == 0) { d.Rci[off + dpos] = i; d.Rva[off + dpos] = 1.0; }
}

template <int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(3))) void k_quad8(Work w) {
  constexpr int NQ = NT / 4;
  __shared__ QuadBuf qbuf[NQ];
  const int tid = threadIdx.x;
  const int qd = tid >> 2;
  const int ql = tid & 3;
  QuadBuf& B = qbuf[qd];
  if (w.cnt->nA == 0) return;
  const int total = w.cnt->total_rows;
  // runs of four rows a quad where there are plenty (the row ahead is loaded
  // within a run), of one on small batches, so that more workgroups have some
  const RowBlocks rbk(total, (total >= 4 * NQ * (int)gridDim.x ? 4 : 1) * NQ);
  int r0, r1;
  if (!rbk.block(0, &r0, &r1)) return;
  RefineMax rmx;
  const int q0 = ql, q1 = ql + 4;  // this lane's rows of K
  // With a bin-A bound of 8 the residual that passes the stopping test is still
  // taken off.  That bound had a solver of eight lanes whose first correction
  // came unchecked; this one's test alone left up to 1.6e-14 of a row where that
  // left 1.6e-16 (300^2 five-point, eps = 1, distance 2; now 1.3e-16).  About 3 us
  // of 175 on 16 matrices of 129^2 to 515^2.
  const bool last = w.GA == 8;
  ChunkCursor cc;

  PendingLinks pend;
  int nx_t = 0, nx_i = 0, nx_off = 0, nx_s = 0;
  int2 nx_nn = make_int2(0, 0);
  for (int jb = 0; rbk.block(jb, &r0, &r1); ++jb) {
  bool ahead = false;
  for (int g = r0 + qd; g < r1; g += NQ) {  // quad-uniform
    int t, i, off, s;
    int2 nn;
    if (ahead) {
      t = nx_t; i = nx_i; off = nx_off; s = nx_s; nn = nx_nn;
    } else {
      cc.seek(w, g);
      if (cc.bins.x == 0) {  // no row of this chunk is ours: on to the next one
        g += (cc.re - g + NQ - 1) / NQ * NQ - NQ;
        continue;
      }
      cc.row(w, g, &t, &i, &off, &s);
      nn = *reinterpret_cast<const int2*>(w.slotA + (cc.fbase + t) * 8 + 2 * ql);
    }
    ahead = g + NQ < r1 && g + NQ < cc.re;
    if (ahead) {
      cc.row(w, g + NQ, &nx_t, &nx_i, &nx_off, &nx_s);
      nx_nn = *reinterpret_cast<const int2*>(w.slotA + (cc.fbase + nx_t) * 8 + 2 * ql);
    }
    if (s > 8 || !cc.live) continue;
    const int c = cc.c;
    MatStatus* st = &w.st[cc.m];
    const GDesc& d = cc.md;
    RowInfo ri;
    ri.m = cc.m;
    ri.i = i;
    ri.r = g - cc.rbase_m;
    ri.off = off;
    ri.s = s;
    ri.fine0 = cc.fine0;
    // one 8-byte load per lane (points 2l, 2l+1), then N_l and N_{l+4} by DPP
    // (quad_perm [0,0,1,1] and [2,2,3,3])
    // (all four moves run in every lane; a move under a lane condition would
    // read switched-off lanes)
    const int lx = __builtin_amdgcn_mov_dpp(nn.x, 0x50, 0xF, 0xF, false);
    const int ly = __builtin_amdgcn_mov_dpp(nn.y, 0x50, 0xF, 0xF, false);
    const int hx = __builtin_amdgcn_mov_dpp(nn.x, 0xFA, 0xF, 0xF, false);
    const int hy = __builtin_amdgcn_mov_dpp(nn.y, 0xFA, 0xF, 0xF, false);
    const int lo = (ql & 1) ? ly : lx;
    const int hi = (ql & 1) ? hy : hx;
    const int n0 = q0 < s ? lo : 0x7fffffff;
    const int n1 = q1 < s ? hi : 0x7fffffff;
    // row bounds: a lane without a point reads row i's
    const i2u bA = *(gptr<const i2u>)(d.rp + (q0 < s ? n0 : i));
    const i2u bB = *(gptr<const i2u>)(d.rp + (q1 < s ? n1 : i));
    const i2u bI = *(gptr<const i2u>)(d.rp + i);
    if (ql == 0) d.Rrp[ri.r] = ri.off;
    B.nb[q0] = n0;
    B.nb[q1] = n1;
#pragma unroll
    for (int u = 0; u < 16; ++u) {  // zero the block, identity on the padding
      const int idx = ql * 16 + u;
      const int rq = idx / 8, cp = idx % 8;
      B.K[idx] = (rq == cp && rq >= s) ? 1.0 : 0.0;
    }
    B.f[q0] = 0.0;
    B.f[q1] = 0.0;
    wave_sync();
    // gather: the quad reads row N_p of A (column p of K) together, four
    // consecutive entries per load, then lane l the fifth entry of rows N_l
    // and N_{l+4}, and four entries of row i: all loads in flight at once.
    // An index past its row reads the row's last entry and is dropped.
    const int ra0 = bA.x, ra1 = q0 < s ? bA.y : bA.x;
    const int rb0 = bB.x, rb1 = q1 < s ? bB.y : bB.x;
    const int i0 = bI.x, i1 = bI.y;
    if (d.nnz > 0) {
      int k[8], kt[2], kf[2];
      double v[8], vt[2], vf[2];
#pragma unroll
      for (int p = 0; p < 8; ++p) {
        const int e = (p < 4 ? qbi(ra0, p) : qbi(rb0, p - 4)) + ql;
        const int e1 = p < 4 ? qbi(ra1, p) : qbi(rb1, p - 4);
        const int ec = max(min(e, e1 - 1), 0);
        const int kk = d.ci[ec];
        v[p] = d.va[ec];
        k[p] = e < e1 ? kk : -1;
      }
      {
        const int ea = max(min(ra0 + 4, ra1 - 1), 0), eb = max(min(rb0 + 4, rb1 - 1), 0);
        const int ka = d.ci[ea], kb = d.ci[eb];
        vt[0] = d.va[ea];
        vt[1] = d.va[eb];
        kt[0] = ra0 + 4 < ra1 ? ka : -1;
        kt[1] = rb0 + 4 < rb1 ? kb : -1;
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int e = i0 + ql + 4 * h;
        const int ec = max(min(e, i1 - 1), 0);
        const int kk = d.ci[ec];
        vf[h] = d.va[ec];
        kf[h] = e < i1 ? kk : -1;
      }
      pend.flush(w);
#pragma unroll
      for (int p = 0; p < 8; ++p) {
        const int qq = find_pos<8>(B.nb, k[p]);
        if (qq >= 0) B.K[qq * 8 + p] = v[p];
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int qq = find_pos<8>(B.nb, kt[h]);
        if (qq >= 0) B.K[qq * 8 + (h ? q1 : q0)] = vt[h];
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int qq = find_pos<8>(B.nb, kf[h]);
        if (qq >= 0) B.f[qq] = -vf[h];
      }
      // rows of more than five entries, row i of more than eight
      int left = max(ra1 - ra0, rb1 - rb0) - 5;
      left = max(left, __builtin_amdgcn_mov_dpp(left, 0xB1, 0xF, 0xF, false));
      left = max(left, __builtin_amdgcn_mov_dpp(left, 0x4E, 0xF, 0xF, false));
      for (int o = 5; left > 0; o += 4, left -= 4) {
#pragma unroll
        for (int p = 0; p < 8; ++p) {
          const int e = (p < 4 ? qbi(ra0, p) : qbi(rb0, p - 4)) + ql + o;
          const int e1 = p < 4 ? qbi(ra1, p) : qbi(rb1, p - 4);
          k[p] = -1;
          if (e < e1) { k[p] = d.ci[e]; v[p] = d.va[e]; }
        }
#pragma unroll
        for (int p = 0; p < 8; ++p) {
          const int qq = find_pos<8>(B.nb, k[p]);
          if (qq >= 0) B.K[qq * 8 + p] = v[p];
        }
      }
      for (int e = i0 + ql + 8; e < i1; e += 4) {
        const int qq = find_pos<8>(B.nb, d.ci[e]);
        if (qq >= 0) B.f[qq] = -d.va[e];
      }
    }
    wave_sync();
    if (s <= 4) {
      // Blocks of at most four points (every row at distance 1 on a
      // five-point graph): lane l owns row l of the 4 x 4 corner of K (the
      // padding rows are identity there as in the full block), so the LU, the
      // substitutions and the residual take four steps instead of eight.
      const int q = ql;
      double kq[4];
      float amax = 0.f;
      double rs = 0.0;
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        kq[p] = B.K[q * 8 + p];
        amax = fmaxf(amax, (float)fabs(kq[p]));
        rs += fabs(kq[p]);
      }
      const double fq = B.f[q];
      const int nq = B.nb[q];  // INT32_MAX on padding rows
      amax = qmaxf(amax);
      const double knorm = qmaxd(rs);
      const double fnorm = qmaxd(fabs(fq));
      int ex = 0;
      frexpf(amax, &ex);
      const double scale = ldexp(1.0, -ex);
      float a[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) a[p] = (float)(kq[p] * scale);
      int bad = !(amax > 0.f) || !(amax < 3.0e38f);
      float ui = 1.f;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        float pr[4];
#pragma unroll
        for (int p = k; p < 4; ++p) pr[p] = qb(a[p], k);
        bad |= !(fabsf(pr[k]) >= 0x1p-24f);
        const float pinv = __builtin_amdgcn_rcpf(pr[k]);
        if (q == k) ui = pinv;
        if (q > k) {
          const float l = a[k] * pinv;
          a[k] = l;
#pragma unroll
          for (int p = k + 1; p < 4; ++p) a[p] = fmaf(-l, pr[p], a[p]);
        }
      }
      bad = qori(bad);
      double z = 0.0;
      int it = 0;
      bool conv = false;
      if (!bad) {
        // K y = rhs for this lane's entry of y
        auto solve4 = [&](float y) {
#pragma unroll
          for (int k = 0; k < 4; ++k) {  // forward, unit lower
            const float yk = qb(y, k);
            if (q > k) y = fmaf(-a[k], yk, y);
          }
#pragma unroll
          for (int k = 3; k >= 0; --k) {  // backward, upper
            if (q == k) y *= ui;
            const float zk = qb(y, k);
            if (q < k) y = fmaf(-a[k], zk, y);
          }
          return y;
        };
        z = solve4((float)(fq * scale));
        for (it = 1; it <= kRefineMax; ++it) {
          double r = fq;
#pragma unroll
          for (int p = 0; p < 4; ++p) r = fma(-kq[p], qbd(z, p), r);
          const double rn = qmaxd(fabs(r));
          const double zn = qmaxd(fabs(z));
          conv = rn <= 0x1p-47 * (knorm * zn + fnorm);
          if (conv && !last) break;
          z += (double)solve4((float)(r * scale));
          if (conv) break;
        }
        conv = conv && (z == z);
        conv = qori(conv ? 0 : 1) == 0;
      }
      if (!conv) {
        if (ql == 0) {
          const int qc = atomicAdd(&w.cnt->nC, 1);
          if (qc < w.capC) w.binC[qc] = c * w.chunk + t;
          else flag_row(st, ST_UNSUPPORTED, i);
        }
        continue;
      }
      if (ql == 0) rmx.add(w, ri.m, it);
      const int below = nq < i ? 1 : 0;
      const int b2 = below + __builtin_amdgcn_mov_dpp(below, 0xB1, 0xF, 0xF, false);
      const int dpos4 = b2 + __builtin_amdgcn_mov_dpp(b2, 0x4E, 0xF, 0xF, false);
      emit_quad(w, d, pend, ri.fine0, ri.off, s, ql, i, dpos4, nq, 0, z, 0.0);
      continue;
    }
    // rows q0, q1 of K (FP64), scaled FP32 copies
    double k0[8], k1[8];
    float amax = 0.f;
    double rs0 = 0.0, rs1 = 0.0;
#pragma unroll
    for (int p = 0; p < 8; ++p) {
      k0[p] = B.K[q0 * 8 + p];
      k1[p] = B.K[q1 * 8 + p];
      amax = fmaxf(amax, fmaxf((float)fabs(k0[p]), (float)fabs(k1[p])));
      rs0 += fabs(k0[p]);
      rs1 += fabs(k1[p]);
    }
    const double f0 = B.f[q0], f1 = B.f[q1];
    amax = qmaxf(amax);
    const double knorm = qmaxd(fmax(rs0, rs1));
    const double fnorm = qmaxd(fmax(fabs(f0), fabs(f1)));
    int ex = 0;
    frexpf(amax, &ex);
    const double scale = ldexp(1.0, -ex);
    float a0[8], a1[8];
#pragma unroll
    for (int p = 0; p < 8; ++p) {
      a0[p] = (float)(k0[p] * scale);
      a1[p] = (float)(k1[p] * scale);
    }
    // LU without pivoting: lane-local rows, pivot rows broadcast in the quad
    int bad = !(amax > 0.f) || !(amax < 3.0e38f);
    float ui0 = 1.f, ui1 = 1.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      float pr[8];
#pragma unroll
      for (int p = k; p < 8; ++p) pr[p] = QB_ROW(a0, a1, k, p);
      const float piv = pr[k];
      bad |= !(fabsf(piv) >= 0x1p-24f);
      const float pinv = __builtin_amdgcn_rcpf(piv);
      if (k < 4 && q0 == k) ui0 = pinv;
      if (k >= 4 && q1 == k) ui1 = pinv;
      if (k < 3 && q0 > k) {
        const float l = a0[k] * pinv;
        a0[k] = l;
#pragma unroll
        for (int p = k + 1; p < 8; ++p) a0[p] = fmaf(-l, pr[p], a0[p]);
      }
      if (q1 > k) {
        const float l = a1[k] * pinv;
        a1[k] = l;
#pragma unroll
        for (int p = k + 1; p < 8; ++p) a1[p] = fmaf(-l, pr[p], a1[p]);
      }
    }
    bad = qori(bad);

    double z0 = 0.0, z1 = 0.0;
    int it = 0;
    bool conv = false;
    if (!bad) {
      // solve K y = rhs for this lane's two entries y0, y1
      auto solve = [&](float y0, float y1, float* o0, float* o1) {
#pragma unroll
        for (int k = 0; k < 8; ++k) {  // forward, unit lower
          const float yk = k < 4 ? qb(y0, k) : qb(y1, k - 4);
          if (k < 3 && q0 > k) y0 = fmaf(-a0[k], yk, y0);
          if (q1 > k) y1 = fmaf(-a1[k], yk, y1);
        }
#pragma unroll
        for (int k = 7; k >= 0; --k) {  // backward, upper
          if (k < 4 && q0 == k) y0 *= ui0;
          if (k >= 4 && q1 == k) y1 *= ui1;
          const float zk = k < 4 ? qb(y0, k) : qb(y1, k - 4);
          if (q0 < k) y0 = fmaf(-a0[k], zk, y0);
          if (k > 4 && q1 < k) y1 = fmaf(-a1[k], zk, y1);
        }
        *o0 = y0;
        *o1 = y1;
      };
      float y0, y1;
      solve((float)(f0 * scale), (float)(f1 * scale), &y0, &y1);
      z0 = y0;
      z1 = y1;
      for (it = 1; it <= kRefineMax; ++it) {
        // r = f - K z in FP64: all of z broadcast in the quad
        // (the FP64 rows are read from LDS again rather than kept live)
        double r0 = f0, r1 = f1;
#pragma unroll
        for (int p = 0; p < 8; ++p) {
          const double zp = p < 4 ? qbd(z0, p) : qbd(z1, p - 4);
          r0 = fma(-B.K[q0 * 8 + p], zp, r0);
          r1 = fma(-B.K[q1 * 8 + p], zp, r1);
        }
        const double rn = qmaxd(fmax(fabs(r0), fabs(r1)));
        const double zn = qmaxd(fmax(fabs(z0), fabs(z1)));
        conv = rn <= 0x1p-47 * (knorm * zn + fnorm);
        if (conv && !last) break;
        float d0, d1;
        solve((float)(r0 * scale), (float)(r1 * scale), &d0, &d1);
        z0 += (double)d0;
        z1 += (double)d1;
        if (conv) break;
      }
      conv = conv && (z0 == z0) && (z1 == z1);
      conv = qori(conv ? 0 : 1) == 0;
    }
    if (!conv) {
      // FP32 factorisation not trusted: the workgroup solver redoes the row in FP64
      if (ql == 0) {
        const int qc = atomicAdd(&w.cnt->nC, 1);
        if (qc < w.capC) w.binC[qc] = c * w.chunk + t;
        else flag_row(st, ST_UNSUPPORTED, i);
      }
      continue;
    }
    if (ql == 0) rmx.add(w, ri.m, it);
    // R row
    const int dpos_l = (n0 < i ? 1 : 0) + (n1 < i ? 1 : 0);
    const int dpos = dpos_l + __builtin_amdgcn_mov_dpp(dpos_l, 0xB1, 0xF, 0xF, false);
    const int dposq = dpos + __builtin_amdgcn_mov_dpp(dpos, 0x4E, 0xF, 0xF, false);
    emit_quad(w, d, pend, ri.fine0, ri.off, s, ql, i, dposq, n0, n1, z0, z1);
  }
  }
  pend.flush(w);
  rmx.flush_wave(w);
}

}  // namespace

hipError_t launch_quad8(const Work& w, int wg_threads, int cus, hipStream_t s) {
#define CLAIR_Q8(NTT)                                                                       \
  if (wg_threads == NTT) {                                                                  \
    const int per = resident_blocks<k_quad8<NTT>, NTT>();                                   \
    if (per < 0) return hipErrorInvalidValue;                                               \
    const int blocks = (std::max(1, per) * cus + 7) / 8 * 8;                               \
    hipLaunchKernelGGL((k_quad8<NTT>), dim3(blocks), dim3(NTT), 0, s, w);                   \
    return hipGetLastError();                                                               \
  }
  CLAIR_Q8(256)
  CLAIR_Q8(128)
  CLAIR_Q8(64)
#undef CLAIR_Q8
  return hipErrorInvalidValue;
}

}  // namespace clair
