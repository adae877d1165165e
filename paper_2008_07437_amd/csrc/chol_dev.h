// Device pieces of the 64-block right-looking Cholesky: the factor and
// inverse of one 64 x 64 block, and the products around it.  Every function
// runs in a workgroup of 256 threads (4 waves); lane l of a wave is
// (l16, lk) = (l % 16, l / 16).
//
// Register layouts of v_mfma_f64_16x16x4 (D += A B, 16 x 4 by 4 x 16): the A
// operand of lane l is A[l16][lk], the B operand B[lk][l16], and element e of
// the result is D[4e + lk][l16].  Written with the operands exchanged,
// D^T += B^T A^T, lane l holds row l16 and columns 4e + lk of a tile: that is
// the A operand of k-step e, so a product's result feeds the next product
// without leaving the registers ("row layout" below).
#pragma once

#include "mvgeo_internal.h"

namespace mvg {

typedef double dbl4 __attribute__((ext_vector_type(4)));

constexpr int CB = 64;             // block of the step kernels
constexpr int CT = 17;             // padded row of the 16 x 16 transposes in LDS
constexpr int CHOL_LDS = 2 * CB * CB + 5 * 16 * CT;  // doubles: two blocks, five tiles (76 KB)

__device__ __forceinline__ dbl4 mfma_f64(double a, double b, dbl4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ double lane_value(double v, int lane) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
  return __hiloint2double(hi, lo);
}

// LDS written by a wave is read by other lanes of the same wave next: the LDS
// pipe keeps a wave's order, so only the compiler has to keep it.
__device__ __forceinline__ void wave_lds_order() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_wave_barrier();
}

// One wave: Cholesky of a 16 x 16 tile and its inverse in one sweep.  Lane
// r < 16 holds row r of the tile in v[0..15], lane 16 + c column c of the
// identity; both see the same elimination v[i] -= l_i v_own.  Afterwards lane
// r holds row r of L (entries 0..r) and lane 16 + c column c of L^-1; piv is
// the pivot of row r before its square root.  1/sqrt(d) is v_rsq_f64 (24 bits
// or more) and one third-order correction, which leaves an error of an ulp.
__device__ __forceinline__ void sweep16(double v[16], int lane, double &piv) {
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const double d = lane_value(v[j], j);
    const double r0 = __builtin_amdgcn_rsq(d);
    const double e = fma(-(d * r0), r0, 1.0);
    const double r = fma(r0 * e, fma(0.375, e, 0.5), r0);
    const double own = v[j] * r;
    double ljj = d * r;
    ljj = fma(fma(-ljj, ljj, d), 0.5 * r, ljj);
    if (lane == j) piv = d;
    v[j] = lane == j ? ljj : own;
#pragma unroll
    for (int i = j + 1; i < 16; ++i) v[i] = fma(-lane_value(own, i), own, v[i]);
  }
}

// Pivot rule of a factorisation: row g fails when its pivot is not above
// tol[g % p] (rows from plim on are padding of unit variance).
struct PivotRule {
  double tol[PMAX];
  int p;
  int64_t row0;  // global row of block 0's first row
  int64_t plim;
};

// Cholesky of a 64 x 64 block and its inverse.  s: the block in row layout,
// wave w holding rows 16 w .. 16 w + 15 (tiles s[0..w] are read).  Lower part
// to S, the inverse (zeros above the diagonal) to W, both column-major.
//
// 16-wide steps: wave q factors and inverts diagonal tile q (sweep16), the
// waves below form their tile of L as a product with that inverse and update
// their row; the waves above, which are done with their rows, build row q of
// the inverse meanwhile (wave j owns column j).  Serial chain per step: one
// sweep, four MFMAs for L, four for the next diagonal tile, and two trips
// through LDS.  lt: 6 x 256 doubles, st: 16 x CT, wi: 4 x 16 x CT of LDS.
__device__ __forceinline__ void potrf64(dbl4 s[4], double *S, int64_t lds, double *W, int64_t ldw,
                                        double *lt, double *st, double *wi, int64_t g0,
                                        const PivotRule &pr, int64_t *info) {
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lk = lane >> 4;
  dbl4 inv[4];  // column w of the inverse, tiles w..3, lane (column l16, rows 4e + lk)
#pragma unroll
  for (int q = 0; q < 4; ++q) inv[q] = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int t = 1; t < 4; ++t)  // zeros above the diagonal
    if (t > w)
#pragma unroll
      for (int e = 0; e < 4; ++e) W[(int64_t)(16 * t + 4 * e + lk) * ldw + 16 * w + l16] = 0.0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    double *wq = wi + q * 16 * CT;
    dbl4 t4 = dbl4{0.0, 0.0, 0.0, 0.0};
    if (w == q) {
#pragma unroll
      for (int e = 0; e < 4; ++e) st[l16 * CT + 4 * e + lk] = s[q][e];
      wave_lds_order();
      double v[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const double x = st[l16 * CT + i];
        v[i] = lane < 16 ? x : (i == lane - 16 ? 1.0 : 0.0);
      }
      wave_lds_order();
      double piv = 1.0;
      sweep16(v, lane, piv);
      if (lane < 16) {
        const int64_t g = g0 + 16 * q + lane;
        const int64_t row = pr.row0 + g;
        const int var = (int)(row % pr.p);
        double tol = pr.tol[0];
#pragma unroll
        for (int i = 1; i < PMAX; ++i) tol = var == i ? pr.tol[i] : tol;
        if (row >= pr.plim) tol = 0x1p-40;
        const bool bad = !(piv > tol) || !(piv > 0.0);
        const uint64_t m = __ballot(bad);
        if (m && lane == __builtin_ctzll(m))
          atomicMin((unsigned long long *)info, (unsigned long long)(row + 1));
#pragma unroll
        for (int c = 0; c < 16; ++c)
          if (c <= lane) S[(int64_t)(16 * q + c) * lds + 16 * q + lane] = v[c];
      } else if (lane < 32) {
#pragma unroll
        for (int i = 0; i < 16; ++i) wq[i * CT + lane - 16] = v[i];
      }
    } else if (w < q) {
      // sum_m L(q, m) inv(m, w), m = w..q-1 (inv is zero for m < w)
#pragma unroll
      for (int m = 0; m < q; ++m)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          t4 = mfma_f64(lt[(q * (q - 1) / 2 + m) * 256 + (4 * e + lk) * 16 + l16], inv[m][e], t4);
    }
    __syncthreads();
    if (w > q) {
      dbl4 x = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int e = 0; e < 4; ++e) x = mfma_f64(wq[l16 * CT + 4 * e + lk], s[q][e], x);
      double *t = lt + (w * (w - 1) / 2 + q) * 256;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        t[(4 * e + lk) * 16 + l16] = x[e];
        S[(int64_t)(16 * q + 4 * e + lk) * lds + 16 * w + l16] = x[e];
      }
      s[q] = x;
#pragma unroll
      for (int tj = q + 1; tj < 4; ++tj)
        if (tj == w)
#pragma unroll
          for (int e = 0; e < 4; ++e) s[tj] = mfma_f64(x[e], -x[e], s[tj]);
    } else {
      // row q of the inverse: -inv(q, q) times the sum, or inv(q, q) itself
      dbl4 r = dbl4{0.0, 0.0, 0.0, 0.0};
      if (w < q) {
#pragma unroll
        for (int e = 0; e < 4; ++e) r = mfma_f64(-wq[l16 * CT + 4 * e + lk], t4[e], r);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = wq[(4 * e + lk) * CT + l16];
      }
      inv[q] = r;
#pragma unroll
      for (int e = 0; e < 4; ++e) W[(int64_t)(16 * w + l16) * ldw + 16 * q + 4 * e + lk] = r[e];
    }
    if (q < 3) __syncthreads();
    if (w > q) {
#pragma unroll
      for (int tj = q + 1; tj < 4; ++tj)
        if (tj < w)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            s[tj] = mfma_f64(lt[(tj * (tj - 1) / 2 + q) * 256 + (4 * e + lk) * 16 + l16], -s[q][e],
                             s[tj]);
    }
  }
}

// Column-major 64 x 64 block to 16 values a thread (one load each, all in
// flight), and those values to LDS as [column][row].
__device__ __forceinline__ void block_load(const double *p, int64_t ld, double v[16]) {
  const int r = threadIdx.x & 63, c = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = p[(int64_t)(c + 4 * i) * ld + r];
}
__device__ __forceinline__ void block_store(double *sm, const double v[16]) {
  const int r = threadIdx.x & 63, c = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < 16; ++i) sm[(c + 4 * i) * CB + r] = v[i];
}

// Rows 16 w .. 16 w + 15 of a column-major 64 x 64 block in row layout.
__device__ __forceinline__ void rows_load(const double *p, int64_t ld, dbl4 v[4]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const double *q = p + 16 * w + (lane & 15) + (int64_t)(lane >> 4) * ld;
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) v[t][e] = q[(int64_t)(16 * t + 4 * e) * ld];
}
__device__ __forceinline__ void rows_store(double *p, int64_t ld, const dbl4 v[4]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  double *q = p + 16 * w + (lane & 15) + (int64_t)(lane >> 4) * ld;
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) q[(int64_t)(16 * t + 4 * e) * ld] = v[t][e];
}

// acc[0..nt) -= a B^T over k < 64: a in row layout (one wave's 16 rows), B a
// 64 x 64 block in LDS as [column][row].
__device__ __forceinline__ void rows_sub_nt(dbl4 acc[4], const dbl4 a[4], const double *sm, int nt) {
  const int lane = threadIdx.x & 63;
  const double *b = sm + (lane >> 4) * CB + (lane & 15);
#pragma unroll
  for (int t = 0; t < 4; ++t)
    if (t < nt)
#pragma unroll
      for (int ks = 0; ks < 16; ++ks)
        acc[t] = mfma_f64(b[4 * ks * CB + 16 * t], -a[ks >> 2][ks & 3], acc[t]);
}

// x = a W^T with W lower triangular (64 x 64 in LDS as [column][row]): tile t
// of x needs k < 16 (t + 1) only.
__device__ __forceinline__ void rows_mul_wt(dbl4 x[4], const dbl4 a[4], const double *sm) {
  const int lane = threadIdx.x & 63;
  const double *b = sm + (lane >> 4) * CB + (lane & 15);
#pragma unroll
  for (int t = 0; t < 4; ++t) x[t] = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int ks = 0; ks < 16; ++ks)
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (ks < 4 * (t + 1)) x[t] = mfma_f64(b[4 * ks * CB + 16 * t], a[ks >> 2][ks & 3], x[t]);
}

// One row block of step t: A1 = A(R, t), P1 = L(R, t-1), P0 = L(t, t-1)
// (both null: no earlier panel), Wt = inv(t, t).  L(R, t) = (A1 - P1 P0^T)
// Wt^T, written over A1.  With S != null, R = t + 1 and the block (R, R) in S
// follows: S -= P1 P1^T + L(R, t) L(R, t)^T, factored and inverted into Wn.
struct RowStep {
  double *A1;
  const double *P1, *P0, *Wt;
  double *S, *Wn;
  int64_t ld, ldw;
};

template <bool CRIT>
__device__ __forceinline__ void row_step(const RowStep &a, double *sm, int64_t g0,
                                         const PivotRule &pr, int64_t *info) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, lk = lane >> 4;
  double *b0 = sm, *b1 = sm + CB * CB, *st = sm + 2 * CB * CB, *wi = st + 16 * CT;
  dbl4 s[4], x[4];
  if (a.A1) {
    dbl4 acc[4], p1[4];
    double v0[16], vw[16];
    // every load of the step is in flight at once
    if (a.P1) {
      block_load(a.P0, a.ld, v0);
      rows_load(a.P1, a.ld, p1);
    }
    rows_load(a.A1, a.ld, acc);
    block_load(a.Wt, a.ldw, vw);
    if (CRIT) rows_load(a.S, a.ld, s);
    if (a.P1) {
      block_store(b0, v0);
      if (CRIT)
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int e = 0; e < 4; ++e) b1[(16 * t + 4 * e + lk) * CB + 16 * w + l16] = p1[t][e];
      __syncthreads();
      rows_sub_nt(acc, p1, b0, 4);
      __syncthreads();
    }
    block_store(b0, vw);
    __syncthreads();
    rows_mul_wt(x, acc, b0);
    rows_store(a.A1, a.ld, x);
    if (CRIT) {
      if (a.P1) rows_sub_nt(s, p1, b1, w + 1);
      __syncthreads();
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) b0[(16 * t + 4 * e + lk) * CB + 16 * w + l16] = x[t][e];
      __syncthreads();
      rows_sub_nt(s, x, b0, w + 1);
    }
  } else if (CRIT) {
    rows_load(a.S, a.ld, s);
  }
  if (CRIT) potrf64(s, a.S, a.ld, a.Wn, a.ldw, b1, st, wi, g0, pr, info);
}

// C -= A B^T for 64 x 64 column-major blocks of leading dimension ld, wave
// (wr, wc) of a 2 x 2 grid on 32 x 32; lower: the strict upper 32 x 32
// quarter is skipped.  The operands go from memory to registers directly
// (the two waves that share a half meet in the CU's cache).
__device__ __forceinline__ void block_sub_nt(double *C, const double *A, const double *B, int64_t ld,
                                             bool lower) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = w & 1, wc = w >> 1, l16 = lane & 15, lk = lane >> 4;
  if (lower && wr < wc) return;
  const double *a = A + 32 * wr + l16 + (int64_t)lk * ld;
  const double *b = B + 32 * wc + l16 + (int64_t)lk * ld;
  double *c = C + 32 * wr + l16 + (int64_t)(32 * wc + lk) * ld;
  double af[16][2], bf[16][2];
  dbl4 acc[2][2];
#pragma unroll
  for (int ks = 0; ks < 16; ++ks)
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      af[ks][t] = a[(int64_t)(4 * ks) * ld + 16 * t];
      bf[ks][t] = b[(int64_t)(4 * ks) * ld + 16 * t];
    }
#pragma unroll
  for (int ti = 0; ti < 2; ++ti)
#pragma unroll
    for (int tj = 0; tj < 2; ++tj)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[ti][tj][e] = c[(int64_t)(16 * tj + 4 * e) * ld + 16 * ti];
#pragma unroll
  for (int ks = 0; ks < 16; ++ks)
#pragma unroll
    for (int ti = 0; ti < 2; ++ti)
#pragma unroll
      for (int tj = 0; tj < 2; ++tj) acc[ti][tj] = mfma_f64(bf[ks][tj], -af[ks][ti], acc[ti][tj]);
#pragma unroll
  for (int ti = 0; ti < 2; ++ti)
#pragma unroll
    for (int tj = 0; tj < 2; ++tj)
#pragma unroll
      for (int e = 0; e < 4; ++e) c[(int64_t)(16 * tj + 4 * e) * ld + 16 * ti] = acc[ti][tj][e];
}

}  // namespace mvg
