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
typedef double dbl2 __attribute__((ext_vector_type(2)));

constexpr int CB = 64;             // block of the step kernels
constexpr int CT = 18;             // padded row of the 16 x 16 transposes in LDS (16-byte rows)
constexpr int CHOL_LDS = 2 * CB * CB + 4 * 256 + 2 * 16 * CT;  // doubles: two blocks, six tiles (76 KB)

__device__ __forceinline__ dbl4 mfma_f64(double a, double b, dbl4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Four 16 x 16 tiles of a wave's 16 rows, and a loop over them with the tile as
// a constant: as an array the compiler joins the tiles into one 32-register
// value and copies it around every branch.
struct Rows {
  dbl4 t0, t1, t2, t3;
  template <int T>
  __device__ __forceinline__ dbl4 &tile() {
    if constexpr (T == 0) return t0;
    else if constexpr (T == 1) return t1;
    else if constexpr (T == 2) return t2;
    else return t3;
  }
  template <int T>
  __device__ __forceinline__ const dbl4 &tile() const {
    return const_cast<Rows *>(this)->tile<T>();
  }
};
template <int T>
struct TileIx {
  static constexpr int value = T;
};
template <class F>
__device__ __forceinline__ void for_tiles(F f) {
  f(TileIx<0>());
  f(TileIx<1>());
  f(TileIx<2>());
  f(TileIx<3>());
}

// v of lane N of the own row of 16 lanes (DPP row_newbcast)
template <int N>
__device__ __forceinline__ double row_lane(double v) {
  const long b = __builtin_amdgcn_update_dpp(0L, (long)__double_as_longlong(v), 0x150 + N, 0xF, 0xF, true);
  return __longlong_as_double(b);
}

// LDS written by a wave is read by other lanes of the same wave next: the LDS
// pipe keeps a wave's order, so only the compiler has to keep it.
__device__ __forceinline__ void wave_lds_order() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_wave_barrier();
}

// One wave: Cholesky of a 16 x 16 tile and its inverse in one sweep.  Lane l
// (mod 16) holds row l of the tile in a[0..15] and column l of the identity in
// x[0..15]; both see the same elimination, a[i] -= l_i l_own and x[i] -= l_i
// x_own, with l_i broadcast from lane i by DPP (the four rows of 16 lanes work
// alike).  Afterwards a holds row l of L (entries 0..l), x column l of L^-1,
// piv the pivot of row l before its square root.  1/sqrt(d) is v_rsq_f64 (24
// bits or more) and one third-order correction, which leaves an error of an
// ulp.
//
// Column J + 1's square root starts as soon as its own entry is updated, under
// the other updates of column J; the scheduling barrier keeps the broadcasts
// of later columns from being hoisted (and spilled).
template <int J>
__device__ __forceinline__ void sweep_update(double (&a)[16], double (&x)[16], double own, double y) {
  if constexpr (J < 16) {
    const double l = row_lane<J>(own);
    a[J] = fma(-l, own, a[J]);
    x[J] = fma(-l, y, x[J]);
    sweep_update<J + 1>(a, x, own, y);
  }
}
template <int J>
__device__ __forceinline__ void sweep_column(double (&a)[16], double (&x)[16], int l16, double &piv) {
  if constexpr (J < 16) {
    const double d = row_lane<J>(a[J]);
    const double r0 = __builtin_amdgcn_rsq(d);
    const double e = fma(-(d * r0), r0, 1.0);
    const double r = fma(r0 * e, fma(0.375, e, 0.5), r0);
    const double own = a[J] * r, y = x[J] * r;
    double ljj = d * r;
    ljj = fma(fma(-ljj, ljj, d), 0.5 * r, ljj);
    if (l16 == J) piv = d;
    a[J] = l16 == J ? ljj : own;
    x[J] = y;
    if constexpr (J < 15) {
      const double l = row_lane<J + 1>(own);
      a[J + 1] = fma(-l, own, a[J + 1]);
      x[J + 1] = fma(-l, y, x[J + 1]);
      __builtin_amdgcn_sched_barrier(0);
      sweep_update<J + 2>(a, x, own, y);
    }
    sweep_column<J + 1>(a, x, l16, piv);
  }
}
__device__ __forceinline__ void sweep16(double (&a)[16], double (&x)[16], int l16, double &piv) {
  sweep_column<0>(a, x, l16, piv);
}

// Pivot rule of a factorisation: row g fails when its pivot is not above
// tol[g % p] (rows from plim on are padding of unit variance).
struct PivotRule {
  double tol[PMAX];
  int p;
  int m0;        // row0 % p
  int64_t row0;  // global row of block 0's first row
  int64_t plim;
};

// Row `row` (in block 0's count) of a factorisation against its pivot rule.
__device__ __forceinline__ void check_pivot(const PivotRule &pr, int64_t g, double piv,
                                            int64_t *info) {
  const unsigned var = ((unsigned)pr.m0 + (unsigned)g) % (unsigned)pr.p;
  double tol = pr.tol[0];
#pragma unroll
  for (int i = 1; i < PMAX; ++i) tol = var == (unsigned)i ? pr.tol[i] : tol;
  if (pr.row0 + g >= pr.plim) tol = 0x1p-40;
  const uint64_t m = __ballot(!(piv > tol) || !(piv > 0.0));
  if (m && (threadIdx.x & 63) == __builtin_ctzll(m))
    atomicMin((unsigned long long *)info, (unsigned long long)(pr.row0 + g + 1));
}

// Cholesky of a 64 x 64 block and its inverse.  s: the block in row layout,
// wave w holding rows 16 w .. 16 w + 15 (tiles s[0..w] are read).  Lower part
// to S, the inverse (zeros above the diagonal) to W, both column-major.
//
// 16-wide steps: wave q factors and inverts diagonal tile q (sweep16), the
// waves below form their tile of L as a product with that inverse and update
// their row; the waves above, which are done with their rows, build row q of
// the inverse meanwhile (wave j owns column j).  The serial chain per step is
// one sweep, four MFMAs for L, four for the next diagonal tile, and two trips
// through LDS; the pivot test and every store to memory are off it.  The steps
// are a rolled loop: straight-line code is fetched once and runs at the pace
// of its instruction misses.  tl: 16 tiles of 256 doubles (L's six below the
// diagonal, ten of the inverse), dl: 4 more (its diagonal tiles), st: 16 x CT,
// wi: 16 x CT of LDS.
__device__ __forceinline__ void potrf64(const Rows &s, double *S, unsigned lds, double *W,
                                        unsigned ldw, double *tl, double *dl, double *st, double *wi,
                                        int64_t g0,
                                        const PivotRule &pr, int64_t *info) {
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lk = lane >> 4;
  double *ti = tl + 6 * 256;  // inverse tiles (q, j), j <= q: lane's element e at 64 e + lane
  double piv = 1.0;
  // to memory: row q of L (tile (q, m) by wave m, the diagonal tile by wave q)
  // and of the inverse (wave w's tile)
  // (32-bit offsets from lane indices that the compiler cannot see through:
  // hoisted out of the loop, the addresses took every register)
  auto store_rows = [&](int q, int m) {
    int r = l16, k = lk;
    asm volatile("" : "+v"(r), "+v"(k));
    if (m < q) {
      const double *t = tl + (q * (q - 1) / 2 + m) * 256;
      double *s0 = S + (unsigned)(16 * m) * lds + 16 * q;
#pragma unroll
      for (int e = 0; e < 4; ++e) s0[(unsigned)(4 * e + k) * lds + r] = t[(4 * e + k) * 16 + r];
    }
    const double *i = ti + (q * (q + 1) / 2 + m) * 256;
    double *w0 = W + (unsigned)(16 * m) * ldw + 16 * q;
#pragma unroll
    for (int e = 0; e < 4; ++e) w0[(unsigned)r * ldw + 4 * e + k] = i[64 * e + 16 * k + r];
  };
  auto store_diag = [&](int q) {
    int r = l16, k = lk;
    asm volatile("" : "+v"(r), "+v"(k));
    double *s0 = S + (unsigned)(16 * q) * lds + 16 * q;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (4 * e + k <= r) s0[(unsigned)(4 * e + k) * lds + r] = dl[q * 256 + (4 * e + k) * 16 + r];
    if (k == 0) check_pivot(pr, g0 + 16 * q + r, piv, info);
  };
  // tiles (w, q), (w, q + 1), (w, q + 2) below the diagonal tile dg
  dbl4 o0 = s.t0, o1 = s.t1, o2 = s.t2, dg = s.t3;
  if (w == 0) dg = s.t0;
  if (w == 1) dg = s.t1;
  if (w == 2) dg = s.t2;
#pragma unroll 1
  for (int t = w + 1; t < 4; ++t)  // zeros of the inverse above the diagonal
#pragma unroll
    for (int e = 0; e < 4; ++e) W[(int64_t)(16 * t + l16) * ldw + 16 * w + 4 * e + lk] = 0.0;
#pragma unroll 1
  for (int q = 0; q < 4; ++q) {
    dbl4 t4 = dbl4{0.0, 0.0, 0.0, 0.0};
    double a[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) a[i] = 0.0;
    if (w == q) {
#pragma unroll
      for (int e = 0; e < 4; ++e) st[l16 * CT + 4 * e + lk] = dg[e];
      wave_lds_order();
      int r = l16;
      asm volatile("" : "+v"(r));  // (the identity is formed here, not held across the loop)
      double x[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        a[i] = st[r * CT + i];
        x[i] = i == r ? 1.0 : 0.0;
      }
      wave_lds_order();
      sweep16(a, x, r, piv);
      // (keeps x's updates from being sunk past the sweep, into the branch)
#pragma unroll
      for (int i = 0; i < 16; ++i) asm volatile("" : "+v"(x[i]));
      if (lane < 16)  // inverse of tile q, column-major, ld CT
#pragma unroll
        for (int i = 0; i < 16; ++i) wi[r * CT + i] = x[i];
    } else if (w < q) {
      store_rows(q - 1, w);
      if (w == q - 1) store_diag(w);
      // sum_m L(q, m) inv(m, w), m = w..q-1
      for (int m = w; m < q; ++m)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          t4 = mfma_f64(tl[(q * (q - 1) / 2 + m) * 256 + (4 * e + lk) * 16 + l16],
                        ti[(m * (m + 1) / 2 + w) * 256 + 64 * e + lane], t4);
    }
    __syncthreads();
    dbl4 x = dbl4{0.0, 0.0, 0.0, 0.0};
    if (w > q) {
#pragma unroll
      for (int e = 0; e < 4; ++e) x = mfma_f64(wi[(4 * e + lk) * CT + l16], o0[e], x);
      double *t = tl + (w * (w - 1) / 2 + q) * 256;
#pragma unroll
      for (int e = 0; e < 4; ++e) t[(4 * e + lk) * 16 + l16] = x[e];
#pragma unroll
      for (int e = 0; e < 4; ++e) dg = mfma_f64(x[e], -x[e], dg);
    } else {
      dbl4 r = dbl4{0.0, 0.0, 0.0, 0.0};
      if (w < q) {  // row q of the inverse: -inv(q, q) times the sum
#pragma unroll
        for (int e = 0; e < 4; ++e) r = mfma_f64(-wi[(4 * e + lk) * CT + l16], t4[e], r);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = wi[l16 * CT + 4 * e + lk];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) ti[(q * (q + 1) / 2 + w) * 256 + 64 * e + lane] = r[e];
      if (w == q && lane < 16)
#pragma unroll
        for (int i = 0; i < 16; ++i) dl[q * 256 + 16 * i + lane] = a[i];
    }
    __syncthreads();
    if (w > q) {  // (w, q + 1), (w, q + 2) -= L(w, q) L(., q)^T
      const double *t1 = tl + ((q + 1) * q / 2 + q) * 256, *t2 = tl + ((q + 2) * (q + 1) / 2 + q) * 256;
      if (q + 1 < w)
#pragma unroll
        for (int e = 0; e < 4; ++e) o1 = mfma_f64(t1[(4 * e + lk) * 16 + l16], -x[e], o1);
      if (q + 2 < w)
#pragma unroll
        for (int e = 0; e < 4; ++e) o2 = mfma_f64(t2[(4 * e + lk) * 16 + l16], -x[e], o2);
      o0 = o1;
      o1 = o2;
    }
  }
  store_rows(3, w);
  if (w == 3) store_diag(3);
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
__device__ __forceinline__ void rows_load(const double *p, int64_t ld, Rows &v) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const double *q = p + 16 * w + (lane & 15) + (int64_t)(lane >> 4) * ld;
  for_tiles([&](auto t) {
    constexpr int T = decltype(t)::value;
#pragma unroll
    for (int e = 0; e < 4; ++e) v.tile<T>()[e] = q[(int64_t)(16 * T + 4 * e) * ld];
  });
}
__device__ __forceinline__ void rows_store(double *p, int64_t ld, const Rows &v) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  double *q = p + 16 * w + (lane & 15) + (int64_t)(lane >> 4) * ld;
  for_tiles([&](auto t) {
    constexpr int T = decltype(t)::value;
#pragma unroll
    for (int e = 0; e < 4; ++e) q[(int64_t)(16 * T + 4 * e) * ld] = v.tile<T>()[e];
  });
}
// ... to a 64 x 64 block in LDS as [column][row]
__device__ __forceinline__ void rows_to_lds(double *sm, const Rows &v) {
  rows_store(sm, CB, v);
}

// acc[0..nt) -= a B^T over k < 64: a in row layout (one wave's 16 rows), B a
// 64 x 64 block in LDS as [column][row].
__device__ __forceinline__ void rows_sub_nt(Rows &acc, const Rows &a, const double *sm, int nt) {
  const int lane = threadIdx.x & 63;
  const double *b = sm + (lane >> 4) * CB + (lane & 15);
  for_tiles([&](auto t) {
    constexpr int T = decltype(t)::value;
    if (T >= nt) return;
    dbl4 c = acc.tile<T>();
    for_tiles([&](auto k) {
      constexpr int K = decltype(k)::value;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        c = mfma_f64(b[(16 * K + 4 * e) * CB + 16 * T], -a.tile<K>()[e], c);
    });
    acc.tile<T>() = c;
  });
}

// x = a W^T with W lower triangular (64 x 64 in LDS as [column][row]): tile t
// of x needs k < 16 (t + 1) only.
__device__ __forceinline__ void rows_mul_wt(Rows &x, const Rows &a, const double *sm) {
  const int lane = threadIdx.x & 63;
  const double *b = sm + (lane >> 4) * CB + (lane & 15);
  for_tiles([&](auto t) {
    constexpr int T = decltype(t)::value;
    dbl4 c = dbl4{0.0, 0.0, 0.0, 0.0};
    for_tiles([&](auto k) {
      constexpr int K = decltype(k)::value;
      if constexpr (K <= T)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          c = mfma_f64(b[(16 * K + 4 * e) * CB + 16 * T], a.tile<K>()[e], c);
    });
    x.tile<T>() = c;
  });
}

// The forward solve beside a row block's step: with v_t complete, y_t = W v_t,
// and v_R -= L(R, t) y_t.  solve_parts sums a quarter of the columns of W (in
// LDS) per wave, four partial sums a row to part; solve_rows, after a barrier,
// adds them in wave order and applies the wave's 16 rows of L (row layout).
__device__ __forceinline__ void solve_parts(const double *sm, const double *vt, double *part) {
  const int c = threadIdx.x & 63, p = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < 16; ++i) s = fma(sm[(16 * p + i) * CB + c], vt[16 * p + i], s);
  part[p * CB + c] = s;
}
__device__ __forceinline__ double solve_y(const double *part, int c) {
  return (part[c] + part[CB + c]) + (part[2 * CB + c] + part[3 * CB + c]);
}
// ys: 64 doubles of LDS of the wave's own
__device__ __forceinline__ void solve_rows(const Rows &x, const double *part, double *ys,
                                           double *vr) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, l16 = lane & 15, lk = lane >> 4;
  ys[lane] = solve_y(part, lane);
  wave_lds_order();
  double s = 0.0;
  for_tiles([&](auto t) {
    constexpr int T = decltype(t)::value;
#pragma unroll
    for (int e = 0; e < 4; ++e) s = fma(x.tile<T>()[e], ys[16 * T + 4 * e + lk], s);
  });
  wave_lds_order();
  s += __shfl_xor(s, 16);
  s += __shfl_xor(s, 32);
  if (lk == 0) vr[16 * w + l16] -= s;
}

// One row block of step t: A1 = A(R, t), P1 = L(R, t-1), P0 = L(t, t-1)
// (both null: no earlier panel), Wt = inv(t, t).  L(R, t) = (A1 - P1 P0^T)
// Wt^T, written over A1.  CRIT: R = t + 1 and the block (R, R) in S follows:
// S -= P1 P1^T + L(R, t) L(R, t)^T, factored and inverted into Wn.  SOLVE:
// the right-hand side too (vt, vr: its blocks t and R), y_t to yt.
struct RowStep {
  double *A1;
  const double *P1, *P0, *Wt;
  double *S, *Wn;
  int64_t ld, ldw;
  const double *vt;
  double *vr, *yt;
};

template <bool CRIT, bool SOLVE = false>
__device__ __forceinline__ void row_step(const RowStep &a, double *sm, int64_t g0,
                                         const PivotRule &pr, int64_t *info) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double *b0 = sm, *b1 = sm + CB * CB, *st = sm + 2 * CB * CB, *wi = st + 16 * CT,
         *dl = wi + 16 * CT;
  Rows s, x;
  if (a.A1) {
    Rows acc, p1;
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
      if (CRIT) rows_to_lds(b1, p1);
      __syncthreads();
      rows_sub_nt(acc, p1, b0, 4);
      __syncthreads();
    }
    block_store(b0, vw);
    __syncthreads();
    if (SOLVE) solve_parts(b0, a.vt, st);
    rows_mul_wt(x, acc, b0);
    rows_store(a.A1, a.ld, x);
    if (CRIT) {
      if (a.P1) rows_sub_nt(s, p1, b1, w + 1);
      __syncthreads();
      rows_to_lds(b0, x);
      if (SOLVE) {
        if (w == 0) a.yt[lane] = solve_y(st, lane);
        solve_rows(x, st, wi + w * CB, a.vr);
      }
      __syncthreads();
      rows_sub_nt(s, x, b0, w + 1);
    }
  } else if (CRIT) {
    rows_load(a.S, a.ld, s);
  }
  if (CRIT)
    potrf64(s, a.S, (unsigned)a.ld, a.Wn, (unsigned)a.ldw, b1, dl, st, wi, g0, pr, info);
}

// C -= sum over n panels of A_p B_p^T for 64 x 64 column-major blocks of
// leading dimension ld; panel(p, A, B) gives the pointers.  Wave (wr, wc) of
// a 2 x 2 grid on 32 x 32; lower: the strict upper 32 x 32 quarter is skipped.
// The operands go from memory to registers directly (the two waves that share
// a half meet in the CU's cache), half a panel ahead of the products.  Row l
// of MFMA tile t is row 2 l + t of the half, so that a load brings both tiles'
// operands: with one tile's a load, the cache's lookups bound the update.
template <class F>
__device__ __forceinline__ void block_sub_nt(double *C, int n, F panel, int64_t ld, bool lower) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = w & 1, wc = w >> 1, l16 = lane & 15, lk = lane >> 4;
  if (lower && wr < wc) return;
  const int64_t oa = 32 * wr + 2 * l16 + (int64_t)lk * ld;
  const int64_t ob = 32 * wc + 2 * l16 + (int64_t)lk * ld;
  double *c = C + 32 * wr + 2 * l16 + (int64_t)(32 * wc + 2 * lk) * ld;
  dbl2 af[2][8], bf[2][8];
  dbl4 acc[2][2];
  auto load = [&](int h, const double *A, const double *B) {
    const double *a = A + oa, *b = B + ob;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      af[h][ks] = *(const dbl2 *)(a + (int64_t)(32 * h + 4 * ks) * ld);
      bf[h][ks] = *(const dbl2 *)(b + (int64_t)(32 * h + 4 * ks) * ld);
    }
  };
  auto mul = [&](int h) {
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
#pragma unroll
      for (int ti = 0; ti < 2; ++ti)
#pragma unroll
        for (int tj = 0; tj < 2; ++tj)
          acc[ti][tj] = mfma_f64(bf[h][ks][tj], -af[h][ks][ti], acc[ti][tj]);
  };
  const double *A, *B;
  panel(0, A, B);
  load(0, A, B);
  load(1, A, B);
#pragma unroll
  for (int tj = 0; tj < 2; ++tj)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const dbl2 v = *(const dbl2 *)(c + (int64_t)(8 * e + tj) * ld);
      acc[0][tj][e] = v[0];
      acc[1][tj][e] = v[1];
    }
  for (int p = 1; p < n; ++p) {
    panel(p, A, B);
    mul(0);
    load(0, A, B);
    mul(1);
    load(1, A, B);
  }
  mul(0);
  mul(1);
#pragma unroll
  for (int tj = 0; tj < 2; ++tj)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      *(dbl2 *)(c + (int64_t)(8 * e + tj) * ld) = dbl2{acc[0][tj][e], acc[1][tj][e]};
}

}  // namespace mvg
