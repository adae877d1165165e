// Right-looking Cholesky in 64-wide steps, one launch per step (the POTRF /
// TRSM / SYRK tasks of Section 5.1 on 64 x 64 blocks), with the inverses
// W_k = L_kk^-1 of the diagonal tiles that the solves use.
//
// A step is a serial chain (the 64 x 64 factor needs the column before it),
// so what it costs is its latency, not its arithmetic.  One launch per step
// keeps the chain short: the workgroup of row block t + 1 forms its block of
// L, updates the diagonal block (t+1, t+1) and factors it in the same launch,
// while the others update the rest.  For that each update lags at least one
// step behind its panel:
//
//   launch t:  rows R > t:     A(R, t) -= L(R, t-1) L(t, t-1)^T
//                              L(R, t)  = A(R, t) W(t, t)^T
//              row t + 1 also: A(t+1, t+1) -= both panels' products, then
//                              L(t+1, t+1) and W(t+1, t+1)
//              row t of W:     W(t, j) = -W(t, t) sum_m L(t, m) W(m, j)
//
// The rest of the matrix is updated by GROUP panels at once, which reads and
// writes it once for them: with u = t - g0, the panels g..g + GROUP - 1 (g a
// multiple of GROUP from g0) go to the columns from g + GROUP + 1 on in
// launches g + GROUP .. g + 2 GROUP - 1, a share of the columns in each, the
// nearest first.  What the next two launches need is updated by itself:
//
//   launch t:  R > t + 1:      A(R, t+1)   -= panels g..t-1 of the group of t
//                              A(t+2, t+2) -= the same
//
// The order of the panels is the same for every block, so the split decides
// nothing about the result.  Every block is written by one workgroup and all
// it reads was finished by the launch before, so there is nothing to wait for
// inside a launch.
//
// Measured: 21 us a step while the chain bounds it, up to 2,000 trailing rows
// (about 4 us of launch, 1.3 of loads, 10 of the 64 x 64 factor, the rest the
// products before it), 29 us at 3,100, 38 at 4,000 and 60 at 6,000, where the
// rank-256 updates do: the matrix cores are busy half of that time, the rest is
// waiting for operands at the blocks' starts and ends.  Before, a step was
// three launches (factor 37 us, panel 5, update 9) and the inverse of a tile 7
// (nb = 512) or 15 more of 12 to 40 us each: 2n = 3,074 took 6.2 ms, now 1.3; a
// 1024 tile 2 ms, now 0.3.
#include <algorithm>
#include <cmath>

#include "chol_dev.h"
#include "tile_dev.h"

namespace mvg {

struct StepArgs {
  TileMap M;
  double *winv;
  int64_t *info;
  PivotRule pr;
  int t, g0, g1;  // step, first block of the region, one past its last
  int s;          // blocks per tile side
  int r0, r1;     // rows of column t (t + 1 .. r0 - 1) and of column t - 1 that are not zero
  int nw, np;     // workgroups for W's row t and for the panel's rows from t + 2
  int l0, nl;     // first panel of t's group; rows of column t + 1 it goes to now, and the diagonal
  int q0;         // first panel of the group before, which goes to columns c0 .. c1 - 1,
  int c0, c1, cr; // rows up to cr - 1
  int nq;         // positions of these (see rest_block)
};

// Whole simulation of 6,400 rows and likelihood of 12,800 (ms): one panel at a
// time 3.93, 16.9; 2 at once 3.47, 16.5; 4: 3.37, 16.2; 6: 3.42, 16.2; 8: 3.56,
// 16.4, the shares then being too few blocks for the chip.
constexpr int GROUP = 4;
constexpr int SUP = 8;  // super-blocks of SUP x SUP blocks share their panels in one L2

// Position b of the rest: rows in strips of SUP, in each the columns up to its
// last row in groups of SUP.  Positions above the diagonal have no block.
__device__ __forceinline__ bool rest_block(const StepArgs &a, int b, int &R, int &C) {
  const int m = a.cr - a.c0, w = a.c1 - a.c0;
  int i = 0, n = 0;
  for (;; ++i) {
    n = min(SUP, m - SUP * i) * min(w, SUP * (i + 1));
    if (b < n) break;
    b -= n;
  }
  const int h = min(SUP, m - SUP * i), j = b / (h * SUP);
  b -= j * h * SUP;
  R = a.c0 + SUP * i + b % h;
  C = a.c0 + SUP * j + b / h;
  return C <= R;
}
static int rest_positions(int m, int w) {
  int n = 0;
  for (int i = 0; SUP * i < m; ++i) n += std::min(SUP, m - SUP * i) * std::min(w, SUP * (i + 1));
  return n;
}

__device__ __forceinline__ double *step_block(const StepArgs &a, int R, int C) {
  return tile_ptr(a.M, R / a.s, C / a.s) + (int64_t)(C % a.s) * CB * a.M.nb + (R % a.s) * CB;
}
// block (i, j) of W_k, i and j in the same tile
__device__ __forceinline__ double *step_inv(const StepArgs &a, int i, int j) {
  const int64_t nb = a.M.nb;
  return a.winv + (int64_t)(i / a.s) * nb * nb + (int64_t)(j % a.s) * CB * nb + (i % a.s) * CB;
}

// 16 columns (quarter cq of block column j) of W(t, j): the waves take the
// earlier blocks m = j + w, j + w + 4, ... and are added in wave order.
__device__ __forceinline__ void inv_row(const StepArgs &a, int j, int cq, double *sm) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, lk = lane >> 4, t = a.t;
  const int64_t nb = a.M.nb;
  dbl4 acc[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) acc[i] = dbl4{0.0, 0.0, 0.0, 0.0};
  for (int m = j + w; m < t; m += 4) {
    const double *L = step_block(a, t, m) + l16 + (int64_t)lk * nb;
    const double *B = step_inv(a, m, j) + (int64_t)(16 * cq + l16) * nb + lk;
    double bf[16], af[16][4];
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) {
      bf[ks] = B[4 * ks];
#pragma unroll
      for (int i = 0; i < 4; ++i) af[ks][i] = L[(int64_t)(4 * ks) * nb + 16 * i];
    }
#pragma unroll
    for (int ks = 0; ks < 16; ++ks)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i] = mfma_f64(af[ks][i], bf[ks], acc[i]);
  }
  // partial sums [wave][row][column] in LDS
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) sm[w * 1024 + (16 * i + 4 * e + lk) * 16 + l16] = acc[i][e];
  // W(t, t): rows 16 w .. of it, k < 16 (w + 1)
  const double *D = step_inv(a, t, t) + 16 * w + l16 + (int64_t)lk * nb;
  double df[16];
#pragma unroll
  for (int ks = 0; ks < 16; ++ks) df[ks] = D[(int64_t)(4 * ks) * nb];
  __syncthreads();
  dbl4 r = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int ks = 0; ks < 16; ++ks) {
    if (ks < 4 * (w + 1)) {
      const double *p = sm + (4 * ks + lk) * 16 + l16;
      const double b = (p[0] + p[1024]) + (p[2048] + p[3072]);
      r = mfma_f64(-df[ks], b, r);
    }
  }
  double *o = step_inv(a, t, j) + (int64_t)(16 * cq + l16) * nb + 16 * w + lk;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[4 * e] = r[e];
}

// First launch of a region (t = g0 - 1): besides the first diagonal block,
// the parts of W that no step writes, that is zeros above the diagonal and,
// in the padding rows, the identity.
__device__ __forceinline__ void inv_init(const StepArgs &a, int b) {
  const int ss = a.s * a.s, tile = b / ss, i = b % ss % a.s, j = b % ss / a.s;
  const int gi = a.g0 + tile * a.s + i, gj = a.g0 + tile * a.s + j;
  if (!(gi < gj || gi >= a.g1)) return;
  double *W = step_inv(a, gi, gj);
  const int r = threadIdx.x & 63;
  for (int c = threadIdx.x >> 6; c < CB; c += 4)
    W[(int64_t)c * a.M.nb + r] = (gi == gj && r == c) ? 1.0 : 0.0;
}

__global__ __launch_bounds__(256, 2) void k_chol_step(StepArgs a) {
  __shared__ double sm[CHOL_LDS];
  const int t = a.t;
  int b = blockIdx.x;
  const int64_t nb = a.M.nb;
  const int ncrit = t + 1 < a.g1 ? 1 : 0;
  if (b < ncrit) {
    RowStep r{};
    r.ld = r.ldw = nb;
    r.S = step_block(a, t + 1, t + 1);
    r.Wn = step_inv(a, t + 1, t + 1);
    if (t >= a.g0 && t + 1 < a.r0) {  // (else the row is zero there: first block, or past the band)
      r.A1 = step_block(a, t + 1, t);
      r.Wt = step_inv(a, t, t);
      if (t > a.g0 && t + 1 < a.r1) {
        r.P1 = step_block(a, t + 1, t - 1);
        r.P0 = step_block(a, t, t - 1);
      }
    }
    row_step<true>(r, sm, (int64_t)(t + 1) * CB, a.pr, a.info);
    return;
  }
  b -= ncrit;
  if (t < a.g0) {
    inv_init(a, b);
    return;
  }
  if (b < a.nw) {
    inv_row(a, t - t % a.s + b / 4, b % 4, sm);
    return;
  }
  b -= a.nw;
  if (b < a.np) {
    const int R = t + 2 + b;
    RowStep r{};
    r.ld = r.ldw = nb;
    r.A1 = step_block(a, R, t);
    r.Wt = step_inv(a, t, t);
    if (t > a.g0 && R < a.r1) {
      r.P1 = step_block(a, R, t - 1);
      r.P0 = step_block(a, t, t - 1);
    }
    row_step<false>(r, sm, 0, a.pr, a.info);
    return;
  }
  b -= a.np;
  int R, C, p0, n;
  if (b < a.nl) {
    R = b + 1 < a.nl ? t + 2 + b : t + 2;
    C = b + 1 < a.nl ? t + 1 : t + 2;
    p0 = a.l0;
    n = t - a.l0;
  } else {
    // a contiguous eighth of the positions to each XCD (workgroups go to them in turn)
    b -= a.nl;
    const int per = (a.nq + 7) >> 3;
    b = (b & 7) * per + (b >> 3);
    if (b >= a.nq || !rest_block(a, b, R, C)) return;
    if (R == t + 1) return;  // (t + 1, t + 1), the critical row's
    p0 = a.q0;
    n = GROUP;
  }
  auto panel = [&](int p, const double *&A, const double *&B) {
    A = step_block(a, R, p0 + p);
    B = step_block(a, C, p0 + p);
  };
  block_sub_nt(step_block(a, R, C), n, panel, nb, R == C);
}

// The first column of share u of GROUP of the lower triangle of m columns:
// equal areas, but no column in a later share than the launch that updates it
// by itself allows.
static int rest_column(int m, int u) {
  if (u == 0 || m <= 0) return 0;
  if (u == GROUP) return m;
  const int c = (int)std::ceil(m * (1.0 - std::sqrt(1.0 - (double)u / GROUP)));
  return std::min(m, std::max(c, GROUP + 1));
}

// Blocks g0..g1-1 (64 rows each) of the matrix, g0 the first block of a tile;
// rows from 64 g1 to the end of the last tile are padding and hold the
// identity.  band: tiles (I, J) with I - J >= band are zero.
static int chol_region(const TileMap &M, int band, int g0, int g1, double *winv, int64_t *d_info,
                       const PivotRule &pr, hipStream_t st) {
  StepArgs a{};
  a.M = M;
  a.winv = winv;
  a.info = d_info;
  a.pr = pr;
  a.g0 = g0;
  a.g1 = g1;
  a.s = M.nb / CB;
  const int tiles = (g1 - g0 + a.s - 1) / a.s;
  auto rows = [&](int c) { return (int)std::min<int64_t>(g1, (int64_t)(c / a.s + band) * a.s); };
  for (int t = g0 - 1; t < g1; ++t) {
    a.t = t;
    int64_t n = t + 1 < g1 ? 1 : 0;
    if (t < g0) {
      n += (int64_t)tiles * a.s * a.s;
    } else {
      a.r0 = rows(t);
      a.r1 = t > g0 ? rows(t - 1) : 0;
      a.nw = 4 * (t % a.s);
      a.np = std::max(0, a.r0 - (t + 2));
      const int u = (t - g0) % GROUP;  // launches since the group's panels began
      a.l0 = t - u;
      a.nl = u > 0 && t + 2 < a.r1 ? a.r1 - (t + 2) + 1 : 0;
      a.nq = 0;
      if (t - g0 >= GROUP) {
        a.q0 = t - u - GROUP;
        a.cr = rows(t - u - 1);
        a.c0 = t - u + 1 + rest_column(a.cr - (t - u + 1), u);
        a.c1 = t - u + 1 + rest_column(a.cr - (t - u + 1), u + 1);
        if (a.c1 > a.c0) a.nq = rest_positions(a.cr - a.c0, a.c1 - a.c0);
      }
      n += a.nw + a.np + a.nl + (a.nq + 7) / 8 * 8;
    }
    if (n <= 0) continue;
    hipLaunchKernelGGL(k_chol_step, dim3((unsigned)n), dim3(256), 0, st, a);
    if (int rc = check_launch("chol_step")) return rc;
  }
  return 0;
}

static PivotRule pivot_rule(const PivotTol &pt, int64_t row0, int64_t plim) {
  PivotRule r{};
  for (int i = 0; i < PMAX; ++i) r.tol[i] = pt.tol[i];
  r.p = pt.p;
  r.row0 = row0;
  r.m0 = (int)(row0 % pt.p);
  r.plim = plim;
  return r;
}

// Factor the diagonal tile (k, k) in place and fill W_k = L_kk^-1.
int diag_factor(const TileMap &M, int k, double *winv, int64_t *d_info, const PivotTol &pt,
                hipStream_t st) {
  const int s = M.nb / CB;
  const int64_t first = pt.gbase >= 0 ? pt.gbase : (int64_t)k * M.nb;  // global row of row 0
  const int64_t plim = std::min<int64_t>(pt.N, first + (pt.lreal > 0 ? pt.lreal : M.nb));
  const int real = (int)std::max<int64_t>(1, (plim - first + CB - 1) / CB);
  return chol_region(M, M.T, k * s, k * s + real, winv, d_info,
                     pivot_rule(pt, first - (int64_t)k * M.nb, plim), st);
}

// Factor the trailing matrix from tile column k on (already updated by the
// columns before), tiles (I, J) with I - J >= band being zero.
int chol_flat(const TileMap &M, int k, int band, double *winv, int64_t *d_info, const PivotTol &pt,
              hipStream_t st) {
  const int s = M.nb / CB;
  return chol_region(M, band, k * s, (int)((pt.N + CB - 1) / CB), winv, d_info,
                     pivot_rule(pt, 0, pt.N), st);
}

}  // namespace mvg
