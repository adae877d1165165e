// Covariance generation for the bivariate parsimonious Matern model (Eq. 2)
// and the cokriging predictor (Eq. 3-5) on gfx950.
//
// K_nu is evaluated by the trapezoidal rule on the integral representation
// K_nu(x) = int_0^inf exp(-x cosh t) cosh(nu t) dt (DLMF 10.32.9), written as
// e^-x * int exp(-x (cosh t - 1)) cosh(nu t) dt so that large x does not
// underflow.  The integrand is analytic in a strip around the real axis, so
// the rule converges geometrically in 1/h; the step is refined with x (levels
// in mvgeo_internal.h) because the integrand narrows like 1/sqrt(x).  One
// exponential per node serves the three orders nu11, nu22, nu12, and the
// node-dependent factors cosh(nu t_k), cosh(t_k) - 1 come from a per-theta
// table held in LDS.  Half-integer orders 1/2, 3/2, 5/2 use their closed forms.
#include <algorithm>
#include <cmath>

#include "matern_dev.h"
#include "tile_dev.h"

namespace mvg {

// 1 / Gamma(nu), nu > 0: Taylor series of 1 / Gamma(1 + z) at |z| <= 1/2 (24
// terms, 2e-16; generated with mpmath) and the recurrence.
static double rgamma(double nu) {
  static const double c[] = {
    1, 0.57721566490153287, -0.6558780715202539,
    -0.042002635034095237, 0.16653861138229148, -0.042197734555544333,
    -0.009621971527876973, 0.0072189432466630999, -0.0011651675918590652,
    -0.00021524167411495098, 0.0001280502823881162, -2.0134854780788239e-05,
    -1.2504934821426706e-06, 1.1330272319816959e-06, -2.0563384169776071e-07,
    6.1160951044814161e-09, 5.0020076444692229e-09, -1.18127457048702e-09,
    1.0434267116911005e-10, 7.7822634399050708e-12, -3.696805618642206e-12,
    5.1003702874544758e-13, -2.0583260535665066e-14, -5.3481225394230178e-15,
    1.2267786282382608e-15,
  };
  const int n = (int)std::floor(nu + 0.5);
  const double z = nu - n;
  double s = 0.0;
  for (int k = (int)(sizeof(c) / sizeof(c[0])) - 1; k >= 0; --k) s = std::fma(s, z, c[k]);
  if (n == 0) return s * z;
  for (int k = 1; k < n; ++k) s /= k + z;
  return s;
}

int matern_setup(const mvg_theta *th, MaternArgs *P, int64_t n_loc) {
  if (!th) return -1;
  const double v[6] = {th->sigma11_sq, th->sigma22_sq, th->a, th->nu11, th->nu22, th->beta};
  for (int i = 0; i < 5; ++i)
    if (!(v[i] > 0.0) || !std::isfinite(v[i])) return -(i + 1);
  if (th->nu11 > 5.0) return -4;
  if (th->nu22 > 5.0) return -5;
  if (!(std::fabs(th->beta) < 1.0)) return -6;
  P->a = th->a;
  P->nu[0] = th->nu11;
  P->nu[1] = th->nu22;
  P->nu[2] = 0.5 * (th->nu11 + th->nu22);
  // colocated correlation for d = 2: Gamma(nu + 1) / Gamma(nu) = nu
  const double rho = th->beta * std::sqrt(th->nu11 * th->nu22) / P->nu[2];
  P->coef[0] = th->sigma11_sq;
  P->coef[1] = th->sigma22_sq;
  P->coef[2] = rho * std::sqrt(th->sigma11_sq) * std::sqrt(th->sigma22_sq);
  P->any_quad = 0;
  for (int o = 0; o < 3; ++o) {
    const double nu = P->nu[o];
    P->lnorm[o] = -((nu - 1.0) * std::log(2.0) + std::lgamma(nu));
    P->norm[o] = std::exp2(1.0 - nu) * rgamma(nu);
    P->closed[o] = nu == 0.5 ? 1 : nu == 1.5 ? 2 : nu == 2.5 ? 3 : 0;
    if (!P->closed[o]) P->any_quad = 1;
  }
  P->table = P->any_quad && n_loc >= TABLE_MIN_LOC;
  return 0;
}

__global__ __launch_bounds__(256) void k_theta_tables(MaternArgs P, double *__restrict__ q) {
  theta_tables(blockIdx.x, P, q);
}

int launch_quad_table(const MaternArgs &P, double *d_qtab, hipStream_t st) {
  hipLaunchKernelGGL(k_theta_tables, dim3(P.table ? (CT_HI - CT_LO) / CT_GROUP : 1), dim3(256), 0,
                     st, P, d_qtab);
  return check_launch("theta_tables");
}

// One workgroup: a 32 x 32 block of location pairs of one lower tile.
// Thread layout: 32 consecutive pair-rows (coalesced column writes) x 8 groups
// of 4 pair-columns.
template <int FORM>
__global__ __launch_bounds__(256) void k_cov_tiles(MaternArgs P, const double *__restrict__ qtab,
                                                   const double *__restrict__ xs,
                                                   const double *__restrict__ ys, int64_t n_loc,
                                                   TileMap M, int tile_first, int spt) {
  __shared__ double ct[cov_lds(FORM)];
  const int nsub = spt * spt;
  const int64_t tile = tile_first + blockIdx.x / nsub;
  const int sub = blockIdx.x % nsub;
  if (M.kind && M.kind[tile] == TK_ZERO) return;  // annihilated DST tile (whole workgroup)
  load_cov_table<FORM>(qtab, ct);
  int J = 0;
  int64_t t = tile;
  while (t >= M.T - J) {
    t -= M.T - J;
    ++J;
  }
  const int I = J + (int)t;
  const int nb = M.nb, hp = nb / 2;
  const int pl = (sub % spt) * 32 + (threadIdx.x & 31);
  if (pl >= hp) return;
  const int pc0 = (sub / spt) * 32 + (threadIdx.x >> 5) * 4;
  const int64_t gl = (int64_t)I * hp + pl;
  const bool lpad = gl >= n_loc;
  const double xl = lpad ? 0.0 : xs[gl], yl = lpad ? 0.0 : ys[gl];
  const int kind = M.kind ? M.kind[tile] : TK_F64;
  char *tb = tile_bytes(M, tile);
  for (int q = 0; q < 4; ++q) {
    const int pr = pc0 + q;
    if (pr >= hp) break;
    const int64_t gr = (int64_t)J * hp + pr;
    double c[3];
    if (lpad || gr >= n_loc) {
      const double d = (gl == gr) ? 1.0 : 0.0;
      c[0] = d;
      c[1] = d;
      c[2] = 0.0;
    } else {
      cross_cov_block<FORM>(xl, yl, xs[gr], ys[gr], P, ct, qtab, c);
    }
    const int64_t e0 = (int64_t)(2 * pr) * nb + 2 * pl;  // (row 2pl, col 2pr)
    if (kind == TK_F64) {
      double *T = reinterpret_cast<double *>(tb);
      *reinterpret_cast<double2 *>(T + e0) = make_double2(c[0], c[2]);
      *reinterpret_cast<double2 *>(T + e0 + nb) = make_double2(c[2], c[1]);
    } else {
      float *T = reinterpret_cast<float *>(tb);
      *reinterpret_cast<float2 *>(T + e0) = make_float2((float)c[0], (float)c[2]);
      *reinterpret_cast<float2 *>(T + e0 + nb) = make_float2((float)c[2], (float)c[1]);
    }
  }
}

int launch_cov_tiles(const MaternArgs &P, const double *d_qtab, const double *d_x,
                     const double *d_y, int64_t n_loc, TileMap M, int tile_first, int tile_count,
                     hipStream_t st) {
  if (tile_count <= 0) return 0;
  const int spt = (M.nb / 2 + 31) / 32;
  const int64_t nwg = (int64_t)tile_count * spt * spt;
  // split very large grids into several launches of < 2^31 workgroups
  const int64_t per = ((int64_t)1 << 30) / (spt * spt);
  for (int64_t t0 = 0; t0 < tile_count; t0 += per) {
    const int64_t cnt = tile_count - t0 < per ? tile_count - t0 : per;
    const dim3 grid((unsigned)(cnt * spt * spt));
#define MVG_FORM(F)                                                                             \
  hipLaunchKernelGGL(k_cov_tiles<F>, grid, dim3(256), 0, st, P, d_qtab, d_x, d_y, n_loc, M,     \
                     (int)(tile_first + t0), spt)
    switch (cov_form(P)) {
      case COV_TABLE: MVG_FORM(COV_TABLE); break;
      case COV_QUAD: MVG_FORM(COV_QUAD); break;
      default: MVG_FORM(COV_CLOSED); break;
    }
#undef MVG_FORM
    int rc = check_launch("cov_tiles");
    if (rc) return rc;
  }
  (void)nwg;
  return 0;
}

// ------------------------------------------------------------ p variables

int matern_setup_p(const mvg_theta_p *th, MaternArgsP *P) {
  if (!th) return -1;
  const int p = th->p;
  if (p < 1 || p > PMAX) return -1;
  for (int i = 0; i < p; ++i)
    if (!(th->sigma_sq[i] > 0.0) || !std::isfinite(th->sigma_sq[i])) return -2;
  if (!(th->a > 0.0) || !std::isfinite(th->a)) return -3;
  for (int i = 0; i < p; ++i)
    if (!(th->nu[i] > 0.0) || !(th->nu[i] <= 5.0)) return -4;
  // beta: symmetric, unit diagonal, positive definite (Cholesky)
  double c[PMAX][PMAX];
  for (int i = 0; i < p; ++i)
    for (int j = 0; j < p; ++j) {
      const double b = th->beta[i * PMAX + j];
      if (!std::isfinite(b) || b != th->beta[j * PMAX + i]) return -5;
      if (i == j && b != 1.0) return -5;
      c[i][j] = b;
    }
  for (int j = 0; j < p; ++j) {
    double d = c[j][j];
    for (int k = 0; k < j; ++k) d -= c[j][k] * c[j][k];
    if (!(d > 0.0)) return -5;
    const double l = std::sqrt(d);
    c[j][j] = l;
    for (int i = j + 1; i < p; ++i) {
      double v = c[i][j];
      for (int k = 0; k < j; ++k) v -= c[i][k] * c[j][k];
      c[i][j] = v / l;
    }
  }
  P->p = p;
  P->no = p * (p + 1) / 2;
  P->a = th->a;
  P->any_quad = 0;
  for (int i = 0; i < p; ++i)
    for (int j = i; j < p; ++j) {
      const int o = pord(i, j, p);
      const double nu = 0.5 * (th->nu[i] + th->nu[j]);
      // colocated correlation for d = 2: Gamma(nu + 1) / Gamma(nu) = nu
      const double rho = i == j ? 1.0 : th->beta[i * PMAX + j] * std::sqrt(th->nu[i] * th->nu[j]) / nu;
      P->nu[o] = nu;
      P->coef[o] = rho * std::sqrt(th->sigma_sq[i]) * std::sqrt(th->sigma_sq[j]);
      P->lnorm[o] = -((nu - 1.0) * std::log(2.0) + std::lgamma(nu));
      P->closed[o] = nu == 0.5 ? 1 : nu == 1.5 ? 2 : nu == 2.5 ? 3 : 0;
      if (!P->closed[o]) P->any_quad = 1;
    }
  return 0;
}

__global__ void k_quad_table_p(MaternArgsP P, double *__restrict__ q) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < QN) quad_entry_p(k, P, q);
}

int launch_quad_table_p(const MaternArgsP &P, double *d_qtab, hipStream_t st) {
  hipLaunchKernelGGL(k_quad_table_p, dim3((QN + 255) / 256), dim3(256), 0, st, P, d_qtab);
  return check_launch("quad_table_p");
}

// One workgroup: up to 32 x 32 location pairs (l, r) whose P x P blocks meet
// lower tile (I, J); a thread takes one l and four r, evaluates all orders of
// a pair at once and writes the entries (P l + i, P r + j) that lie in the
// tile.  Every tile entry belongs to exactly one pair, so each is written
// once.  Rows / columns at or beyond N = P n are the identity padding.
template <int P>
__global__ __launch_bounds__(256) void k_cov_tiles_p(MaternArgsP A, const double *__restrict__ qtab,
                                                     const double *__restrict__ xs,
                                                     const double *__restrict__ ys, int64_t n_loc,
                                                     TileMap M, int64_t tile_first, int spt) {
  constexpr int NO = P * (P + 1) / 2;
  __shared__ double sq[(1 + NO) * QN];
  const int nsub = spt * spt;
  const int64_t tile = tile_first + blockIdx.x / nsub;
  const int sub = blockIdx.x % nsub;
  const int kind = M.kind ? M.kind[tile] : TK_F64;
  if (kind == TK_ZERO) return;  // annihilated DST tile (whole workgroup)
  for (int i = threadIdx.x; i < (1 + NO) * QN; i += blockDim.x) sq[i] = qtab[i];
  __syncthreads();
  int J = 0;
  int64_t t = tile;
  while (t >= M.T - J) {
    t -= M.T - J;
    ++J;
  }
  const int I = J + (int)t;
  const int nb = M.nb;
  const int64_t N = (int64_t)P * n_loc;
  const int64_t g0 = (int64_t)I * nb, c0 = (int64_t)J * nb;  // first row / column of the tile
  const int64_t lr0 = g0 / P, lr1 = (g0 + nb - 1) / P;       // row locations meeting the tile
  const int64_t lc0 = c0 / P, lc1 = (c0 + nb - 1) / P;
  const int64_t l = lr0 + (sub % spt) * 32 + (threadIdx.x & 31);
  if (l > lr1) return;
  const bool lreal = l < n_loc;
  const double xl = lreal ? xs[l] : 0.0, yl = lreal ? ys[l] : 0.0;
  char *tb = tile_bytes(M, tile);
  const int64_t rbase = lc0 + (sub / spt) * 32 + (threadIdx.x >> 5) * 4;
  for (int q = 0; q < 4; ++q) {
    const int64_t r = rbase + q;
    if (r > lc1) break;
    const bool real = lreal && r < n_loc;
    double Mv[NO];
    bool zero_h = false;
    if (real) {
      const double dx = xl - xs[r], dy = yl - ys[r];
      const double h = sqrt(dx * dx + dy * dy);
      zero_h = h == 0.0;
      if (!zero_h) matern_p<NO>(h / A.a, A, sq, Mv);
    }
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const int64_t g = (int64_t)P * l + i;
      if (g < g0 || g >= g0 + nb) continue;
#pragma unroll
      for (int j = 0; j < P; ++j) {
        const int64_t c = (int64_t)P * r + j;
        if (c < c0 || c >= c0 + nb) continue;
        double v;
        if (g >= N || c >= N) {
          v = g == c ? 1.0 : 0.0;
        } else {
          const int o = i <= j ? pord(i, j, P) : pord(j, i, P);
          v = zero_h ? A.coef[o] : A.coef[o] * Mv[o];
        }
        const int64_t e = (c - c0) * nb + (g - g0);
        if (kind == TK_F64)
          reinterpret_cast<double *>(tb)[e] = v;
        else
          reinterpret_cast<float *>(tb)[e] = (float)v;
      }
    }
  }
}

int launch_cov_tiles_p(const MaternArgsP &P, const double *d_qtab, const double *d_x,
                       const double *d_y, int64_t n_loc, TileMap M, hipStream_t st) {
  const int64_t nt = (int64_t)M.T * (M.T + 1) / 2;
  const int p = P.p;
  const int spt = (int)(((M.nb - 1) / p + 2 + 31) / 32);  // location rows per tile <= (nb-1)/p + 2
  const int64_t per = ((int64_t)1 << 30) / (spt * spt);
  for (int64_t t0 = 0; t0 < nt; t0 += per) {
    const int64_t cnt = std::min<int64_t>(per, nt - t0);
    const dim3 grid((unsigned)(cnt * spt * spt));
    switch (p) {
      case 1:
        hipLaunchKernelGGL(k_cov_tiles_p<1>, grid, dim3(256), 0, st, P, d_qtab, d_x, d_y, n_loc, M,
                           t0, spt);
        break;
      case 2:
        hipLaunchKernelGGL(k_cov_tiles_p<2>, grid, dim3(256), 0, st, P, d_qtab, d_x, d_y, n_loc, M,
                           t0, spt);
        break;
      case 3:
        hipLaunchKernelGGL(k_cov_tiles_p<3>, grid, dim3(256), 0, st, P, d_qtab, d_x, d_y, n_loc, M,
                           t0, spt);
        break;
      case 4:
        hipLaunchKernelGGL(k_cov_tiles_p<4>, grid, dim3(256), 0, st, P, d_qtab, d_x, d_y, n_loc, M,
                           t0, spt);
        break;
      default:
        set_error("p = %d variables is not supported", p);
        return MVG_ERR_STATE;
    }
    if (int rc = check_launch("cov_tiles_p")) return rc;
  }
  return 0;
}

// ---------------------------------------------------------------- cokriging

// Locations per partial sum: 256, more only where that makes over 64 sums a
// target.  From n_loc alone: how many targets share a call may not change the
// order of a target's sum.
int cokrige_span(int64_t n_loc) {
  return 256 * (int)((n_loc + 256 * 64 - 1) / (256 * 64));
}

// v summed over the 16 lanes of a row (DPP row_ror), in every lane
template <int N>
__device__ __forceinline__ double row_ror(double v) {
  return __longlong_as_double(
      __builtin_amdgcn_update_dpp(0L, (long)__double_as_longlong(v), 0x120 + N, 0xF, 0xF, true));
}
__device__ __forceinline__ double row_sum(double v) {
  v += row_ror<8>(v);
  v += row_ror<4>(v);
  v += row_ror<2>(v);
  return v + row_ror<1>(v);
}

constexpr int COK_TARGETS = 16;  // targets of a workgroup at most

// part[chunk 2m + 2t + j] = sum over the chunk's locations r and i in {0,1} of
// C_ij(||s0_t - s_r||) w[2r+i].  A workgroup takes one chunk and tg targets one
// after another, its table and its locations held; the sums do not depend on tg.
// Bound by the pairs' polynomials (LDS reads).  Whole predictions of 100 and
// 4,000 targets on 5,000 locations take 41 and 146 us; with one target and a
// chunk of 256 to 2,048 locations a workgroup, chosen from both counts, 45 and 169.
template <int FORM>
__global__ __launch_bounds__(256) void k_cokrige_dot(MaternArgs P, const double *__restrict__ qtab,
                                                     const double *__restrict__ xs,
                                                     const double *__restrict__ ys, int64_t n_loc,
                                                     const double *__restrict__ x0,
                                                     const double *__restrict__ y0, int64_t m,
                                                     const double *__restrict__ w,
                                                     double *__restrict__ part, int nchunk, int span,
                                                     int tg) {
  __shared__ double ct[cov_lds(FORM)];
  __shared__ double red[COK_TARGETS][2][16];
  load_cov_table<FORM>(qtab, ct);
  const int tid = threadIdx.x, chunk = blockIdx.x % nchunk;
  const int64_t t0 = (int64_t)(blockIdx.x / nchunk) * tg;
  const int nt = (int)min((int64_t)tg, m - t0);
  const int64_t r0 = (int64_t)chunk * span + tid, r1 = min(n_loc, (int64_t)(chunk + 1) * span);
  const int64_t rc = min(r0, n_loc - 1);
  const double xr = xs[rc], yr = ys[rc], w0 = w[2 * rc], w1 = w[2 * rc + 1];
  for (int t = 0; t < nt; ++t) {
    const double xt = x0[t0 + t], yt = y0[t0 + t];
    double a0 = 0.0, a1 = 0.0, c[3];
    if (r0 < r1) {
      cross_cov_block<FORM>(xt, yt, xr, yr, P, ct, qtab, c);
      a0 = c[0] * w0 + c[2] * w1;  // Zhat_1 += C11 w_1 + C21 w_2
      a1 = c[2] * w0 + c[1] * w1;  // Zhat_2 += C12 w_1 + C22 w_2
    }
    for (int64_t r = r0 + 256; r < r1; r += 256) {
      cross_cov_block<FORM>(xt, yt, xs[r], ys[r], P, ct, qtab, c);
      a0 += c[0] * w[2 * r] + c[2] * w[2 * r + 1];
      a1 += c[2] * w[2 * r] + c[1] * w[2 * r + 1];
    }
    a0 = row_sum(a0);
    a1 = row_sum(a1);
    if ((tid & 15) == 0) {
      red[t][0][tid >> 4] = a0;
      red[t][1][tid >> 4] = a1;
    }
  }
  __syncthreads();
  if (tid < 2 * nt) {
    double s = 0.0;
#pragma unroll
    for (int g = 0; g < 16; ++g) s += red[tid >> 1][tid & 1][g];
    part[(int64_t)chunk * 2 * m + 2 * t0 + tid] = s;
  }
}

int launch_cokrige_dot(const MaternArgs &P, const double *d_qtab, const double *d_x,
                       const double *d_y, int64_t n_loc, const double *d_x0, const double *d_y0,
                       int64_t m, const double *d_w, double *d_part, int nchunk, hipStream_t st) {
  // about 1,024 workgroups (four to a CU)
  const int tg = (int)std::min<int64_t>(COK_TARGETS, (m * nchunk + 1023) / 1024);
  const dim3 grid((unsigned)((m + tg - 1) / tg * nchunk));
  const int span = cokrige_span(n_loc);
#define MVG_FORM(F)                                                                              \
  hipLaunchKernelGGL(k_cokrige_dot<F>, grid, dim3(256), 0, st, P, d_qtab, d_x, d_y, n_loc, d_x0, \
                     d_y0, m, d_w, d_part, nchunk, span, tg)
  switch (cov_form(P)) {
    case COV_TABLE: MVG_FORM(COV_TABLE); break;
    case COV_QUAD: MVG_FORM(COV_QUAD); break;
    default: MVG_FORM(COV_CLOSED); break;
  }
#undef MVG_FORM
  return check_launch("cokrige_dot");
}

// c0 columns for the MSE: V[(2t + j) * Np + 2r + i] = C_ij(||s0_t - s_r||),
// padded rows 0.
template <int FORM>
__global__ __launch_bounds__(256) void k_cokrige_c0(MaternArgs P, const double *__restrict__ qtab,
                                                    const double *__restrict__ xs,
                                                    const double *__restrict__ ys, int64_t n_loc,
                                                    int64_t Np, const double *__restrict__ x0,
                                                    const double *__restrict__ y0,
                                                    double *__restrict__ V) {
  __shared__ double ct[cov_lds(FORM)];
  load_cov_table<FORM>(qtab, ct);
  const int64_t t = blockIdx.y;
  const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (2 * r >= Np) return;
  double c[3] = {0.0, 0.0, 0.0};
  if (r < n_loc) cross_cov_block<FORM>(x0[t], y0[t], xs[r], ys[r], P, ct, qtab, c);
  double *v0 = V + (2 * t) * Np, *v1 = V + (2 * t + 1) * Np;
  v0[2 * r] = c[0];
  v0[2 * r + 1] = c[2];
  v1[2 * r] = c[2];
  v1[2 * r + 1] = c[1];
}

int launch_cokrige_c0(const MaternArgs &P, const double *d_qtab, const double *d_x,
                      const double *d_y, int64_t n_loc, int64_t Np, const double *d_x0,
                      const double *d_y0, int64_t m, double *d_c0, hipStream_t st) {
  const int64_t npair = Np / 2;
  const dim3 grid((unsigned)((npair + 255) / 256), (unsigned)m);
#define MVG_FORM(F)                                                                             \
  hipLaunchKernelGGL(k_cokrige_c0<F>, grid, dim3(256), 0, st, P, d_qtab, d_x, d_y, n_loc, Np,   \
                     d_x0, d_y0, d_c0)
  switch (cov_form(P)) {
    case COV_TABLE: MVG_FORM(COV_TABLE); break;
    case COV_QUAD: MVG_FORM(COV_QUAD); break;
    default: MVG_FORM(COV_CLOSED); break;
  }
#undef MVG_FORM
  return check_launch("cokrige_c0");
}

// The same, transposed: V[(2r + i) ld + 2t + j] = C_ij(||s0_t - s_r||), zero for
// padded rows and targets.  64 targets by 32 locations per workgroup, a row's
// targets side by side.
template <int FORM>
__global__ __launch_bounds__(256) void k_cokrige_c0t(MaternArgs P, const double *__restrict__ qtab,
                                                     const double *__restrict__ xs,
                                                     const double *__restrict__ ys, int64_t n_loc,
                                                     int64_t Np, const double *__restrict__ x0,
                                                     const double *__restrict__ y0, int64_t m, int ld,
                                                     double *__restrict__ V) {
  __shared__ double ct[cov_lds(FORM)];
  load_cov_table<FORM>(qtab, ct);
  const int64_t t = (int64_t)blockIdx.x * 64 + (threadIdx.x & 63);
  const bool real = t < m;
  const double xt = real ? x0[t] : 0.0, yt = real ? y0[t] : 0.0;
  for (int q = threadIdx.x >> 6; q < 32; q += 4) {
    const int64_t r = (int64_t)blockIdx.y * 32 + q;
    if (2 * r >= Np) break;
    double c[3] = {0.0, 0.0, 0.0};
    if (real && r < n_loc) cross_cov_block<FORM>(xt, yt, xs[r], ys[r], P, ct, qtab, c);
    double *v = V + 2 * r * ld + 2 * t;
    *reinterpret_cast<double2 *>(v) = make_double2(c[0], c[2]);
    *reinterpret_cast<double2 *>(v + ld) = make_double2(c[2], c[1]);
  }
}

int launch_cokrige_c0t(const MaternArgs &P, const double *d_qtab, const double *d_x,
                       const double *d_y, int64_t n_loc, int64_t Np, const double *d_x0,
                       const double *d_y0, int64_t m, int ld, double *d_c0, hipStream_t st) {
  const dim3 grid((unsigned)(ld / 128), (unsigned)((Np / 2 + 31) / 32));
#define MVG_FORM(F)                                                                              \
  hipLaunchKernelGGL(k_cokrige_c0t<F>, grid, dim3(256), 0, st, P, d_qtab, d_x, d_y, n_loc, Np,   \
                     d_x0, d_y0, m, ld, d_c0)
  switch (cov_form(P)) {
    case COV_TABLE: MVG_FORM(COV_TABLE); break;
    case COV_QUAD: MVG_FORM(COV_QUAD); break;
    default: MVG_FORM(COV_CLOSED); break;
  }
#undef MVG_FORM
  return check_launch("cokrige_c0t");
}

}  // namespace mvg
