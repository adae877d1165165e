// Device-side evaluation of the bivariate Matern covariance (Eq. 2): the
// per-theta quadrature table and the 2 x 2 covariance block of two locations.
// Shared by the generation, cokriging and batched small-problem kernels.
//
// K_nu is evaluated by the trapezoidal rule on the integral representation
// K_nu(x) = int_0^inf exp(-x cosh t) cosh(nu t) dt (DLMF 10.32.9), written as
// e^-x * int exp(-x (cosh t - 1)) cosh(nu t) dt; see mvgeo_internal.h for the
// step levels.
#pragma once

#include "mvgeo_internal.h"

namespace mvg {

// Table entry k of the per-theta table q (4 x QN): cosh t_k - 1 and
// cosh(nu_o t_k) for the three orders.
__device__ __forceinline__ void quad_entry(int k, const MaternArgs &P, double *__restrict__ q) {
  int j = -1;
  for (int l = 0; l < QLEV; ++l)
    if (k >= qlev_off(l) && k < qlev_off(l) + qlev_cnt(l)) j = l;
  double cm1 = 0.0, c0 = 0.0, c1 = 0.0, c2 = 0.0;
  if (j >= 0) {
    const double t = (double)(k - qlev_off(j)) * qlev_h(j);
    const double s = sinh(0.5 * t);
    cm1 = 2.0 * s * s;  // cosh t - 1 without cancellation
    c0 = cosh(P.nu[0] * t);
    c1 = cosh(P.nu[1] * t);
    c2 = cosh(P.nu[2] * t);
  }
  q[k] = cm1;
  q[QN + k] = c0;
  q[2 * QN + k] = c1;
  q[3 * QN + k] = c2;
}

// Trapezoidal sums of the three orders at x > 0 (x within the levels) in
// units of the level's step, which is returned.
__device__ __forceinline__ double quad_sums(double x, const double *__restrict__ sq, double s[3]) {
  double s0 = 0.5, s1 = 0.5, s2 = 0.5;
  const int j = x <= qlev_xmax(0) ? 0 : x <= qlev_xmax(1) ? 1 : x <= qlev_xmax(2) ? 2
              : x <= qlev_xmax(3) ? 3 : 4;
  const int off = qlev_off(j), cnt = qlev_cnt(j);
  // nodes in pairs, the stopping test on the second of each pair (the
  // test costs six FP64 operations against the node's ~25)
  for (int k = 1; k < cnt; k += 2) {
    const double e = exp(-x * sq[off + k]);
    s0 += e * sq[QN + off + k];
    s1 += e * sq[2 * QN + off + k];
    s2 += e * sq[3 * QN + off + k];
    if (k + 1 >= cnt) break;
    const double e2 = exp(-x * sq[off + k + 1]);
    const double t0 = e2 * sq[QN + off + k + 1];
    const double t1 = e2 * sq[2 * QN + off + k + 1];
    const double t2 = e2 * sq[3 * QN + off + k + 1];
    s0 += t0;
    s1 += t1;
    s2 += t2;
    if (t0 <= 1e-17 * s0 && t1 <= 1e-17 * s1 && t2 <= 1e-17 * s2) break;
  }
  s[0] = s0;
  s[1] = s1;
  s[2] = s2;
  return qlev_h(j);
}

// The same for x below the polynomials' first octave, from the table in memory
// (their kernels hold the polynomials in LDS instead): all lanes of a wave are at
// the same node, of level 0, so a node's values come by scalar loads.  Sigma of
// 6,400 locations all that close (a = 1e5 on the unit square): 3.3 ms with vector
// loads, 1.9 so (a pair of nodes loaded ahead takes registers: 2.6); the
// quadrature alone, without polynomials, 2.2.
static_assert(qlev_cnt(0) % 2 == 1, "nodes 1 .. cnt - 1 in pairs");
__device__ __forceinline__ void quad_sums_near(double x, const double *qt, double s[3]) {
  typedef const __attribute__((address_space(4))) double cdouble;
  cdouble *q = (cdouble *)qt;
  double s0 = 0.5, s1 = 0.5, s2 = 0.5;
  for (int k = 1; k < qlev_cnt(0); k += 2) {
    double u[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      u[2 * i] = q[i * QN + k];
      u[2 * i + 1] = q[i * QN + k + 1];
    }
    const double e = exp(-x * u[0]);
    s0 += e * u[2];
    s1 += e * u[4];
    s2 += e * u[6];
    const double e2 = exp(-x * u[1]);
    const double t0 = e2 * u[3];
    const double t1 = e2 * u[5];
    const double t2 = e2 * u[7];
    s0 += t0;
    s1 += t1;
    s2 += t2;
    if (t0 <= 1e-17 * s0 && t1 <= 1e-17 * s1 && t2 <= 1e-17 * s2) break;
  }
  s[0] = s0;
  s[1] = s1;
  s[2] = s2;
}

// Normalised Matern M(x; nu_o) of the three orders from the closed forms or the
// quadrature's sums s (times the step, of logarithm logh).
__device__ __forceinline__ void matern3_orders(double x, const MaternArgs &P, const double s[3],
                                               double logh, double M[3]) {
  const double ex = exp(-x), lx = log(x);
#pragma unroll
  for (int o = 0; o < 3; ++o) {
    switch (P.closed[o]) {
      case 1: M[o] = ex; break;
      case 2: M[o] = (1.0 + x) * ex; break;
      case 3: M[o] = (1.0 + x + x * x * (1.0 / 3.0)) * ex; break;
      default: M[o] = exp(P.nu[o] * lx - x + P.lnorm[o] + logh) * s[o]; break;
    }
  }
}

// The same for x > 0, by the closed forms and (QUAD: some order needs it) the
// quadrature (sq: its table).
template <bool QUAD>
__device__ __forceinline__ void matern3(double x, const MaternArgs &P,
                                        const double *__restrict__ sq, double M[3]) {
  if (x > qlev_xmax(QLEV - 1)) {
    M[0] = M[1] = M[2] = 0.0;
    return;
  }
  double s[3] = {0.5, 0.5, 0.5}, logh = 0.0;
  if (QUAD) logh = log(quad_sums(x, sq, s));
  matern3_orders(x, P, s, logh, M);
}

// T_k(z) as powers of z: p[k][j]
struct ChebyshevPowers {
  short p[CT_NODES][CT_NODES] = {};
  constexpr ChebyshevPowers() {
    p[0][0] = 1;
    p[1][1] = 1;
    for (int k = 2; k < CT_NODES; ++k)
      for (int j = 0; j <= k; ++j)
        p[k][j] = (short)((j > 0 ? 2 * p[k - 1][j - 1] : 0) - p[k - 2][j]);
  }
};
static __device__ __constant__ constexpr ChebyshevPowers cheb_powers{};

// A theta's tables q (QTAB doubles): group `grp` of CT_GROUP octaves of the
// polynomials by one workgroup of 256 threads, the quadrature table by group
// 0's (each forms it for itself in LDS).  Values of g_o at the nodes of the
// parts, one node a thread; Chebyshev coefficients (whose rounding errors stay
// those of the values); then powers of z (the coefficients fall like 18^-k, so
// the change of basis loses nothing).  Bound by the latency of the longest sum
// (70 nodes at x = 2^-14).
__device__ __forceinline__ void theta_tables(int grp, const MaternArgs &P, double *__restrict__ q) {
  constexpr int NP = CT_GROUP * CT_SUB;  // parts of a group
  static_assert(NP * CT_NODES <= 256, "one node a thread");
  __shared__ double sq[4 * QN], val[NP * CT_ROW], che[NP * CT_ROW], cosine[4 * CT_NODES];
  const int tid = threadIdx.x;
  for (int k = tid; k < QN; k += 256) quad_entry(k, P, sq);
  if (tid < 4 * CT_NODES) cosine[tid] = cospi(tid / (2.0 * CT_NODES));
  __syncthreads();
  if (grp == 0)
    for (int i = tid; i < 4 * QN; i += 256) q[i] = sq[i];
  if (!P.table) return;
  if (tid < NP * CT_NODES) {
    const int part = tid / CT_NODES, k = tid % CT_NODES;
    const double scale = ldexp(1.0, CT_LO + grp * CT_GROUP + part / CT_SUB);
    const double x = scale * (1.0 + (part % CT_SUB + 0.5 + 0.5 * cosine[2 * k + 1]) / CT_SUB);
    double s[3];
    const double h = quad_sums(x, sq, s);
#pragma unroll
    for (int o = 0; o < 3; ++o) {
      double g;
      switch (P.closed[o]) {
        case 1: g = 1.0; break;
        case 2: g = 1.0 + x; break;
        case 3: g = 1.0 + x + x * x * (1.0 / 3.0); break;
        default: g = pow(x, P.nu[o]) * (P.norm[o] * (h * s[o])); break;
      }
      val[part * CT_ROW + k * 3 + o] = g;
    }
  }
  __syncthreads();
  for (int i = tid; i < NP * CT_ROW; i += 256) {
    const int part = i / CT_ROW, k = i % CT_ROW / 3, o = i % 3;
    double c = 0.0;
    for (int n = 0; n < CT_NODES; ++n)
      c = fma(val[part * CT_ROW + n * 3 + o], cosine[k * (2 * n + 1) % (4 * CT_NODES)], c);
    che[i] = c * ((k == 0 ? 1.0 : 2.0) / CT_NODES);
  }
  __syncthreads();
  double *out = q + 4 * QN + grp * NP * CT_ROW;
  for (int i = tid; i < NP * CT_ROW; i += 256) {
    const int part = i / CT_ROW, j = i % CT_ROW / 3, o = i % 3;
    double a = 0.0;
    for (int k = CT_DEG - ((CT_DEG - j) & 1); k >= j; k -= 2)
      a = fma(che[part * CT_ROW + k * 3 + o], (double)cheb_powers.p[k][j], a);
    out[i] = a;
  }
}

// Normalised Matern of the three orders at x > 0 from the polynomials ct
// (LDS), outside of them by the quadrature (qt).
__device__ __forceinline__ void matern3_tab(double x, const MaternArgs &P,
                                            const double *__restrict__ ct,
                                            const double *__restrict__ qt, double M[3]) {
  const int hi = __double2hiint(x);
  const int row = (hi >> 18) - ((1023 + CT_LO) << 2);  // octave and its quarter
  static_assert(CT_SUB == 4, "the two leading mantissa bits name the part");
  if ((unsigned)row >= (unsigned)((CT_HI - CT_LO) * CT_SUB)) {
    if (x > qlev_xmax(QLEV - 1)) {
      M[0] = M[1] = M[2] = 0.0;
      return;
    }
    double s[3], h = qlev_h(0);
    if (row < 0) quad_sums_near(x, qt, s);
    else h = quad_sums(x, qt, s);
    matern3_orders(x, P, s, log(h), M);
    return;
  }
  const double m = __hiloint2double((hi & 0xFFFFF) | 0x3FF00000, __double2loint(x));  // [1, 2)
  const double z = (m - (1.125 + 0.25 * (row & 3))) * 8.0;
  const double *c = ct + row * CT_ROW;
  double g0 = c[3 * CT_DEG], g1 = c[3 * CT_DEG + 1], g2 = c[3 * CT_DEG + 2];
#pragma unroll
  for (int k = CT_DEG - 1; k >= 0; --k) {
    g0 = fma(g0, z, c[3 * k]);
    g1 = fma(g1, z, c[3 * k + 1]);
    g2 = fma(g2, z, c[3 * k + 2]);
  }
  const double ex = exp(-x);
  M[0] = g0 * ex;
  M[1] = g1 * ex;
  M[2] = g2 * ex;
}

// How a theta's covariances are evaluated: every order closed, the quadrature
// at each pair, or the polynomials.
enum CovForm { COV_CLOSED = 0, COV_QUAD = 1, COV_TABLE = 2 };
__host__ __device__ inline int cov_form(const MaternArgs &P) {
  return P.table ? COV_TABLE : P.any_quad ? COV_QUAD : COV_CLOSED;
}
__host__ __device__ constexpr int cov_lds(int form) {  // doubles of LDS
  return form == COV_TABLE ? CT_SIZE : form == COV_QUAD ? 4 * QN : 1;
}

// The form's table into LDS (whole workgroup).
template <int FORM>
__device__ __forceinline__ void load_cov_table(const double *__restrict__ qt, double *ct) {
  if (FORM == COV_CLOSED) return;
  for (int i = threadIdx.x; i < cov_lds(FORM); i += blockDim.x)
    ct[i] = qt[i + (FORM == COV_TABLE ? 4 * QN : 0)];
  __syncthreads();
}

// 2x2 block C(||s_l - s_r||) of Representation I: c[0]=C11, c[1]=C22, c[2]=C12.
// ct: the table in LDS (load_cov_table), qt: the theta's tables in memory.
template <int FORM>
__device__ __forceinline__ void cross_cov_block(double xl, double yl, double xr, double yr,
                                                const MaternArgs &P, const double *ct,
                                                const double *qt, double c[3]) {
  const double dx = xl - xr, dy = yl - yr;
  const double h = sqrt(dx * dx + dy * dy);
  if (h == 0.0) {
    c[0] = P.coef[0];
    c[1] = P.coef[1];
    c[2] = P.coef[2];
    return;
  }
  double M[3];
  if (FORM == COV_TABLE) matern3_tab(h / P.a, P, ct, qt, M);
  else matern3<FORM != COV_CLOSED>(h / P.a, P, ct, M);
  c[0] = P.coef[0] * M[0];
  c[1] = P.coef[1] * M[1];
  c[2] = P.coef[2] * M[2];
}

// ------------------------------------------------------------ p variables

// Table entry k of the p-variate table ((1 + no) x QN).
__device__ __forceinline__ void quad_entry_p(int k, const MaternArgsP &P, double *__restrict__ q) {
  int j = -1;
  for (int l = 0; l < QLEV; ++l)
    if (k >= qlev_off(l) && k < qlev_off(l) + qlev_cnt(l)) j = l;
  double t = 0.0, cm1 = 0.0;
  if (j >= 0) {
    t = (double)(k - qlev_off(j)) * qlev_h(j);
    const double s = sinh(0.5 * t);
    cm1 = 2.0 * s * s;
  }
  q[k] = cm1;
  for (int o = 0; o < P.no; ++o) q[(1 + o) * QN + k] = j >= 0 ? cosh(P.nu[o] * t) : 0.0;
}

// Normalised Matern M(x; nu_o) for all NO orders of the p-variate model,
// x > 0 (one exponential per node for every order).
template <int NO>
__device__ __forceinline__ void matern_p(double x, const MaternArgsP &P,
                                         const double *__restrict__ sq, double M[NO]) {
  if (x > qlev_xmax(QLEV - 1)) {
#pragma unroll
    for (int o = 0; o < NO; ++o) M[o] = 0.0;
    return;
  }
  const double ex = exp(-x);
  double s[NO];
#pragma unroll
  for (int o = 0; o < NO; ++o) s[o] = 0.5;
  double logh = 0.0;
  if (P.any_quad) {
    const int j = x <= qlev_xmax(0) ? 0 : x <= qlev_xmax(1) ? 1 : x <= qlev_xmax(2) ? 2
                : x <= qlev_xmax(3) ? 3 : 4;
    const int off = qlev_off(j), cnt = qlev_cnt(j);
    logh = log(qlev_h(j));
    // nodes in pairs, the stopping test on the second of each pair
    for (int k = 1; k < cnt; k += 2) {
      const double e = exp(-x * sq[off + k]);
#pragma unroll
      for (int o = 0; o < NO; ++o) s[o] += e * sq[(1 + o) * QN + off + k];
      if (k + 1 >= cnt) break;
      const double e2 = exp(-x * sq[off + k + 1]);
      bool small = true;
#pragma unroll
      for (int o = 0; o < NO; ++o) {
        const double tt = e2 * sq[(1 + o) * QN + off + k + 1];
        s[o] += tt;
        small = small && tt <= 1e-17 * s[o];
      }
      if (small) break;
    }
  }
  const double lx = log(x);
#pragma unroll
  for (int o = 0; o < NO; ++o) {
    switch (P.closed[o]) {
      case 1: M[o] = ex; break;
      case 2: M[o] = (1.0 + x) * ex; break;
      case 3: M[o] = (1.0 + x + x * x * (1.0 / 3.0)) * ex; break;
      default: M[o] = exp(P.nu[o] * lx - x + P.lnorm[o] + logh) * s[o]; break;
    }
  }
}

}  // namespace mvg
