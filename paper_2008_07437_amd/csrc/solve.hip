// Triangular solves and products with a factored tile matrix (Eq. (1):
// L^-1 Z; Eq. (3)-(5) and Algorithm 1 of Section 5.4: L^-1 c0, Sigma^-1 c0,
// L^T w) for one or many right-hand sides, on dense FP64, mixed and TLR
// factors.
#include <algorithm>

#include "mvgeo_internal.h"
#include "tile_dev.h"
#include "tlr.h"

namespace mvg {

constexpr int VB = 64;  // rows per workgroup chunk of the per-column kernels

// ------------------------------------------------------- triangular solves
//
// Vectors are padded to Np = T nb; nrhs right-hand sides are stored column
// after column with leading dimension ldv, blockIdx.z selects the column.
// The diagonal tiles are solved with the inverses W_k kept by the
// factorisation: each step is a dense triangular matrix-vector product.

// One step is two launches on the serial chain (the tile's W_k, then its
// column), so each is cut for latency: 32 output rows (or 16 output columns
// of a transposed product) per workgroup, two rows a load, eight or more loads
// of a lane in flight, sums in a fixed order.  Before (64 rows a workgroup, a
// quarter of the columns per wave two at a time): 36 us for the tile and 19
// for the column at nb = 512 and 6 tiles, now 5 and 5; at nb = 1024 and 49 tiles
// 112 and 74 forward, 115 and 133 backward, now 9 and 40, 6 and 38 (5 TB/s over
// the column's bytes).
constexpr int SR = 32;  // output rows of a forward workgroup
constexpr int SC = 16;  // output columns of a transposed one
constexpr int SU = 8;   // loads of a lane in flight

template <class T>
struct Pair;
template <>
struct Pair<double> {
  typedef double2 type;
};
template <>
struct Pair<float> {
  typedef float2 type;
};

// sum over columns c < nc of A[r][c] x[c] for the 32 rows at A (column-major,
// ld nb); x in LDS, nc a multiple of 16.  Thread (pair p of rows, group g)
// takes columns g, g + 16, ...; the groups are added in order by the threads
// below 32, which get their row's sum.
template <class T>
__device__ __forceinline__ double rows_dot(const T *A, int nb, int nc, const double *x,
                                           double (*part)[SR]) {
  const int p = threadIdx.x & 15, g = threadIdx.x >> 4;
  const int n = nc / 16;
  double s0 = 0.0, s1 = 0.0;
  for (int i = 0; i < n; i += SU) {
    typename Pair<T>::type v[SU];
#pragma unroll
    for (int u = 0; u < SU; ++u)
      v[u] = *reinterpret_cast<const typename Pair<T>::type *>(
          A + (int64_t)(g + 16 * min(i + u, n - 1)) * nb + 2 * p);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < SU; ++u) {
      const double xc = i + u < n ? x[g + 16 * min(i + u, n - 1)] : 0.0;
      s0 = fma((double)v[u].x, xc, s0);
      s1 = fma((double)v[u].y, xc, s1);
    }
  }
  part[g][2 * p] = s0;
  part[g][2 * p + 1] = s1;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x < SR)
#pragma unroll
    for (int q = 0; q < 16; ++q) s += part[q][threadIdx.x];
  return s;
}

// sum over rows r < nr of A[r][c] x[r] for the 16 columns at A (column-major,
// ld nb); x in LDS, nr even.  A wave takes four columns, its lanes row pairs;
// every lane gets the four sums.
template <class T>
__device__ __forceinline__ void cols_dot(const T *A, int nb, int nr, const double *x, double s[4]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const T *a = A + (int64_t)(4 * w) * nb;
#pragma unroll
  for (int c = 0; c < 4; ++c) s[c] = 0.0;
  for (int r0 = 0; r0 < nr; r0 += 256) {
    typename Pair<T>::type v[2][4];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        v[u][c] = *reinterpret_cast<const typename Pair<T>::type *>(
            a + (int64_t)c * nb + min(r0 + 128 * u + 2 * lane, nr - 2));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int r = r0 + 128 * u + 2 * lane;
      const double x0 = r < nr ? x[min(r, nr - 2)] : 0.0, x1 = r < nr ? x[min(r, nr - 2) + 1] : 0.0;
#pragma unroll
      for (int c = 0; c < 4; ++c)
        s[c] = fma((double)v[u][c].y, x1, fma((double)v[u][c].x, x0, s[c]));
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1)
#pragma unroll
    for (int c = 0; c < 4; ++c) s[c] += __shfl_xor(s[c], o);
}

// y_k = W_k x_k (W_k lower triangular with its zeros stored, column-major):
// 32 output rows per workgroup.  Reads x from X, writes y to Y (out of place:
// other workgroups still read x).
__global__ __launch_bounds__(256) void k_trsv_tile_fwd(int nb, int k, const double *__restrict__ winv,
                                                       const double *__restrict__ X,
                                                       double *__restrict__ Y, int64_t ldv) {
  __shared__ double v[1024], part[16][SR];
  const int r0 = blockIdx.x * SR;
  const int64_t off = (int64_t)blockIdx.z * ldv + (int64_t)k * nb;
  const int nc = r0 + SR;  // columns that meet rows r0 .. r0 + 31
  for (int c = threadIdx.x; c < nc; c += 256) v[c] = X[off + c];
  __syncthreads();
  const double s = rows_dot(winv + (int64_t)k * nb * nb + r0, nb, nc, v, part);
  if (threadIdx.x < SR) Y[off + r0 + threadIdx.x] = s;
}

// v_i -= L_ik y_k for tiles i in (k, T), y_k read from Y: 32 rows per
// workgroup.
__global__ __launch_bounds__(256) void k_gemv_fwd(TileMap M, int k, double *__restrict__ V,
                                                 const double *__restrict__ Y, int64_t ldv) {
  __shared__ double y[1024], part[16][SR];
  const int nb = M.nb, chunks = nb / SR;
  const int i = k + 1 + blockIdx.x / chunks, r0 = (blockIdx.x % chunks) * SR;
  const int64_t off = (int64_t)blockIdx.z * ldv;
  for (int c = threadIdx.x; c < nb; c += 256) y[c] = Y[off + (int64_t)k * nb + c];
  __syncthreads();
  const double s = tile_is_f32(M, i, k)  // mixed precision: off-band tiles in FP32
                       ? rows_dot(tile_ptr_f32(M, i, k) + r0, nb, nb, y, part)
                       : rows_dot(tile_ptr(M, i, k) + r0, nb, nb, y, part);
  if (threadIdx.x < SR) V[off + (int64_t)i * nb + r0 + threadIdx.x] -= s;
}

// y_k = W_k^T x_k: 16 outputs per workgroup, rows from the outputs' own 64-row
// block on (zeros above the diagonal are stored).  Out of place.
__global__ __launch_bounds__(256) void k_trsv_tile_bwd(int nb, int k, const double *__restrict__ winv,
                                                       const double *__restrict__ X,
                                                       double *__restrict__ Y, int64_t ldv) {
  __shared__ double v[1024];
  const int c0 = blockIdx.x * SC, rb = c0 / 64 * 64;
  const int64_t off = (int64_t)blockIdx.z * ldv + (int64_t)k * nb;
  for (int r = threadIdx.x; r < nb - rb; r += 256) v[r] = X[off + rb + r];
  __syncthreads();
  double s[4];
  cols_dot(winv + (int64_t)k * nb * nb + (int64_t)c0 * nb + rb, nb, nb - rb, v, s);
  const int lane = threadIdx.x & 63;
  const double o = lane == 0 ? s[0] : lane == 1 ? s[1] : lane == 2 ? s[2] : s[3];
  if (lane < 4) Y[off + c0 + 4 * (threadIdx.x >> 6) + lane] = o;
}

// v_j -= L_kj^T w_k for tiles j in [0, k), w_k read from Y: 16 columns per
// workgroup.
__global__ __launch_bounds__(256) void k_gemv_bwd(TileMap M, int k, double *__restrict__ V,
                                                 const double *__restrict__ Y, int64_t ldv) {
  __shared__ double w[1024];
  const int nb = M.nb, cb = nb / SC;
  const int j = blockIdx.x / cb, c0 = (blockIdx.x % cb) * SC;
  const int64_t off = (int64_t)blockIdx.z * ldv;
  for (int r = threadIdx.x; r < nb; r += 256) w[r] = Y[off + (int64_t)k * nb + r];
  __syncthreads();
  double s[4];
  if (tile_is_f32(M, k, j)) cols_dot(tile_ptr_f32(M, k, j) + (int64_t)c0 * nb, nb, nb, w, s);
  else cols_dot(tile_ptr(M, k, j) + (int64_t)c0 * nb, nb, nb, w, s);
  const int lane = threadIdx.x & 63;
  const double o = lane == 0 ? s[0] : lane == 1 ? s[1] : lane == 2 ? s[2] : s[3];
  if (lane < 4) V[off + (int64_t)j * nb + c0 + 4 * (threadIdx.x >> 6) + lane] -= o;
}

// Scratch of the per-column solves: the solved tiles (Np x nrhs).
static int solve_scratch(const mvg_mat *A, int nrhs, double **Y, hipStream_t st) {
  if (malloc_async((void **)Y, sizeof(double) * A->Np * nrhs, st) != hipSuccess) {
    hipGetLastError();
    set_error("solve workspace of %.3f GB failed", A->Np * nrhs * 8.0 / 1e9);
    return MVG_ERR_ALLOC;
  }
  return 0;
}

// Copy the solution back into V and release the scratch.
static int solve_finish(const mvg_mat *A, double *V, double *Y, int nrhs, int rc, hipStream_t st) {
  if (!rc && hipMemcpyAsync(V, Y, sizeof(double) * A->Np * nrhs, hipMemcpyDeviceToDevice, st) !=
                 hipSuccess)
    rc = MVG_ERR_LAUNCH;
  hipFreeAsync(Y, st);
  return rc;
}

static int solve_args_ok(const mvg_mat *A) {
  if (A->nb > 1024 || A->nb % VB || !A->d_winv) {
    set_error("triangular solve needs nb <= 1024, nb %% 64 == 0 and a factored matrix");
    return MVG_ERR_STATE;
  }
  return 0;
}

// Right-hand sides go in gridDim.z, at most 65535 per launch.
constexpr int MAX_RHS_LAUNCH = 65535;

// Many right-hand sides on an FP64 factor: the tile steps become GEMMs on
// FP64 MFMA (one pass over L for all columns instead of one per column).
//   forward  L X = B:   Y_k = W_k X_k,   X_i -= L_ik Y_k  (i > k)
//   backward L^T X = B: Y_k = W_k^T X_k, X_j -= L_kj^T Y_k (j < k)
//   product  Y = L^T X: Y_J = sum_{I >= J} L_IJ^T X_I, one launch per
//                       tile diagonal d = I - J (distinct outputs per task)
// Y (Np x nrhs) is the solution of the solves, copied back into X.
constexpr int GEMM_RHS_MIN = 4;
enum { TS_FORWARD = 0, TS_BACKWARD = 1, TS_TRMM_T = 2 };

static bool gemm_solve_ok(const mvg_mat *A, int nrhs) {
  return (A->precision == MVG_FP64 || A->precision == MVG_DST) && !A->tlr && A->h_off &&
         nrhs >= GEMM_RHS_MIN;
}

static int tile_gemm_solve(const mvg_mat *A, double *X, double *Y, int nrhs, int mode,
                           hipStream_t st) {
  const int T = A->T, nb = A->nb;
  const int ld = (int)A->Np;
  auto L = [&](int I, int J) {
    return (const double *)(A->arena + A->h_off[tidx(I, J, T)]);
  };
  auto W = [&](int k) { return (const double *)A->d_winv + (int64_t)k * nb * nb; };
  auto zero = [&](int I, int J) { return A->h_kind && A->h_kind[tidx(I, J, T)] == TK_ZERO; };
  auto task = [&](const double *a, int ta, int tri, const double *b, double *c, double alpha,
                  double beta) {
    return GemmTask{a, b, c, nb, nrhs, nb, nb, ld, ld, ta, 0, alpha, beta, tri};
  };
  // every launch: a segment of one task list (starts relative to the segment)
  std::vector<GemmTask> tasks;
  std::vector<int64_t> start;
  std::vector<int> seg;          // first task of each launch
  std::vector<int64_t> blocks;   // blocks of each launch
  auto close = [&](size_t first) {
    int64_t nbk = 0;
    for (size_t i = first; i < tasks.size(); ++i) {
      start.push_back(nbk);
      nbk += gemm_blocks(tasks[i]);
    }
    seg.push_back((int)first);
    blocks.push_back(nbk);
  };
  const int64_t tstride = (int64_t)nb;
  if (mode == TS_FORWARD) {
    for (int k = 0; k < T; ++k) {
      size_t f = tasks.size();
      tasks.push_back(task(W(k), 0, 1, X + k * tstride, Y + k * tstride, 1.0, 0.0));
      close(f);
      if (k + 1 < T) {
        f = tasks.size();
        for (int i = k + 1; i < T; ++i)
          if (!zero(i, k))
            tasks.push_back(task(L(i, k), 0, 0, Y + k * tstride, X + i * tstride, -1.0, 1.0));
        close(f);
      }
    }
  } else if (mode == TS_BACKWARD) {
    for (int k = T - 1; k >= 0; --k) {
      size_t f = tasks.size();
      tasks.push_back(task(W(k), 1, 1, X + k * tstride, Y + k * tstride, 1.0, 0.0));
      close(f);
      if (k > 0) {
        f = tasks.size();
        for (int j = 0; j < k; ++j)
          if (!zero(k, j))
            tasks.push_back(task(L(k, j), 1, 0, Y + k * tstride, X + j * tstride, -1.0, 1.0));
        close(f);
      }
    }
  } else {
    for (int d = 0; d < T; ++d) {
      const size_t f = tasks.size();
      for (int J = 0; J + d < T; ++J)
        if (d == 0 || !zero(J + d, J))
          tasks.push_back(task(L(J + d, J), 1, d == 0, X + (J + d) * tstride, Y + J * tstride,
                               1.0, d == 0 ? 0.0 : 1.0));
      close(f);
    }
  }
  HostLists H;
  int rc = 0;
  const GemmTask *dt =
      (const GemmTask *)H.stage(tasks.data(), tasks.size() * sizeof(GemmTask), st, &rc);
  const int64_t *ds = (const int64_t *)H.stage(start.data(), start.size() * 8, st, &rc);
  for (size_t s = 0; !rc && s < seg.size(); ++s) {
    const int n = (int)((s + 1 < seg.size() ? seg[s + 1] : (int)tasks.size()) - seg[s]);
    rc = launch_gemm_batched(dt + seg[s], ds + seg[s], n, blocks[s], st);
  }
  if (!rc && mode != TS_TRMM_T &&
      hipMemcpyAsync(X, Y, sizeof(double) * A->Np * nrhs, hipMemcpyDeviceToDevice, st) !=
          hipSuccess)
    rc = MVG_ERR_LAUNCH;
  H.release(st);
  return rc;
}

static int gemm_solve_inplace(const mvg_mat *A, double *d_V, int nrhs, int mode, hipStream_t st) {
  double *Y = nullptr;
  if (malloc_async((void **)&Y, sizeof(double) * A->Np * nrhs, st) != hipSuccess) {
    hipGetLastError();
    set_error("solve workspace of %.2f GB failed", A->Np * nrhs * 8.0 / 1e9);
    return MVG_ERR_ALLOC;
  }
  const int rc = tile_gemm_solve(A, d_V, Y, nrhs, mode, st);
  hipFreeAsync(Y, st);
  return rc;
}

int trsm_forward_multi(const mvg_mat *A, double *d_V, int nrhs, hipStream_t st) {
  if (A->tlr) return tlr_trsm_forward(A, d_V, nrhs, A->Np, st);
  if (int rc = solve_args_ok(A)) return rc;
  if (gemm_solve_ok(A, nrhs)) return gemm_solve_inplace(A, d_V, nrhs, TS_FORWARD, st);
  if (nrhs > MAX_RHS_LAUNCH) {
    for (int c = 0; c < nrhs; c += MAX_RHS_LAUNCH)
      if (int rc = trsm_forward_multi(A, d_V + (int64_t)c * A->Np, std::min(MAX_RHS_LAUNCH, nrhs - c),
                                      st))
        return rc;
    return 0;
  }
  // solved tiles go to Y (the tile solve is out of place), the updates to V;
  // Y is copied back at the end
  double *Y = nullptr;
  if (int rc = solve_scratch(A, nrhs, &Y, st)) return rc;
  const TileMap M = A->map();
  const int chunks = M.nb / SR;
  int rc = 0;
  for (int k = 0; k < M.T && !rc; ++k) {
    hipLaunchKernelGGL(k_trsv_tile_fwd, dim3(chunks, 1, nrhs), dim3(256), 0, st, M.nb, k,
                       (const double *)A->d_winv, (const double *)d_V, Y, A->Np);
    rc = check_launch("trsv_tile_fwd");
    if (!rc && k + 1 < M.T) {
      hipLaunchKernelGGL(k_gemv_fwd, dim3((M.T - k - 1) * chunks, 1, nrhs), dim3(256), 0, st, M, k,
                         d_V, (const double *)Y, A->Np);
      rc = check_launch("gemv_fwd");
    }
  }
  return solve_finish(A, d_V, Y, nrhs, rc, st);
}

int trsv_forward(const mvg_mat *A, double *d_v, hipStream_t st) {
  return trsm_forward_multi(A, d_v, 1, st);
}

int trsm_backward_multi(const mvg_mat *A, double *d_V, int nrhs, hipStream_t st) {
  if (A->tlr) {
    for (int c = 0; c < nrhs; ++c)
      if (int rc = tlr_trsv_backward(A, d_V + (int64_t)c * A->Np, st)) return rc;
    return 0;
  }
  if (int rc = solve_args_ok(A)) return rc;
  if (gemm_solve_ok(A, nrhs)) return gemm_solve_inplace(A, d_V, nrhs, TS_BACKWARD, st);
  if (nrhs > MAX_RHS_LAUNCH) {
    for (int c = 0; c < nrhs; c += MAX_RHS_LAUNCH)
      if (int rc = trsm_backward_multi(A, d_V + (int64_t)c * A->Np,
                                       std::min(MAX_RHS_LAUNCH, nrhs - c), st))
        return rc;
    return 0;
  }
  double *Y = nullptr;
  if (int rc = solve_scratch(A, nrhs, &Y, st)) return rc;
  const TileMap M = A->map();
  const int nb = M.nb;
  int rc = 0;
  for (int k = M.T - 1; k >= 0 && !rc; --k) {
    hipLaunchKernelGGL(k_trsv_tile_bwd, dim3(nb / SC, 1, nrhs), dim3(256), 0, st, nb, k,
                       (const double *)A->d_winv, (const double *)d_V, Y, A->Np);
    rc = check_launch("trsv_tile_bwd");
    if (!rc && k > 0) {
      hipLaunchKernelGGL(k_gemv_bwd, dim3(k * (nb / SC), 1, nrhs), dim3(256), 0, st, M, k, d_V,
                         (const double *)Y, A->Np);
      rc = check_launch("gemv_bwd");
    }
  }
  return solve_finish(A, d_V, Y, nrhs, rc, st);
}

int trsv_backward(const mvg_mat *A, double *d_v, hipStream_t st) {
  return trsm_backward_multi(A, d_v, 1, st);
}

// Y = L^T X for nrhs columns (ld Np), L the factor's lower tiles: output tile
// J, column c: sum_{I >= J} sum_r L_IJ[r][c] X_I[r] (rows r >= c in the
// diagonal tile).  One workgroup per (J, 64 output columns, right-hand side),
// one wave per output column at a time, lanes over rows; fixed order.
__global__ __launch_bounds__(256) void k_trmm_t(TileMap M, const double *__restrict__ X,
                                                double *__restrict__ Y, int64_t ldv) {
  const int nb = M.nb, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int cb = nb / 64;
  const int J = blockIdx.x / cb;
  const int c0 = (blockIdx.x % cb) * 64;
  const double *Xc = X + (int64_t)blockIdx.z * ldv;
  double *Yc = Y + (int64_t)blockIdx.z * ldv;
  const bool f32 = M.kind != nullptr;
  for (int c = c0 + wave; c < c0 + 64; c += 4) {
    double s = 0.0;
    for (int I = J; I < M.T; ++I) {
      const double *x = Xc + (int64_t)I * nb;
      const int r0 = (I == J) ? c : 0;
      if (f32 && tile_is_f32(M, I, J)) {
        const float *col = tile_ptr_f32(M, I, J) + (int64_t)c * nb;
        for (int r = r0 + lane; r < nb; r += 64) s += (double)col[r] * x[r];
      } else {
        const double *col = tile_ptr(M, I, J) + (int64_t)c * nb;
        for (int r = r0 + lane; r < nb; r += 64) s += col[r] * x[r];
      }
    }
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (lane == 0) Yc[(int64_t)J * nb + c] = s;
  }
}

int launch_trmm_t(const mvg_mat *A, const double *d_X, double *d_Y, int nrhs, hipStream_t st) {
  if (A->tlr) {
    set_error("L^T products are not available for TLR factors");
    return MVG_ERR_STATE;
  }
  if (int rc = solve_args_ok(A)) return rc;
  if (gemm_solve_ok(A, nrhs))
    return tile_gemm_solve(A, const_cast<double *>(d_X), d_Y, nrhs, TS_TRMM_T, st);
  const TileMap M = A->map();
  for (int c = 0; c < nrhs; c += MAX_RHS_LAUNCH) {
    const int64_t off = (int64_t)c * A->Np;
    hipLaunchKernelGGL(k_trmm_t, dim3(M.T * (M.nb / 64), 1, std::min(MAX_RHS_LAUNCH, nrhs - c)),
                       dim3(256), 0, st, M, d_X + off, d_Y + off, A->Np);
    if (int rc = check_launch("trmm_t")) return rc;
  }
  return 0;
}

// out[c] = sum_i A[c Np + i] B[c Np + i] for ncols columns (fixed order)
__global__ __launch_bounds__(256) void k_dot_cols(const double *__restrict__ A,
                                                  const double *__restrict__ B, int64_t Np,
                                                  double *__restrict__ out) {
  __shared__ double r[256];
  const double *a = A + (int64_t)blockIdx.x * Np, *b = B + (int64_t)blockIdx.x * Np;
  double s = 0.0;
  for (int64_t i = threadIdx.x; i < Np; i += 256) s += a[i] * b[i];
  r[threadIdx.x] = s;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if (threadIdx.x < k) r[threadIdx.x] += r[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[blockIdx.x] = r[0];
}

int launch_dot_cols(const double *d_A, const double *d_B, int64_t Np, int ncols, double *d_out,
                    hipStream_t st) {
  hipLaunchKernelGGL(k_dot_cols, dim3(ncols), dim3(256), 0, st, d_A, d_B, Np, d_out);
  return check_launch("dot_cols");
}

// z = L eps: 32 rows by up to TRMV_COLS columns (whole tiles) per workgroup,
// part[chunk][row], then the chunks added in order, TRMV_CHUNKS at a time: the
// workspace is at most that many vectors (all 47 of 48,000 rows at once: 1.59
// ms, 32: 1.60; 16 cost 4 % at 18,000), and the sums are the same for any
// number.  The diagonal tile's upper part is scratch and not used.  Bound by the
// factor's bytes; one thread per row before: 1.5 ms at 2n = 6,400, now 0.03.
constexpr int TRMV_COLS = 1024, TRMV_CHUNKS = 32;

// (chunks from c0 on; row tiles from the first that they reach)
__global__ __launch_bounds__(256) void k_trmv_part(TileMap M, const double *__restrict__ eps,
                                                   double *__restrict__ out, int64_t Np, int c0) {
  __shared__ double x[1024], part[16][SR];
  const int nb = M.nb, chunks = nb / SR, per = max(1, TRMV_COLS / nb);
  const int I = c0 * per + blockIdx.x / chunks, r0 = (blockIdx.x % chunks) * SR;
  const int J0 = (c0 + blockIdx.y) * per, J1 = min(I + 1, J0 + per);
  if (J0 > I) return;
  const int p = threadIdx.x & 15, g = threadIdx.x >> 4;
  double s = 0.0;
  for (int J = J0; J < J1; ++J) {
    const double *A = tile_ptr(M, I, J) + r0;
    const int nc = J < I ? nb : r0;
    __syncthreads();  // the last tile's x and partial sums are used up
    for (int c = threadIdx.x; c < nb; c += 256) x[c] = eps[(int64_t)J * nb + c];
    __syncthreads();
    if (nc > 0) s += rows_dot(A, nb, nc, x, part);
    if (J == I) {  // the 32 x 32 block on the diagonal, c <= r
      double s0 = 0.0, s1 = 0.0;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int c = g + 16 * u;
        const double2 v = *reinterpret_cast<const double2 *>(A + (int64_t)(r0 + c) * nb + 2 * p);
        s0 = fma(c <= 2 * p ? v.x : 0.0, x[r0 + c], s0);
        s1 = fma(c <= 2 * p + 1 ? v.y : 0.0, x[r0 + c], s1);
      }
      __syncthreads();
      part[g][2 * p] = s0;
      part[g][2 * p + 1] = s1;
      __syncthreads();
      if (threadIdx.x < SR)
#pragma unroll
        for (int q = 0; q < 16; ++q) s += part[q][threadIdx.x];
    }
  }
  if (threadIdx.x < SR)
    out[(int64_t)blockIdx.y * Np + (int64_t)I * nb + r0 + threadIdx.x] = s;
}

// the rows of tile rows c0 per .. on: chunks c0 .. c0 + nc - 1 added to z
__global__ void k_trmv_sum(const double *__restrict__ part, int64_t Np, int nb, int64_t N, int c0,
                           int nc, double *__restrict__ z) {
  const int per = max(1, TRMV_COLS / nb);
  const int64_t g = (int64_t)c0 * per * nb + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= N) return;
  const int n = min(nc, (int)(g / nb) / per + 1 - c0);
  double s = c0 > 0 ? z[g] : 0.0;
  for (int c = 0; c < n; ++c) s += part[c * Np + g];
  z[g] = s;
}

int launch_trmv(const mvg_mat *A, const double *d_eps, double *d_z, hipStream_t st) {
  // eps is read up to the padded length: a zero-padded copy, then the parts
  const int nb = A->nb, per = std::max(1, TRMV_COLS / nb), chunks = (A->T + per - 1) / per;
  double *ep = nullptr;
  if (malloc_async((void **)&ep, sizeof(double) * A->Np * (1 + std::min(chunks, TRMV_CHUNKS)), st) !=
      hipSuccess) {
    hipGetLastError();
    set_error("trmv workspace allocation failed");
    return MVG_ERR_ALLOC;
  }
  double *part = ep + A->Np;
  int rc = launch_fill_f64(ep, 0.0, A->Np, st);
  if (!rc) hipMemcpyAsync(ep, d_eps, sizeof(double) * A->N, hipMemcpyDeviceToDevice, st);
  for (int c0 = 0; c0 < chunks && !rc; c0 += TRMV_CHUNKS) {
    const int nc = std::min(TRMV_CHUNKS, chunks - c0);
    hipLaunchKernelGGL(k_trmv_part, dim3((A->T - c0 * per) * (nb / SR), nc), dim3(256), 0, st,
                       A->map(), (const double *)ep, part, A->Np, c0);
    const int64_t rows = A->N - (int64_t)c0 * per * nb;
    hipLaunchKernelGGL(k_trmv_sum, dim3((unsigned)((rows + 255) / 256)), dim3(256), 0, st,
                       (const double *)part, A->Np, nb, A->N, c0, nc, d_z);
    rc = check_launch("trmv");
  }
  hipFreeAsync(ep, st);
  return rc;
}

}  // namespace mvg
