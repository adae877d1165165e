// Many small likelihoods at once (Eq. 1 per task).
//
// Each task is one (dataset, theta) pair with 2n <= SMALL_MAX rows, padded to
// 64-row blocks (identity).  All tasks of a group advance together, one
// launch per 64 columns: a launch gives every task the workgroups of its step
// (several per task, so that a few tasks fill the chip as well as many do),
// and what a workgroup reads was finished by the launch before.  Left-looking
// by 64-block columns, so that a block of L is read, not read and written,
// once per later column:
//
//   launch t:  rows R > t + 1:  L(R, t) = (A(R, t) - sum_{m<t} L(R, m) L(t, m)^T)
//                                         W(t, t)^T
//              row t + 1:       the same; its sums over m < t - 1 were formed
//                               ahead by the launch before, so the serial chain
//                               (row, diagonal block, 64 x 64 factor) has the
//                               same length at every step
//              ahead:           A(t+2, t+1) and A(t+2, t+2) -= their sums over m < t
//
// The forward solve rides along (v_R -= L(R, t) y_t beside each row block) and
// a last launch per task sums the log-determinant and the quadratic form in a
// fixed order.  A task's arithmetic depends on its own data alone, so results
// are the same alone and in any batch.
//
// Bound by the FP64 matrix units and, with few tasks, by the chain of steps.
// Measured against one workgroup per task in a persistent launch: 1024 theta
// at n = 400 12.7 -> 7.5 ms (1.3 of it generation, 6.0 the steps, with the matrix
// units 51 % busy, 17 GB read and 4 written), 192 tasks of n = 20..512 7.3 -> 1.8
// ms (the largest task's latency on its one workgroup had set it).
#include <algorithm>
#include <cmath>

#include "chol_dev.h"
#include "matern_dev.h"

namespace mvg {

constexpr int SMALL_GROUP = 1024;  // tasks that advance together at most

__host__ __device__ inline int small_blocks(int64_t n) { return (int)((2 * n + CB - 1) / CB); }

// One task's workspace, sized by its own n (at SmallTask::ws): lower 64 x 64 blocks of the matrix (column-major
// inside, rows of blocks one after another), inverses of the diagonal blocks,
// right-hand side, solution, quadrature table, pivot info.
struct SmallSlot {
  double *base;
  int nk;
  __device__ SmallSlot(double *ws, const SmallTask &t) : base(ws + t.ws), nk(small_blocks(t.n)) {}
  __device__ double *blk(int R, int C) const { return base + (int64_t)(R * (R + 1) / 2 + C) * CB * CB; }
  __device__ double *inv(int k) const {
    return base + (int64_t)(nk * (nk + 1) / 2 + k) * CB * CB;
  }
  __device__ double *v() const { return inv(nk); }
  __device__ double *y() const { return v() + CB * nk; }
  __device__ double *qtab() const { return y() + CB * nk; }
  __device__ int64_t *info() const { return reinterpret_cast<int64_t *>(qtab() + QTAB); }
};

size_t small_workspace_doubles(int64_t n) {
  const size_t k = small_blocks(n);
  return (k * (k + 1) / 2 + k) * CB * CB + 2 * CB * k + QTAB + 32;
}

size_t small_layout(SmallTask *tasks, int ntask, size_t limit) {
  size_t most = 0, used = 0;
  for (int i = 0, first = 0; i < ntask; ++i) {
    const size_t w = small_workspace_doubles(tasks[i].n);
    if (i > first && (used + w > limit || i - first == SMALL_GROUP)) {
      first = i;
      used = 0;
    }
    tasks[i].ws = (int64_t)used;
    used += w;
    most = std::max(most, used);
  }
  return most;
}

// Workgroup index b of a list of ntask x per workgroups, the tasks dealt to
// the XCDs (workgroups go to them round robin), so that a task's workgroups
// share one L2.
__device__ __forceinline__ bool task_of(int b, int ntask, int per, int &task, int &item) {
  const int q = b >> 3;
  task = q / per * 8 + (b & 7);
  item = q % per;
  return task < ntask;
}

__global__ __launch_bounds__(256) void k_small_prep(const SmallTask *__restrict__ tasks, double *ws,
                                                    int groups) {
  const int task = blockIdx.x / groups, grp = blockIdx.x % groups;
  const SmallTask &tk = tasks[task];
  const SmallSlot s(ws, tk);
  if (grp > 0 && !tk.P.table) return;
  theta_tables(grp, tk.P, s.qtab());
  if (grp > 0) return;
  const int N = 2 * (int)tk.n;
  for (int i = threadIdx.x; i < CB * s.nk; i += 256) s.v()[i] = i < N ? tk.z[i] : 0.0;
  if (threadIdx.x == 0) *s.info() = INT64_MAX;
}

// Workgroups of a task in k_small_cov: one per 64 x 64 block where the task's
// polynomials are used; else (few locations, or closed orders) one per 256
// pairs l >= r, so that no thread is spent on padding or on the upper half.
__host__ __device__ inline int small_cov_items(int64_t n, bool table) {
  const int nk = small_blocks(n);
  return table ? nk * (nk + 1) / 2 : (int)((n * (n + 1) / 2 + 255) / 256);
}

// Sigma's 2 x 2 block of the pair (l, r) into its 64 x 64 block.
__device__ __forceinline__ void small_put(const SmallSlot &s, int l, int r, const double c[3]) {
  double *B = s.blk(l / 32, r / 32) + (2 * (r % 32)) * CB + 2 * (l % 32);
  *reinterpret_cast<double2 *>(B) = make_double2(c[0], c[2]);
  *reinterpret_cast<double2 *>(B + CB) = make_double2(c[2], c[1]);
}

// Pair q of the n (n + 1) / 2 pairs l >= r: columns r and n - 1 - r together
// hold n + 1 pairs, one folded row of them.
template <int FORM>
__device__ __forceinline__ void small_pairs(const SmallTask &tk, const SmallSlot &s, int item,
                                            double *ct) {
  const int n = (int)tk.n, q = item * 256 + threadIdx.x;
  load_cov_table<FORM>(s.qtab(), ct);
  if (q < n * (n + 1) / 2) {
    const int fi = q / (n + 1), fc = q % (n + 1);
    const bool first = fc < n - fi;
    const int r = first ? fi : n - 1 - fi, l = first ? fi + fc : r + (fc - (n - fi));
    double c[3];
    cross_cov_block<FORM>(tk.x[l], tk.y[l], tk.x[r], tk.y[r], tk.P, ct, s.qtab(), c);
    small_put(s, l, r, c);
  }
  // padding locations n .. 32 nk - 1: unit diagonal, zeros before it
  const int pad = 32 * s.nk - n, items = small_cov_items(n, false);
  for (int i = q; i < pad * 32 * s.nk; i += 256 * items) {
    const int l = n + i / (32 * s.nk), r = i % (32 * s.nk);
    const double d = l == r ? 1.0 : 0.0, c[3] = {d, d, 0.0};
    if (r <= l) small_put(s, l, r, c);
  }
}

__global__ __launch_bounds__(256) void k_small_cov(const SmallTask *__restrict__ tasks, int ntask,
                                                   double *ws, int per) {
  __shared__ double ct[CT_SIZE];
  int task, item;
  if (!task_of(blockIdx.x, ntask, per, task, item)) return;
  const SmallTask &tk = tasks[task];
  const SmallSlot s(ws, tk);
  if (item >= small_cov_items(tk.n, tk.P.table)) return;
  if (!tk.P.table) {
    if (tk.P.any_quad) small_pairs<COV_QUAD>(tk, s, item, ct);
    else small_pairs<COV_CLOSED>(tk, s, item, ct);
    return;
  }
  const MaternArgs P = tk.P;
  load_cov_table<COV_TABLE>(s.qtab(), ct);
  int R = (int)((sqrtf(8.0f * (float)item + 1.0f) - 1.0f) * 0.5f);
  while ((R + 1) * (R + 2) / 2 <= item) ++R;
  while (R * (R + 1) / 2 > item) --R;
  const int C = item - R * (R + 1) / 2, n = (int)tk.n;
  const int pl = threadIdx.x & 31, gl = 32 * R + pl;
  const double xl = gl < n ? tk.x[gl] : 0.0, yl = gl < n ? tk.y[gl] : 0.0;
  double *B = s.blk(R, C) + 2 * pl;
  for (int q = 0; q < 4; ++q) {
    const int pr = (threadIdx.x >> 5) * 4 + q, gr = 32 * C + pr;
    double c[3];
    if (gl >= n || gr >= n) {
      c[0] = c[1] = gl == gr ? 1.0 : 0.0;
      c[2] = 0.0;
    } else {
      cross_cov_block<COV_TABLE>(xl, yl, tk.x[gr], tk.y[gr], P, ct, s.qtab(), c);
    }
    *reinterpret_cast<double2 *>(B + 2 * pr * CB) = make_double2(c[0], c[2]);
    *reinterpret_cast<double2 *>(B + (2 * pr + 1) * CB) = make_double2(c[2], c[1]);
  }
}

// acc (16 rows of block row R per wave, row layout) -= sum_{m<nm} L(R, m)
// L(C, m)^T: the C blocks go through LDS, two in turn, one barrier each, the
// next pair of blocks in flight under the products.
__device__ __forceinline__ void left_sum(Rows &acc, const double *LR, const double *LC, int nm,
                                         double *sm) {
  if (nm <= 0) return;
  double v[16];
  Rows a;
  block_load(LC, CB, v);
  rows_load(LR, CB, a);
  for (int m = 0; m < nm; ++m) {
    double *b = sm + (m & 1) * CB * CB;
    const Rows c = a;
    block_store(b, v);
    __syncthreads();
    const int64_t nx = (int64_t)min(m + 1, nm - 1) * CB * CB;
    block_load(LC + nx, CB, v);
    rows_load(LR + nx, CB, a);
    rows_sub_nt(acc, c, b, 4);
  }
}

// Log-determinant, quadratic form and Eq. (1) of a factored task.
__device__ __forceinline__ void small_finish(const SmallSlot &s, int n, double *sm, double *o) {
  const int tid = threadIdx.x, last = s.nk - 1;
  double *part = sm + 2 * CB * CB, *r0 = sm, *r1 = sm + 256;
  double v[16];
  block_load(s.inv(last), CB, v);
  block_store(sm, v);
  __syncthreads();
  solve_parts(sm, s.v() + CB * last, part);
  __syncthreads();
  double ld = 0.0, q = 0.0;
  for (int i = tid; i < CB * s.nk; i += 256) {
    const int k = i / CB, r = i % CB;
    const double y = k == last ? solve_y(part, r) : s.y()[i];
    ld += log(s.blk(k, k)[r * CB + r]);  // padding rows: log 1, y = 0
    q += y * y;
  }
  r0[tid] = ld;
  r1[tid] = q;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (tid < h) {
      r0[tid] += r0[tid + h];
      r1[tid] += r1[tid + h];
    }
    __syncthreads();
  }
  if (tid == 0) {
    const int64_t fail = *s.info();
    const double logdet = 2.0 * r0[0], quad = r1[0];
    const bool ok = fail == INT64_MAX;
    o[0] = ok ? -(double)n * log(2.0 * M_PI) - 0.5 * logdet - 0.5 * quad : -INFINITY;
    o[1] = ok ? logdet : NAN;
    o[2] = ok ? quad : NAN;
    o[3] = ok ? 0.0 : (double)fail;
  }
}

// Step t of every task: first each task's row t + 1 (the serial chain) or, at
// its end, its sums; then the other rows and the two blocks ahead.
__global__ __launch_bounds__(256, 2) void k_small_step(const SmallTask *__restrict__ tasks, int ntask,
                                                       double *ws, int t, int per,
                                                       double *__restrict__ out) {
  __shared__ double sm[CHOL_LDS];
  int b = blockIdx.x;
  if (b < ntask) {
    const SmallTask &tk = tasks[b];
    const SmallSlot s(ws, tk);
    if (t + 1 < s.nk) {
      RowStep r{};
      r.ld = r.ldw = CB;
      r.S = s.blk(t + 1, t + 1);
      r.Wn = s.inv(t + 1);
      if (t >= 0) {
        r.A1 = s.blk(t + 1, t);
        r.Wt = s.inv(t);
        r.vt = s.v() + CB * t;
        r.vr = s.v() + CB * (t + 1);
        r.yt = s.y() + CB * t;
        if (t > 0) {
          r.P1 = s.blk(t + 1, t - 1);
          r.P0 = s.blk(t, t - 1);
        }
      }
      PivotRule pr{};
      pr.tol[0] = tk.t0;
      pr.tol[1] = tk.t1;
      pr.p = 2;
      pr.plim = 2 * tk.n;
      row_step<true, true>(r, sm, (int64_t)(t + 1) * CB, pr, s.info());
    } else if (t + 1 == s.nk) {
      small_finish(s, (int)tk.n, sm, out + 4 * (int64_t)b);
    }
    return;
  }
  int task, item;
  if (!task_of(b - ntask, ntask, per, task, item)) return;
  const SmallSlot s(ws, tasks[task]);
  if (item < 2) {  // ahead: (t + 2, t + 1), (t + 2, t + 2)
    const int R = t + 2, C = t + 1 + item;
    if (R >= s.nk || t < 1) return;
    Rows acc;
    rows_load(s.blk(R, C), CB, acc);
    left_sum(acc, s.blk(R, 0), s.blk(C, 0), t, sm);
    rows_store(s.blk(R, C), CB, acc);
    return;
  }
  const int R = t + item;  // rows t + 2 on
  if (R >= s.nk) return;
  Rows acc, x;
  double v[16];
  double *w = sm + (t & 1) * CB * CB, *part = sm + 2 * CB * CB;
  rows_load(s.blk(R, t), CB, acc);
  block_load(s.inv(t), CB, v);  // in flight under the sum
  left_sum(acc, s.blk(R, 0), s.blk(t, 0), t, sm);
  block_store(w, v);  // the buffer that the last product did not read
  __syncthreads();
  solve_parts(w, s.v() + CB * t, part);
  rows_mul_wt(x, acc, w);
  rows_store(s.blk(R, t), CB, x);
  __syncthreads();
  solve_rows(x, part, part + 16 * CT + (threadIdx.x >> 6) * CB, s.v() + CB * R);
}

int launch_small_loglik(const SmallTask *d_tasks, const SmallTask *h_tasks, int ntask, double *d_ws,
                        double *d_out, hipStream_t st) {
  for (int g = 0, cnt = 0; g < ntask; g += cnt) {
    for (cnt = 1; g + cnt < ntask && h_tasks[g + cnt].ws > 0;) ++cnt;
    const int cnt8 = (cnt + 7) / 8 * 8;
    const SmallTask *tk = d_tasks + g;
    int64_t big = 1;
    int per = 1, tables = 0;
    for (int i = 0; i < cnt; ++i) {
      const SmallTask &t = h_tasks[g + i];
      big = std::max(big, t.n);
      per = std::max(per, small_cov_items(t.n, t.P.table));
      tables |= t.P.table;
    }
    if (2 * big > SMALL_MAX) {
      set_error("batched small likelihood: 2n = %lld above %d", (long long)(2 * big), SMALL_MAX);
      return MVG_ERR_LIMIT;
    }
    const int nk = small_blocks(big), groups = tables ? (CT_HI - CT_LO) / CT_GROUP : 1;
    hipLaunchKernelGGL(k_small_prep, dim3(cnt * groups), dim3(256), 0, st, tk, d_ws, groups);
    hipLaunchKernelGGL(k_small_cov, dim3(cnt8 * per), dim3(256), 0, st, tk, cnt, d_ws, per);
    if (int rc = check_launch("small_cov")) return rc;
    for (int t = -1; t < nk; ++t) {
      const int rows = t < 0 ? 0 : std::max(0, nk - (t + 2));  // rows R >= t + 2
      const int p = rows ? rows + 2 : 0;
      hipLaunchKernelGGL(k_small_step, dim3(cnt + cnt8 * p), dim3(256), 0, st, tk, cnt, d_ws, t,
                         std::max(1, p), d_out + 4 * (int64_t)g);
      if (int rc = check_launch("small_step")) return rc;
    }
  }
  return 0;
}

}  // namespace mvg
