// Vector, sparse and reduction kernels of the IPM (gfx950): row jobs with A, A'
// and P (residuals, eq. residuals-objectives; KKT products), fused axpys,
// ordered block reductions, and the assembly of the KKT Schur complement.
#include "hc_vec.h"

#include <cmath>

namespace hc {

// max that propagates NaN (a NaN residual must never pass a test)
__device__ inline double nmax(double a, double b) { return (a != a || b != b) ? NAN : (a > b ? a : b); }

// lanes per row of a sparse product, from the mean row length
int choose_lanes(double mean_nnz) {
  if (mean_nnz <= 6.0) return 1;
  if (mean_nnz <= 24.0) return 4;
  if (mean_nnz <= 96.0) return 16;
  return 64;
}

// dense rows (row-major nd x n; column t is variable cols[t], or t when cols
// is null): y[rows[r]] += alpha * Ad[r, :] x   (one workgroup per row)
__global__ __launch_bounds__(256) void k_dense_rows(int64_t n, const double* __restrict__ Ad,
                                                    const int32_t* __restrict__ rows,
                                                    const int32_t* __restrict__ cols, const double* __restrict__ x,
                                                    double* __restrict__ y, double alpha) {
  __shared__ double red[256];
  const int r = blockIdx.x;
  double acc = 0;
  for (int64_t j = threadIdx.x; j < n; j += 256) acc += Ad[(int64_t)r * n + j] * x[cols ? cols[j] : j];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) y[rows[r]] += alpha * red[0];
}

void dense_rows_gemv(int nd, int64_t n, const double* Ad, const int32_t* rows, const int32_t* cols, const double* x,
                     double* y, double alpha, hipStream_t st) {
  if (nd == 0) return;
  hipLaunchKernelGGL(k_dense_rows, dim3(nd), dim3(256), 0, st, n, Ad, rows, cols, x, y, alpha);
  HC_LAUNCH_CHECK();
}

// y[cols[j]] += alpha * sum_r Ad[r, j] v[rows[r]]  (cols null: y[j]; cols is
// one-to-one).  The rows are split into chunks of DRT_ROWS: workgroup (x, c)
// sums chunk c for 256 columns (coalesced row reads) into part[c][j], and a
// second kernel adds the chunks in order, so the result does not depend on
// scheduling.  part holds dense_rows_t_parts(nd) * n doubles.
constexpr int DRT_ROWS = 64;
int64_t dense_rows_t_parts(int nd) { return ceil_div(nd, DRT_ROWS); }

__global__ __launch_bounds__(256) void k_dense_rows_t(int nd, int64_t n, const double* __restrict__ Ad,
                                                      const int32_t* __restrict__ rows, const double* __restrict__ v,
                                                      double* __restrict__ part) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int r0 = blockIdx.y * DRT_ROWS, r1 = min(nd, r0 + DRT_ROWS);
  if (j >= n) return;
  double acc = 0;
  for (int r = r0; r < r1; ++r) acc += Ad[(int64_t)r * n + j] * v[rows[r]];
  part[(int64_t)blockIdx.y * n + j] = acc;
}

__global__ __launch_bounds__(256) void k_dense_rows_t_sum(int64_t n, int nparts, const double* __restrict__ part,
                                                          const int32_t* __restrict__ cols, double* __restrict__ y,
                                                          double alpha) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  double acc = 0;
  for (int c = 0; c < nparts; ++c) acc += part[(int64_t)c * n + j];
  y[cols ? cols[j] : j] += alpha * acc;
}

void dense_rows_gemv_t(int nd, int64_t n, const double* Ad, const int32_t* rows, const int32_t* cols,
                       const double* v, double* y, double alpha, double* part, hipStream_t st) {
  if (nd == 0) return;
  const int np = (int)dense_rows_t_parts(nd);
  hipLaunchKernelGGL(k_dense_rows_t, dim3((unsigned)ceil_div(n, 256), (unsigned)np), dim3(256), 0, st, nd, n, Ad, rows,
                     v, part);
  HC_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_dense_rows_t_sum, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, st, n, np, part, cols, y,
                     alpha);
  HC_LAUNCH_CHECK();
}

// ---------------------------------------------------------------------------
// elementwise
// ---------------------------------------------------------------------------
__global__ void k_axpby(int64_t n, double a, const double* __restrict__ x, double b, double* __restrict__ y) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] = a * x[i] + (b == 0.0 ? 0.0 : b * y[i]);
}
void vaxpby(int64_t n, double a, const double* x, double b, double* y, hipStream_t st) {
  if (n == 0) return;
  hipLaunchKernelGGL(k_axpby, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, st, n, a, x, b, y);
  HC_LAUNCH_CHECK();
}
// z = a x + b y + c w  (any of y, w may be null)
__global__ void k_lin3(int64_t n, double a, const double* __restrict__ x, double b, const double* __restrict__ y,
                       double c, const double* __restrict__ w, double* __restrict__ z) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double v = a * x[i];
  if (y) v += b * y[i];
  if (w) v += c * w[i];
  z[i] = v;
}
void vlin3(int64_t n, double a, const double* x, double b, const double* y, double c, const double* w, double* z,
           hipStream_t st) {
  if (n == 0) return;
  hipLaunchKernelGGL(k_lin3, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, st, n, a, x, b, y, c, w, z);
  HC_LAUNCH_CHECK();
}
__global__ void k_fill(int64_t n, double v, double* __restrict__ y) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] = v;
}
void vfill(int64_t n, double v, double* y, hipStream_t st) {
  if (n == 0) return;
  hipLaunchKernelGGL(k_fill, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, st, n, v, y);
  HC_LAUNCH_CHECK();
}
// ---------------------------------------------------------------------------
// reductions: per-block partials, combined in block order by k_collect
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_reduce(int64_t n, RedOps ops, double* __restrict__ partial) {
  __shared__ double red[256];
  for (int o = 0; o < ops.nops; ++o) {
    const RedOp op = ops.op[o];
    const bool is_sum = (op.kind == RED_DOT);
    double acc = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
      if (op.kind == RED_DOT) {
        acc += op.x[i] * op.y[i];
      } else {
        double v = op.x[i];
        if (op.y) v += op.yc * op.y[i];
        if (op.w) v = (op.kind == RED_MAX_MUL) ? v * op.w[i] : v / op.w[i];
        acc = nmax(acc, fabs(v));
      }
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
      if ((int)threadIdx.x < off)
        red[threadIdx.x] = is_sum ? red[threadIdx.x] + red[threadIdx.x + off] : nmax(red[threadIdx.x], red[threadIdx.x + off]);
      __syncthreads();
    }
    if (threadIdx.x == 0) partial[(int64_t)blockIdx.x * ops.nops + o] = red[0];
    __syncthreads();
  }
}

int reduce_launch(int64_t n, const RedOps& ops, double* partial, hipStream_t st) {
  const int nb = (int)std::min<int64_t>(512, std::max<int64_t>(1, ceil_div(n, 256)));
  hipLaunchKernelGGL(k_reduce, dim3(nb), dim3(256), 0, st, n, ops, partial);
  HC_LAUNCH_CHECK();
  return nb;
}

// ---------------------------------------------------------------------------
// Row jobs: the sparse products, sums and residuals of a refinement step (of
// both of its systems), side by side in one launch.  At the sizes where a
// solve is a chain of short kernels each costs its launch (about 4 us of host
// time) whatever it does; at the large ones each reads its matrix once.  With the cone applications of both systems in one launch and
// the norms read back by k_collect, a small LP (n 50) went from 12.6 to
// 4.7 ms, an MPC problem of 100 stages from 31 to 15.5 ms per solve.
// ---------------------------------------------------------------------------
RowJob::RowJob(int kind_, const Csr& A, const double* x_, double* y_)
    : kind(kind_), nrows(A.nrows), lanes(A.lanes), long_nnz(A.long_nnz), nlong(A.nlong), rp(A.rowptr), ci(A.col),
      longrows(A.longrows), v(A.val), x(x_), y(y_) {}
int RowJob::row_blocks() const {
  return (int)std::min<int64_t>(2048, ceil_div((int64_t)nrows * (kind == ROW_LIN ? 1 : lanes), 256));
}
int RowJob::blocks() const { return row_blocks() + (kind == ROW_LIN ? 0 : std::min(nlong, 512)); }

__device__ inline double row_finish(const RowJob& j, int64_t row, double acc, double p) {
  double y;
  if (j.kind == ROW_MUL) y = j.alpha * acc + (j.beta == 0.0 ? 0.0 : j.beta * j.c[row]);
  else {
    y = acc + (j.addp ? j.addp[row] : p);
    if (j.kind == ROW_RESID) y = j.c[row] - y;
  }
  j.y[row] = y;
  return fabs(y);
}

template <int LPR>
__device__ inline double row_range(const RowJob& j, int blk, int nblk) {
  double mx = 0.0;
  const int sub = threadIdx.x % LPR;
  for (int64_t row = ((int64_t)blk * 256 + threadIdx.x) / LPR; row < j.nrows; row += (int64_t)nblk * 256 / LPR) {
    const int32_t b = j.rp[row], e = j.rp[row + 1];
    if (e - b > j.long_nnz) continue;
    double acc = 0.0, p = 0.0;
    for (int32_t k = b + sub; k < e; k += LPR) acc += j.v[k] * j.x[j.ci[k]];
    if (j.rp2 && sub < j.lanes2)
      for (int32_t k = j.rp2[row] + sub, e2 = j.rp2[row + 1]; k < e2; k += j.lanes2) p += j.v2[k] * j.x2[j.ci2[k]];
#pragma unroll
    for (int off = LPR / 2; off > 0; off >>= 1) {
      acc += __shfl_xor(acc, off, 64);
      p += __shfl_xor(p, off, 64);
    }
    if (sub == 0) mx = nmax(mx, row_finish(j, row, acc, p));
  }
  return mx;
}

// k_reduce's tree: across the four waves lane by lane, then within one
// (the sum is wave 0's; red holds 192)
__device__ inline double block_sum(double v, double* red) {
  const int t = threadIdx.x;
  __syncthreads();   // red's previous readers are done
  if (t >= 64) red[t - 64] = v;
  __syncthreads();
  if (t < 64) {
    v = (v + red[t + 64]) + (red[t] + red[t + 128]);
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  }
  return v;
}
__device__ inline double block_nmax(double v, double* red) {
  for (int off = 32; off > 0; off >>= 1) v = nmax(v, __shfl_xor(v, off, 64));
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return nmax(nmax(red[0], red[1]), nmax(red[2], red[3]));
}

// Rounds of 1,024 entries of a long row in flight.  A long row is one workgroup's
// latency: with its four entries a round under a condition each (the compiler
// then waits for every load) the KKT solves of eight iterations with 20 columns
// of 200,000 entries took 27.3 ms, with one round loaded together 11.1, two 8.1,
// four 7.9; two leave the eight waves per SIMD that the short rows had.
constexpr int LONG_AHEAD = 2;
__global__ __launch_bounds__(256, 8) void k_row_jobs(RowJobs J) {
  __shared__ double red[16];
  int q = 0;
  while (q + 1 < J.n && (int)blockIdx.x >= J.first[q + 1]) ++q;
  const RowJob& j = J.j[q];
  const int blk = blockIdx.x - J.first[q], nblk = J.rows[q];
  double mx = 0.0;
  if (j.kind == ROW_LIN) {
    for (int64_t i = (int64_t)blk * 256 + threadIdx.x; i < j.nrows; i += (int64_t)nblk * 256) {
      double y = j.alpha * j.x[i];
      if (j.beta != 0.0) y = fma(j.beta, j.c[i], y);
      j.y[i] = y;
      mx = nmax(mx, fabs(y));
    }
  } else if (blk < nblk) {
    switch (j.lanes) {
      case 1: mx = row_range<1>(j, blk, nblk); break;
      case 4: mx = row_range<4>(j, blk, nblk); break;
      case 16: mx = row_range<16>(j, blk, nblk); break;
      default: mx = row_range<64>(j, blk, nblk); break;
    }
  } else {
    const int nl = J.first[q + 1] - J.first[q] - nblk;   // long rows: one workgroup each
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int l = blk - nblk; l < j.nlong; l += nl) {
      const int32_t row = j.longrows[l];
      double acc[4] = {}, p = 0.0;   // the row is summed by 1,024 lanes, four to a thread
      const int32_t b = j.rp[row], e = j.rp[row + 1];
      int32_t k = b + threadIdx.x;
      for (; e - k > 1024 * (LONG_AHEAD - 1) + 768; k += 1024 * LONG_AHEAD) {
        int32_t col[4 * LONG_AHEAD];
        double v[4 * LONG_AHEAD], x[4 * LONG_AHEAD];
#pragma unroll
        for (int q = 0; q < 4 * LONG_AHEAD; ++q) col[q] = j.ci[k + 256 * q];
#pragma unroll
        for (int q = 0; q < 4 * LONG_AHEAD; ++q) v[q] = j.v[k + 256 * q];
#pragma unroll
        for (int q = 0; q < 4 * LONG_AHEAD; ++q) x[q] = j.x[col[q]];
#pragma unroll
        for (int q = 0; q < 4 * LONG_AHEAD; ++q) acc[q % 4] += v[q] * x[q];
      }
      for (; k < e; k += 1024)
#pragma unroll
        for (int h = 0; h < 4; ++h)
          if (k + 256 * h < e) acc[h] += j.v[k + 256 * h] * j.x[j.ci[k + 256 * h]];
      if (j.rp2 && (int)threadIdx.x < j.lanes2)
        for (int32_t k = j.rp2[row] + threadIdx.x, e2 = j.rp2[row + 1]; k < e2; k += j.lanes2)
          p += j.v2[k] * j.x2[j.ci2[k]];
      __syncthreads();
      for (int h = 0; h < 4; ++h) {
        for (int off = 32; off > 0; off >>= 1) acc[h] += __shfl_xor(acc[h], off, 64);
        if (lane == 0) red[4 * h + w] = acc[h];
      }
      for (int off = 32; off > 0; off >>= 1) p += __shfl_xor(p, off, 64);
      __syncthreads();
      if (threadIdx.x == 0) {
        double sum = 0.0;
        for (int i = 0; i < 16; ++i) sum += red[i];
        mx = nmax(mx, row_finish(j, row, sum, p));
      }
    }
  }
  if (j.pmax) {
    mx = block_nmax(mx, red);
    if (threadIdx.x == 0) j.pmax[blk] = mx;
  }
}

void row_jobs(RowJobs& J, hipStream_t st) {
  int nb = 0;
  for (int i = 0; i < J.n; ++i) {
    J.first[i] = nb;
    J.rows[i] = J.j[i].row_blocks();
    nb += J.j[i].blocks();
  }
  J.first[J.n] = nb;
  if (nb == 0) return;
  hipLaunchKernelGGL(k_row_jobs, dim3((unsigned)nb), dim3(256), 0, st, J);
  HC_LAUNCH_CHECK();
}

__global__ __launch_bounds__(256) void k_resid(ResidArgs a, int nbn, double* __restrict__ partial) {
  __shared__ double red[192];
  double v[RESID_VALS] = {};
  if ((int)blockIdx.x < nbn) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < a.n; i += (int64_t)nbn * 256) {
      const double px = a.Px[i], at = a.Atz[i], x = a.x[i], q = a.q[i], d = a.D[i];
      const double r = (px + at) + a.tau * q;
      a.rd[i] = r;
      a.r1[i] = -r;
      v[0] += x * px;
      v[1] += q * x;
      v[2] = nmax(v[2], fabs(r / d));
      v[3] = nmax(v[3], fabs(x * d));
      v[4] = nmax(v[4], fabs(at / d));
      v[5] = nmax(v[5], fabs(px / d));
      v[6] = nmax(v[6], fabs(r));
    }
  } else {
    const int nbm = gridDim.x - nbn, blk = blockIdx.x - nbn;
    for (int64_t i = (int64_t)blk * 256 + threadIdx.x; i < a.m; i += (int64_t)nbm * 256) {
      const double ax = a.Ax[i], s = a.s[i], z = a.z[i], b = a.b[i], e = a.E[i];
      const double r = (-ax - s) + a.tau * b, r2 = r + s;
      a.rp[i] = r;
      a.r2[i] = r2;
      v[0] += b * z;
      v[1] += s * z;
      v[2] = nmax(v[2], fabs(r / e));
      v[3] = nmax(v[3], fabs(s / e));
      v[4] = nmax(v[4], fabs(z * e));
      v[5] = nmax(v[5], fabs((ax + s) / e));
      v[6] = nmax(v[6], fabs(r2));
    }
  }
#pragma unroll
  for (int o = 0; o < RESID_VALS; ++o) {
    const double t = o < 2 ? block_sum(v[o], red) : block_nmax(v[o], red);
    if (threadIdx.x == 0) partial[(int64_t)blockIdx.x * 8 + o] = t;
  }
}
static int vec_blocks(int64_t n) { return (int)std::min<int64_t>(512, std::max<int64_t>(1, ceil_div(n, 256))); }
void resid_launch(const ResidArgs& a, double* partial, int* nbn, int* nbm, hipStream_t st) {
  *nbn = vec_blocks(a.n);
  *nbm = vec_blocks(a.m);
  hipLaunchKernelGGL(k_resid, dim3((unsigned)(*nbn + *nbm)), dim3(256), 0, st, a, *nbn, partial);
  HC_LAUNCH_CHECK();
}

// a x rounded, then + y
__device__ inline double lin_rounded(double a, double x, double y) {
#pragma clang fp contract(off)
  return a * x + y;
}
__global__ __launch_bounds__(256) void k_dir_dots(int64_t n, int64_t m, double pc, const double* __restrict__ Px,
                                                  const double* __restrict__ q, const double* __restrict__ x1,
                                                  const double* __restrict__ x2, const double* __restrict__ b,
                                                  const double* __restrict__ z1, const double* __restrict__ z2,
                                                  int nbn, double* __restrict__ partial) {
  __shared__ double red[192];
  double v0 = 0.0, v1 = 0.0;
  if ((int)blockIdx.x < nbn) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)nbn * 256) {
      const double w = lin_rounded(pc, Px[i], q[i]);
      v0 += w * x1[i];
      v1 += w * x2[i];
    }
  } else {
    const int nbm = gridDim.x - nbn;
    for (int64_t i = (int64_t)(blockIdx.x - nbn) * 256 + threadIdx.x; i < m; i += (int64_t)nbm * 256) {
      v0 += b[i] * z1[i];
      v1 += b[i] * z2[i];
    }
  }
  v0 = block_sum(v0, red);
  v1 = block_sum(v1, red);
  if (threadIdx.x == 0) {
    partial[2 * (int64_t)blockIdx.x] = v0;
    partial[2 * (int64_t)blockIdx.x + 1] = v1;
  }
}
void dir_dots(int64_t n, int64_t m, double pc, const double* Px, const double* q, const double* x1, const double* x2,
              const double* b, const double* z1, const double* z2, double* partial, int* nbn, int* nbm,
              hipStream_t st) {
  *nbn = vec_blocks(n);
  *nbm = vec_blocks(m);
  hipLaunchKernelGGL(k_dir_dots, dim3((unsigned)(*nbn + *nbm)), dim3(256), 0, st, n, m, pc, Px, q, x1, x2, b, z1, z2,
                     *nbn, partial);
  HC_LAUNCH_CHECK();
}

__device__ inline double combine(int kind, double a, double v) {
  return kind == COLLECT_MAX ? nmax(a, v) : kind == COLLECT_MIN ? fmin(a, v) : fmax(a, v);
}
// one wave per op.  Extrema: lane-strided, then a shuffle tree; sums: partial
// after partial (at most 512 of them, from LDS: 8 cycles each), the order they
// had on the host.  Each value is one store of its own that the host waits for
// (COLLECT_EMPTY until then), with no fence and no flag behind them: 4.9 -> 3.1 us.
__global__ __launch_bounds__(64 * MAX_COLLECT) void k_collect(Collect c, double* out) {
  extern __shared__ double part[];   // 512 per op, where any is a sum
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (w >= c.n) return;
  const CollectOp op = c.op[w];
  double acc = op.kind == COLLECT_MIN ? INFINITY : op.kind == COLLECT_TOP ? -INFINITY : 0.0;
  if (op.kind == COLLECT_INT) {
    acc = (double)*(const int*)op.p;
  } else if (op.kind == COLLECT_SUM) {
    double* ls = part + 512 * w;
    for (int i0 = 0; i0 < op.cnt; i0 += 512) {
      const int k = min(512, op.cnt - i0);
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int i = 64 * q + lane;
        const double v = op.p[(int64_t)(i0 + min(i, k - 1)) * op.stride];
        ls[i] = i < k ? v : 0.0;
      }
      __builtin_amdgcn_wave_barrier();   // read across lanes of the wave
      for (int i = 0; i < k; i += 8)
#pragma unroll
        for (int l = 0; l < 8; ++l) acc += ls[i + l];
    }
  } else {
    for (int i = lane; i < op.cnt; i += 512) {
      double v[8];   // the last partial more than once changes no extremum
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = op.p[(int64_t)min(i + 64 * q, op.cnt - 1) * op.stride];
#pragma unroll
      for (int q = 0; q < 8; ++q) acc = combine(op.kind, acc, v[q]);
    }
    for (int off = 32; off > 0; off >>= 1) acc = combine(op.kind, acc, __shfl_xor(acc, off, 64));
  }
  if (lane == 0) {
    unsigned long long u = (unsigned long long)__double_as_longlong(acc);
    if (u == COLLECT_EMPTY) u = 0x7ff8000000000000ull;   // any other NaN
    __hip_atomic_store((unsigned long long*)(out + w), u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}
void collect(const Collect& c, double* out, hipStream_t st) {
  bool sum = false;
  for (int i = 0; i < c.n; ++i) sum = sum || c.op[i].kind == COLLECT_SUM;
  hipLaunchKernelGGL(k_collect, dim3(1), dim3(64 * c.n), sum ? 512 * c.n * sizeof(double) : 0, st, c, out);
  HC_LAUNCH_CHECK();
}

// device-side max of partials into out[0] (no host round trip); used to scale
// FP32 right-hand sides
__global__ void k_combine_max(int nb, const double* __restrict__ partial, double* __restrict__ out) {
  __shared__ double red[256];
  double acc = 0;
  for (int i = threadIdx.x; i < nb; i += 256) acc = fmax(acc, partial[i]);
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + off]);
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = (red[0] > 0.0) ? red[0] : 1.0;
}
void combine_max(int nb, const double* partial, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_combine_max, dim3(1), dim3(256), 0, st, nb, partial, out);
  HC_LAUNCH_CHECK();
}

// FP64 <-> FP32 with a device-side scale
__global__ void k_to_f32(int64_t n, const double* __restrict__ x, const double* __restrict__ scale,
                         float* __restrict__ y) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] = (float)(x[i] / scale[0]);
}
__global__ void k_from_f32(int64_t n, const float* __restrict__ x, const double* __restrict__ scale,
                           double* __restrict__ y) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] = (double)x[i] * scale[0];
}
void to_f32(int64_t n, const double* x, const double* scale, float* y, hipStream_t st) {
  hipLaunchKernelGGL(k_to_f32, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, st, n, x, scale, y);
  HC_LAUNCH_CHECK();
}
void from_f32(int64_t n, const float* x, const double* scale, double* y, hipStream_t st) {
  hipLaunchKernelGGL(k_from_f32, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, st, n, x, scale, y);
  HC_LAUNCH_CHECK();
}
// lower triangle (including diagonal) of a column-major n x n FP64 matrix -> FP32
__global__ void k_lower_to_f32(int64_t n, int64_t ld, const double* __restrict__ S, float* __restrict__ S32) {
  const int64_t j = blockIdx.y;
  for (int64_t i = j + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    S32[i + j * ld] = (float)S[i + j * ld];
}
void lower_to_f32(int64_t n, int64_t ld, const double* S, float* S32, hipStream_t st) {
  if (n == 0) return;
  hipLaunchKernelGGL(k_lower_to_f32, dim3((unsigned)std::min<int64_t>(64, ceil_div(n, 256)), (unsigned)n), dim3(256),
                     0, st, n, ld, S, S32);
  HC_LAUNCH_CHECK();
}

// ---------------------------------------------------------------------------
// Schur complement assembly  S = P + delta I + A' M A  (lower triangle)
// ---------------------------------------------------------------------------
__global__ void k_fill_lower_zero(int64_t n, int64_t ld, double* __restrict__ S) {
  const int64_t j = blockIdx.y;
  for (int64_t i = j + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    S[i + j * ld] = 0.0;
}
void fill_lower_zero(int64_t n, int64_t ld, double* S, hipStream_t st) {
  if (n == 0) return;
  hipLaunchKernelGGL(k_fill_lower_zero, dim3((unsigned)std::min<int64_t>(64, ceil_div(n, 256)), (unsigned)n),
                     dim3(256), 0, st, n, ld, S);
  HC_LAUNCH_CHECK();
}

// P (full CSR) lower part + delta on the diagonal
__global__ void k_add_P(int32_t n, const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                        const double* __restrict__ v, double delta, int64_t ld, double* __restrict__ S) {
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  S[i + (int64_t)i * ld] += delta;
  if (!rp) return;
  for (int32_t p = rp[i]; p < rp[i + 1]; ++p) {
    const int32_t j = ci[p];
    if (j <= i) S[i + (int64_t)j * ld] += v[p];
  }
}
void add_P_delta(const Csr& P, int64_t n, double delta, int64_t ld, double* S, hipStream_t st) {
  hipLaunchKernelGGL(k_add_P, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, st, (int32_t)n, P.rowptr, P.col, P.val,
                     delta, ld, S);
  HC_LAUNCH_CHECK();
}

// One task, an unordered pair of rows (ra >= rb, same cone) with the index of
// m = M_c[ra, rb], adds m (a_ra a_rb' + a_rb a_ra') (m a_ra a_ra' when ra = rb) to
// the lower triangle of S by hardware FP64 atomics.  Short tasks run one lane
// each; long ones (rows with hundreds of entries) one wave each, the lanes
// striding over the entries of row ra, so no single lane issues the whole row's
// quadratic update.
template <bool WIDE>
__global__ __launch_bounds__(256) void k_assemble_pairs(int64_t ntask, const int32_t* __restrict__ tra,
                                                        const int32_t* __restrict__ trb,
                                                        const int64_t* __restrict__ tm,
                                                        const double* __restrict__ mval, const int32_t* __restrict__ rp,
                                                        const int32_t* __restrict__ ci, const double* __restrict__ av,
                                                        int64_t ld, double* __restrict__ S) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t t = WIDE ? gid / 64 : gid;
  const int lane = WIDE ? (int)(threadIdx.x & 63) : 0, nl = WIDE ? 64 : 1;
  if (t >= ntask) return;
  const int32_t ra = tra[t], rb = trb[t];
  const double m = mval[tm[t]];
  if (m == 0.0) return;
  const int32_t ba = rp[ra], ea = rp[ra + 1], bb = rp[rb], eb = rp[rb + 1];
  if (ra == rb) {
    for (int32_t p = ba + lane; p < ea; p += nl) {
      const int32_t j = ci[p];
      const double mj = m * av[p];
      for (int32_t q = ba; q <= p; ++q) atomicAdd(&S[j + (int64_t)ci[q] * ld], mj * av[q]);
    }
  } else {
    for (int32_t p = ba + lane; p < ea; p += nl) {
      const int32_t j = ci[p];
      const double mj = m * av[p];
      for (int32_t q = bb; q < eb; ++q) {
        const int32_t k = ci[q];
        double v = mj * av[q];
        if (j == k) v *= 2.0;
        const int32_t hi = j > k ? j : k, lo = j > k ? k : j;
        atomicAdd(&S[hi + (int64_t)lo * ld], v);
      }
    }
  }
}
void assemble_pairs(int64_t ntask, const int32_t* tra, const int32_t* trb, const int64_t* tm, const double* mval,
                    const Csr& A, int64_t ld, double* S, bool wide, hipStream_t st) {
  if (ntask == 0) return;
  if (wide)
    hipLaunchKernelGGL(k_assemble_pairs<true>, dim3((unsigned)ceil_div(ntask * 64, 256)), dim3(256), 0, st, ntask,
                       tra, trb, tm, mval, A.rowptr, A.col, A.val, ld, S);
  else
    hipLaunchKernelGGL(k_assemble_pairs<false>, dim3((unsigned)ceil_div(ntask, 256)), dim3(256), 0, st, ntask, tra,
                       trb, tm, mval, A.rowptr, A.col, A.val, ld, S);
  HC_LAUNCH_CHECK();
}

// T[e, j] = sum_b M_c[a, b] A[row b of cone c, j] for segment row e = c dim + a
// (M_c symmetric, stored as its lower triangle: entry (a, b), a >= b, at
// moff + (a (a + 1) / 2 + b) count + c).  One workgroup per cone and PT_ROWS rows
// of T: those rows of M_c are staged in LDS (M is packed by cone, so its entries
// lie `count` apart), a thread takes a column the cone touches and loads each of
// its entries, in row order, once for all PT_ROWS rows; with a row of
// T per workgroup, every term was two loads of scattered lines.  30 cones each
// of sides 20 and 32 on 1,800 columns, both segments: 826 -> 241 us.
constexpr int PT_ROWS = 8;
__global__ __launch_bounds__(256) void k_psd_dense_T(int32_t dim, int64_t count, int64_t coff, int64_t moff,
                                                     const double* __restrict__ mval, PsdCols pc,
                                                     const double* __restrict__ av, int64_t n,
                                                     double* __restrict__ T) {
  extern __shared__ double ms[];   // row b of the cone: PT_ROWS entries M[a0 .., b]
  const int64_t nblk = (dim + PT_ROWS - 1) / PT_ROWS;
  for (int64_t w = blockIdx.x; w < count * nblk; w += gridDim.x) {
    const int64_t c = w / nblk;
    const int a0 = (int)(w % nblk) * PT_ROWS, na = min(PT_ROWS, dim - a0);
    __syncthreads();   // the previous rows' readers are done
    for (int i = threadIdx.x; i < PT_ROWS * dim; i += 256) {
      const int q = i / dim, b = i - q * dim, a = a0 + min(q, na - 1);
      const int hi = a > b ? a : b, lo = a > b ? b : a;
      ms[b * PT_ROWS + q] = mval[moff + ((int64_t)hi * (hi + 1) / 2 + lo) * count + c];
    }
    __syncthreads();
    const int64_t u1 = pc.cu_off[coff + c + 1];
    for (int64_t u = pc.cu_off[coff + c] + threadIdx.x; u < u1; u += 256) {
      double acc[PT_ROWS] = {};
      for (int64_t k = pc.cu_ptr[u]; k < pc.cu_ptr[u + 1]; ++k) {
        const double* m = ms + pc.cu_b[k] * PT_ROWS;
        const double x = av[pc.cu_p[k]];
#pragma unroll
        for (int q = 0; q < PT_ROWS; ++q) acc[q] += m[q] * x;
      }
      double* t = T + (c * dim + a0) * n + pc.cu_col[u];
#pragma unroll
      for (int q = 0; q < PT_ROWS; ++q)
        if (q < na) t[q * n] = acc[q];
    }
  }
}
void psd_dense_T(int32_t dim, int64_t count, int64_t coff, int64_t moff, const double* mval, const PsdCols& pc,
                 const double* av, int64_t n, double* T, hipStream_t st) {
  const int64_t wgs = count * ceil_div(dim, PT_ROWS);
  if (wgs == 0) return;
  hipLaunchKernelGGL(k_psd_dense_T, dim3((unsigned)std::min<int64_t>(wgs, 65536)), dim3(256),
                     (size_t)dim * PT_ROWS * sizeof(double), st, dim, count, coff, moff, mval, pc, av, n, T);
  HC_LAUNCH_CHECK();
}

template <bool WIDE>
__global__ __launch_bounds__(256) void k_ordered_sum(OrderedSum os, int64_t first, int64_t cnt,
                                                     const double* __restrict__ mval, const double* __restrict__ av,
                                                     const double* __restrict__ slot, double* b0, double* b1,
                                                     double* b2) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t i = WIDE ? gid / 64 : gid;
  const int lane = WIDE ? (int)(threadIdx.x & 63) : 0, nl = WIDE ? 64 : 1;
  if (i >= cnt) return;   // wide: one destination per wave, so whole waves leave together
  const int64_t d = first + i;
  const int64_t k0 = os.ptr[d], k1 = os.ptr[d + 1];
  double acc = 0.0;
  if (os.pm) {
    for (int64_t k = k0 + lane; k < k1; k += nl) {
      int32_t q = os.pq[k];
      const bool two = q < 0;
      if (two) q = ~q;
      double v = mval[os.pm[k]] * av[os.pp[k]] * av[q];
      if (two) v *= 2.0;
      acc += v;
    }
  } else {
    for (int64_t k = k0 + lane; k < k1; k += nl) acc += slot[os.pp[k]];
  }
  if (WIDE)
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if (lane == 0) {
    const int64_t e = os.dst[d];
    const int sel = (int)((uint64_t)e >> 62);
    double* base = sel == 0 ? b0 : sel == 1 ? b1 : b2;
    base[e & ((int64_t(1) << 62) - 1)] += acc;
  }
}
void ordered_sum(const OrderedSum& os, const double* mval, const double* av, const double* slot, double* b0,
                 double* b1, double* b2, hipStream_t st) {
  const int64_t ns = os.nshort, nl = os.nd - os.nshort;
  if (ns > 0) {
    hipLaunchKernelGGL(k_ordered_sum<false>, dim3((unsigned)ceil_div(ns, 256)), dim3(256), 0, st, os, (int64_t)0,
                       ns, mval, av, slot, b0, b1, b2);
    HC_LAUNCH_CHECK();
  }
  if (nl > 0) {
    hipLaunchKernelGGL(k_ordered_sum<true>, dim3((unsigned)ceil_div(nl * 64, 256)), dim3(256), 0, st, os, ns, nl,
                       mval, av, slot, b0, b1, b2);
    HC_LAUNCH_CHECK();
  }
}

// S[j, k] += sum_e A[row(e), j] T[e, k] for k <= j: a workgroup takes TG_COLS
// columns j of A (rows j of S) and 256 columns k of S, a thread one k, so each
// entry has one writer, the T rows are read contiguously and a thread writes
// TG_COLS neighbours of S's column k (one entry each, the writes of a wave went
// to 64 lines; the workload of psd_dense_T: 436 -> 373 us, 1.3 GB of T).
constexpr int TG_COLS = 8;
__global__ __launch_bounds__(256) void k_dense_T_gather(int64_t n, const int32_t* __restrict__ erp,
                                                        const int32_t* __restrict__ ee, const int32_t* __restrict__ ep,
                                                        const double* __restrict__ atval,
                                                        const double* __restrict__ T, int64_t ld,
                                                        double* __restrict__ S) {
  const int64_t j0 = (int64_t)blockIdx.x * TG_COLS, k = (int64_t)blockIdx.y * 256 + threadIdx.x;
  const int64_t j1 = std::min<int64_t>(n, j0 + TG_COLS);
  if ((int64_t)blockIdx.y * 256 >= j1) return;
  const double* Tk = T + std::min<int64_t>(k, n - 1);
  for (int64_t j = j0; j < j1; ++j) {
    double s = 0.0;
    int32_t p = erp[j];
    const int32_t e = erp[j + 1];
    if (p == e) continue;
    for (; p + 8 <= e; p += 8) {
      double t[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) t[q] = Tk[(int64_t)ee[p + q] * n];
#pragma unroll
      for (int q = 0; q < 8; ++q) s += atval[ep[p + q]] * t[q];
    }
    for (; p < e; ++p) s += atval[ep[p]] * Tk[(int64_t)ee[p] * n];
    if (k <= j) S[j + k * ld] += s;
  }
}
void dense_T_gather(int64_t n, const int32_t* erp, const int32_t* ee, const int32_t* ep, const double* atval,
                    const double* T, int64_t ld, double* S, hipStream_t st) {
  if (n == 0) return;
  hipLaunchKernelGGL(k_dense_T_gather, dim3((unsigned)ceil_div(n, TG_COLS), (unsigned)ceil_div(n, 256)), dim3(256), 0,
                     st, n, erp, ee, ep, atval, T, ld, S);
  HC_LAUNCH_CHECK();
}

// Small groups: a wave each.
__global__ __launch_bounds__(64) void k_group_T(GroupPlan gp, const double* __restrict__ mval,
                                                const double* __restrict__ av) {
  const int lane = threadIdx.x;
  for (int64_t g = blockIdx.x; g < gp.ng; g += gridDim.x) {
    const int64_t nr = gp.rows_off[g + 1] - gp.rows_off[g];
    const int64_t uo = gp.u_off[g], s = gp.u_off[g + 1] - uo;
    if (nr * s >= GROUP_WIDE) continue;
    const int64_t* gm = gp.gm + gp.m_off[g];
    double* T = gp.T + gp.t_off[g];
    for (int64_t a = 0; a < nr; ++a)
      for (int64_t t = lane; t < s; t += 64) {
        double v = 0.0;
        for (int64_t e = gp.c_ptr[uo + t]; e < gp.c_ptr[uo + t + 1]; ++e) {
          const int64_t mi = gm[a * nr + gp.c_b[e]];
          if (mi >= 0) v += mval[mi] * av[gp.c_k[e]];
        }
        T[a * s + t] = v;
      }
  }
}
// The groups of at least GROUP_WIDE entries of T: a workgroup per group and
// GT_ROWS of its rows, whose part of M_g is staged in LDS (the index table gm
// read once, in order) up to GT_ROWS_MAX rows per group; a thread takes a
// column and loads its entries once for GT_ROWS rows.  A wave per group followed
// gm -> mval for every term: 2,000 cones of 55 rows on 421 columns, 1.04 ms ->
// 175 us (370 MB of T).
constexpr int GT_ROWS = 8, GT_ROWS_MAX = 512;
__global__ __launch_bounds__(256) void k_group_T_wide(GroupPlan gp, const double* __restrict__ mval,
                                                      const double* __restrict__ av) {
  extern __shared__ double ms[];   // row b of the group: GT_ROWS entries M[a0 .., b]
  const int64_t g = gp.wide[blockIdx.x];
  const int nr = (int)(gp.rows_off[g + 1] - gp.rows_off[g]);
  const int64_t uo = gp.u_off[g], s = gp.u_off[g + 1] - uo;
  const int64_t* gm = gp.gm + gp.m_off[g];
  for (int a0 = blockIdx.y * GT_ROWS; a0 < nr; a0 += gridDim.y * GT_ROWS) {
    const int na = min(GT_ROWS, nr - a0);
    double* T = gp.T + gp.t_off[g] + (int64_t)a0 * s;
    if (nr <= GT_ROWS_MAX) {
      __syncthreads();   // the previous rows' readers are done
      for (int i = threadIdx.x; i < GT_ROWS * nr; i += 256) {
        const int q = i / nr, b = i - q * nr;
        const int64_t mi = q < na ? gm[(int64_t)(a0 + q) * nr + b] : -1;
        ms[b * GT_ROWS + q] = mi >= 0 ? mval[mi] : 0.0;
      }
      __syncthreads();
    }
    for (int64_t t = threadIdx.x; t < s; t += 256) {
      double v[GT_ROWS] = {};
      for (int64_t e = gp.c_ptr[uo + t]; e < gp.c_ptr[uo + t + 1]; ++e) {
        const int b = gp.c_b[e];
        const double x = av[gp.c_k[e]];
        if (nr <= GT_ROWS_MAX) {
#pragma unroll
          for (int q = 0; q < GT_ROWS; ++q) v[q] += ms[b * GT_ROWS + q] * x;
        } else {
#pragma unroll
          for (int q = 0; q < GT_ROWS; ++q) {
            const int64_t mi = q < na ? gm[(int64_t)(a0 + q) * nr + b] : -1;
            if (mi >= 0) v[q] += mval[mi] * x;
          }
        }
      }
#pragma unroll
      for (int q = 0; q < GT_ROWS; ++q)
        if (q < na) T[q * s + t] = v[q];
    }
  }
}
void group_T(const GroupPlan& gp, const double* mval, const Csr& A, hipStream_t st) {
  if (gp.ng > gp.nwide) {
    hipLaunchKernelGGL(k_group_T, dim3((unsigned)std::min<int64_t>(gp.ng, 65536)), dim3(64), 0, st, gp, mval, A.val);
    HC_LAUNCH_CHECK();
  }
  if (gp.nwide > 0) {
    const int rows = std::min(gp.wide_rows, GT_ROWS_MAX);
    hipLaunchKernelGGL(k_group_T_wide,
                       dim3((unsigned)gp.nwide, (unsigned)std::min<int64_t>(ceil_div(gp.wide_rows, GT_ROWS), 16)),
                       dim3(256), (size_t)rows * GT_ROWS * sizeof(double), st, gp, mval, A.val);
    HC_LAUNCH_CHECK();
  }
}

// value of one lane (wave-uniform index), as a scalar
__device__ inline int lane_i(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ inline int64_t lane_l(int64_t v, int l) {
  const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)v, l), hi = __builtin_amdgcn_readlane((int)(v >> 32), l);
  return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ inline double lane_d(double v, int l) { return __longlong_as_double(lane_l(__double_as_longlong(v), l)); }
// One wave per column j, its rows in order.  Each row adds a run of (index,
// value) pairs to the column in LDS; the runs are cut into segments of 64 and
// GG_AHEAD segments are in flight, since a wave that waits for each row's run
// spends its time on memory latency: 2,000 cones of 55 rows on 421 of 5,000
// columns, 4.08 -> 0.78 ms (2.1 GB of T and indices; a column's runs start at its
// own diagonal).  Chunks trade passes over a column's runs against LDS, that is
// waves on a CU: GATHER_CHUNK rows are 40 KB, four waves, and every further chunk
// reads the runs again, so a column has as few chunks as that allows and they
// have equal lengths.  800 cones of 55 rows on 4,600 / 5,200 / 5,700 / 6,400 /
// 7,200 / 8,000 / 10,000 columns: 351 / 325 / 344 / 423 / 520 / 570 / 823 us; with
// chunks of 5,120 rows and a rest 350 / 391 / 447 / 518 / 579 / 649 / 823, of 4,096
// 378 / 449 / 493 / 557 / 615 / 674 / 883.  SOCs of three rows, 11,000 to 16,000 of
// them on 5,620 / 6,920 / 8,120 columns: 136 / 243 / 416 us, 186 / 268 / 403 and
// 199 / 282 / 412.
constexpr int GG_AHEAD = 8;
__global__ __launch_bounds__(64) void k_group_gather(GroupPlan gp, int64_t n, int chunk,
                                                     const int32_t* __restrict__ atrp,
                                                     const double* __restrict__ atv, int64_t ld,
                                                     double* __restrict__ S) {
  extern __shared__ double acc[];   // chunk rows
  const int lane = threadIdx.x;
  for (int64_t j = blockIdx.x; j < n; j += gridDim.x) {
    const int32_t p0 = atrp[j], p1 = atrp[j + 1];
    if (p0 == p1) continue;
    for (int64_t c0 = j; c0 < n; c0 += chunk) {
      const int len = (int)std::min<int64_t>(n - c0, chunk);
      for (int i = lane; i < len; i += 64) acc[i] = 0.0;
      for (int32_t pb = p0; pb < p1; pb += 64) {
        // 64 rows' runs: a lane each, then picked by index
        const int32_t p = std::min(pb + lane, p1 - 1);
        const int rs = pb + lane < p1 ? gp.e_s[p] : 0;
        const int64_t ru = gp.e_u[p], rt = gp.e_t[p];
        const double rc = atv[p];
        int nseg = (rs + 63) >> 6;
        for (int off = 32; off > 0; off >>= 1) nseg += __shfl_xor(nseg, off, 64);
        nseg = lane_i(nseg, 0);
        int row = -1, t0 = 0, s = 0;   // the run being fetched
        const int32_t* ui = gp.u;
        const double* tv = gp.T;
        double cf = 0.0;
        int i_q[GG_AHEAD], l_q[GG_AHEAD];
        double v_q[GG_AHEAD], c_q[GG_AHEAD];
        auto fetch = [&](int q) {   // always two loads: the waits count them
          while (t0 >= s && row < 63) {
            ++row;
            t0 = 0;
            s = lane_i(rs, row);
            if (s > 0) {
              ui = gp.u + lane_l(ru, row);
              tv = gp.T + lane_l(rt, row);
              cf = lane_d(rc, row);
            }
          }
          const int t = std::max(0, std::min(t0 + lane, s - 1));
          i_q[q] = ui[t] - (int)c0;
          v_q[q] = tv[t];
          c_q[q] = cf;
          l_q[q] = t0 + lane < s ? len : 0;
          t0 += 64;
        };
#pragma unroll
        for (int q = 0; q < GG_AHEAD; ++q) fetch(q);
        for (int done = 0; done < nseg; done += GG_AHEAD) {
#pragma unroll
          for (int q = 0; q < GG_AHEAD; ++q) {
            if ((unsigned)i_q[q] < (unsigned)l_q[q]) acc[i_q[q]] += c_q[q] * v_q[q];
            fetch(q);
          }
        }
      }
      for (int i = lane; i < len; i += 64) {
        const double v = acc[i];
        if (v != 0.0) S[c0 + i + j * ld] += v;
      }
    }
  }
}
void group_gather(const GroupPlan& gp, int64_t n, const Csr& At, int64_t ld, double* S, hipStream_t st) {
  if (gp.ng == 0 || n == 0) return;
  const int chunk = (int)ceil_div(n, ceil_div(n, GATHER_CHUNK));
  hipLaunchKernelGGL(k_group_gather, dim3((unsigned)std::min<int64_t>(n, 16384)), dim3(64),
                     (size_t)chunk * sizeof(double), st, gp, n, chunk, At.rowptr, At.val, ld, S);
  HC_LAUNCH_CHECK();
}

// B (nd x n row-major, i.e. n x nd column-major with ld n) = sqrt|m_r| Ad[r, :];
// rows with midx < 0 are padding and stay zero
__global__ void k_scale_dense_rows(int nd, int64_t n, const double* __restrict__ Ad, const int64_t* __restrict__ midx,
                                   const double* __restrict__ mval, double* __restrict__ B) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int r = blockIdx.y;
  const int64_t mi = midx[r];
  if (j < n) B[(int64_t)r * n + j] = mi < 0 ? 0.0 : sqrt(fabs(mval[mi])) * Ad[(int64_t)r * n + j];
}
void scale_dense_rows(int nd, int64_t n, const double* Ad, const int64_t* midx, const double* mval, double* B,
                      hipStream_t st) {
  if (nd == 0) return;
  hipLaunchKernelGGL(k_scale_dense_rows, dim3((unsigned)ceil_div(n, 256), (unsigned)nd), dim3(256), 0, st, nd, n, Ad,
                     midx, mval, B);
  HC_LAUNCH_CHECK();
}

// transpose between cone-by-cone (AoS) and component-major layouts (test entry points)
__global__ void k_aos_to_cm(int64_t count, int dim, const double* __restrict__ a, double* __restrict__ c, int inverse) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= count * dim) return;
  const int64_t i = t / dim;
  const int j = (int)(t % dim);
  if (!inverse) c[j * count + i] = a[t];
  else c[t] = a[j * count + i];
}
void aos_to_cm(int64_t count, int dim, const double* a, double* c, bool inverse, hipStream_t st) {
  if (count == 0) return;
  hipLaunchKernelGGL(k_aos_to_cm, dim3((unsigned)ceil_div(count * dim, 256)), dim3(256), 0, st, count, dim, a, c,
                     inverse ? 1 : 0);
  HC_LAUNCH_CHECK();
}

}  // namespace hc
