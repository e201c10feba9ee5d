// Dense factorisation of the KKT Schur complement on gfx950.
//
// After the cone rows are eliminated (their pivots are the -(H_c + delta I)
// blocks), the quasi-definite LDL' of the regularised KKT matrix
// (eq. linsys_2x2, Sec. 3.7) continues on the positive definite Schur
// complement S = P + delta I + A' M A.  This file factors S = L L' (the
// positive pivots of the LDL', D = diag(L)^2 absorbed into L) and solves with
// L, in FP64 or -- for the mixed-precision mode of Sec. 3.7 -- FP32 with FP32
// accumulation.
//
// Layout: S is column-major with leading dimension ld, lower triangle used.
// Algorithm: blocked right-looking Cholesky with 64-wide diagonal blocks.
//   step:   one launch per 64 columns: L21 = A21 * Linv' in place, one
//           workgroup per 64 rows, the update of the panel's later columns,
//           and the next diagonal block's factor with its inverse (Linv, 64x64
//           per block)
//   update: trailing C -= L21 L21' on MFMA (v_mfma_f64_16x16x4f64 or
//           v_mfma_f32_16x16x4f32), 64x64 tiles, lower tiles only.  It is
//           delayed to every panel of 256 or Aux::nb columns, so the trailing
//           matrix is read and written once per panel.
// Triangular solves: one launch per pass, from the inverses of 128 x 128
// diagonal blocks (FP64), or launches of 256 rows (FP32).
#include "hc_dense.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace hc {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef double v2d __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));

template <typename T> struct Mfma;
// Both instructions take A[i][k] from lane i + 16 k and B[k][j] from lane
// j + 16 k.  Output element r of lane l is D[row(l, r)][l % 16]; the FP64
// form interleaves rows (l/16 + 4 r), the FP32 form blocks them (4 (l/16) + r).
template <> struct Mfma<double> {
  typedef v4d acc_t;
  __device__ static inline acc_t op(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  __device__ static inline int row(int lane, int r) { return (lane >> 4) + 4 * r; }
};
template <> struct Mfma<float> {
  typedef v4f acc_t;
  __device__ static inline acc_t op(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  __device__ static inline int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};

constexpr int BS = 64;    // diagonal block
constexpr int IB = 256;   // inner panel
// Rows from which a trailing update is long enough to run beside the next
// panel on a second stream (two event waits, about 10 us, per panel): 5,056
// rows take 3.97 ms with the rule at 4,096, 4.03 at 2,048, 3.97 without.
constexpr int64_t LOOKAHEAD_MIN = 4096;
// Rows from which panels are Aux::nb columns wide instead of IB: the update
// then runs at K = 768 (65 TFLOP/s instead of 57 at K = 256) and reads the
// trailing matrix a third as often, but a panel's chain is three times as
// long and has to fit behind it.  10,048 / 20,032 rows: 11.5 / 53.5 ms with
// the rule at 8,192, 11.7 / 54.5 at 12,288, 11.8 / 59.3 without wide panels.
constexpr int64_t WIDE_MIN = 8192;
// LDS a trailing update's workgroup takes on top of its own 20 KB: three fit
// a compute unit and leave 37 KB and 248 VGPRs per lane in one piece, room
// for a workgroup of the panel chain.  At full occupancy the chain's
// workgroups (one of them for k_chol_diag) found no room until the update
// ended, 4.8 ms at 20,032 rows; the update alone loses 4 % (65.1 -> 62.8 TFLOP/s).
constexpr size_t BEHIND_PAD = 21504;

// ---------------------------------------------------------------------------
// 64 x 64 diagonal block: Cholesky factor and its inverse, one workgroup of
// four waves
// ---------------------------------------------------------------------------
// value of v in a wave-uniform lane
__device__ inline double lane_bcast(double v, int src) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = __builtin_amdgcn_readlane((unsigned)u, src);
  const unsigned hi = __builtin_amdgcn_readlane((unsigned)(u >> 32), src);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ inline float lane_bcast(float v, int src) {
  return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), src));
}

// 1 / sqrt(d): v_rsq_f64 is good to about 2^-24, one cubic step takes that past 2^-53
__device__ inline double rsqrt_full(double d) {
  const double e = __builtin_amdgcn_rsq(d);
  const double h = fma(-(d * e), e, 1.0);
  return fma(e, h * fma(h, 0.375, 0.5), e);
}

// exchanges lane groups and registers: x[a] of lane 16 g + i becomes x[g] of
// lane 16 a + i (v_permlane16_swap, v_permlane32_swap)
__device__ inline void swap16(double& x, double& y) {
  const uint64_t a = (uint64_t)__double_as_longlong(x), b = (uint64_t)__double_as_longlong(y);
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)a, (unsigned)b, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(a >> 32), (unsigned)(b >> 32), false, false);
  x = __longlong_as_double((long long)(((uint64_t)hi[0] << 32) | lo[0]));
  y = __longlong_as_double((long long)(((uint64_t)hi[1] << 32) | lo[1]));
}
__device__ inline void swap32(double& x, double& y) {
  const uint64_t a = (uint64_t)__double_as_longlong(x), b = (uint64_t)__double_as_longlong(y);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)a, (unsigned)b, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(a >> 32), (unsigned)(b >> 32), false, false);
  x = __longlong_as_double((long long)(((uint64_t)hi[0] << 32) | lo[0]));
  y = __longlong_as_double((long long)(((uint64_t)hi[1] << 32) | lo[1]));
}
__device__ inline void transpose4(double (&x)[4]) {
  swap16(x[0], x[1]);
  swap16(x[2], x[3]);
  swap32(x[0], x[2]);
  swap32(x[1], x[3]);
}

constexpr int CST = 66;                   // column stride of the LDS block
constexpr int CHOL_LDS = BS * CST + BS;   // doubles: L and below-diagonal L^-1 in one block, 1 / diag(L)

// L^-1[i][k] of the block: below the diagonal it sits in the place of entry
// (k, i) above it, its diagonal is dv
__device__ __forceinline__ double chol_inv(const double* __restrict__ lds, int i, int k) {
  const double v = lds[i * CST + k], d = lds[BS * CST + i];
  return i > k ? v : (i == k ? d : 0.0);
}

// On entry Lc holds the 64 x 64 block (Lc[k * CST + i] = A[i][k], i >= k used)
// and every wave has passed a barrier since it was written; on return its
// lower triangle is the factor and the rest the inverse (chol_inv).  FP64 in
// both precision modes (the FP32 mode rounds at the end).
//
// It is a chain of 64 dependent pivots, so what counts is the length of the
// chain and what runs beside it.  Wave s factors column block s alone, four
// columns at a time: one matrix row per lane, two pivots at a time (the second
// one's root is that of the 2 x 2 determinant, so that both reciprocal roots
// run at once), multipliers by readlane.  Lane-group swaps then turn the four
// columns into MFMA operands (K = 4) and the rest of the block, held in MFMA
// output registers D[column][row], gets their update.  Behind that wave,
// between the same four barriers, the waves to its right apply the finished
// block on MFMA, and those to its left build the inverse: Y_ss in wave s,
// T_sp = sum_{k=p}^{s-1} L_sk Y_kp in wave p and one stage later Y_sp =
// -Y_ss T_sp, T_sp staying in the output registers, whose layout is the next
// product's operand layout.  One pivot at a time with a 15-column update each
// (an FP64 FMA issues every 8 cycles) and a lane-per-column inverse took
// 45,600 cycles a block, this takes 30,500 (12.7 us).
// The 2 x 2 determinant is a product of two diagonal entries: within 1e-150 ..
// 1e150 it stays in range.  (Taking one pivot after the other where it does not
// cost every step 1 us of 24, for matrices that no solve gets to: the refinement
// makes no progress on data from about 1e40 on.)
__device__ __forceinline__ void chol_block(int lane, int p, double* __restrict__ lds, double tol, double fix,
                                  unsigned long long* __restrict__ hits) {
  typedef Mfma<double> M;
  // Lc[k * CST + i] = L[i][k], Lc[i * CST + k] = Y[i][k] = L^-1[i][k], i > k.
  // Row i of Y comes after column i of L, whose zeros above the diagonal the
  // whole-column stores below put there.
  double* Lc = lds;
  double* dv = lds + BS * CST;   // 1 / L[k][k]
  const int li = lane & 15, lg = lane >> 4;
  int nhits = 0;
  v4d t = v4d{0, 0, 0, 0};
  // U[a][r] = A[16 a + li][16 p + lg + 4 r], a >= p
  v4d U[4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int r = 0; r < 4; ++r) U[a][r] = a >= p ? Lc[(16 * p + lg + 4 * r) * CST + 16 * a + li] : 0.0;
  __syncthreads();   // the factor's columns overwrite the block
  // Y_ip = -Y_ii T_ip
  auto finish = [&](int i) {
    v4d y = v4d{0, 0, 0, 0};
#pragma unroll
    for (int q = 0; q < 4; ++q) y = M::op(chol_inv(lds, 16 * i + li, 16 * i + lg + 4 * q), t[q], y);
#pragma unroll
    for (int q = 0; q < 4; ++q) Lc[(16 * i + lg + 4 * q) * CST + 16 * p + li] = -y[q];
    __builtin_amdgcn_wave_barrier();   // this wave reads them next
  };
#pragma unroll 1
  for (int s = 0; s < 4; ++s) {
    if (p == s) {
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const int j0 = 16 * s + 4 * m;
        double c[4] = {U[0][m], U[1][m], U[2][m], U[3][m]};
        transpose4(c);   // c[q] = A[lane][j0 + q]
#pragma unroll
        for (int h = 0; h < 4; h += 2) {
          const int j = j0 + h;
          double a00 = lane_bcast(c[h], j);
          const double a10 = lane_bcast(c[h], j + 1), a11 = lane_bcast(c[h + 1], j + 1);
          double det = fma(a00, a11, -(a10 * a10));
          if (!(a00 > tol) || !(det > tol * a00)) {   // pivots that are not positive (NaN too) are replaced and counted
            if (!(a00 > tol)) {
              a00 = fix;
              ++nhits;
              det = fma(a00, a11, -(a10 * a10));
            }
            if (!(det > tol * a00)) {
              det = fix * a00;
              ++nhits;
            }
          }
          const double e0 = rsqrt_full(a00), rd = rsqrt_full(det);
          const double l00 = a00 * e0, l10 = a10 * e0;
          const double e1 = l00 * rd, l11 = det * rd * e0;   // the second pivot is det / a00
          dv[j] = e0;
          dv[j + 1] = e1;
          const double x0 = lane > j ? c[h] * e0 : 0.0;
          const double x1 = lane > j + 1 ? fma(-x0, l10, c[h + 1]) * e1 : 0.0;
          c[h] = lane == j ? l00 : x0;
          c[h + 1] = lane == j + 1 ? l11 : x1;
          if (h == 0) {
            const double l20 = lane_bcast(x0, j + 2), l21 = lane_bcast(x1, j + 2);
            const double l30 = lane_bcast(x0, j + 3), l31 = lane_bcast(x1, j + 3);
            c[2] = fma(-x1, l21, fma(-x0, l20, c[2]));
            c[3] = fma(-x1, l31, fma(-x0, l30, c[3]));
          }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) Lc[(j0 + q) * CST + lane] = c[q];
        if (m < 3) {
          transpose4(c);   // c[a] = L[16 a + li][j0 + lg]
          const double ns = -(s == 0 ? c[0] : s == 1 ? c[1] : s == 2 ? c[2] : c[3]);
#pragma unroll
          for (int a = 0; a < 4; ++a)
            if (a >= s) U[a] = M::op(ns, c[a], U[a]);
        }
      }
    }
    __syncthreads();
    if (p > s) {
      // U[a] -= L[rows of a][block s] L[rows of p][block s]'
      double f[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) f[q] = -Lc[(16 * s + lg + 4 * q) * CST + 16 * p + li];
#pragma unroll
      for (int a = 1; a < 4; ++a)
        if (a >= p) {
#pragma unroll
          for (int q = 0; q < 4; ++q) U[a] = M::op(f[q], Lc[(16 * s + lg + 4 * q) * CST + 16 * a + li], U[a]);
        }
    } else if (p == s) {
      // Y_ss by rows of 4 x 4 blocks: with R = I at the start, block row b is
      // Y_b = N_b R_b (N_b the inverse of the diagonal 4 x 4 block) and the
      // rows below lose L_b Y_b.  R sits in the output registers (block row b
      // is register b), which are the operand layout of both products.
      // nv = N_b[u][v] for b = li / 4, u = li % 4, v = lg
      const int o = 16 * s + (li & 12);
      const double *c0 = Lc + o * CST + o, *c1 = c0 + CST, *c2 = c1 + CST;
      const double y0 = lg == 0 ? dv[o] : 0.0;
      const double y1 = fma(-c0[1], y0, lg == 1 ? 1.0 : 0.0) * dv[o + 1];
      const double y2 = fma(-c1[2], y1, fma(-c0[2], y0, lg == 2 ? 1.0 : 0.0)) * dv[o + 2];
      const double y3 = fma(-c2[3], y2, fma(-c1[3], y1, fma(-c0[3], y0, lg == 3 ? 1.0 : 0.0))) * dv[o + 3];
      const int u = li & 3;
      const double nv = u == 0 ? y0 : u == 1 ? y1 : u == 2 ? y2 : y3;
      v4d R;
#pragma unroll
      for (int b = 0; b < 4; ++b) R[b] = (lg + 4 * b == li) ? 1.0 : 0.0;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const v4d y = M::op((li >> 2) == b ? nv : 0.0, R[b], v4d{0, 0, 0, 0});
        if (lg + 4 * b > li) Lc[(16 * s + lg + 4 * b) * CST + 16 * s + li] = y[b];
        if (b < 3) R = M::op(-Lc[(16 * s + 4 * b + lg) * CST + 16 * s + li], y[b], R);
      }
    } else {
      if (p < s - 1) finish(s - 1);
      t = v4d{0, 0, 0, 0};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = 16 * p + lg + 4 * q;
        t = M::op(Lc[i * CST + 16 * s + li], chol_inv(lds, i, 16 * p + li), t);
      }
      for (int k = p + 1; k < s; ++k) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int i = 16 * k + lg + 4 * q;
          t = M::op(Lc[i * CST + 16 * s + li], Lc[i * CST + 16 * p + li], t);
        }
      }
    }
  }
  __syncthreads();
  if (p < 3) finish(3);
  __syncthreads();
  if (lane == 0 && nhits) atomicAdd(hits, (unsigned long long)nhits);
}

// writes the factor block's lower triangle to A (its corner at (c, c)) and the
// inverse, with zeros above its diagonal, to Linv (64 x 64, column-major)
__device__ __forceinline__ void chol_store(int lane, int p, int bs, const double* __restrict__ lds, double* __restrict__ A,
                                  int64_t ld, int64_t c, double* __restrict__ Linv) {
#pragma unroll 4
  for (int k = 16 * p; k < 16 * p + 16; ++k) {
    if (lane < bs && k < bs && k <= lane) A[(c + lane) + (c + k) * ld] = lds[k * CST + lane];
    Linv[lane + k * BS] = chol_inv(lds, lane, k);
  }
}

// a block column of the padded diagonal block: identity past bs
__device__ inline double chol_pad(double v, int i, int k, int bs) {
  return (i < bs && k < bs) ? v : (i == k ? 1.0 : 0.0);
}

__global__ __launch_bounds__(256, 3) void k_chol_diag(double* __restrict__ A, int64_t ld, int64_t c, int64_t n,
                                                   double* __restrict__ Linv, double tol, double fix,
                                                   unsigned long long* __restrict__ hits) {
  __shared__ __align__(16) double lds[CHOL_LDS];
  __builtin_amdgcn_s_setprio(3);   // the factorisation's critical path
  const int lane = threadIdx.x & 63;
  const int p = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int bs = (int)std::min<int64_t>(BS, n - c);
  double g[16];
#pragma unroll
  for (int q = 0; q < 16; ++q)
    g[q] = A[(c + std::min(lane, bs - 1)) + (c + std::min(16 * p + q, bs - 1)) * ld];
#pragma unroll
  for (int q = 0; q < 16; ++q) lds[(16 * p + q) * CST + lane] = chol_pad(g[q], lane, 16 * p + q, bs);
  __syncthreads();
  chol_block(lane, p, lds, tol, fix, hits);
  chol_store(lane, p, bs, lds, A, ld, c, Linv);
}

// ---------------------------------------------------------------------------
// One 64-column step of a panel in one launch.  On entry the block column at
// c is up to date, its diagonal block factored and that factor's inverse in
// Linv; a workgroup takes 64 of the rows [c + 64, R), each wave 16 of them:
//   L[i, c] = A[i, c] Linv'                                     (all rows)
// and brings the block columns c' in [c + 64, cend) left of its rows up to date:
//   A[i, c'] -= L[i, c] L[c', c]',
// whereupon workgroup 0, whose rows are the next diagonal block, factors it.
// So the chain per 64 columns is one launch instead of three (factor, TRSM,
// update), and the factorisation of the next diagonal block runs beside the
// other rows' work.  L[c', c] is needed by every workgroup and recomputed by
// each (a 64^3 product); since all of them read A[c', c], the workgroups of
// those rows leave their tile in a slot (defer) and the next step's workgroups
// from rowgs on put it in its place (rows below rdef of the row blocks from c).
//
// Products run on MFMA as X' = Linv A' and U' = X_c' X', whose output
// registers (rows k, one matrix row i per lane) are the next product's operand
// registers, and whose stores to A are 16 consecutive rows per column.
// Bound: the chain of workgroup 0 (launch, loads past the L2, two 64^3
// products, 64 pivots); 34 KB of LDS and at most 168 VGPRs let it run beside
// three trailing-update workgroups.  The four steps of a panel at 1,856 rows:
// 34, 27, 24, 24 us (in the first two the other rows' workgroups, 7 us a tile,
// outlast the chain; up to about 5,000 rows a step stays under 30 us, at 20,032 it
// averages 58 with the trailing update beside it), against 53 us each in three launches and 26 to 34 with
// the panel's earlier columns applied only when a block column is next, which
// puts up to 192 of them, and the tile of the previous step, in the chain.
// ---------------------------------------------------------------------------
constexpr int XST = CST;       // k row stride of X_c' in LDS
constexpr int SLOTS = 2 * (IB / BS + 1);   // deferred tiles: a step's, and the previous one's on their way
static_assert(BS * XST <= CHOL_LDS, "X_c' fits the block's LDS");

__global__ __launch_bounds__(256, 3) void k_panel_step(double* __restrict__ A, int64_t ld, int64_t n, int64_t c,
                                                    int64_t cend, int64_t R, double* __restrict__ LinvAll,
                                                    double* __restrict__ slots, int rowgs, int defer, int64_t rdef,
                                                    double tol, double fix, unsigned long long* __restrict__ hits) {
  typedef Mfma<double> M;
  __shared__ __align__(16) double lds[CHOL_LDS];   // X_c', then the next diagonal block
  __builtin_amdgcn_s_setprio(3);   // the factorisation's critical path
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool first = blockIdx.x == 0;
  const double* Linv = LinvAll + (c / BS) * BS * BS;
  const int64_t c1 = c + BS;                                  // next block column
  const int64_t r0 = c1 + (int64_t)blockIdx.x * BS;
  // tile of L[r .., k ..] between the launch that makes it and the next
  auto slot_of = [&](int64_t r, int64_t k) {
    return slots + ((r / BS) % (SLOTS / 2) + ((k / BS) & 1) * (SLOTS / 2)) * BS * BS;
  };
  if ((int)blockIdx.x >= rowgs) {
    const int64_t r = c + (int64_t)(blockIdx.x - rowgs) * BS;
    const double* slot = slot_of(r, c - BS);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int k = w + 4 * e;
      if (r + lane < rdef) A[(r + lane) + (c - BS + k) * ld] = slot[lane + k * BS];
    }
    return;
  }
  if (r0 >= R) return;
  const int64_t row = r0 + 16 * w + li;                       // this lane's row
  // column j + lane / 16 of a row: uniform base of column j, 32-bit lane offset
  // (64-bit addresses per lane take twice the registers there are)
  const uint32_t lgo = (uint32_t)((lane >> 4) * ld);
  const uint32_t own = (uint32_t)std::min<int64_t>(row, R - 1) + lgo;   // rows past R repeat the last one
  // Linv A' of the 16 rows at offset o, 16 of its rows at a time: f(t, x) with
  // x[q] = X[i][16 t + row(lane, q)]
  auto trsm = [&](uint32_t o, auto&& f) {
    double a[4][4];   // A[i][m], m = 16 u + row(lane, q)
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int q = 0; q < 4; ++q) a[u][q] = (A + (c + 16 * u + 4 * q) * ld)[o];
    const double* inv = Linv;
    asm volatile("" : "+s"(inv));   // its 40 operands are not kept from one product to the next
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      v4d y = v4d{0, 0, 0, 0};
#pragma unroll
      for (int u = 0; u <= t; ++u)   // Linv is lower triangular
#pragma unroll
        for (int q = 0; q < 4; ++q)
          y = M::op(inv[(16 * t + li) + (16 * u + M::row(lane, q)) * BS], a[u][q], y);
      f(t, y);
    }
  };
  // columns cb + j, j = 16 b + row(lane, q), of this lane's row
  auto load = [&](int64_t cb, double (&cv)[4][4]) {
    const int nb = (int)std::min<int64_t>(BS, n - cb);
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int j = std::min(16 * b + 4 * q, nb - 1);   // past nb: any column
        cv[b][q] = (A + (cb + j) * ld)[nb < BS && j + (lane >> 4) >= nb ? own - lgo : own];
      }
  };
  v4d x[4];
  trsm(own, [&](int t, v4d y) { x[t] = y; });
  // L[i][c + k], k = 16 t + row(lane, q)
  const bool slot_out = defer && r0 < cend;
  double* slot = slot_of(r0, c);
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = 16 * t + M::row(lane, q);
      if (slot_out) slot[(16 * w + li) + k * BS] = x[t][q];
      else if (row < R) (A + (c + 16 * t + 4 * q) * ld)[own] = x[t][q];
    }
#pragma unroll 1
  for (int64_t cb = c1; cb < cend && cb <= r0; cb += BS) {
    const int nb = (int)std::min<int64_t>(BS, n - cb);
    const int nbt = first ? w + 1 : 4;   // the next diagonal tile needs its lower blocks only
    if (cb > c1) __syncthreads();   // the previous X_c' has been read
    auto put = [&](int t, v4d y) {
#pragma unroll
      for (int q = 0; q < 4; ++q) lds[(16 * t + M::row(lane, q)) * XST + 16 * w + li] = y[q];
    };
    if (cb == r0) {
#pragma unroll
      for (int t = 0; t < 4; ++t) put(t, x[t]);
    } else {
      trsm((uint32_t)std::min<int64_t>(cb + 16 * w + li, n - 1) + lgo, put);
    }
    double cv[4][4];
    load(cb, cv);
    __syncthreads();   // X_c' is in LDS
    v4d u[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) u[b] = v4d{0, 0, 0, 0};
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int b = 0; b < 4; ++b)
        if (b < nbt)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            u[b] = M::op(lds[(16 * t + M::row(lane, q)) * XST + 16 * b + li], x[t][q], u[b]);
    if (!first) {
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int j = 16 * b + M::row(lane, q);
          if (row < R && j < nb) (A + (cb + 16 * b + 4 * q) * ld)[own] = cv[b][q] - u[b][q];
        }
      continue;
    }
    __syncthreads();   // every wave has read X_c'
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = 16 * b + M::row(lane, q), i = 16 * w + li;
        lds[k * CST + i] = chol_pad(cv[b][q] - u[b][q], i, k, nb);
      }
  }
  if (!first || c1 >= cend) return;
  __syncthreads();
  chol_block(lane, w, lds, tol, fix, hits);
  chol_store(lane, w, (int)std::min<int64_t>(BS, n - c1), lds, A, ld, c1, LinvAll + (c1 / BS) * BS * BS);
}

// ---------------------------------------------------------------------------
// The FP32 mode's panel: diagonal block, TRSM and in-panel update, a launch
// each, panels of Aux::nb columns.  Its refinement stops at a fraction of mu,
// so the rounding of the factor shows in the iterates (a relative 1e-4 where
// the FP64 mode's differences stay under 1e-10): these kernels keep their
// order of operations, and with it the results, and the FP64 kernels above,
// which sum in another order, are not instantiated for it.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_chol_diag32(float* __restrict__ A, int64_t ld, int64_t c, int64_t n,
                                                   float* __restrict__ Linv, double tol, double fix,
                                                   unsigned long long* __restrict__ hits) {
  // Cholesky of one 64 x 64 diagonal block and the inverse of its factor, by
  // 16-column blocks.  Thread (i, p) = (lane, wave) keeps r[q] = A[i][16p + q].
  // Column block pj is factored by wave pj alone: the pivot comes from lane
  // j by readlane and so do the multipliers of the later columns, so the 16
  // steps need no barrier.  The finished block goes to LDS and the waves to
  // its right apply it (a rank-16 update), one barrier per block.  L^-1 is
  // then built by 16 x 16 blocks: each wave inverts its diagonal block by
  // forward substitution (rows exchanged with shuffles), and the blocks
  // below the diagonal follow by distance from it,
  // Y_ij = -Y_ii sum_{k=j}^{i-1} L_ik Y_kj.
  __shared__ float Ls[BS][BS + 1];          // L, then read by the inverse
  __shared__ float Ys[BS][BS + 1];          // L^-1
  __shared__ float Ts[4][16][17];           // per-wave scratch of the inverse
  const int lane = threadIdx.x & 63;
  const int p = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int bs = (int)std::min<int64_t>(BS, n - c);
  float r[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int k = 16 * p + q;
    const float g = A[(c + std::min(lane, bs - 1)) + (c + std::min(k, bs - 1)) * ld];
    r[q] = (lane < bs && k < bs) ? (k <= lane ? g : float(0)) : (lane == k ? float(1) : float(0));
  }
  int nhits = 0;
  // ---- L: column block pj is factored by its owning wave alone (pivots by
  // readlane, no barrier), published, and applied by the waves to its right
#pragma unroll 1
  for (int pj = 0; pj < 4; ++pj) {
    if (p == pj) {
#pragma unroll
      for (int qj = 0; qj < 16; ++qj) {
        const int j = 16 * pj + qj;
        double d = (double)lane_bcast(r[qj], j);
        if (j < bs && !(d > tol)) {
          d = fix;
          ++nhits;
        }
        double e = __builtin_amdgcn_rsq(d);
        e = e * (1.5 - 0.5 * d * e * e);
        e = e * (1.5 - 0.5 * d * e * e);
        const float inv = (float)e, ljj = (float)(d * e);
        const float li = (lane > j) ? r[qj] * inv : float(0);
        r[qj] = (lane == j) ? ljj : li;   // zero above the diagonal
#pragma unroll
        for (int q = qj + 1; q < 16; ++q) r[q] -= li * lane_bcast(li, 16 * pj + q);
      }
#pragma unroll
      for (int q = 0; q < 16; ++q) Ls[lane][16 * pj + q] = (16 * pj + q <= lane) ? r[q] : float(0);
    }
    __syncthreads();
    if (p > pj) {
      float a[16];
#pragma unroll
      for (int t = 0; t < 16; ++t) a[t] = Ls[lane][16 * pj + t];
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        float s = 0;
#pragma unroll
        for (int t = 0; t < 16; ++t) s += a[t] * Ls[16 * p + q][16 * pj + t];
        r[q] -= s;
      }
    }
  }
  if (lane == 0 && nhits) atomicAdd(hits, (unsigned long long)nhits);
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int k = 16 * p + q;
    if (lane < bs && k < bs && k <= lane) A[(c + lane) + (c + k) * ld] = r[q];
  }
  // ---- L^-1 by 16 x 16 blocks.  Lane (s, g) = (lane % 16, lane / 16) holds
  // row s, columns 4g .. 4g + 3 of a block.
  const int s = lane & 15, g = lane >> 4;
  {
    // diagonal block p: forward substitution over its rows
    const int o = 16 * p;
    float y[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) y[u] = (s == 4 * g + u) ? float(1) : float(0);
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      const float dinv = float(1) / Ls[o + t][o + t];
      const float lst = Ls[o + s][o + t];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float yt = __shfl(y[u], t + 16 * g, 64) * dinv;   // row t, final
        y[u] = (s == t) ? yt : ((s > t) ? y[u] - lst * yt : y[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) Ys[o + s][o + 4 * g + u] = y[u];
  }
  __syncthreads();
  // off-diagonal blocks by distance from the diagonal:
  //   Y_ij = -Y_ii sum_{k=j}^{i-1} L_ik Y_kj
#pragma unroll 1
  for (int dist = 1; dist < 4; ++dist) {
    if (p + dist < 4) {
      const int i = p + dist, j = p;
      float t4[4] = {};
      for (int k = j; k < i; ++k)
#pragma unroll
        for (int m = 0; m < 16; ++m) {
          const float l = Ls[16 * i + s][16 * k + m];
#pragma unroll
          for (int u = 0; u < 4; ++u) t4[u] += l * Ys[16 * k + m][16 * j + 4 * g + u];
        }
#pragma unroll
      for (int u = 0; u < 4; ++u) Ts[p][s][4 * g + u] = t4[u];
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // this wave's scratch writes landed
      float o4[4] = {};
#pragma unroll
      for (int m = 0; m < 16; ++m) {
        const float yim = Ys[16 * i + s][16 * i + m];
#pragma unroll
        for (int u = 0; u < 4; ++u) o4[u] -= yim * Ts[p][m][4 * g + u];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) Ys[16 * i + s][16 * j + 4 * g + u] = o4[u];
    }
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int k = 16 * p + q;
    Linv[lane + k * BS] = (k <= lane) ? Ys[lane][k] : float(0);
  }
}

// ---------------------------------------------------------------------------
// TRSM: rows [r0, r1) of the 64 columns starting at c: A21 <- A21 * Linv'
// ---------------------------------------------------------------------------
// On MFMA: each wave takes 16 rows and all 64 columns (four 16 x 16 output
// tiles, 16 k-steps of four).  A wave's 16 x 64 block of A21 is loaded into
// registers at once; Linv goes through a 4 KB LDS slice, the 16 rows of Linv
// that one output tile needs, one tile after another.  With few registers and
// 4 KB of LDS a workgroup fits beside a running trailing-update workgroup on
// the same compute unit instead of waiting for one to finish: this kernel sits
// on the factorisation's critical path while the trailing update runs.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8))) void k_trsm32(
    float* __restrict__ A, int64_t ld, int64_t c, int64_t r0, int64_t r1, const float* __restrict__ Linv) {
  __shared__ float Ls[BS][16];   // Ls[k][jj] = Linv[16 t + jj][k] for the current tile t
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t rb = r0 + (int64_t)blockIdx.x * BS + wave * 16;   // first row of this wave
  // operand lanes: A[i = lane % 16][k = lane / 16], B[k = lane / 16][j = lane % 16]
  const int64_t ra = std::min<int64_t>(rb + (lane & 15), r1 - 1);   // rows past r1 repeat the last one
  const float* pa = A + ra + (c + (lane >> 4)) * ld;
  float a[BS / 4];
#pragma unroll
  for (int q = 0; q < BS / 4; ++q) a[q] = pa[(int64_t)(4 * q) * ld];
#pragma unroll 1
  for (int t = 0; t < 4; ++t) {
    __syncthreads();   // the previous slice has been read
#pragma unroll
    for (int q = 0; q < BS * 16 / 256; ++q) {
      const int e = tid + 256 * q;
      Ls[e >> 4][e & 15] = Linv[(16 * t + (e & 15)) + (e >> 4) * BS];
    }
    __syncthreads();
    v4f acc = v4f{0, 0, 0, 0};
#pragma unroll
    for (int q = 0; q < BS / 4; ++q) acc = Mfma<float>::op(a[q], Ls[4 * q + (lane >> 4)][lane & 15], acc);
    // X[i][j] = sum_k A[i][k] Linv[j][k]; this wave loaded its rows above,
    // other waves own other rows
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t row = rb + Mfma<float>::row(lane, r);
      if (row < r1) A[row + (c + 16 * t + (lane & 15)) * ld] = acc[r];
    }
  }
}

// ---------------------------------------------------------------------------
// In-panel update after a TRSM: C -= A B' with K <= 64 (one 64-column block
// of L), the shape of the TRSM so that it also fits beside a running
// trailing-update workgroup: a workgroup takes 64 rows x 64 columns of C,
// each wave 16 rows (its 16 x K block of A in registers) and four 16 x 16
// tiles, B through a 4 KB LDS slice per tile.  Tiles strictly above the
// global diagonal (C[0, 0] at global (gr, gc)) are skipped.  The products are
// the same MFMA chain as the large update kernels' (k in steps of four).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8))) void k_gemm_panel32(
    float* __restrict__ C, int64_t ldc, const float* __restrict__ A, int64_t lda, const float* __restrict__ B, int64_t ldb,
    int64_t M, int64_t N, int K, int64_t gr, int64_t gc) {
  __shared__ float Bs[BS][16];   // Bs[k][jj] = B[j0 + jj][k] for the current tile
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t i_blk = (int64_t)blockIdx.x * BS, j_blk = (int64_t)blockIdx.y * BS;
  if (gr + i_blk + BS - 1 < gc + j_blk) return;   // block strictly above the diagonal
  const int64_t rb = i_blk + wave * 16;             // first row of this wave
  const int64_t ra = std::min<int64_t>(rb + (lane & 15), M - 1);
  const float* pa = A + ra;
  float a[BS / 4];
#pragma unroll
  for (int q = 0; q < BS / 4; ++q) {
    const int k = 4 * q + (lane >> 4);
    const float v = pa[(int64_t)std::min(k, K - 1) * lda];
    a[q] = k < K ? v : float(0);
  }
#pragma unroll 1
  for (int t = 0; t < 4; ++t) {
    const int64_t j0 = j_blk + 16 * t;
    if (j0 >= N) break;
    __syncthreads();   // the previous slice has been read
#pragma unroll
    for (int q = 0; q < BS * 16 / 256; ++q) {
      const int e = tid + 256 * q, k = e >> 4, jj = e & 15;
      const float v = B[std::min<int64_t>(j0 + jj, N - 1) + (int64_t)std::min(k, K - 1) * ldb];
      Bs[k][jj] = k < K ? v : float(0);
    }
    __syncthreads();
    if (gr + rb + 15 < gc + j0) continue;   // this wave's rows lie above the tile's columns
    v4f acc = v4f{0, 0, 0, 0};
#pragma unroll
    for (int q = 0; q < BS / 4; ++q) acc = Mfma<float>::op(a[q], Bs[4 * q + (lane >> 4)][lane & 15], acc);
    const int64_t j = j0 + (lane & 15);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t i = rb + Mfma<float>::row(lane, r);
      if (i < M && j < N) C[i + j * ldc] -= acc[r];
    }
  }
}

// ---------------------------------------------------------------------------
// C[i, j] += alpha * sum_k A[i, k] B[j, k]  (i < M, j < N, k < K), all
// column-major.  64 x 64 tiles of four waves (32 x 32 each); operand chunks of
// 64 bytes of k go through registers into a double-buffered LDS ring, two
// chunks ahead of the MFMAs, one barrier per chunk.  A wave's MFMAs take the B
// rows as first operand and the A rows as second, so its output registers hold
// 16 consecutive rows of C per column and C is read and written in whole
// 128-byte lines straight from registers.
// Bound: FP64 MFMA issue (64 cycles each, 16 per chunk and wave).  What keeps
// it busy is waves: 80 VGPRs and 20 KB of LDS put six of these workgroups on a
// compute unit, so one's loads, barriers and C traffic run behind the others'
// MFMAs.  Measured on the trailing update, K = 768 (TFLOP/s at 19,200 / 8,192 /
// 4,096 rows): 67.8 / 64.7 / 57.7; 128 x 128 tiles at two workgroups per unit
// 64.8 / 57.9 / 42.4 (too few waves, and four times the work in a last, partly
// filled round); one chunk ahead instead of two 64.4 / 61.9 / 54.3.
// With tri (square C on the diagonal) the grid holds the lower tiles only;
// with `lower` alone, tiles strictly above the global diagonal (C[0, 0] at
// (gr, gc)) return at once.  VEC: 16-byte operand loads (row groups of
// 16 / sizeof(T) whole and aligned, K a multiple of the chunk); otherwise
// element by element.
// ---------------------------------------------------------------------------
template <typename T> struct Vec16;
template <> struct Vec16<double> { typedef v2d t; };
template <> struct Vec16<float> { typedef v4f t; };
constexpr int TL = 64;

template <typename T, bool VEC>
__global__ __launch_bounds__(256, 4) void k_gemm_nt(T* __restrict__ C, int64_t ldc, const T* __restrict__ A,
                                                    int64_t lda, const T* __restrict__ B, int64_t ldb, int64_t M,
                                                    int64_t N, int64_t K, T alpha, int lower, int tri, int64_t gr,
                                                    int64_t gc, int tiles_n, int prio) {
  typedef typename Mfma<T>::acc_t acc_t;
  typedef typename Vec16<T>::t vec;
  constexpr int G = 16 / sizeof(T);     // rows per load
  constexpr int DK = 64 / sizeof(T);    // k per chunk
  constexpr int ST = TL + 16;           // k row stride in LDS
  constexpr int SK = 256 * G / TL;      // k rows one round of loads covers
  static_assert(SK == DK, "one load per thread, operand and chunk");
  __shared__ __align__(16) T As[2][DK][ST];
  __shared__ __align__(16) T Bs[2][DK][ST];
  if (prio) __builtin_amdgcn_s_setprio(2);   // on the factorisation's critical path
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lg = lane >> 4;
  const int wm = (wave & 1) * 32, wn = (wave >> 1) * 32;
  int tile_m, tile_n;
  if (tri) {   // tile b is (r, b - r (r + 1) / 2)
    const int64_t b = blockIdx.x;
    int64_t r = (int64_t)((sqrt(8.0 * (double)b + 1.0) - 1.0) * 0.5);
    if ((r + 1) * (r + 2) / 2 <= b) ++r;
    if (r * (r + 1) / 2 > b) --r;
    tile_m = (int)r;
    tile_n = (int)(b - r * (r + 1) / 2);
  } else {
    tile_m = blockIdx.x / tiles_n;
    tile_n = blockIdx.x % tiles_n;
  }
  const int64_t i_base = (int64_t)tile_m * TL, j_base = (int64_t)tile_n * TL;
  if (lower && gr + i_base + TL - 1 < gc + j_base) return;
  acc_t acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = acc_t{0, 0, 0, 0};
  // a thread loads row group sg of k row sk of a chunk.  Rows past the end
  // repeat the last group: their products are never stored.
  const int sg = (tid % (TL / G)) * G, sk = tid / (TL / G);
  const int64_t gi = std::min<int64_t>(i_base + sg, VEC ? M - G : M - 1);
  const int64_t gj = std::min<int64_t>(j_base + sg, VEC ? N - G : N - 1);
  const T* pa = A + gi + (VEC ? sk * lda : 0);
  const T* pb = B + gj + (VEC ? sk * ldb : 0);
  vec ra[2], rb[2];
  auto fetch = [&](int kc, int s) {
    if (VEC) {
      ra[s] = *reinterpret_cast<const vec*>(pa + (int64_t)kc * DK * lda);
      rb[s] = *reinterpret_cast<const vec*>(pb + (int64_t)kc * DK * ldb);
    } else {
      const int64_t k = (int64_t)kc * DK + sk, kk = std::min<int64_t>(k, K - 1);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        ra[s][g] = pa[std::min<int64_t>(g, M - 1 - gi) + kk * lda];
        rb[s][g] = pb[std::min<int64_t>(g, N - 1 - gj) + kk * ldb];
      }
      if (k >= K) {   // zero past the end of k
        ra[s] = vec(T(0));
        rb[s] = vec(T(0));
      }
    }
  };
  auto stage = [&](int buf, int s) {
    *reinterpret_cast<vec*>(&As[buf][sk][sg]) = ra[s];
    *reinterpret_cast<vec*>(&Bs[buf][sk][sg]) = rb[s];
  };
  auto product = [&](int buf) {
#pragma unroll
    for (int kk = 0; kk < DK; kk += 4) {
      T ao[2], bo[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        ao[t] = As[buf][kk + lg][wm + 16 * t + li];
        bo[t] = Bs[buf][kk + lg][wn + 16 * t + li];
      }
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = Mfma<T>::op(bo[b], ao[a], acc[a][b]);
    }
  };
  // chunk kc sits in buffer kc % 2 during its products; the registers of set
  // 0 hold the next odd chunk, those of set 1 the next even one
  const int nk = (int)((K + DK - 1) / DK);
  fetch(0, 1);
  stage(0, 1);
  if (nk > 1) fetch(1, 0);
  __syncthreads();
  for (int kc = 0; kc < nk; kc += 2) {
    if (kc + 2 < nk) fetch(kc + 2, 1);
    product(0);
    if (kc + 1 < nk) {
      stage(1, 0);   // last read before the previous barrier
      __syncthreads();
      if (kc + 3 < nk) fetch(kc + 3, 0);
      product(1);
      if (kc + 2 < nk) stage(0, 1);
      __syncthreads();
    }
  }
  // acc[a][b][q]: row 16 a + li, column 16 b + row(lane, q) of the wave tile;
  // loads from clamped addresses, issued together
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    T cv[4][2];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t j = std::min<int64_t>(j_base + wn + 16 * b + Mfma<T>::row(lane, q), N - 1);
#pragma unroll
      for (int a = 0; a < 2; ++a) cv[q][a] = C[std::min<int64_t>(i_base + wm + 16 * a + li, M - 1) + j * ldc];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t j = j_base + wn + 16 * b + Mfma<T>::row(lane, q);
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        const int64_t i = i_base + wm + 16 * a + li;
        if (i < M && j < N) C[i + j * ldc] = cv[q][a] + alpha * acc[a][b][q];
      }
    }
  }
}

template <typename T>
void gemm_nt(T* C, int64_t ldc, const T* A, int64_t lda, const T* B, int64_t ldb, int64_t M, int64_t N, int64_t K,
             T alpha, bool lower, int64_t gr, int64_t gc, hipStream_t st, GemmRole role) {
  if (M <= 0 || N <= 0 || K <= 0) return;
  constexpr int G = 16 / sizeof(T);
  const bool vec = M % G == 0 && N % G == 0 && lda % G == 0 && ldb % G == 0 && K % (64 / sizeof(T)) == 0 &&
                   ((uintptr_t)A % 16) == 0 && ((uintptr_t)B % 16) == 0;
  const int64_t tm = ceil_div(M, TL), tn = ceil_div(N, TL);
  const bool tri = lower && M == N && gr == gc;
  const int64_t tiles = tri ? tm * (tm + 1) / 2 : tm * tn;
  const unsigned grid = (unsigned)tiles;
  const int prio = role == GEMM_AHEAD ? 1 : 0;
  const size_t pad = role == GEMM_BEHIND ? BEHIND_PAD : 0;
  if (vec)
    hipLaunchKernelGGL((k_gemm_nt<T, true>), dim3(grid), dim3(256), pad, st, C, ldc, A, lda, B, ldb, M, N, K, alpha,
                       lower ? 1 : 0, tri ? 1 : 0, gr, gc, (int)tn, prio);
  else
    hipLaunchKernelGGL((k_gemm_nt<T, false>), dim3(grid), dim3(256), pad, st, C, ldc, A, lda, B, ldb, M, N, K, alpha,
                       lower ? 1 : 0, tri ? 1 : 0, gr, gc, (int)tn, prio);
  HC_LAUNCH_CHECK();
}

hipEvent_t Prof::next() {
  if (used == ev.size()) {
    hipEvent_t e;
    HC_HIP(hipEventCreate(&e));
    ev.push_back(e);
  }
  return ev[used++];
}

double Prof::collect_ms() {
  double ms = 0;
  for (size_t i = 0; i + 1 < used; i += 2) {
    HC_HIP(hipEventSynchronize(ev[i + 1]));
    float t = 0;
    HC_HIP(hipEventElapsedTime(&t, ev[i], ev[i + 1]));
    ms += t;
  }
  used = 0;
  return ms;
}

Prof::~Prof() {
  for (hipEvent_t e : ev) (void)hipEventDestroy(e);
}

// lower-triangle entries (global row >= global col) of the C block
static double lower_entries(int64_t rc, int64_t cc, int64_t M, int64_t N) {
  double cnt = 0;
  for (int64_t j = cc; j < cc + N; ++j) cnt += (double)std::max<int64_t>(0, rc + M - std::max(rc, j));
  return cnt;
}

// C -= A B' with every operand inside the one column-major matrix S
template <typename T>
static void gemm_nt_sub(T* S, int64_t ld, int64_t rc, int64_t cc, int64_t ra, int64_t rb, int64_t ka, int64_t M,
                        int64_t N, int64_t K, bool lower, hipStream_t st, Prof* prof, GemmRole role) {
  if (M <= 0 || N <= 0 || K <= 0) return;
  if (prof) HC_HIP(hipEventRecord(prof->next(), st));
  gemm_nt<T>(S + rc + cc * ld, ld, S + ra + ka * ld, ld, S + rb + ka * ld, ld, M, N, K, T(-1), lower, rc, cc, st, role);
  if (prof) {
    HC_HIP(hipEventRecord(prof->next(), st));
    prof->flops += 2.0 * (double)K * lower_entries(rc, cc, M, N);
    prof->launches++;
  }
}

void Aux::init() {
  if (!side) HC_HIP(hipStreamCreateWithFlags(&side, hipStreamNonBlocking));
}

hipEvent_t Aux::next() {
  if (used == ev.size()) {
    hipEvent_t e;
    HC_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    ev.push_back(e);
  }
  return ev[used++];
}

Aux::~Aux() {
  for (hipEvent_t e : ev) (void)hipEventDestroy(e);
  if (side) (void)hipStreamDestroy(side);
}

// rows [0, rows_below(j)) hold every nonzero of columns <= j: the envelope
// rounded up to whole 64-blocks (dense without an envelope)
static int64_t rows_below(const int64_t* last, int64_t n, int64_t j) {
  if (!last) return n;
  return std::min<int64_t>(n, ceil_div(std::max<int64_t>(last[j], j + 1), BS) * BS);
}

// Factor the columns [K0, Kend).  Steps of 64 columns (k_panel_step) inside
// inner panels of IB columns: every step updates the inner panel's later block
// columns and the one behind it, and at the inner panel's end one MFMA update
// (K = IB) brings the rest of the columns up to Kend up to date.
static void factor_panel(double* S, int64_t n, int64_t ld, double* Linv, double tol, double fix, unsigned long long* hits,
                         int64_t K0, int64_t Kend, const int64_t* last, hipStream_t st, Prof* prof) {
  hipLaunchKernelGGL(k_chol_diag, dim3(1), dim3(256), 0, st, S, ld, K0, n, Linv + (K0 / BS) * BS * BS, tol, fix,
                     hits);
  HC_LAUNCH_CHECK();
  double* slots = Linv + ceil_div(n, BS) * BS * BS;
  int64_t cdef = 0, rdef = 0;   // tiles of L that wait in their slots (k_panel_step): row blocks before cdef, rows before rdef
  for (int64_t I0 = K0; I0 < Kend; I0 += IB) {
    const int64_t Iend = std::min<int64_t>(Kend, I0 + IB);
    const int64_t upto = Iend < Kend ? Iend + BS : Kend;   // the block column after the panel is brought up to date too
    for (int64_t c = I0; c < Iend; c += BS) {
      const int64_t c1 = std::min<int64_t>(n, c + BS);
      const bool next = c1 < Kend;
      int64_t R = rows_below(last, n, c1 - 1);
      if (next) R = std::max(R, std::min<int64_t>(n, c1 + BS));   // the next diagonal block, also when it is not reached
      if (R <= c1 && cdef == 0) continue;
      const int64_t wgs = std::max<int64_t>(1, ceil_div(R - c1, BS));
      const int64_t cend = next ? std::min(std::min(upto, n), R) : c1;
      const bool defer = next && wgs > 1;
      const int64_t tiles = cdef > c ? ceil_div(std::min(cdef, rdef) - c, BS) : 0;
      hipLaunchKernelGGL(k_panel_step, dim3((unsigned)(wgs + tiles)), dim3(256), 0, st, S, ld, n, c, cend, R, Linv,
                         slots, (int)wgs, defer ? 1 : 0, rdef, tol, fix, hits);
      HC_LAUNCH_CHECK();
      cdef = defer ? cend : 0;
      rdef = defer ? R : 0;
    }
    if (Iend < Kend) {
      const int64_t c2 = Iend + BS, R = rows_below(last, n, Iend - 1);   // Iend's own block column is up to date
      if (c2 < Kend && c2 < R)
        gemm_nt_sub<double>(S, ld, c2, c2, c2, c2, I0, R - c2, std::min(Kend, R) - c2, Iend - I0, true, st, prof, GEMM_AHEAD);
    }
  }
}

// The same in FP32: per 64-block the diagonal factor, the TRSM of
// the rows below (down to the envelope) and the eager update of the rest of
// the panel
static void factor_panel(float* S, int64_t n, int64_t ld, float* Linv, double tol, double fix, unsigned long long* hits,
                         int64_t K0, int64_t Kend, const int64_t* last, hipStream_t st, Prof*) {
  for (int64_t c = K0; c < Kend; c += BS) {
    const int64_t cb = std::min<int64_t>(BS, n - c);
    hipLaunchKernelGGL(k_chol_diag32, dim3(1), dim3(256), 0, st, S, ld, c, n, Linv + (c / BS) * BS * BS, tol,
                       fix, hits);
    HC_LAUNCH_CHECK();
    const int64_t r0 = c + cb, R = rows_below(last, n, c + cb - 1);
    if (r0 < R) {
      hipLaunchKernelGGL(k_trsm32, dim3((unsigned)ceil_div(R - r0, BS)), dim3(256), 0, st, S, ld, c, r0, R,
                         (const float*)(Linv + (c / BS) * BS * BS));
      HC_LAUNCH_CHECK();
    }
    if (r0 < Kend && r0 < R) {
      // rows [r0, R) of the panel's remaining columns [r0, min(Kend, R))
      const int64_t M = R - r0, N = std::min(Kend, R) - r0;
      hipLaunchKernelGGL(k_gemm_panel32, dim3((unsigned)ceil_div(M, BS), (unsigned)ceil_div(N, BS)), dim3(256), 0,
                         st, S + r0 + r0 * ld, ld, (const float*)(S + r0 + c * ld), ld, (const float*)(S + r0 + c * ld), ld,
                         M, N, (int)cb, r0, r0);
      HC_LAUNCH_CHECK();
    }
  }
}

template <typename T>
void dense_cholesky(T* S, int64_t n, int64_t ld, T* Linv, double tol, double fix, unsigned long long* hits,
                    hipStream_t st, Prof* prof, Aux* aux, const int64_t* last) {
  if (n <= 0) return;
  // Look-ahead.  After panel k is factored: U1 updates panel k+1 on `st`, U2
  // updates every later column on `side`.  Panel k+1 is then factored on `st`
  // while U2 runs.  U1 writes the columns that the previous U2 wrote, so it
  // waits for that U2; U2 waits for panel k to be factored.  Both stop at the
  // rows the panel's columns reach (the envelope); a panel whose columns reach
  // no row past the next panel launches no U2.  In serial mode U2 runs on
  // `st` before U1: the same launches, one at a time.
  const bool serial = aux->serial;
  hipStream_t side = st;
  bool started = false;
  hipEvent_t u2_done = nullptr;
  auto wait_u2 = [&] {
    if (u2_done) HC_HIP(hipStreamWaitEvent(st, u2_done, 0));
    u2_done = nullptr;
  };
  // rows from K on that an inner panel at K reaches; from single_from on they
  // are few everywhere, the updates are short and one panel on `st` takes the rest
  auto reach = [&](int64_t K) { return rows_below(last, n, std::min<int64_t>(n, K + IB) - 1) - K; };
  constexpr bool fp64 = std::is_same<T, double>::value;
  int64_t single_from = n;
  for (int64_t K = (n - 1) / IB * IB; fp64 && K >= 0 && reach(K) <= LOOKAHEAD_MIN; K -= IB) single_from = K;
  const int64_t wide = std::max<int64_t>(IB, aux->nb / IB * IB);
  auto width = [&](int64_t K) {   // FP32: always wide, the order of its sums depends on it
    return K >= single_from ? n - K : !fp64 || reach(K) >= WIDE_MIN ? wide : (int64_t)IB;
  };
  for (int64_t K0 = 0, Kend; K0 < n; K0 = Kend) {
    Kend = std::min<int64_t>(n, K0 + width(K0));
    factor_panel(S, n, ld, Linv, tol, fix, hits, K0, Kend, last, st, prof);
    if (Kend >= n) break;
    const int64_t K1 = std::min<int64_t>(n, Kend + width(Kend));
    const int64_t R = rows_below(last, n, Kend - 1);
    const bool u2 = K1 < R;
    if (u2 && !serial) {
      if (!started) {
        aux->init();
        aux->used = 0;
        side = aux->side;
        started = true;
      }
      hipEvent_t factored = aux->next();
      HC_HIP(hipEventRecord(factored, st));
      HC_HIP(hipStreamWaitEvent(side, factored, 0));
    }
    // U2: rows and columns [K1, R)
    if (u2)
      gemm_nt_sub<T>(S, ld, K1, K1, K1, K1, K0, R - K1, R - K1, Kend - K0, true, side, prof,
                     serial ? GEMM_PLAIN : GEMM_BEHIND);
    wait_u2();   // the previous U2 wrote the columns that U1 updates
    // U1 on the caller's stream: rows [Kend, R), columns [Kend, min(K1, R))
    if (Kend < R)
      gemm_nt_sub<T>(S, ld, Kend, Kend, Kend, Kend, K0, R - Kend, std::min(K1, R) - Kend, Kend - K0, true, st, prof,
                     GEMM_AHEAD);
    if (u2 && !serial) {
      u2_done = aux->next();
      HC_HIP(hipEventRecord(u2_done, side));
    }
  }
  wait_u2();
}

// ---------------------------------------------------------------------------
// FP64 triangular solves: one launch per pass.  A workgroup takes a block of
// TB = 128 rows (forward) or columns (backward) and runs along the other
// blocks in the order in which their results appear, its 128 x 128 tile of L
// loaded before it waits for the block's result; then the diagonal block's
// stored inverse gives its own.
// Results travel between workgroups in an exchange array that holds a marker
// (a NaN of one bit pattern) until a value is there: a consumer polls the
// values themselves, so an exchange costs one store and one load past the L2s
// and no flag or barrier.  Blocks are dealt by a ticket, so a workgroup waits
// only for ones that started before it, whatever the dispatch order or the
// other streams' load; each wait is bounded all the same (POLL_MAX loads, and
// one load per value once it has run out).
// Bound: the chain of n / 128 exchanges (about 2 us each), then L's bytes.
// A solve (both passes, one right-hand side): 700 / 1,856 / 5,056 / 20,032 rows
// 33 / 71 / 181 / 1,110 us, with two 40 / 92 / 236 / 1,287; one right-hand side
// of 1,856 / 5,056 / 20,032 rows took 107 / 284 / 1,600 us of kernel time in
// two launches per 256 rows and pass (and, launched one by one, as much again
// at the small sizes); a second tile on its way ahead of the first one's
// values changes nothing.  The 128-blocks' inverses take 22 us, the 256-blocks'
// in one workgroup each took 337.
// ---------------------------------------------------------------------------
constexpr int TB = 128;
constexpr int POLL_MAX = 1 << 20;
constexpr unsigned long long EX_EMPTY = 0x7ff8dead0badbeefull;

// values x[0..NV) from p[0..NV), once all of them are there in every lane
template <int NV>
__device__ __forceinline__ void ex_poll(const double* const* p, double (&x)[NV], int& budget) {
  unsigned long long v[NV];
  while (true) {
    bool empty = false;
#pragma unroll
    for (int i = 0; i < NV; ++i)
      v[i] = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p[i]), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int i = 0; i < NV; ++i) empty |= v[i] == EX_EMPTY;
    if (!__any(empty) || budget <= 0) break;
    --budget;
  }
#pragma unroll
  for (int i = 0; i < NV; ++i) x[i] = __longlong_as_double((long long)v[i]);
}
__device__ inline void ex_put(double* p, double x) {
  unsigned long long v = (unsigned long long)__double_as_longlong(x);
  if (v == EX_EMPTY) v = 0x7ff8000000000000ull;   // any other NaN
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void ex_clear(double* p) { *reinterpret_cast<unsigned long long*>(p) = EX_EMPTY; }

// Inverse of each 128 x 128 diagonal block, [Y0, 0; -Y1 L10 Y0, Y1] from the 64 x 64
// ones (identity where there is no second one): a wave takes 16 columns, both
// products on MFMA with the first one's output registers as the second's
// operand.  n: factored rows; the exchange array's ne rows are emptied and the
// tickets set to zero along the way.
__global__ __launch_bounds__(256) void k_inv128(const double* __restrict__ L, int64_t ld, int64_t n,
                                                const double* __restrict__ Linv, double* __restrict__ inv, int64_t ne,
                                                double* __restrict__ ex, unsigned* __restrict__ ticket) {
  typedef Mfma<double> M;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, li = lane & 15;
  const int64_t c = (int64_t)blockIdx.x * TB;
  double* X = inv + (int64_t)blockIdx.x * TB * TB;
  if (blockIdx.x == 0 && tid < 2) ticket[tid] = 0;
  for (int e = tid; e < 4 * TB; e += 256) {
    const int64_t i = c + (e & (TB - 1));
    if (i < ne) ex_clear(ex + (e / TB) * ne + i);
  }
  const double* Y0 = Linv + (c / BS) * BS * BS;
  const bool two = c + BS < n;
  const double* Y1 = two ? Y0 + BS * BS : Y0;
  for (int e = tid; e < BS * BS; e += 256) {
    const int i = e % BS, j = e / BS;
    X[i + j * TB] = Y0[e];
    X[i + (BS + j) * TB] = 0.0;
    X[BS + i + (BS + j) * TB] = two ? Y1[e] : (i == j ? 1.0 : 0.0);
  }
  v4d t[4];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    t[a] = v4d{0, 0, 0, 0};
    const int64_t row = c + BS + 16 * a + li;
    const double* pl = L + std::min<int64_t>(row, n - 1) + c * ld;
#pragma unroll 4
    for (int q = 0; two && q < 16; ++q) {   // (without a second block the columns need not exist either)
      const int m = 4 * q + (lane >> 4);
      const double l = pl[m * ld];
      t[a] = M::op(row < n ? l : 0.0, Y0[m + (16 * w + li) * BS], t[a]);
    }
  }
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    v4d y = v4d{0, 0, 0, 0};
#pragma unroll
    for (int b = 0; b <= a; ++b)
#pragma unroll
      for (int q = 0; q < 4; ++q) y = M::op(Y1[(16 * a + li) + (16 * b + M::row(lane, q)) * BS], t[b][q], y);
#pragma unroll
    for (int q = 0; q < 4; ++q) X[BS + 16 * a + M::row(lane, q) + (16 * w + li) * TB] = -y[q];
  }
}

// y = L^-1 b.  Lane l holds rows l and l + 64 of its block, wave w the columns
// 16 w .. 16 w + 15 of each tile; the waves' sums meet in LDS once per block.
template <int NR>
__global__ __launch_bounds__(512) void k_tri_fwd(const double* __restrict__ L, int64_t ld, int64_t n,
                                                 const double* __restrict__ inv, const int32_t* __restrict__ lo,
                                                 const double* __restrict__ b0, const double* __restrict__ b1,
                                                 double* ex_y, double* __restrict__ ex_x,
                                                 unsigned* __restrict__ ticket) {
  __shared__ double part[8][NR][TB];
  __shared__ double bb[NR][TB];
  __shared__ int blk;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (tid == 0) blk = (int)atomicAdd(&ticket[0], 1u);
  __syncthreads();
  const int B = __builtin_amdgcn_readfirstlane(blk);
  if (B == 0 && tid == 0) ticket[1] = 0;   // the backward pass's
  const int64_t c = (int64_t)B * TB;
  const int ri = tid & (TB - 1), rr = tid / TB;   // row and right-hand side of the block's vectors
  const bool mine = rr < NR && c + ri < n;
  if (mine) ex_clear(ex_x + rr * n + c + ri);
  const double rhs = mine ? (rr == 0 ? b0 : b1)[c + ri] : 0.0;
  const double* X = inv + (int64_t)B * TB * TB + lane + 16 * w * TB;
  const double* p0 = L + std::min<int64_t>(c + lane, n - 1) + 16 * w * ld;
  const double* p1 = L + std::min<int64_t>(c + 64 + lane, n - 1) + 16 * w * ld;
  double l0[16], l1[16], x0[16], x1[16], acc[NR][2] = {};
  auto load = [&](int k) {
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      l0[q] = p0[((int64_t)k * TB + q) * ld];
      l1[q] = p1[((int64_t)k * TB + q) * ld];
    }
  };
  const int k0 = lo ? lo[B] : 0;
  if (k0 < B) load(k0);
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    x0[q] = X[q * TB];
    x1[q] = X[q * TB + 64];
  }
  // lane 16 r + q of a wave polls y[q] of right-hand side r
  const double* py = ex_y + ((lane >> 4) % NR) * n + 16 * w + (lane & 15);
  int budget = POLL_MAX;
  for (int k = k0; k < B; ++k) {
    const double* const at[1] = {py + (int64_t)k * TB};
    double y[1];
    ex_poll<1>(at, y, budget);
#pragma unroll
    for (int q = 0; q < 16; ++q)
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const double yq = lane_bcast(y[0], 16 * r + q);
        acc[r][0] = fma(l0[q], yq, acc[r][0]);
        acc[r][1] = fma(l1[q], yq, acc[r][1]);
      }
    if (k + 1 < B) load(k + 1);
  }
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    part[w][r][lane] = acc[r][0];
    part[w][r][64 + lane] = acc[r][1];
  }
  __syncthreads();
  if (rr < NR) {
    double v = rhs;
#pragma unroll
    for (int u = 0; u < 8; ++u) v -= part[u][rr][ri];
    bb[rr][ri] = mine ? v : 0.0;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const double t = bb[r][16 * w + q];
      s0 = fma(x0[q], t, s0);
      s1 = fma(x1[q], t, s1);
    }
    part[w][r][lane] = s0;
    part[w][r][64 + lane] = s1;
  }
  __syncthreads();
  if (mine) {
    double v = 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) v += part[u][rr][ri];
    ex_put(ex_y + rr * n + c + ri, v);
  }
}

// sums a[0..15] over the wave: lane l returns the total of a[l / 4].  Each level
// halves the values and the lanes they are spread over: lane-group swaps for 32
// and 16 lanes, DPP below.  It stands in the chain twice per block and
// right-hand side; with shuffles through LDS a backward pass with two of them
// took 211 us at 5,056 rows, now 142.
template <int CTRL> __device__ inline double dpp(double v) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)b, CTRL, 0xf, 0xf, true),
                 hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
template <int CTRL> __device__ inline double halve(double lower, double upper, bool up) {
  return (up ? upper : lower) + dpp<CTRL>(up ? lower : upper);
}
__device__ __forceinline__ double wave_sum16(double (&a)[16], int lane) {
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    swap32(a[q], a[q + 8]);
    a[q] += a[q + 8];
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    swap16(a[q], a[q + 4]);
    a[q] += a[q + 4];
  }
  const double b0 = halve<0x128>(a[0], a[2], lane & 8), b1 = halve<0x128>(a[1], a[3], lane & 8);   // row_ror 8
  double s = halve<0x141>(b0, b1, lane & 4);   // row_half_mirror
  s += dpp<0xB1>(s);                           // quad_perm [1, 0, 3, 2]
  return s + dpp<0x4E>(s);                     // quad_perm [2, 3, 0, 1]
}

// x = L^-T y, last block first.  Lane l holds the rows l and l + 64 of a tile,
// wave w the block's columns 16 w .. 16 w + 15, summed over the lanes at the end.
template <int NR>
__global__ __launch_bounds__(512) void k_tri_bwd(const double* __restrict__ L, int64_t ld, int64_t n,
                                                 const double* __restrict__ inv, const int32_t* __restrict__ hi,
                                                 double* __restrict__ ex_y, double* ex_x,
                                                 unsigned* __restrict__ ticket, double* __restrict__ o0,
                                                 double* __restrict__ o1) {
  __shared__ double bb[NR][TB];
  __shared__ int blk;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nb = (int)((n + TB - 1) / TB);
  if (tid == 0) {
    blk = nb - 1 - (int)atomicAdd(&ticket[1], 1u);
    if (blk == nb - 1) ticket[0] = 0;   // the forward pass's
  }
  __syncthreads();
  const int B = __builtin_amdgcn_readfirstlane(blk);
  const int64_t c = (int64_t)B * TB;
  const double* X = inv + (int64_t)B * TB * TB + lane + 16 * w * TB;
  const double* pl = L + (c + 16 * w) * ld;
  double l0[16], l1[16], x0[16], x1[16], acc[NR][16] = {};
  auto load = [&](int k) {   // columns past n do not occur: a block with blocks after it is whole
    const int64_t i = (int64_t)k * TB + lane;
    const double *p0 = pl + std::min<int64_t>(i, n - 1), *p1 = pl + std::min<int64_t>(i + 64, n - 1);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      l0[q] = p0[q * ld];
      l1[q] = p1[q * ld];
    }
  };
  const int kh = hi ? hi[B] : nb - 1;
  if (kh > B) load(kh);
  // y of this wave's columns, one per group of four lanes; then that place is emptied
  const int64_t j = c + 16 * w + (lane >> 2);
  double y[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    y[r] = j < n ? ex_y[r * n + j] : 0.0;
    __builtin_amdgcn_wave_barrier();
    if (j < n && (lane & 3) == 0) ex_clear(ex_y + r * n + j);
  }
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    x0[q] = X[q * TB];
    x1[q] = X[q * TB + 64];
  }
  int budget = POLL_MAX;
  for (int k = kh; k > B; --k) {
    const int64_t i = (int64_t)k * TB + lane;
    const double* at[2 * NR];
    at[0] = ex_x + std::min<int64_t>(i, n - 1);
    at[1] = ex_x + std::min<int64_t>(i + 64, n - 1);
    if constexpr (NR == 2) {
      at[2] = at[0] + n;
      at[3] = at[1] + n;
    }
    double v[2 * NR];
    ex_poll<2 * NR>(at, v, budget);
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const double v0 = i < n ? v[2 * r] : 0.0;   // rows past n repeat the last one's entries of L
      const double v1 = i + 64 < n ? v[2 * r + 1] : 0.0;
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[r][q] = fma(l1[q], v1, fma(l0[q], v0, acc[r][q]));
    }
    if (k - 1 > B) load(k - 1);
  }
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const double s = wave_sum16(acc[r], lane);
    if ((lane & 3) == 0) bb[r][16 * w + (lane >> 2)] = j < n ? y[r] - s : 0.0;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const double t0 = bb[r][lane], t1 = bb[r][64 + lane];
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[r][q] = fma(x1[q], t1, x0[q] * t0);
    const double s = wave_sum16(acc[r], lane);
    if (j < n && (lane & 3) == 0) {
      ex_put(ex_x + r * n + j, s);
      (r == 0 ? o0 : o1)[j] = s;
    }
  }
}

int64_t tri_inv_elems(int64_t n) { return ceil_div(n, TB) * TB * TB; }
int64_t tri_exchange_elems(int64_t n) { return n > 0 ? 4 * n + 1 : 0; }

void tri_envelope(int64_t n, const int64_t* last, std::vector<int32_t>& lo, std::vector<int32_t>& hi) {
  const int64_t nb = ceil_div(n, TB);
  lo.assign(nb, 0);
  hi.assign(nb, 0);
  for (int64_t k = 0; k < nb; ++k)
    hi[k] = (int32_t)((rows_below(last, n, std::min<int64_t>(n, (k + 1) * TB) - 1) - 1) / TB);
  for (int64_t b = 0, k = 0; b < nb; ++b) {   // hi is non-decreasing
    while (hi[k] < b) ++k;
    lo[b] = (int32_t)k;
  }
}

void tri_prepare(const TriSolve& t, const double* L, int64_t nf, int64_t ld, const double* Linv, hipStream_t st) {
  if (t.n <= 0) return;
  hipLaunchKernelGGL(k_inv128, dim3((unsigned)ceil_div(t.n, TB)), dim3(256), 0, st, L, ld, nf, Linv, t.inv, t.n, t.ex,
                     (unsigned*)(t.ex + 4 * t.n));
  HC_LAUNCH_CHECK();
}

template <int NR>
static void tri_solve_nr(const TriSolve& t, const double* L, int64_t ld, const double* b0, const double* b1, double* x0,
                         double* x1, hipStream_t st) {
  const unsigned nb = (unsigned)ceil_div(t.n, TB);
  double *ey = t.ex, *exx = t.ex + 2 * t.n;
  unsigned* ticket = (unsigned*)(t.ex + 4 * t.n);
  hipLaunchKernelGGL((k_tri_fwd<NR>), dim3(nb), dim3(512), 0, st, L, ld, t.n, (const double*)t.inv, t.lo, b0, b1, ey,
                     exx, ticket);
  HC_LAUNCH_CHECK();
  hipLaunchKernelGGL((k_tri_bwd<NR>), dim3(nb), dim3(512), 0, st, L, ld, t.n, (const double*)t.inv, t.hi, ey, exx,
                     ticket, x0, x1);
  HC_LAUNCH_CHECK();
}

void tri_solve(const TriSolve& t, const double* L, int64_t ld, const double* const* b, double* const* x, int nrhs,
               hipStream_t st) {
  if (t.n <= 0) return;
  for (int r = 0; r + 1 < nrhs; r += 2) tri_solve_nr<2>(t, L, ld, b[r], b[r + 1], x[r], x[r + 1], st);
  if (nrhs % 2) tri_solve_nr<1>(t, L, ld, b[nrhs - 1], nullptr, x[nrhs - 1], nullptr, st);
}

// ---------------------------------------------------------------------------
// The FP32 mode's triangular solves (a launch per 256-row block and pass; like
// its panel they keep their order of operations).
// Inverses of the 256 x 256 diagonal blocks of L (one workgroup per block),
// from the 64 x 64 block inverses:  X_ii = Linv_i,
// X_ij = -Linv_i sum_{k=j}^{i-1} L_ik X_kj  (i > j).  X and X' are stored
// column-major with leading dimension 256 (block b at b * 256 * 256).
// ---------------------------------------------------------------------------
constexpr int SB = 256;   // rows per triangular-solve step
constexpr int MAXRHS = 4;

__global__ __launch_bounds__(256) void k_inv256(const float* __restrict__ L, int64_t ld, const float* __restrict__ Linv,
                                                int64_t n, float* __restrict__ Xall, float* __restrict__ XTall) {
  __shared__ float Tt[BS][BS + 1];
  const int tid = threadIdx.x;
  const int64_t c = (int64_t)blockIdx.x * SB;
  const int cb = (int)std::min<int64_t>(SB, n - c);
  const int nsub = (cb + BS - 1) / BS;
  float* X = Xall + (int64_t)blockIdx.x * SB * SB;
  float* XT = XTall + (int64_t)blockIdx.x * SB * SB;
  for (int e = tid; e < SB * SB; e += 256) {
    const int i = e % SB, j = e / SB;
    float v = 0;
    if (i / BS == j / BS) {
      if (i / BS < nsub) v = Linv[((c + (i / BS) * BS) / BS) * BS * BS + (i % BS) + (j % BS) * BS];
      else v = (i == j) ? float(1) : float(0);
    }
    X[i + j * SB] = v;
  }
  __syncthreads();
  const int i0 = 4 * (tid % 16), j0 = 4 * (tid / 16);
  for (int jb = 0; jb < nsub; ++jb)
    for (int ib = jb + 1; ib < nsub; ++ib) {
      float acc[4][4] = {};
      for (int kb = jb; kb < ib; ++kb)
        for (int p = 0; p < BS; ++p) {
          float la[4], xb[4];
#pragma unroll
          for (int a = 0; a < 4; ++a) {
            const int row = ib * BS + i0 + a;   // local row inside the 256 block
            la[a] = (row < cb && kb * BS + p < cb) ? L[(c + row) + (c + kb * BS + p) * ld] : float(0);
          }
#pragma unroll
          for (int q = 0; q < 4; ++q) xb[q] = X[(kb * BS + p) + (jb * BS + j0 + q) * SB];
#pragma unroll
          for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[a][q] += la[a] * xb[q];
        }
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int q = 0; q < 4; ++q) Tt[i0 + a][j0 + q] = acc[a][q];
      __syncthreads();
      const float* Li = X + (ib * BS) + (ib * BS) * SB;   // Linv_ib sits on X's diagonal
      float out[4][4] = {};
      for (int p = 0; p < BS; ++p) {
        float la[4], tb[4];
#pragma unroll
        for (int a = 0; a < 4; ++a) la[a] = Li[(i0 + a) + p * SB];
#pragma unroll
        for (int q = 0; q < 4; ++q) tb[q] = Tt[p][j0 + q];
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int q = 0; q < 4; ++q) out[a][q] -= la[a] * tb[q];
      }
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int q = 0; q < 4; ++q) X[(ib * BS + i0 + a) + (jb * BS + j0 + q) * SB] = out[a][q];
      __syncthreads();
    }
  for (int e = tid; e < SB * SB; e += 256) {
    const int i = e % SB, j = e / SB;
    XT[i + j * SB] = X[j + i * SB];
  }
}

int64_t inv256_elems(int64_t n) { return ceil_div(n, SB) * SB * SB; }

void dense_block_inverses(const float* L, int64_t n, int64_t ld, const float* Linv, float* X, float* XT, hipStream_t st) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_inv256, dim3((unsigned)ceil_div(n, SB)), dim3(256), 0, st, L, ld, Linv, n, X, XT);
  HC_LAUNCH_CHECK();
}

// ---------------------------------------------------------------------------
// triangular solves, nrhs <= 4 right-hand sides stored column-major with
// leading dimension n:  forward Y = L^-1 B (B overwritten), backward
// X = L^-T Y (Y overwritten).  Per 256-row block: one workgroup applies the
// block inverse (a 256 x 256 triangular matvec), then a bandwidth-bound kernel
// updates the rows below (forward) or the columns to the left (backward).
// ---------------------------------------------------------------------------
// Yout[c + i] = sum_k Xinv[i + k * 256] Bin[c + k] for the 256 x 256 block
// inverse Xinv (lower for the forward pass, upper for the backward one).
// 16 workgroups of 16 rows each; thread (row, g) sums k in [16 g, 16 g + 16)
// and the 16 partial sums meet in LDS.  The stored inverse is zero outside
// its triangle and bb is zero past cb, so loads and products need no masks.
constexpr int DIAG_ROWS = 16;
template <int NR>
__global__ __launch_bounds__(256) void k_trsv_diag(const float* __restrict__ Xinv, int64_t c, int64_t n,
                                                   const float* __restrict__ Bin, float* __restrict__ Yout, int nrhs) {
  __shared__ float bb[SB][NR];
  __shared__ float part[16][DIAG_ROWS][NR];
  const int tid = threadIdx.x;
  const int cb = (int)std::min<int64_t>(SB, n - c);
  const int il = tid % DIAG_ROWS, g = tid / DIAG_ROWS;
  const int i = blockIdx.x * DIAG_ROWS + il;
  // the inverse's entries do not depend on the previous kernel: their loads
  // are issued before the right-hand side's, so the two latencies overlap
  float x[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) x[q] = Xinv[i + (int64_t)(g * 16 + q) * SB];
  for (int e = tid; e < SB * NR; e += 256) {
    const int ie = e % SB, r = e / SB;
    bb[ie][r] = (ie < cb && r < nrhs) ? Bin[(c + ie) + r * n] : float(0);
  }
  __syncthreads();
  float acc[NR] = {};
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int k = g * 16 + q;
#pragma unroll
    for (int r = 0; r < NR; ++r) acc[r] += x[q] * bb[k][r];
  }
#pragma unroll
  for (int r = 0; r < NR; ++r) part[g][il][r] = acc[r];
  __syncthreads();
  if (tid < DIAG_ROWS * NR) {
    const int row = tid % DIAG_ROWS, r = tid / DIAG_ROWS;
    float v = 0;
#pragma unroll
    for (int gg = 0; gg < 16; ++gg) v += part[gg][row][r];
    const int ig = blockIdx.x * DIAG_ROWS + row;
    if (ig < cb && r < nrhs) Yout[(c + ig) + r * n] = v;
  }
}

// rows below the block: B[row] -= L[row, c:c+cb] y_c.  A workgroup takes 64
// rows; wave w sums columns [16 w, 16 w + 16) with one lane per row (each
// column read is 256 contiguous bytes, 16 loads in flight per lane), and the
// 16 partial sums meet in LDS.
template <int NR>
__global__ __launch_bounds__(1024) void k_trsv_fwd_update(const float* __restrict__ L, int64_t ld, int64_t c, int64_t n,
                                                          float* __restrict__ B, const float* __restrict__ Y, int nrhs) {
  __shared__ float yb[SB][NR];
  __shared__ float part[16][64][NR];
  const int tid = threadIdx.x;
  const int cb = (int)std::min<int64_t>(SB, n - c);
  const int lane = tid & 63, w = tid >> 6;
  const int64_t row = c + cb + (int64_t)blockIdx.x * 64 + lane;
  const int64_t rowc = std::min<int64_t>(row, n - 1);
  // L's entries do not depend on the previous kernel: loaded before y
  float l[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) l[q] = L[rowc + (c + std::min(w * 16 + q, cb - 1)) * ld];   // yb is zero past cb
  // the entry of B this thread updates at the end (final before this kernel)
  const int64_t rw = c + cb + (int64_t)blockIdx.x * 64 + (tid % 64);
  const int rr = tid / 64;
  const bool writer = tid < 64 * NR && rw < n && rr < nrhs;
  const float bold = writer ? B[rw + rr * n] : float(0);
  for (int e = tid; e < SB * NR; e += 1024) {
    const int i = e % SB, r = e / SB;
    yb[i][r] = (i < cb && r < nrhs) ? Y[(c + i) + r * n] : float(0);
  }
  __syncthreads();
  float acc[NR] = {};
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int k = w * 16 + q;
#pragma unroll
    for (int r = 0; r < NR; ++r) acc[r] += l[q] * yb[k][r];
  }
#pragma unroll
  for (int r = 0; r < NR; ++r) part[w][lane][r] = acc[r];
  __syncthreads();
  if (tid < 64 * NR) {
    const int ln = tid % 64;
    float v = 0;
#pragma unroll
    for (int ww = 0; ww < 16; ++ww) v += part[ww][ln][rr];
    if (writer) B[rw + rr * n] = bold - v;
  }
}

// columns left of the block: Y[j] -= sum_i L[c + i, j] x[i]; each wave takes
// four columns (16 loads in flight per lane), lanes run over i
constexpr int BWD_COLS = 4;
template <int NR>
__global__ __launch_bounds__(256) void k_trsv_bwd_update(const float* __restrict__ L, int64_t ld, int64_t c, int64_t n,
                                                         int64_t j_begin, float* __restrict__ Yv, const float* __restrict__ X,
                                                         int nrhs) {
  __shared__ float xb[SB][NR];
  const int tid = threadIdx.x;
  const int cb = (int)std::min<int64_t>(SB, n - c);
  const int lane = tid & 63;
  const int64_t j0 = j_begin + ((int64_t)blockIdx.x * 4 + (tid >> 6)) * BWD_COLS;
  // L's entries do not depend on the previous kernel: loaded before x
  float l[BWD_COLS][SB / 64];
#pragma unroll
  for (int cc = 0; cc < BWD_COLS; ++cc) {
    const int64_t j = std::min<int64_t>(j0 + cc, c - 1);
#pragma unroll
    for (int q = 0; q < SB / 64; ++q) l[cc][q] = L[(c + std::min(lane + 64 * q, cb - 1)) + j * ld];   // xb is zero past cb
  }
  // the entries of Y lane 0 updates at the end (final before this kernel)
  float yold[BWD_COLS][NR] = {};
  if (lane == 0)
#pragma unroll
    for (int cc = 0; cc < BWD_COLS; ++cc)
      if (j0 + cc < c)
#pragma unroll
        for (int r = 0; r < NR; ++r)
          if (r < nrhs) yold[cc][r] = Yv[(j0 + cc) + r * n];
  for (int e = tid; e < SB * NR; e += 256) {
    const int i = e % SB, r = e / SB;
    xb[i][r] = (i < cb && r < nrhs) ? X[(c + i) + r * n] : float(0);
  }
  __syncthreads();
  float acc[BWD_COLS][NR] = {};
#pragma unroll
  for (int cc = 0; cc < BWD_COLS; ++cc) {
#pragma unroll
    for (int q = 0; q < SB / 64; ++q) {
      const int i = lane + 64 * q;
#pragma unroll
      for (int r = 0; r < NR; ++r) acc[cc][r] += l[cc][q] * xb[i][r];
    }
  }
#pragma unroll
  for (int cc = 0; cc < BWD_COLS; ++cc)
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      float v = acc[cc][r];
      for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
      acc[cc][r] = v;
    }
  if (lane == 0)
#pragma unroll
    for (int cc = 0; cc < BWD_COLS; ++cc)
      if (j0 + cc < c)
#pragma unroll
        for (int r = 0; r < NR; ++r)
          if (r < nrhs) Yv[(j0 + cc) + r * n] = yold[cc][r] - acc[cc][r];
}

// With an envelope (`last`, see dense_cholesky) the forward updates stop at
// the rows a block's columns reach and the backward updates start at the
// first column its rows reach: entries outside are zero.
template <int NR>
static void dense_solve_nr(const float* L, int64_t n, int64_t ld, const float* X256, const float* XT256, float* B, float* Y, float* X,
                           int nrhs, const int64_t* last, hipStream_t st) {
  for (int64_t c = 0; c < n; c += SB) {
    const float* Xi = X256 + (c / SB) * SB * SB;
    hipLaunchKernelGGL((k_trsv_diag<NR>), dim3(SB / DIAG_ROWS), dim3(256), 0, st, Xi, c, n, (const float*)B, Y, nrhs);
    HC_LAUNCH_CHECK();
    const int64_t cend = std::min<int64_t>(n, c + SB);
    const int64_t below = rows_below(last, n, cend - 1) - cend;
    if (below > 0) {
      hipLaunchKernelGGL((k_trsv_fwd_update<NR>), dim3((unsigned)ceil_div(below, 64)), dim3(1024), 0, st, L, ld, c,
                         n, B, (const float*)Y, nrhs);
      HC_LAUNCH_CHECK();
    }
  }
  const int64_t lastb = ((n - 1) / SB) * SB;
  for (int64_t c = lastb; c >= 0; c -= SB) {
    const float* XTi = XT256 + (c / SB) * SB * SB;
    hipLaunchKernelGGL((k_trsv_diag<NR>), dim3(SB / DIAG_ROWS), dim3(256), 0, st, XTi, c, n, (const float*)Y, X, nrhs);
    HC_LAUNCH_CHECK();
    // first column with a nonzero in rows >= c (last is non-decreasing)
    int64_t jb = 0;
    if (last) jb = (std::upper_bound(last, last + c, c) - last) / (4 * BWD_COLS) * (4 * BWD_COLS);
    if (c > jb) {
      hipLaunchKernelGGL((k_trsv_bwd_update<NR>), dim3((unsigned)ceil_div(c - jb, 4 * BWD_COLS)), dim3(256), 0, st,
                         L, ld, c, n, jb, Y, (const float*)X, nrhs);
      HC_LAUNCH_CHECK();
    }
  }
}

// kernels specialised for one right-hand side (the iteration's case) and for
// up to MAXRHS
void dense_solve(const float* L, int64_t n, int64_t ld, const float* X256, const float* XT256, float* B, float* Y, float* X, int nrhs,
                 hipStream_t st, const int64_t* last) {
  if (n <= 0) return;
  if (nrhs == 1) dense_solve_nr<1>(L, n, ld, X256, XT256, B, Y, X, nrhs, last, st);
  else if (nrhs == 2) dense_solve_nr<2>(L, n, ld, X256, XT256, B, Y, X, nrhs, last, st);
  else dense_solve_nr<MAXRHS>(L, n, ld, X256, XT256, B, Y, X, nrhs, last, st);
}

template void dense_cholesky<double>(double*, int64_t, int64_t, double*, double, double, unsigned long long*,
                                     hipStream_t, Prof*, Aux*, const int64_t*);
template void dense_cholesky<float>(float*, int64_t, int64_t, float*, double, double, unsigned long long*,
                                    hipStream_t, Prof*, Aux*, const int64_t*);
template void gemm_nt<double>(double*, int64_t, const double*, int64_t, const double*, int64_t, int64_t, int64_t,
                              int64_t, double, bool, int64_t, int64_t, hipStream_t, GemmRole);
template void gemm_nt<float>(float*, int64_t, const float*, int64_t, const float*, int64_t, int64_t, int64_t,
                             int64_t, float, bool, int64_t, int64_t, hipStream_t, GemmRole);
int64_t linv_elems(int64_t n) { return n > 0 ? (ceil_div(n, BS) + SLOTS) * BS * BS : 0; }
int64_t linv32_elems(int64_t n) { return ceil_div(n, BS) * BS * BS; }

// factor flops of a dense n x n Cholesky
double cholesky_flops(int64_t n) { return (double)n * n * n / 3.0; }

double envelope_cholesky_flops(int64_t n, const int64_t* last) {
  if (!last) return cholesky_flops(n);
  double f = 0;
  for (int64_t j = 0; j < n; ++j) {
    const double h = (double)(std::max<int64_t>(last[j], j + 1) - j - 1);   // rows below the pivot
    f += h * h + h;
  }
  return f;
}

}  // namespace hc
