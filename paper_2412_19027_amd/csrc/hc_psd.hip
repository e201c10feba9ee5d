// PSD cones (gfx950): scaling, products with H, d_s, step lengths, and the
// explicit inverse blocks.
//
// Every kernel but the blocks' takes one workgroup per cone (step lengths: per
// half of one): one wave up to side 16, four above.  The matrices are at most
// 32 x 32, so a cone is a chain of short dependent operations and what counts
// is the length of that chain: contractions run on MFMA (v_mfma_f64_16x16x4f64,
// one 16 x 16 tile per wave), factorisations keep their matrix in registers
// (four entries a thread) and exchange one column per step through LDS, and all
// segments of a size class share a launch.
#include "hc_cones.h"

namespace hc {
constexpr int PSD_SMALL = 16, PSD_LARGE = 32;   // sides of the two size classes

// matrices sit in LDS as KM rows of LD, zero outside k x k
template <int KM> struct Psd {
  static constexpr int NT = KM <= 16 ? 64 : 256;
  static constexpr int RS = NT / KM;   // thread t owns column t % KM, rows t / KM + RS q, q < 4
  static constexpr int LD = KM + 1, MAT = KM * LD;
  static constexpr int G = NT / (KM / 2) >= 16 ? 16 : 8;   // lanes per pair of columns (Jacobi)
};
template <int KM> struct PsdShared {
  double ca[2][KM], cb[2][KM], td[KM], te[KM];
};

// 1/sqrt(x), 1/x: the hardware's estimate and one third-order step
__device__ inline double rsqrt_step(double x) {
  const double y = __builtin_amdgcn_rsq(x), e = fma(-(x * y), y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}
__device__ inline double rcp_step(double x) {
  const double y = __builtin_amdgcn_rcp(x), e = fma(-x, y, 1.0);
  return fma(y, fma(e, e, e), y);
}

template <int CTRL> __device__ inline double dpp(double v) {
  const int64_t b = __double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)b, CTRL, 0xf, 0xf, true),
                 hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double((int64_t)(((uint64_t)hi << 32) | lo));
}
// sum over aligned groups of W lanes (8, 16 or 32), the same bits on each
template <int W> __device__ inline double group_sum(double v) {
  v += dpp<0xB1>(v);    // quad_perm [1, 0, 3, 2]
  v += dpp<0x4E>(v);    // quad_perm [2, 3, 0, 1]
  v += dpp<0x141>(v);   // row_half_mirror
  if (W > 8) v += dpp<0x140>(v);   // row_mirror
  if (W > 16) v += __shfl_xor(v, 16, 64);
  return v;
}

// (i, j) of entry e of the packed triangle i >= j (row by row)
__device__ inline void tri_index(int e, int& i, int& j) {
  i = (int)((sqrt(8.0 * e + 1.0) - 1.0) / 2.0);
  while (i * (i + 1) / 2 > e) --i;
  while ((i + 1) * (i + 2) / 2 <= e) ++i;
  j = e - i * (i + 1) / 2;
}
// entry (i, j) of smat(v)
__device__ inline double smat_at(const double* v, int i, int j) {
  const int hi = max(i, j), lo = min(i, j);
  return v[hi * (hi + 1) / 2 + lo] * (i == j ? 1.0 : 0.70710678118654752440);
}

// calls f(i, l, in) for the thread's four entries; in: inside k x k
template <int KM, typename F> __device__ inline void psd_each(int k, F&& f) {
  const int l = threadIdx.x % KM, i0 = threadIdx.x / KM;
#pragma unroll
  for (int q = 0; q < 4; ++q) f(i0 + Psd<KM>::RS * q, l, i0 + Psd<KM>::RS * q < k && l < k);
}

// e with 2^e times the largest magnitude of the workgroup's entries in [1, 2)
// (less for subnormal ones; 0 beside an infinity or a NaN), the same in every
// thread, from the entries' upper words; w: LDS that nobody reads any more
template <int KM> __device__ inline int psd_unit_exp(const double (&d)[4], double* w) {
  int h = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) h = max(h, __double2hiint(d[q]) & 0x7fffffff);
  h = max(h, __builtin_amdgcn_mov_dpp(h, 0xB1, 0xf, 0xf, true));    // as group_sum
  h = max(h, __builtin_amdgcn_mov_dpp(h, 0x4E, 0xf, 0xf, true));
  h = max(h, __builtin_amdgcn_mov_dpp(h, 0x141, 0xf, 0xf, true));
  h = max(h, __builtin_amdgcn_mov_dpp(h, 0x140, 0xf, 0xf, true));
  h = max(max(__builtin_amdgcn_readlane(h, 0), __builtin_amdgcn_readlane(h, 16)),
          max(__builtin_amdgcn_readlane(h, 32), __builtin_amdgcn_readlane(h, 48)));
  if (Psd<KM>::NT > 64) {
    int* hw = reinterpret_cast<int*>(w);
    if ((threadIdx.x & 63) == 0) hw[threadIdx.x >> 6] = h;
    __syncthreads();
    h = max(max(hw[0], hw[1]), max(hw[2], hw[3]));
  }
  return h < 0x7ff00000 ? 1023 - max(h >> 20, 1) : 0;
}

// C = op(X) op(Y), tx / ty transpose X / Y (C is neither; one 16 x 16 tile per
// wave).  Lane l holds A[l % 16][l / 16] and B[l / 16][l % 16] of a step and
// rows l / 16 + 4 r of column l % 16 of the result.
typedef double v4d __attribute__((ext_vector_type(4)));
template <int KM>
__device__ inline void psd_mm(const double* X, bool tx, const double* Y, bool ty, int k, double* C) {
  constexpr int LD = Psd<KM>::LD;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int i = (w >> 1) * 16 + (lane & 15), j = (w & 1) * 16 + (lane & 15), p0 = lane >> 4;
  v4d c = {0.0, 0.0, 0.0, 0.0};
  for (int p = p0; p - p0 < k; p += 4) {
    const double a = tx ? X[p * LD + i] : X[i * LD + p], b = ty ? Y[j * LD + p] : Y[p * LD + j];
    c = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) C[((w >> 1) * 16 + p0 + 4 * r) * LD + j] = c[r];
  __syncthreads();
}

// smallest eigenvalue of the symmetric matrix whose entry (i, l) the threads
// hold in d: Householder reduction to tridiagonal form, then multisection: 64
// shifts a round, each lane testing one by the signs of the leading minors of
// T - x (three-term recurrence, rescaled).  Nine rounds leave 2^-54 of the
// initial interval, which lies in [-b, b] for b the largest row sum of T.  The
// matrix is first scaled by a power of two to entries below 2, so that neither
// squares nor the reflection's reciprocal leave the range of a double: a column
// whose squares add up to less than 1e-280 (entries under 1e-140 of the largest
// one, which move no eigenvalue) counts as reduced.
// k reductions of two barriers each; two-sided Jacobi took about seven sweeps
// of k - 1 rounds with three barriers and twice the matrix through LDS.
template <int KM> __device__ __forceinline__ double psd_min_eig(double (&d)[4], int k, PsdShared<KM>& sh) {
  const int l = threadIdx.x % KM, lane = threadIdx.x & 63;
  __syncthreads();   // the exchange buffers' previous readers are done
  const int unit = psd_unit_exp<KM>(d, sh.td);
#pragma unroll
  for (int q = 0; q < 4; ++q) d[q] = ldexp(d[q], unit);
  for (int j = 0; j < k - 2; ++j) {
    double *x = sh.ca[j & 1], *pv = sh.cb[j & 1];
    int q = 0;
    psd_each<KM>(k, [&](int i, int, bool in) {
      if (in && l == j && i >= j) x[i] = d[q];
      ++q;
    });
    __syncthreads();
    const double xl = l > j && l < k ? x[l] : 0.0, x1 = x[j + 1];
    const double s2 = group_sum<KM>(l > j + 1 ? xl * xl : 0.0);
    if (threadIdx.x == 0) sh.td[j] = x[j];
    if (s2 < 1e-280) {   // nothing to reflect (every thread has the same s2)
      if (threadIdx.x == 0) sh.te[j] = x1;
      continue;
    }
    // I - t v v' with v = (x1 - a, rest) takes the column to (a, 0, ...)
    const double n2 = x1 * x1 + s2, a = -copysign(n2 * rsqrt_step(n2), x1), v1 = x1 - a, t = -rcp_step(a * v1);
    const double vl = l == j + 1 ? v1 : xl;
    double p[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) p[r] = t * group_sum<KM>(d[r] * vl);
    q = 0;
    psd_each<KM>(k, [&](int i, int, bool) {
      if (l == 0 && i < k) pv[i] = p[q];
      ++q;
    });
    __syncthreads();
    const double pl = l > j && l < k ? pv[l] : 0.0;
    const double K = 0.5 * t * group_sum<KM>(pl * vl), wl = pl - K * vl;
    if (threadIdx.x == 0) sh.te[j] = a;
    q = 0;
    psd_each<KM>(k, [&](int i, int, bool) {
      const bool on = i > j && i < k;
      const double vi = !on ? 0.0 : i == j + 1 ? v1 : x[i], wi = on ? p[q] - K * vi : 0.0;
      const bool up = i >= l;   // (i, l) and (l, i) get the same bits
      d[q] -= fma(up ? vi : vl, up ? wl : wi, (up ? wi : wl) * (up ? vl : vi));
      ++q;
    });
  }
  {
    int q = 0;
    psd_each<KM>(k, [&](int i, int, bool in) {
      if (in && i == l && i >= k - 2) sh.td[i] = d[q];
      if (in && i == l + 1 && i == k - 1) sh.te[l] = d[q];
      ++q;
    });
  }
  __syncthreads();
  double b = 0.0, dmin = INFINITY;
  if (lane < k) {
    dmin = sh.td[lane];
    b = fabs(dmin) + (lane > 0 ? fabs(sh.te[lane - 1]) : 0.0) + (lane < k - 1 ? fabs(sh.te[lane]) : 0.0);
  }
  const bool bad = __any(!(b < INFINITY));
  for (int off = 32; off > 0; off >>= 1) {
    b = fmax(b, __shfl_xor(b, off, 64));
    dmin = fmin(dmin, __shfl_xor(dmin, off, 64));
  }
  if (bad || b == 0.0 || k == 1) return ldexp(dmin, -unit);
  const int ex = ilogb(b) + 1;   // scaled by a power of two into (-1, 1)
  __syncthreads();
  if (threadIdx.x < KM && (int)threadIdx.x < k) {
    sh.td[threadIdx.x] = ldexp(sh.td[threadIdx.x], -ex);
    const double e = ldexp((int)threadIdx.x < k - 1 ? sh.te[threadIdx.x] : 0.0, -ex);
    sh.te[threadIdx.x] = e * e;
  }
  __syncthreads();
  double lo = -1.0, hi = ldexp(dmin, -ex);
  for (int round = 0; round < 9; ++round) {
    const double w = (hi - lo) * (1.0 / 65.0), x = lo + w * (lane + 1);
    double p0 = 1.0, p1 = sh.td[0] - x;
    bool neg = !(p1 > 0.0);
    for (int i = 1; i < k; ++i) {
      const double p2 = (sh.td[i] - x) * p1 - sh.te[i - 1] * p0;
      p0 = p1;
      p1 = p2;
      neg |= !(p2 > 0.0);
      if ((i & 3) == 0) {
        const double sc = fmax(fabs(p0), fabs(p1)) < 1e-100 ? 1e100 : 1.0;
        p0 *= sc;
        p1 *= sc;
      }
    }
    const uint64_t mask = __ballot(neg);   // shifts above the smallest eigenvalue
    const int t = mask ? __builtin_ctzll(mask) : 64;
    const double nlo = t > 0 ? lo + w * t : lo, nhi = t < 64 ? lo + w * (t + 1) : hi;
    lo = nlo;
    hi = nhi;
  }
  return ldexp(0.5 * (lo + hi), ex - unit);
}

// largest alpha with x + alpha dx PSD (INFINITY if unbounded): Cholesky
// L L' = x together with dx -> L^-1 dx L^-T (one column and one barrier a
// step), then the smallest eigenvalue; 0 when x has a pivot that is not positive
template <int KM> __device__ __forceinline__ double psd_step_one(const double* x, const double* dx, int k, PsdShared<KM>& sh) {
  const int l = threadIdx.x % KM;
  double a[4], d[4];
  int q = 0;
  psd_each<KM>(k, [&](int i, int, bool in) {
    a[q] = in ? smat_at(x, i, l) : 0.0;
    d[q] = in ? smat_at(dx, i, l) : 0.0;
    ++q;
  });
  __syncthreads();   // the exchange buffers' previous readers are done
  for (int p = 0; p < k; ++p) {
    double *ca = sh.ca[p & 1], *cd = sh.cb[p & 1];
    q = 0;
    psd_each<KM>(k, [&](int i, int, bool) {
      if (l == p) {
        ca[i] = a[q];
        cd[i] = d[q];
      }
      ++q;
    });
    __syncthreads();
    const double piv = ca[p];
    if (!(piv > 0.0)) return 0.0;
    // row / column p scaled is w, its multiples L(., p) leave the others
    const double r = rsqrt_step(piv), g = cd[p] * r * r;
    const double ll = l > p ? ca[l] * r : 0.0, wl = cd[l] * r;
    q = 0;
    psd_each<KM>(k, [&](int i, int, bool) {
      const double li = i > p ? ca[i] * r : 0.0, wi = cd[i] * r;
      a[q] -= li * ll;
      const bool up = i >= l;   // (i, l) and (l, i) get the same bits
      const double l0 = up ? li : ll, l1 = up ? ll : li, w0 = up ? wi : wl, w1 = up ? wl : wi;
      const double v = fma(l0 * l1, g, fma(-l1, w0, fma(-l0, w1, d[q])));
      d[q] = i == p ? (l == p ? g : fma(-ll, g, wl)) : l == p ? fma(-li, g, wi) : v;
      ++q;
    });
  }
  const double lmin = psd_min_eig<KM>(d, k, sh);
  return lmin < 0.0 ? -1.0 / lmin : INFINITY;
}

// workgroups of a segment and this one's place among them
__device__ inline const SegDev& psd_seg(const SegTable& tb, int64_t& blk, int64_t& nblk) {
  int q = 0;
  while (q + 1 < tb.nseg && (int)blockIdx.x >= tb.first[q + 1]) ++q;
  blk = blockIdx.x - tb.first[q];
  nblk = tb.first[q + 1] - tb.first[q];
  return tb.g[q];
}

// per-workgroup minimum over its cones, or per cone (capped at amax) when
// per_cone.  The s and z halves of a cone are separate tasks, so twice as many
// waves share the chip.  30 cones each of sides 8, 20 and 32: 1.53 ms in three
// launches -> 96 us in two; 2,000 cones of side 10: 282 -> 54 us.
template <int KM>
__global__ __launch_bounds__(Psd<KM>::NT) void k_psd_step(SegTable tb, const double* __restrict__ s,
                                                          const double* __restrict__ z, const double* __restrict__ ds,
                                                          const double* __restrict__ dz, double amax, int per_cone,
                                                          double* __restrict__ out) {
  __shared__ PsdShared<KM> sh;
  int64_t blk, nblk;
  const SegDev& g = psd_seg(tb, blk, nblk);
  double best = INFINITY;
  for (int64_t u = 0;; ++u) {
    const int64_t t = per_cone ? 2 * (blk + (u >> 1) * nblk) + (u & 1) : blk + u * nblk;
    if (t >= 2 * g.count) break;
    const int64_t o = g.base + (t >> 1) * g.dim;
    const bool zh = (t & 1) != 0;
    best = fmin(best, psd_step_one<KM>((zh ? z : s) + o, (zh ? dz : ds) + o, g.k, sh));
    if (per_cone && zh) {
      if (threadIdx.x == 0) out[t >> 1] = fmin(amax, best);
      best = INFINITY;
    }
  }
  if (!per_cone && threadIdx.x == 0) out[blockIdx.x] = best;
}

// per workgroup the largest -lambda_min of its cones
template <int KM>
__global__ __launch_bounds__(Psd<KM>::NT) void k_psd_max_neg_eig(SegTable tb, const double* __restrict__ v,
                                                                 double* __restrict__ out) {
  __shared__ PsdShared<KM> sh;
  int64_t blk, nblk;
  const SegDev& g = psd_seg(tb, blk, nblk);
  double a = -INFINITY;
  for (int64_t c = blk; c < g.count; c += nblk) {
    double d[4];
    int q = 0;
    psd_each<KM>(g.k, [&](int i, int l, bool in) {
      d[q] = in ? smat_at(v + g.base + c * g.dim, i, l) : 0.0;
      ++q;
    });
    a = fmax(a, -psd_min_eig<KM>(d, g.k, sh));
  }
  if (threadIdx.x == 0) out[blockIdx.x] = a;
}

// pair of round r on kk indices (circle method: index kk - 1 fixed, the others
// turning, so the kk / 2 pairs of a round are disjoint and a sweep is kk - 1
// rounds)
__device__ inline void rr_pair(int kk, int r, int i, int& p, int& q) {
  const int n = kk - 1;
  int u = r + i, v = r - i + n;
  if (u >= n) u -= n;
  if (v >= n) v -= n;
  if (i == 0) u = n, v = r;
  p = min(u, v);
  q = max(u, v);
}

// one-sided Jacobi (Hestenes) on the columns of B (k x k): on return the
// columns are orthogonal and W accumulates 2^e B_in W = B_out, e the returned
// power that takes B's largest entry into [1, 2) (squares of products of
// columns stay in range).  G lanes per pair, two rows each; a pair is skipped
// when |b_p'b_q| <= 1e-15 |b_p||b_q|.
template <int KM>
__device__ __forceinline__ int psd_jacobi_cols(double* B, int k, double* W, int* flag, PsdShared<KM>& sh) {
  constexpr int LD = Psd<KM>::LD, G = Psd<KM>::G;
  double d[4];
  int n = 0;
  __syncthreads();   // B is complete
  psd_each<KM>(k, [&](int i, int l, bool in) { d[n++] = in ? B[i * LD + l] : 0.0; });
  const int e = psd_unit_exp<KM>(d, sh.td);
  n = 0;
  psd_each<KM>(k, [&](int i, int l, bool in) {
    if (in) B[i * LD + l] = ldexp(d[n], e);
    W[i * LD + l] = in && i == l ? 1.0 : 0.0;
    ++n;
  });
  const int kk = (k + 1) & ~1, np = kk / 2, grp = threadIdx.x / G, sub = threadIdx.x % G;
  for (int sweep = 0; sweep < 60; ++sweep) {
    bool any = false;
    __syncthreads();
    if (threadIdx.x == 0) *flag = 0;
    for (int r = 0; r < kk - 1; ++r) {
      __syncthreads();
      int p, q;
      rr_pair(kk, r, min(grp, np - 1), p, q);
      const bool on = grp < np && q < k;
      double bp[2], bq[2], wp[2], wq[2], a = 0, b = 0, gg = 0;
#pragma unroll
      for (int h = 0; h < 2; ++h) {   // rows from k on are zero
        const int o = min(sub + G * h, KM - 1) * LD;
        const bool in = on && sub + G * h < k;
        bp[h] = in ? B[o + p] : 0.0;
        bq[h] = in ? B[o + q] : 0.0;
        wp[h] = in ? W[o + p] : 0.0;
        wq[h] = in ? W[o + q] : 0.0;
        a = fma(bp[h], bp[h], a);
        b = fma(bq[h], bq[h], b);
        gg = fma(bp[h], bq[h], gg);
      }
      a = group_sum<G>(a);
      b = group_sum<G>(b);
      gg = group_sum<G>(gg);
      if (gg * gg > 1e-30 * (a * b)) {
        // tan of the angle: 2 g / (d + sign(d) sqrt(d^2 + 4 g^2)), d = |b_q|^2 - |b_p|^2
        const double dd = b - a, h2 = fma(dd, dd, 4.0 * gg * gg);
        const double t = 2.0 * gg * rcp_step(dd + copysign(h2 * rsqrt_step(h2), dd));
        const double cs = rsqrt_step(fma(t, t, 1.0)), sn = cs * t;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int o = (sub + G * h) * LD;
          if (sub + G * h >= k) continue;
          B[o + p] = cs * bp[h] - sn * bq[h];
          B[o + q] = sn * bp[h] + cs * bq[h];
          W[o + p] = cs * wp[h] - sn * wq[h];
          W[o + q] = sn * wp[h] + cs * wq[h];
        }
        any = true;
      }
    }
    if (any) *flag = 1;
    __syncthreads();
    if (!*flag) break;
  }
  __syncthreads();
  return e;
}

// squared norms of B's columns
template <int KM> __device__ inline double psd_col_norm2(const double* B, int k, int col) {
  double acc = 0;
  for (int r = 0; r < k; ++r) acc += B[r * Psd<KM>::LD + col] * B[r * Psd<KM>::LD + col];
  return acc;
}

// Scaling: Cholesky factors L_s, L_z (both in one loop); the SVD of
// L_z' L_s = U diag(lam) V' gives R = L_s V lam^-1/2 and R^-1 = lam^-1/2 U' L_z';
// a second one-sided Jacobi on R' gives M = R R' = Q diag(m) Q'.  State of a
// cone: R (k*k row-major) | R^-1 | Q | lambda (k) | m (k), cone after cone.
// Bound by the rounds of the two Jacobi iterations (a dot product over G lanes
// by DPP, one tangent and one rotation each).  30 cones each of sides 8, 20 and
// 32: 1.40 ms in three launches -> 0.42 ms in two; 2,000 cones of side 10:
// 337 -> 106 us.
template <int KM>
__global__ __launch_bounds__(Psd<KM>::NT) void k_psd_scale(SegTable tb, const double* __restrict__ s,
                                                           const double* __restrict__ z, double* __restrict__ hdiag) {
  constexpr int LD = Psd<KM>::LD, MAT = Psd<KM>::MAT;
  __shared__ double Ls[MAT], Lz[MAT], B[MAT], W[MAT], R[MAT], Ri[MAT], lam[KM], m[KM];
  __shared__ PsdShared<KM> sh;
  __shared__ int flag;
  int64_t c, nblk;
  const SegDev& g = psd_seg(tb, c, nblk);
  const int tid = threadIdx.x, l = tid % KM, k = g.k, sd = g.dim;
  const double *sc = s + g.base + c * sd, *zc = z + g.base + c * sd;
  double a[4], b[4];
  int q = 0;
  psd_each<KM>(k, [&](int i, int, bool in) {
    a[q] = in ? smat_at(sc, i, l) : 0.0;
    b[q] = in ? smat_at(zc, i, l) : 0.0;
    Ls[i * LD + l] = a[q];   // stands where a pivot is not positive
    Lz[i * LD + l] = b[q];
    ++q;
  });
  bool oks = true, okz = true;
  for (int p = 0; p < k; ++p) {
    double *ca = sh.ca[p & 1], *cb = sh.cb[p & 1];
    q = 0;
    psd_each<KM>(k, [&](int i, int, bool) {
      if (l == p) {
        ca[i] = a[q];
        cb[i] = b[q];
      }
      ++q;
    });
    __syncthreads();
    const double ps = ca[p], pz = cb[p];
    oks = oks && ps > 0.0;
    okz = okz && pz > 0.0;
    const double rs = rsqrt_step(ps), rz = rsqrt_step(pz);
    const double ls = l > p ? ca[l] * rs : 0.0, lz = l > p ? cb[l] * rz : 0.0;
    q = 0;
    psd_each<KM>(k, [&](int i, int, bool in) {
      const double is = i > p ? ca[i] * rs : i == p ? ps * rs : 0.0, iz = i > p ? cb[i] * rz : i == p ? pz * rz : 0.0;
      if (in && l == p && oks) Ls[i * LD + p] = is;
      if (in && l == p && okz) Lz[i * LD + p] = iz;
      if (i > p) {
        a[q] -= is * ls;
        b[q] -= iz * lz;
      }
      ++q;
    });
  }
  __syncthreads();
  psd_mm<KM>(Lz, true, Ls, false, k, B);   // B = Lz' Ls
  const int eb = psd_jacobi_cols<KM>(B, k, W, &flag, sh);   // B W = U diag(lam) (now 2^eb of it), V = W
  if (tid < k) lam[tid] = ldexp(sqrt(psd_col_norm2<KM>(B, k, tid)), -eb);
  __syncthreads();
  // R = Ls V lam^-1/2 ; Rinv = lam^-1/2 U' Lz' with U = B diag(1/lam)
  psd_mm<KM>(Ls, false, W, false, k, R);
  psd_mm<KM>(B, true, Lz, true, k, Ri);
  psd_each<KM>(k, [&](int i, int, bool in) {
    const double r = in ? R[i * LD + l] / sqrt(lam[l]) : 0.0;
    R[i * LD + l] = r;
    if (in) Ri[i * LD + l] = ldexp(Ri[i * LD + l], -eb) / lam[i] / sqrt(lam[i]);
    // M = R R' = Q diag(m) Q': one-sided Jacobi on the columns of R' (in Ls) gives Q (in W)
    Ls[l * LD + i] = r;
  });
  const int em = psd_jacobi_cols<KM>(Ls, k, W, &flag, sh);
  if (tid < k) m[tid] = ldexp(psd_col_norm2<KM>(Ls, k, tid), -2 * em);
  __syncthreads();
  double* st = g.state + c * (3 * k * k + 2 * k);
  psd_each<KM>(k, [&](int i, int, bool in) {
    if (!in) return;
    st[i * k + l] = R[i * LD + l];
    st[k * k + i * k + l] = Ri[i * LD + l];
    st[2 * k * k + i * k + l] = W[i * LD + l];
  });
  if (tid < k) {
    st[3 * k * k + tid] = lam[tid];
    st[3 * k * k + k + tid] = m[tid];
  }
  psd_mm<KM>(R, false, R, true, k, B);     // Mm = R R'
  for (int p = tid; p < sd; p += Psd<KM>::NT) {       // diag of H in svec coordinates
    int j, i;
    tri_index(p, j, i);
    hdiag[g.base + c * sd + p] =
        i == j ? B[i * LD + i] * B[i * LD + i] : B[i * LD + i] * B[j * LD + j] + B[i * LD + j] * B[i * LD + j];
  }
}

// combined-step d_s:
//   A = R^-1 dS R^-T, B = R' dZ R, V = (A B + B A)/2 + diag(lam^2) - sm I,
//   X_ij = 2 V_ij / (lam_i + lam_j), ds = svec(R X R')
// 30 cones each of sides 8, 20 and 32: 225 us in three launches -> 23 us in two.
template <int KM>
__global__ __launch_bounds__(Psd<KM>::NT) void k_psd_ds(SegTable tb, const double* __restrict__ dsa,
                                                        const double* __restrict__ dza, double sm,
                                                        double* __restrict__ ds) {
  constexpr int LD = Psd<KM>::LD, MAT = Psd<KM>::MAT;
  __shared__ double R[MAT], Ri[MAT], dS[MAT], dZ[MAT], T[MAT], lam[KM];
  int64_t c, nblk;
  const SegDev& g = psd_seg(tb, c, nblk);
  const int tid = threadIdx.x, k = g.k, sd = g.dim;
  const double* st = g.state + c * (3 * k * k + 2 * k);
  const int64_t o = g.base + c * sd;
  psd_each<KM>(k, [&](int i, int l, bool in) {
    R[i * LD + l] = in ? st[i * k + l] : 0.0;
    Ri[i * LD + l] = in ? st[k * k + i * k + l] : 0.0;
    dS[i * LD + l] = in ? smat_at(dsa + o, i, l) : 0.0;
    dZ[i * LD + l] = in ? smat_at(dza + o, i, l) : 0.0;
  });
  if (tid < k) lam[tid] = st[3 * k * k + tid];
  __syncthreads();
  psd_mm<KM>(Ri, false, dS, false, k, T);   // Ri dS
  psd_mm<KM>(T, false, Ri, true, k, dS);    // A = (Ri dS) Ri'
  psd_mm<KM>(R, true, dZ, false, k, T);     // R' dZ
  psd_mm<KM>(T, false, R, false, k, dZ);    // B = (R' dZ) R
  psd_mm<KM>(dS, false, dZ, false, k, T);   // A B
  // V from A B and its transpose, so X is exactly symmetric before the large
  // 1/(lam_i + lam_j) factors
  psd_each<KM>(k, [&](int i, int l, bool in) {
    if (!in) return;
    double v = 0.5 * (T[i * LD + l] + T[l * LD + i]);
    if (i == l) v += lam[i] * lam[i] - sm;
    dS[i * LD + l] = 2.0 * v / (lam[i] + lam[l]);
  });
  __syncthreads();
  psd_mm<KM>(R, false, dS, false, k, T);    // R X
  psd_mm<KM>(T, false, R, true, k, dZ);     // (R X) R'
  for (int p = tid; p < sd; p += Psd<KM>::NT) {
    int j, i;
    tri_index(p, j, i);
    ds[o + p] = dZ[i * LD + j] * (i == j ? 1.0 : 1.41421356237309504880);
  }
}

// Spectral application of H (mode 0) or (H + delta I)^-1: Q (f .* (Q' X Q)) Q'.
// blockIdx.y selects the vector.  30 cones each of sides 20 and 32: 36 us in
// two launches -> 10.5 us in one.
template <int KM>
__global__ __launch_bounds__(Psd<KM>::NT) void k_psd_apply(SegTable tb, int mode, double delta, int epi,
                                                           ApplySys2 ss) {
  constexpr int LD = Psd<KM>::LD, MAT = Psd<KM>::MAT;
  __shared__ double Q[MAT], X[MAT], T[MAT], U[MAT], m[KM];
  int64_t c, nblk;
  const SegDev& g = psd_seg(tb, c, nblk);
  const ApplySys& sy = ss.s[blockIdx.y];
  const int tid = threadIdx.x, k = g.k, sd = g.dim;
  const double* st = g.state + c * (3 * k * k + 2 * k);
  const int64_t o = g.base + c * sd;
  psd_each<KM>(k, [&](int i, int l, bool in) {
    Q[i * LD + l] = in ? st[2 * k * k + i * k + l] : 0.0;
    X[i * LD + l] = in ? smat_at(sy.x + o, i, l) : 0.0;
  });
  if (tid < k) m[tid] = st[3 * k * k + k + tid];
  __syncthreads();
  psd_mm<KM>(X, false, Q, false, k, T);   // X Q
  psd_mm<KM>(Q, true, T, false, k, U);    // Q' X Q
  // average the two roundings of each eigen-coefficient, then scale
  psd_each<KM>(k, [&](int i, int l, bool in) {
    const double h = in ? m[i] * m[l] : 0.0;
    T[i * LD + l] = in ? 0.5 * (U[i * LD + l] + U[l * LD + i]) * (mode == 0 ? h : 1.0 / (h + delta)) : 0.0;
  });
  __syncthreads();
  psd_mm<KM>(T, false, Q, true, k, U);
  psd_mm<KM>(Q, false, U, false, k, X);
  for (int p = tid; p < sd; p += Psd<KM>::NT) {   // svec of the upper triangle
    int j, i;
    tri_index(p, j, i);
    const double v = X[i * LD + j] * (i == j ? 1.0 : 1.41421356237309504880);
    sy.y[o + p] = epi == EPI_NEG ? -sy.a[o + p] - v : v;
  }
}

// Explicit lower-triangle entries of M = (H + delta I)^-1, packed index
// p = a (a + 1) / 2 + b for a >= b, stored mblk[p * count + cone].  With
// f(i,j) = 1/(m_i m_j + delta) and svec index a = (ia, ja),
//   M_ab = (c_a c_b / 2) sum_i Q[ia][i] (Q[ib][i] G_i[ja][jb] + Q[jb][i] G_i[ja][ib]),
//   G_i[q][s] = sum_j f(i,j) Q[q][j] Q[s][j],
// (c = 1 on the diagonal, sqrt2 off it), which is sum_e svec(E_e)_a svec(E_e)_b f_e
// over the eigenvectors E_e = (q_i q_j' + q_j q_i')/sqrt2 of H, expanded by the
// Kronecker structure: k^4 flops for the G_i and 2k per entry instead of k(k+1)/2
// per entry.  G (k^3 per cone) lives in the caller's work buffer.
__global__ __launch_bounds__(256) void k_psd_mblock_g(SegDev g, double delta, double* __restrict__ G) {
  constexpr int LQ = PSD_LARGE + 1;
  __shared__ double Q[PSD_LARGE * LQ], f[PSD_LARGE];
  const int k = g.k, i = blockIdx.y;
  const int64_t kk = (int64_t)k * k, c = blockIdx.x;
  const double* st = g.state + c * (3 * kk + 2 * k);
  for (int e = threadIdx.x; e < k * k; e += blockDim.x) Q[(e / k) * LQ + e % k] = st[2 * kk + e];
  if ((int)threadIdx.x < k) f[threadIdx.x] = 1.0 / (st[3 * kk + k + i] * st[3 * kk + k + threadIdx.x] + delta);
  __syncthreads();
  double* Gi = G + (c * k + i) * kk;
  for (int e = threadIdx.x; e < k * k; e += blockDim.x) {
    const int q = e / k, sx = e % k;
    double acc = 0;
    for (int j = 0; j < k; ++j) acc += Q[q * LQ + j] * Q[sx * LQ + j] * f[j];
    Gi[e] = acc;
  }
}

// one thread per (cone, packed entry p = a (a + 1) / 2 + b): the grid's y
// dimension covers a cone's entries, so even a few large cones fill the chip
__global__ __launch_bounds__(256) void k_psd_mblock(SegDev g, const double* __restrict__ G) {
  constexpr int LQ = PSD_LARGE + 1;
  __shared__ double Q[PSD_LARGE * LQ];
  const int k = g.k, sd = g.dim;
  const int64_t N = g.count, kk = (int64_t)k * k, c = blockIdx.x;
  const double* st = g.state + c * (3 * kk + 2 * k);
  for (int e = threadIdx.x; e < k * k; e += blockDim.x) Q[(e / k) * LQ + e % k] = st[2 * kk + e];
  __syncthreads();
  const int np = sd * (sd + 1) / 2;
  const int p = (int)blockIdx.y * (int)blockDim.x + (int)threadIdx.x;
  if (p >= np) return;
  int a, b, ja, ia, jb, ib;
  tri_index(p, a, b);
  tri_index(a, ja, ia);
  tri_index(b, jb, ib);
  const double ca = (ia == ja) ? 1.0 : 1.41421356237309504880, cb = (ib == jb) ? 1.0 : 1.41421356237309504880;
  const double* Gc = G + c * k * kk + (int64_t)ja * k;
  double acc = 0;
  for (int i = 0; i < k; ++i) {
    const double* Gi = Gc + (int64_t)i * kk;
    acc += Q[ia * LQ + i] * (Q[ib * LQ + i] * Gi[jb] + Q[jb * LQ + i] * Gi[ib]);
  }
  g.mblk[(int64_t)p * N + c] = 0.5 * ca * cb * acc;
}
void psd_mblock(const SegDev& g, double delta, double* work, hipStream_t st) {
  hipLaunchKernelGGL(k_psd_mblock_g, dim3((unsigned)g.count, (unsigned)g.k), dim3(256), 0, st, g, delta, work);
  HC_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_psd_mblock, dim3((unsigned)g.count, (unsigned)ceil_div((int64_t)g.dim * (g.dim + 1) / 2, 256)),
                     dim3(256), 0, st, g, (const double*)work);
  HC_LAUNCH_CHECK();
}

// the scaling of s = z = I
__global__ __launch_bounds__(256) void k_psd_identity(SegDev g, double* __restrict__ hdiag) {
  const int k = g.k, kk = k * k, sd = 3 * kk + 2 * k;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < g.count * sd; e += (int64_t)gridDim.x * 256) {
    const int f = (int)(e % sd);
    g.state[e] = f >= 3 * kk || (f % kk) / k == (f % kk) % k ? 1.0 : 0.0;
  }
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < g.count * g.dim; e += (int64_t)gridDim.x * 256)
    hdiag[g.base + e] = 1.0;
}
void psd_identity(const SegDev& g, double* hdiag, hipStream_t st) {
  const int64_t n = g.count * (3 * (int64_t)g.k * g.k + 2 * g.k);
  hipLaunchKernelGGL(k_psd_identity, dim3((unsigned)std::min<int64_t>(2048, ceil_div(n, 256))), dim3(256), 0, st, g,
                     hdiag);
  HC_LAUNCH_CHECK();
}

// The PSD segments of one size class, up to FUSED_SEGS to a launch:
// blocks(g) workgroups each, launch(table, workgroups)
template <typename Blocks, typename Launch>
static void psd_launches(const std::vector<SegDev>& segs, bool small, Blocks&& blocks, Launch&& launch) {
  SegTable tb{};
  int nb = 0;
  auto flush = [&]() {
    if (tb.nseg == 0) return;
    tb.first[tb.nseg] = nb;
    launch(tb, nb);
    HC_LAUNCH_CHECK();
    tb.nseg = 0;
    nb = 0;
  };
  for (const SegDev& g : segs) {
    if (g.kind != HC_CONE_PSD || g.count == 0 || (g.k <= PSD_SMALL) != small) continue;
    const int64_t b = blocks(g);
    if (tb.nseg == FUSED_SEGS || nb + b > 0x7fffffff) flush();
    tb.g[tb.nseg] = g;
    tb.first[tb.nseg++] = nb;
    nb += (int)b;
  }
  flush();
}
static int64_t all_cones(const SegDev& g) { return g.count; }

void psd_scale(const std::vector<SegDev>& segs, const double* s, const double* z, double* hdiag, hipStream_t st) {
  psd_launches(segs, true, all_cones, [&](const SegTable& tb, int nb) {
    hipLaunchKernelGGL(k_psd_scale<PSD_SMALL>, dim3(nb), dim3(Psd<PSD_SMALL>::NT), 0, st, tb, s, z, hdiag);
  });
  psd_launches(segs, false, all_cones, [&](const SegTable& tb, int nb) {
    hipLaunchKernelGGL(k_psd_scale<PSD_LARGE>, dim3(nb), dim3(Psd<PSD_LARGE>::NT), 0, st, tb, s, z, hdiag);
  });
}
void psd_ds(const std::vector<SegDev>& segs, const double* dsa, const double* dza, double sm, double* ds,
            hipStream_t st) {
  psd_launches(segs, true, all_cones, [&](const SegTable& tb, int nb) {
    hipLaunchKernelGGL(k_psd_ds<PSD_SMALL>, dim3(nb), dim3(Psd<PSD_SMALL>::NT), 0, st, tb, dsa, dza, sm, ds);
  });
  psd_launches(segs, false, all_cones, [&](const SegTable& tb, int nb) {
    hipLaunchKernelGGL(k_psd_ds<PSD_LARGE>, dim3(nb), dim3(Psd<PSD_LARGE>::NT), 0, st, tb, dsa, dza, sm, ds);
  });
}
void psd_apply(const std::vector<SegDev>& segs, int mode, double delta, int epi, const ApplySys2& ss, int ns,
               hipStream_t st) {
  psd_launches(segs, true, all_cones, [&](const SegTable& tb, int nb) {
    hipLaunchKernelGGL(k_psd_apply<PSD_SMALL>, dim3(nb, ns), dim3(Psd<PSD_SMALL>::NT), 0, st, tb, mode, delta, epi, ss);
  });
  psd_launches(segs, false, all_cones, [&](const SegTable& tb, int nb) {
    hipLaunchKernelGGL(k_psd_apply<PSD_LARGE>, dim3(nb, ns), dim3(Psd<PSD_LARGE>::NT), 0, st, tb, mode, delta, epi, ss);
  });
}
int64_t psd_step(const std::vector<SegDev>& segs, const double* s, const double* z, const double* ds, const double* dz,
                 double amax, bool per_cone, double* out, hipStream_t st) {
  int64_t off = 0;
  auto blocks = [&](const SegDev& g) { return std::min<int64_t>((per_cone ? 1 : 2) * g.count, PSD_STEP_GRID); };
  psd_launches(segs, true, blocks, [&](const SegTable& tb, int nb) {
    hipLaunchKernelGGL(k_psd_step<PSD_SMALL>, dim3(nb), dim3(Psd<PSD_SMALL>::NT), 0, st, tb, s, z, ds, dz, amax,
                       per_cone ? 1 : 0, out + off);
    off += nb;
  });
  psd_launches(segs, false, blocks, [&](const SegTable& tb, int nb) {
    hipLaunchKernelGGL(k_psd_step<PSD_LARGE>, dim3(nb), dim3(Psd<PSD_LARGE>::NT), 0, st, tb, s, z, ds, dz, amax,
                       per_cone ? 1 : 0, out + off);
    off += nb;
  });
  return off;
}
int64_t psd_max_neg_eig(const std::vector<SegDev>& segs, const double* v, double* out, hipStream_t st) {
  int64_t off = 0;
  auto blocks = [](const SegDev& g) { return std::min<int64_t>(g.count, PSD_STEP_GRID); };
  psd_launches(segs, true, blocks, [&](const SegTable& tb, int nb) {
    hipLaunchKernelGGL(k_psd_max_neg_eig<PSD_SMALL>, dim3(nb), dim3(Psd<PSD_SMALL>::NT), 0, st, tb, v, out + off);
    off += nb;
  });
  psd_launches(segs, false, blocks, [&](const SegTable& tb, int nb) {
    hipLaunchKernelGGL(k_psd_max_neg_eig<PSD_LARGE>, dim3(nb), dim3(Psd<PSD_LARGE>::NT), 0, st, tb, v, out + off);
    off += nb;
  });
  return off;
}
}  // namespace hc
