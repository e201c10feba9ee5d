// Leaf blocks of the two-level Schur factorisation (gfx950): assembly through
// the column map, batched per-leaf Cholesky and coupling, leaf solves.
#include "hc_leaf.h"

#include <algorithm>
#include <cmath>

namespace hc {

// address of S[j, k] (either order) inside the two-level storage
__device__ inline double* dest(const ColMap& cm, int32_t j, int32_t k) {
  const int32_t bj = cm.leaf[j], bk = cm.leaf[k];
  const int32_t lj = cm.loc[j], lk = cm.loc[k];
  if (bj < 0 && bk < 0) {
    const int32_t hi = lj > lk ? lj : lk, lo = lj > lk ? lk : lj;
    return cm.ST + hi + (int64_t)lo * cm.ldt;
  }
  if (bj >= 0 && bk >= 0) {
    if (bj != bk) return cm.sink;   // cannot happen: leaves are connected components
    const int32_t l = cm.lsize[bj];
    const int32_t hi = lj > lk ? lj : lk, lo = lj > lk ? lk : lj;
    return cm.lval + cm.lval_off[bj] + hi + (int64_t)lo * l;
  }
  const int32_t b = bj >= 0 ? bj : bk;
  const int32_t l = bj >= 0 ? lj : lk;
  const int32_t t = bj >= 0 ? lk : lj;
  const int32_t* cl = cm.clist + cm.clist_off[b];
  int lo = 0, hi = cm.ccnt[b] - 1;
  while (lo <= hi) {
    const int mid = (lo + hi) >> 1;
    const int32_t v = cl[mid];
    if (v == t) return cm.cval + cm.cval_off[b] + mid + (int64_t)l * cm.ccnt[b];
    if (v < t) lo = mid + 1;
    else hi = mid - 1;
  }
  return cm.sink;   // cannot happen: the coupling list holds every neighbour
}

// pair tasks through the column map (lane per task, or wave per long task:
// see k_assemble_pairs)
template <bool WIDE>
__global__ __launch_bounds__(256) void k_assemble_pairs_map(int64_t ntask, const int32_t* __restrict__ tra,
                                                            const int32_t* __restrict__ trb,
                                                            const int64_t* __restrict__ tm,
                                                            const double* __restrict__ mval,
                                                            const int32_t* __restrict__ rp,
                                                            const int32_t* __restrict__ ci,
                                                            const double* __restrict__ av, ColMap cm) {
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
      const double mj = m * av[p];
      for (int32_t q = ba; q <= p; ++q) atomicAdd(dest(cm, ci[p], ci[q]), mj * av[q]);
    }
  } else {
    for (int32_t p = ba + lane; p < ea; p += nl) {
      const int32_t j = ci[p];
      const double mj = m * av[p];
      for (int32_t q = bb; q < eb; ++q) {
        const int32_t k = ci[q];
        double v = mj * av[q];
        if (j == k) v *= 2.0;
        atomicAdd(dest(cm, j, k), v);
      }
    }
  }
}

void assemble_pairs_map(int64_t ntask, const int32_t* tra, const int32_t* trb, const int64_t* tm, const double* mval,
                        const Csr& A, const ColMap& cm, bool wide, hipStream_t st) {
  if (ntask == 0) return;
  if (wide)
    hipLaunchKernelGGL(k_assemble_pairs_map<true>, dim3((unsigned)ceil_div(ntask * 64, 256)), dim3(256), 0, st,
                       ntask, tra, trb, tm, mval, A.rowptr, A.col, A.val, cm);
  else
    hipLaunchKernelGGL(k_assemble_pairs_map<false>, dim3((unsigned)ceil_div(ntask, 256)), dim3(256), 0, st, ntask,
                       tra, trb, tm, mval, A.rowptr, A.col, A.val, cm);
  HC_LAUNCH_CHECK();
}

__global__ void k_add_P_map(int32_t n, const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                            const double* __restrict__ v, double delta, ColMap cm) {
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  *dest(cm, i, i) += delta;   // each diagonal entry has exactly one writer here
  if (!rp) return;
  for (int32_t p = rp[i]; p < rp[i + 1]; ++p) {
    const int32_t j = ci[p];
    if (j <= i) atomicAdd(dest(cm, i, j), v[p]);
  }
}

void add_P_delta_map(const Csr& P, int64_t n, double delta, const ColMap& cm, hipStream_t st) {
  if (n == 0) return;
  hipLaunchKernelGGL(k_add_P_map, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, st, (int32_t)n, P.rowptr, P.col,
                     P.val, delta, cm);
  HC_LAUNCH_CHECK();
}

// ---------------------------------------------------------------------------
// one wave per leaf
// ---------------------------------------------------------------------------
// One wave per leaf, of at most LM columns: with LM = LEAF_SMALL a wave takes
// 3 KB of LDS instead of 25 (six waves on a CU then); 100,500 leaves coupled to
// 10 tail columns each: 270 -> 84 us.
template <int LM>
__global__ __launch_bounds__(64) void k_leaf_factor(ColMap cm, const int32_t* __restrict__ list, double tol, double fix,
                                                    unsigned long long* __restrict__ hits) {
  __shared__ double Lb[LM][LM + 1];
  __shared__ double W[LEAF_CPL_MAX][LM + 1];
  const int b = list[blockIdx.x], lane = threadIdx.x;
  const int l = cm.lsize[b], cnt = cm.ccnt[b];
  double* lv = cm.lval + cm.lval_off[b];
  double* cv = cm.cval + cm.cval_off[b];
  const int32_t* cl = cm.clist + cm.clist_off[b];
  for (int e = lane; e < l * l; e += 64) {
    const int i = e % l, j = e / l;
    Lb[i][j] = (i >= j) ? lv[e] : 0.0;
  }
  for (int e = lane; e < cnt * l; e += 64) W[e % cnt][e / cnt] = cv[e];
  __syncthreads();
  int nh = 0;
  for (int j = 0; j < l; ++j) {
    double d = Lb[j][j];
    if (!(d > tol)) {
      d = fix;
      ++nh;
    }
    const double ljj = sqrt(d);
    __syncthreads();
    if (lane == j) Lb[j][j] = ljj;
    if (lane > j && lane < l) Lb[lane][j] /= ljj;
    __syncthreads();
    for (int k = j + 1; k < l; ++k)
      if (lane >= k && lane < l) Lb[lane][k] -= Lb[lane][j] * Lb[k][j];
    __syncthreads();
  }
  if (lane == 0 && nh) atomicAdd(hits, (unsigned long long)nh);
  // row a of W solves L_b w = s_a:  w_j = (s_aj - sum_{k<j} L_jk w_k) / L_jj
  if (lane < cnt)
    for (int j = 0; j < l; ++j) {
      double v = W[lane][j];
      for (int k = 0; k < j; ++k) v -= Lb[j][k] * W[lane][k];
      W[lane][j] = v / Lb[j][j];
    }
  __syncthreads();
  for (int e = lane; e < l * l; e += 64) {
    const int i = e % l, j = e / l;
    lv[e] = (i >= j) ? Lb[i][j] : 0.0;
  }
  for (int e = lane; e < cnt * l; e += 64) cv[e] = W[e % cnt][e / cnt];
  // S_TT[cl[a], cl[c]] -= sum_j W[a][j] W[c][j] for a >= c (cl ascending, so
  // the target is in the lower triangle)
  const int npair = cnt * (cnt + 1) / 2;
  for (int p = lane; p < npair; p += 64) {
    int a = (int)((sqrtf(8.0f * p + 1.0f) - 1.0f) * 0.5f);   // p < 2,080
    while (a * (a + 1) / 2 > p) --a;
    while ((a + 1) * (a + 2) / 2 <= p) ++a;
    const int c = p - a * (a + 1) / 2;
    double v = 0.0;
    for (int j = 0; j < l; ++j) v += W[a][j] * W[c][j];
    if (cm.lslot) cm.lslot[cm.lp_off[b] + p] = -v;
    else atomicAdd(&cm.ST[cl[a] + (int64_t)cl[c] * cm.ldt], -v);
  }
}

void leaf_factor(const ColMap& cm, double tol, double fix, unsigned long long* hits, hipStream_t st) {
  if (cm.nleaf == 0) return;
  if (cm.nsmall) {
    hipLaunchKernelGGL(k_leaf_factor<LEAF_SMALL>, dim3((unsigned)cm.nsmall), dim3(64), 0, st, cm, cm.small, tol, fix, hits);
    HC_LAUNCH_CHECK();
  }
  if (cm.nlarge) {
    hipLaunchKernelGGL(k_leaf_factor<LEAF_MAX>, dim3((unsigned)cm.nlarge), dim3(64), 0, st, cm, cm.large, tol, fix, hits);
    HC_LAUNCH_CHECK();
  }
}

// Leaf solves, for one or two right-hand sides side by side (NR), which share
// the reads of L and W.  Leaves of at most LEAF_SMALL columns run one lane each
// (their L and coupling rows read straight from memory), larger ones one wave
// each: lane i keeps entry i, the current entry is divided by the pivot and
// broadcast by readlane, the others lose their multiple of it.  (With the
// substitution in one lane a leaf of 32 columns took 16 us a pass; a launch per
// kind, right-hand side and copy of the tail made ten of a solve's three.)
__device__ inline double lane_value(double v, int l) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l),
                 hi = (uint32_t)__builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
constexpr int LEAF_AHEAD = 8;   // columns of L loaded together

template <int NR>
__device__ inline void leaf_fwd_small(const ColMap& cm, int64_t k, const LeafVecs& w) {
  const int b = cm.small[k];
  const int l = cm.lsize[b];
  const double* lv = cm.lval + cm.lval_off[b];   // L_b column-major: L[i][j] = lv[i + j l]
  const int32_t* cols = cm.lcols + cm.lcol_off[b];
  double yb[NR][LEAF_SMALL];
#pragma unroll
  for (int j = 0; j < LEAF_SMALL; ++j) {
    if (j < l) {
      double lr[LEAF_SMALL];
#pragma unroll
      for (int q = 0; q <= j; ++q) lr[q] = lv[j + q * l];
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        double v = w.u[r][cols[j]];
#pragma unroll
        for (int q = 0; q < j; ++q) v -= lr[q] * yb[r][q];
        yb[r][j] = v / lr[j];
        w.x[r][cols[j]] = yb[r][j];
      }
    }
  }
}
template <int NR>
__device__ inline void leaf_fwd_wave(const ColMap& cm, int b, int lane, const LeafVecs& w) {
  const int l = cm.lsize[b], i = min(lane, l - 1);
  const double* lv = cm.lval + cm.lval_off[b] + i;
  const int col = cm.lcols[cm.lcol_off[b] + i];
  double v[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) v[r] = w.u[r][col];
  for (int k0 = 0; k0 < l; k0 += LEAF_AHEAD) {
    double lr[LEAF_AHEAD];
#pragma unroll
    for (int q = 0; q < LEAF_AHEAD; ++q) lr[q] = lv[(int64_t)min(k0 + q, l - 1) * l];
#pragma unroll
    for (int q = 0; q < LEAF_AHEAD; ++q) {
      const int k = k0 + q;
      if (k >= l) break;
      const double d = lane_value(lr[q], k);
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const double y = lane_value(v[r], k) / d;
        v[r] = lane == k ? y : lane > k ? v[r] - lr[q] * y : v[r];
      }
    }
  }
  if (lane < l)
#pragma unroll
    for (int r = 0; r < NR; ++r) w.x[r][col] = v[r];
}
// workgroups: small leaves (256 each), then large ones (four each)
template <int NR>
__global__ __launch_bounds__(256) void k_leaf_fwd(ColMap cm, LeafVecs w) {
  const int64_t ns = (cm.nsmall + 255) / 256;
  if ((int64_t)blockIdx.x < ns) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k < cm.nsmall) leaf_fwd_small<NR>(cm, k, w);
    return;
  }
  const int64_t k = ((int64_t)blockIdx.x - ns) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (k < cm.nlarge) leaf_fwd_wave<NR>(cm, cm.large[k], threadIdx.x & 63, w);
}

// uT[t] = u[tcols[t]] - sum over the couplings (b, a) of t of sum_j W_b[a][j]
// y_b[j]: one workgroup per tail index, of cm.tail_threads threads, its W
// entries (flattened at set-up into (cval index, leaf column) pairs, so each
// costs two independent gathers) split over the threads; per-wave shuffle sums
// meet in LDS in a fixed order
constexpr int TAIL_THREADS_MAX = 1024;
template <int NR>
__global__ __launch_bounds__(TAIL_THREADS_MAX) void k_leaf_tail(ColMap cm, LeafVecs w) {
  __shared__ double part[NR][TAIL_THREADS_MAX / 64];
  const int64_t t = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, nthr = blockDim.x;
  const int64_t e0 = cm.tc_ptr[t], e1 = cm.tc_ptr[t + 1];
  double acc[NR] = {};
  for (int64_t e = e0 + tid; e < e1; e += nthr) {
    const double c = cm.cval[cm.te_cv[e]];
    const int32_t j = cm.te_y[e];
#pragma unroll
    for (int r = 0; r < NR; ++r) acc[r] += c * w.x[r][j];
  }
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    for (int o = 32; o > 0; o >>= 1) acc[r] += __shfl_xor(acc[r], o, 64);
    if (lane == 0) part[r][tid >> 6] = acc[r];
  }
  __syncthreads();
  if (tid < NR) {
    const double u = w.u[tid][cm.tcols[t]];
    double s = 0.0;
    for (int k = 0; k < nthr / 64; ++k) s += part[tid][k];
    w.uT[tid][t] = e1 > e0 ? u - s : u;
  }
}

template <int NR>
__device__ inline void leaf_bwd_small(const ColMap& cm, int64_t k, const LeafVecs& w) {
  const int b = cm.small[k];
  const int l = cm.lsize[b], cnt = cm.ccnt[b];
  const double* lv = cm.lval + cm.lval_off[b];
  const int32_t* cols = cm.lcols + cm.lcol_off[b];
  const int32_t* cl = cm.clist + cm.clist_off[b];
  const double* cv = cm.cval + cm.cval_off[b];
  double vb[NR][LEAF_SMALL];
#pragma unroll
  for (int j = 0; j < LEAF_SMALL; ++j) {
    if (j < l) {
#pragma unroll
      for (int r = 0; r < NR; ++r) vb[r][j] = w.x[r][cols[j]];
      for (int a = 0; a < cnt; ++a) {
        const double c = cv[a + (int64_t)j * cnt];
        const int32_t t = cl[a];
#pragma unroll
        for (int r = 0; r < NR; ++r) vb[r][j] -= c * w.xT[r][t];
      }
    }
  }
#pragma unroll
  for (int j = LEAF_SMALL - 1; j >= 0; --j) {
    if (j < l) {
      double lr[LEAF_SMALL];
#pragma unroll
      for (int q = j; q < LEAF_SMALL; ++q) lr[q] = q < l ? lv[q + j * l] : 0.0;
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        double v = vb[r][j];
#pragma unroll
        for (int q = j + 1; q < LEAF_SMALL; ++q)
          if (q < l) v -= lr[q] * vb[r][q];
        vb[r][j] = v / lr[j];
        w.x[r][cols[j]] = vb[r][j];
      }
    }
  }
}
template <int NR>
__device__ inline void leaf_bwd_wave(const ColMap& cm, int b, int lane, const LeafVecs& w) {
  const int l = cm.lsize[b], cnt = cm.ccnt[b], i = min(lane, l - 1);
  const double* lv = cm.lval + cm.lval_off[b] + (int64_t)i * l;   // column i of L
  const int col = cm.lcols[cm.lcol_off[b] + i];
  const double* cv = cm.cval + cm.cval_off[b] + (int64_t)i * cnt;
  double v[NR], xt[NR];   // lane a: the tail entry of coupling a
  const int32_t t = cnt > 0 ? cm.clist[cm.clist_off[b] + min(lane, cnt - 1)] : 0;
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    v[r] = w.x[r][col];
    xt[r] = cnt > 0 ? w.xT[r][t] : 0.0;
  }
  for (int a0 = 0; a0 < cnt; a0 += LEAF_AHEAD) {
    double c[LEAF_AHEAD];
#pragma unroll
    for (int q = 0; q < LEAF_AHEAD; ++q) c[q] = cv[min(a0 + q, cnt - 1)];
#pragma unroll
    for (int q = 0; q < LEAF_AHEAD; ++q) {
      if (a0 + q >= cnt) break;
#pragma unroll
      for (int r = 0; r < NR; ++r) v[r] -= c[q] * lane_value(xt[r], a0 + q);
    }
  }
  for (int k0 = l - 1; k0 >= 0; k0 -= LEAF_AHEAD) {
    double lr[LEAF_AHEAD];
#pragma unroll
    for (int q = 0; q < LEAF_AHEAD; ++q) lr[q] = lv[max(k0 - q, 0)];
#pragma unroll
    for (int q = 0; q < LEAF_AHEAD; ++q) {
      const int k = k0 - q;
      if (k < 0) break;
      const double d = lane_value(lr[q], k);
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const double y = lane_value(v[r], k) / d;
        v[r] = lane == k ? y : lane < k ? v[r] - lr[q] * y : v[r];
      }
    }
  }
  if (lane < l)
#pragma unroll
    for (int r = 0; r < NR; ++r) w.x[r][col] = v[r];
}
// workgroups: small leaves, large leaves (as k_leaf_fwd), then the tail's
// entries of x
template <int NR>
__global__ __launch_bounds__(256) void k_leaf_bwd(ColMap cm, LeafVecs w) {
  const int64_t ns = (cm.nsmall + 255) / 256, nl = (cm.nlarge + 3) / 4;
  if ((int64_t)blockIdx.x < ns) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k < cm.nsmall) leaf_bwd_small<NR>(cm, k, w);
  } else if ((int64_t)blockIdx.x < ns + nl) {
    const int64_t k = ((int64_t)blockIdx.x - ns) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (k < cm.nlarge) leaf_bwd_wave<NR>(cm, cm.large[k], threadIdx.x & 63, w);
  } else {
    const int64_t t = ((int64_t)blockIdx.x - ns - nl) * 256 + threadIdx.x;
    if (t < cm.nt)
#pragma unroll
      for (int r = 0; r < NR; ++r) w.x[r][cm.tcols[t]] = w.xT[r][t];
  }
}

template <int NR> static void leaf_forward_n(const ColMap& cm, const LeafVecs& w, hipStream_t st) {
  const int64_t wgs = ceil_div(cm.nsmall, 256) + ceil_div(cm.nlarge, 4);
  if (wgs > 0) {
    hipLaunchKernelGGL(k_leaf_fwd<NR>, dim3((unsigned)wgs), dim3(256), 0, st, cm, w);
    HC_LAUNCH_CHECK();
  }
  if (cm.nt) {
    const int thr = cm.tail_threads == 1024 || cm.tail_threads == 256 ? cm.tail_threads : 64;
    hipLaunchKernelGGL(k_leaf_tail<NR>, dim3((unsigned)cm.nt), dim3(thr), 0, st, cm, w);
    HC_LAUNCH_CHECK();
  }
}
void leaf_forward(const ColMap& cm, const LeafVecs& w, int nr, hipStream_t st) {
  if (nr == 1) leaf_forward_n<1>(cm, w, st);
  else leaf_forward_n<2>(cm, w, st);
}

template <int NR> static void leaf_backward_n(const ColMap& cm, const LeafVecs& w, hipStream_t st) {
  const int64_t wgs = ceil_div(cm.nsmall, 256) + ceil_div(cm.nlarge, 4) + ceil_div(cm.nt, 256);
  if (wgs == 0) return;
  hipLaunchKernelGGL(k_leaf_bwd<NR>, dim3((unsigned)wgs), dim3(256), 0, st, cm, w);
  HC_LAUNCH_CHECK();
}
void leaf_backward(const ColMap& cm, const LeafVecs& w, int nr, hipStream_t st) {
  if (nr == 1) leaf_backward_n<1>(cm, w, st);
  else leaf_backward_n<2>(cm, w, st);
}

}  // namespace hc
