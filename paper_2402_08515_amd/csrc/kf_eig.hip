// Float64 eigensolver for the projected pencil of Section 2.1 (eq. projevp).
//
// The basis is M-orthonormal, so the projected pencil is (H, G) with
// G = I up to rounding; the solver works on the symmetric H (its distance
// from the generalized problem is bounded by |G - I| |theta|, reported as the
// orthogonality error).  Steps:
//   1. Householder reduction of H to tridiagonal form (one launch per
//      reflector, the last 128 and small matrices in one workgroup; the
//      reflectors stay in the lower triangle of the work matrix);
//   2. all eigenvalues by Sturm-count bisection, one wavefront per eigenvalue;
//   3. eigenvectors for the selected eigenvalues only, by inverse iteration
//      on the tridiagonal matrix (LU with partial pivoting), re-orthogonalised
//      inside clusters of nearly equal values;
//   4. back-transformation with the stored reflectors, one wavefront per
//      vector held in registers.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <cmath>
#include <vector>

#include "kf_internal.h"

namespace kf {

namespace {

inline int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

// matrices of this order and larger are reduced by k_tri_step
constexpr int kTriMultiFrom = 48;

__device__ __forceinline__ double wave_sum_e(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// Sum over the wavefront through the DPP paths of the vector unit (row shifts,
// then the two row broadcasts), the same value in every lane: six dependent
// adds instead of six trips through the LDS permute unit.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xF, true);
  return v + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double lane_value(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}
__device__ __forceinline__ double wave_total(double v) {
  v = dpp_add<0x111, 0xF>(v);  // row_shr:1, 2, 4, 8
  v = dpp_add<0x112, 0xF>(v);
  v = dpp_add<0x114, 0xF>(v);
  v = dpp_add<0x118, 0xF>(v);
  v = dpp_add<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
  v = dpp_add<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
  return lane_value(v, 63);
}

// The same sum as wave_sum_e, bit for bit (lanes 32 apart first, then 16, 8,
// 4, 2, 1), without its trips through the LDS permute unit: half-wave and row
// swaps, then row rotations (after the step for 8 a row repeats every 8 lanes,
// so a rotation by 4 reads the lane an exchange by 4 would, and so on).
__device__ __forceinline__ double wave_butterfly(double v) {
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  u32x2 lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
  u32x2 hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
  v = __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
  lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
  hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
  v = __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
  v = dpp_add<0x128, 0xF>(v);  // row_ror:8, 4, 2, 1
  v = dpp_add<0x124, 0xF>(v);
  v = dpp_add<0x122, 0xF>(v);
  return dpp_add<0x121, 0xF>(v);
}

// Sum over the workgroup, same value and summation order in every thread.
__device__ double block_sum(double v, double* red) {
  v = wave_sum_e(v);
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  __syncthreads();
  if (l == 0) red[w] = v;
  __syncthreads();
  double s = 0.0;
  const int nw = blockDim.x >> 6;
  for (int i = 0; i < nw; ++i) s += red[i];
  return s;
}

__global__ __launch_bounds__(256) void k_copy_square(int k, const double* __restrict__ H, int64_t ldh,
                                                     double* __restrict__ A) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)k * k) return;
  const int64_t j = t / k, i = t - j * k;
  A[t] = H[i + j * ldh];
}

// Householder reduction to tridiagonal form, one workgroup, full symmetric
// storage in global memory (L2 resident), one row per thread.  Step k uses
// the reflector v_k (v_k[k+1] = 1) with scalar tau_k and w_k = p - (tau/2)(p.v)v,
// p = tau A22 v.  The rank-2 update of step k and the product p of step k+1
// share one pass over the trailing matrix: column k+1 is updated first, v_{k+1}
// is formed from it, then every remaining entry is updated and immediately
// multiplied into p_{k+1}.  Reflector k is stored below the subdiagonal of
// column k.
__global__ __launch_bounds__(1024) void k_tridiag(int m, double* __restrict__ A, double* __restrict__ d,
                                                  double* __restrict__ e, double* __restrict__ tau) {
  extern __shared__ double sh[];
  double* vb[2] = {sh, sh + m};
  double* wb[2] = {sh + 2 * m, sh + 3 * m};
  double* red = sh + 4 * m;
  const int tid = threadIdx.x, nt = blockDim.x;
  if (m == 1) {
    if (tid == 0) d[0] = A[0];
    return;
  }
  if (m == 2) {
    if (tid == 0) {
      d[0] = A[0];
      d[1] = A[3];
      e[0] = A[1];
      tau[0] = 0.0;
    }
    return;
  }
  // reflector from column k (entries k+1..m-1) into v (absolute indexing);
  // returns tau (0 when the column is already reduced) and sets e[k]
  auto make_reflector = [&](int k, double* v) -> double {
    const double* col = A + (int64_t)k * m;
    double s = 0.0;
    for (int i = k + 2 + tid; i < m; i += nt) s = fma(col[i], col[i], s);
    s = block_sum(s, red);
    const double alpha = col[k + 1];
    double beta = alpha, tk = 0.0, v0 = 1.0;
    if (s > 0.0) {
      const double mu = sqrt(alpha * alpha + s);
      beta = alpha <= 0.0 ? mu : -mu;
      v0 = alpha - beta;
      tk = (beta - alpha) / beta;
    }
    for (int i = tid; i < m; i += nt) v[i] = (i <= k) ? 0.0 : (i == k + 1 ? 1.0 : (tk == 0.0 ? 0.0 : col[i] / v0));
    if (tid == 0) {
      e[k] = beta;
      tau[k] = tk;
    }
    __syncthreads();
    return tk;
  };
  // w = p - (tau/2)(p.v) v with p already in w (scaled by tau)
  auto finish_w = [&](int k, double tk, double* v, double* w) {
    double pv = 0.0;
    for (int i = k + 1 + tid; i < m; i += nt) pv = fma(w[i], v[i], pv);
    pv = block_sum(pv, red);
    const double K = 0.5 * tk * pv;
    for (int i = tid; i < m; i += nt) w[i] = (i <= k) ? 0.0 : w[i] - K * v[i];
    __syncthreads();
  };

  // step 0: reflector and the plain product p = tau A22 v
  if (tid == 0) d[0] = A[0];
  double tk = make_reflector(0, vb[0]);
  {
    double* v = vb[0];
    double* w = wb[0];
    for (int i = 1 + tid; i < m; i += nt) {
      double acc = 0.0;
#pragma unroll 8
      for (int j = 1; j < m; ++j) acc = fma(A[i + (int64_t)j * m], v[j], acc);
      w[i] = tk * acc;
    }
    __syncthreads();
    finish_w(0, tk, v, w);
  }
  int cur = 0;
  for (int k = 0; k + 2 < m; ++k) {
    double* v = vb[cur];
    double* w = wb[cur];
    // store reflector k below the subdiagonal of column k
    for (int i = k + 2 + tid; i < m; i += nt) A[i + (int64_t)k * m] = v[i];
    // rank-2 update of column k+1 (rows k+1..m-1)
    const int c = k + 1;
    for (int i = c + tid; i < m; i += nt) A[i + (int64_t)c * m] -= v[i] * w[c] + w[i] * v[c];
    __syncthreads();
    if (tid == 0) d[c] = A[c + (int64_t)c * m];
    if (c + 2 > m - 1) {
      // last 2 x 2 block: update the remaining entry and finish
      if (tid == 0) {
        const int j = c + 1;
        const double a = A[j + (int64_t)j * m] - 2.0 * v[j] * w[j];
        A[j + (int64_t)j * m] = a;
        d[j] = a;
        e[c] = A[j + (int64_t)c * m];
        tau[c] = 0.0;
      }
      break;
    }
    double* vn = vb[cur ^ 1];
    double* wn = wb[cur ^ 1];
    const double tn = make_reflector(c, vn);
    // fused pass: update rows/cols >= c+1 with step k, accumulate p_{k+1}
    for (int i = c + 1 + tid; i < m; i += nt) {
      const double vi = v[i], wi = w[i];
      double acc = 0.0;
      double* __restrict__ ai = A + i;
      int j = c + 1;
      // eight independent loads in flight before the dependent updates
      for (; j + 8 <= m; j += 8) {
        double a[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) a[u] = ai[(int64_t)(j + u) * m];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          a[u] = a[u] - vi * w[j + u] - wi * v[j + u];
          ai[(int64_t)(j + u) * m] = a[u];
          acc = fma(a[u], vn[j + u], acc);
        }
      }
      for (; j < m; ++j) {
        const double a = ai[(int64_t)j * m] - vi * w[j] - wi * v[j];
        ai[(int64_t)j * m] = a;
        acc = fma(a, vn[j], acc);
      }
      wn[i] = tn * acc;
    }
    __syncthreads();
    finish_w(c, tn, vn, wn);
    cur ^= 1;
  }
}

// One step of the same Householder reduction spread over many workgroups
// (one launch per reflector; used for larger matrices, where a single
// workgroup is latency-bound).  Launch k:
//   * every workgroup finishes w_{k-1} = p_{k-1} - (tau_{k-1}/2)(p_{k-1}.v_{k-1}) v_{k-1}
//     from the previous launch's p, applies reflector k-1 to column k on the
//     fly and forms reflector k from it (the same arithmetic in the same
//     order in every workgroup, so all agree bit for bit);
//   * workgroup 0 records d_k, e_k, tau_k and v_k, and stores v_{k-1} below
//     the subdiagonal of column k-1 (no workgroup reads that column here);
//   * each wavefront owns whole columns j > k: it applies reflector k-1 to
//     rows > k of column j (the matrix is symmetric, so a column is a row and
//     the lanes read consecutive addresses) and forms p_k[j] = tau_k (A v_k)_j.
// Column k is only read in launch k; columns > k are only touched by their
// owner, so no two workgroups write the same entry.
__global__ __launch_bounds__(256) void k_tri_step(int m, int k, double* __restrict__ A, double* __restrict__ d,
                                                  double* __restrict__ e, double* __restrict__ tau,
                                                  double* __restrict__ pv) {
  extern __shared__ double sh[];
  double* vp = sh;           // v_{k-1}
  double* w = sh + m;        // w_{k-1}
  double* vk = sh + 2 * m;   // column k after reflector k-1, then v_k
  double* red = sh + 3 * m;
  const int tid = threadIdx.x, nt = blockDim.x;
  const double* pprev = pv + (int64_t)((k + 1) & 1) * m;
  double* pcur = pv + (int64_t)(k & 1) * m;
  const double* vprev_g = pv + (int64_t)(2 + ((k + 1) & 1)) * m;
  double* vcur_g = pv + (int64_t)(2 + (k & 1)) * m;
  // w_{k-1}
  if (k == 0) {
    for (int i = tid; i < m; i += nt) {
      vp[i] = 0.0;
      w[i] = 0.0;
    }
    __syncthreads();
  } else {
    double s = 0.0;
    for (int i = tid; i < m; i += nt) {
      const double v = i >= k ? vprev_g[i] : 0.0;
      vp[i] = v;
      if (i >= k) s = fma(pprev[i], v, s);
    }
    s = block_sum(s, red);
    const double K = 0.5 * tau[k - 1] * s;
    for (int i = tid; i < m; i += nt) w[i] = i >= k ? pprev[i] - K * vp[i] : 0.0;
    __syncthreads();
  }
  // column k after reflector k-1, and reflector k
  const double wk = w[k], vpk = vp[k];
  double s = 0.0;
  for (int i = tid; i < m; i += nt) {
    const double a = i >= k ? A[i + (int64_t)k * m] - vp[i] * wk - w[i] * vpk : 0.0;
    vk[i] = a;
    if (i >= k + 2) s = fma(a, a, s);
  }
  s = block_sum(s, red);
  const double dk = vk[k];
  const double alpha = k + 1 < m ? vk[k + 1] : 0.0;
  double beta = alpha, tk = 0.0, v0 = 1.0;
  if (s > 0.0) {
    const double mu = sqrt(alpha * alpha + s);
    beta = alpha <= 0.0 ? mu : -mu;
    v0 = alpha - beta;
    tk = (beta - alpha) / beta;
  }
  __syncthreads();
  for (int i = tid; i < m; i += nt) vk[i] = (i <= k) ? 0.0 : (i == k + 1 ? 1.0 : (tk == 0.0 ? 0.0 : vk[i] / v0));
  __syncthreads();
  if (blockIdx.x == 0) {
    if (tid == 0) {
      d[k] = dk;
      e[k] = beta;
      tau[k] = tk;
    }
    for (int i = tid; i < m; i += nt) vcur_g[i] = vk[i];
    if (k >= 1)
      for (int i = k + 1 + tid; i < m; i += nt) A[i + (int64_t)(k - 1) * m] = vp[i];
  }
  // owned columns
  const int lane = tid & 63;
  const int nwaves = gridDim.x * (nt >> 6);
  for (int j = k + 1 + blockIdx.x * (nt >> 6) + (tid >> 6); j < m; j += nwaves) {
    double* __restrict__ col = A + (int64_t)j * m;
    const double wj = w[j], vj = vp[j];
    double dot = 0.0;
    int i = k + 1 + lane;
    for (; i + 192 < m; i += 256) {
      double a[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) a[u] = col[i + 64 * u];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int r = i + 64 * u;
        a[u] = a[u] - vp[r] * wj - w[r] * vj;
        col[r] = a[u];
        dot = fma(a[u], vk[r], dot);
      }
    }
    for (; i < m; i += 64) {
      const double a = col[i] - vp[i] * wj - w[i] * vj;
      col[i] = a;
      dot = fma(a, vk[i], dot);
      if (k == m - 2 && i == m - 1) d[m - 1] = a;
    }
    dot = wave_sum_e(dot);
    if (lane == 0) pcur[j] = tk * dot;
  }
}

// The same step, bit for bit, in registers, one column per wavefront.  The
// four wavefronts form the two sums of k_tri_step exactly as it does (element
// tid + 256 u per thread, rows from base = k rounded down to 256), and each
// holds the rows k + 1 + lane + 64 u of w_{k-1}, v_{k-1} and reflector k, where
// its own column j > k is updated.  Every load of the launch (p, v and column k
// in both arrangements, the owned column) is issued at once, so a launch is its
// own latency, one trip to memory and three sums: 6.0 -> 4.5 us at order 440.
// MT: 64 MT rows cover base .. m.
template <int MT>
__global__ __launch_bounds__(256) void k_tri_wave(int m, int k, double* __restrict__ A, double* __restrict__ d,
                                                  double* __restrict__ e, double* __restrict__ tau,
                                                  double* __restrict__ pv) {
  __shared__ double red[2][4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int gw = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + wave));
  const int j = min(k + 1 + gw, m - 1);
  const bool own = k + 1 + gw < m;
  const int base = k & ~255;
  const double* __restrict__ pprev = pv + (int64_t)((k + 1) & 1) * m;
  const double* __restrict__ vprev = pv + (int64_t)(2 + ((k + 1) & 1)) * m;
  double* __restrict__ pcur = pv + (int64_t)(k & 1) * m;
  double* __restrict__ vcur = pv + (int64_t)(2 + (k & 1)) * m;
  const double* __restrict__ colk = A + (int64_t)k * m;
  double* __restrict__ colj = A + (int64_t)j * m;
  const bool some = k > 0;
  constexpr int MA = (MT + 3) / 4;
  double pa[MA], va[MA], ca[MA], w[MT], v[MT], c[MT], x[MT];
#pragma unroll
  for (int t = 0; t < MA; ++t) {
    const int i = base + (int)threadIdx.x + 256 * t;
    const bool ok = i >= k && i < m;
    pa[t] = ok && some ? pprev[i] : 0.0;
    va[t] = ok && some ? vprev[i] : 0.0;
    ca[t] = ok ? colk[i] : 0.0;
  }
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    const int i = k + 1 + lane + 64 * t;
    const bool ok = i < m;
    w[t] = ok && some ? pprev[i] : 0.0;
    v[t] = ok && some ? vprev[i] : 0.0;
    c[t] = ok ? colk[i] : 0.0;
    x[t] = ok ? colj[i] : 0.0;
  }
  const double pk = some ? pprev[k] : 0.0, vpk = some ? vprev[k] : 0.0, ck = colk[k];
  const double pj = some ? pprev[j] : 0.0, vj = some ? vprev[j] : 0.0;
  const double tprev = some ? tau[k - 1] : 0.0;
  auto total = [&](double part, double* r) -> double {
    part = wave_butterfly(part);
    if (lane == 0) r[wave] = part;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) s += r[q];
    return s;
  };
  // w_{k-1} = p - (tau/2)(p.v) v
  double part = 0.0;
#pragma unroll
  for (int t = 0; t < MA; ++t) part = fma(pa[t], va[t], part);
  const double K = 0.5 * tprev * total(part, red[0]);
  const double wk = pk - K * vpk, wj = pj - K * vj;
  // column k after reflector k-1, and reflector k
  part = 0.0;
#pragma unroll
  for (int t = 0; t < MA; ++t) {
    const double wa = pa[t] - K * va[t];
    const double a = ca[t] - va[t] * wk - wa * vpk;
    if (base + (int)threadIdx.x + 256 * t >= k + 2) part = fma(a, a, part);
  }
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    w[t] = w[t] - K * v[t];
    c[t] = c[t] - v[t] * wk - w[t] * vpk;
  }
  const double s = total(part, red[1]);
  const double dk = ck - vpk * wk - wk * vpk;
  const double alpha = lane_value(c[0], 0);
  double beta = alpha, tk = 0.0, v0 = 1.0;
  if (s > 0.0) {
    const double mu = sqrt(alpha * alpha + s);
    beta = alpha <= 0.0 ? mu : -mu;
    v0 = alpha - beta;
    tk = (beta - alpha) / beta;
  }
#pragma unroll
  for (int t = 0; t < MT; ++t) c[t] = (t == 0 && lane == 0) ? 1.0 : (tk == 0.0 ? 0.0 : c[t] / v0);
  if (gw == 0) {
    if (lane == 0) {
      d[k] = dk;
      e[k] = beta;
      tau[k] = tk;
    }
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const int i = k + 1 + lane + 64 * t;
      if (i < m) {
        vcur[i] = c[t];
        if (some) A[i + (int64_t)(k - 1) * m] = v[t];
      }
    }
  }
  if (!own) return;
  double dot = 0.0;
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    const int i = k + 1 + lane + 64 * t;
    if (i < m) {
      const double a = x[t] - v[t] * wj - w[t] * vj;
      colj[i] = a;
      dot = fma(a, c[t], dot);
      if (k == m - 2) d[m - 1] = a;
    }
  }
  dot = wave_butterfly(dot);
  if (lane == 0) pcur[j] = tk * dot;
}

// The last reflectors (trailing order n = m - k0 <= kTriTail, k0 >= 1) in one
// workgroup with the trailing matrix in LDS, again with every sum and product
// of k_tri_step: the rows are elements (i mod 256) of the four parts of its
// sums.  Three barriers and the LDS traffic of the matrix per reflector, 2.6 us
// on average, against 3.6 us for a launch of k_tri_wave.
constexpr int kTriTail = 128;
constexpr size_t tri_tail_lds(int n) { return sizeof(double) * ((size_t)n * n + 5 * kTriTail + 8); }
__global__ __launch_bounds__(1024) void k_tri_tail(int m, int k0, double* __restrict__ A, double* __restrict__ d,
                                                   double* __restrict__ e, double* __restrict__ tau,
                                                   const double* __restrict__ pv) {
  extern __shared__ double sh[];
  const int n = m - k0, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  double* a = sh;               // a[c * n + r], columns and rows k0 ..
  double* p = a + n * n;        // p_{k-1}, then p_k
  double* v = p + kTriTail;     // v_{k-1}
  double* w = v + kTriTail;
  double* y = w + kTriTail;     // column k after reflector k-1
  double* vn = y + kTriTail;    // v_k
  double* red = vn + kTriTail;  // 2 x 4
  {
    const double* __restrict__ pp = pv + (int64_t)((k0 + 1) & 1) * m;
    const double* __restrict__ vp = pv + (int64_t)(2 + ((k0 + 1) & 1)) * m;
    for (int c = wave; c < n; c += 16)
      for (int r = lane; r < n; r += 64) a[c * n + r] = A[(k0 + r) + (int64_t)(k0 + c) * m];
    for (int r = tid; r < n; r += 1024) {
      p[r] = pp[k0 + r];
      v[r] = vp[k0 + r];
    }
  }
  double tprev = tau[k0 - 1];
  // the row of this thread's element of the four-part sums (threads 0 .. 255)
  const int row = ((tid - k0) & 255);  // (k0 + row) mod 256 == tid
  __syncthreads();
  for (int k = 0; k + 2 <= n; ++k) {
    const bool mine = tid < 256 && row >= k && row < n;
    double part = mine ? fma(p[row], v[row], 0.0) : 0.0;
    if (tid < 256) {
      part = wave_butterfly(part);
      if (lane == 0) red[wave] = part;
    }
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) s += red[q];
    const double K = 0.5 * tprev * s;
    const double vpk = v[k], wk = p[k] - K * vpk;
    if (tid < 256) {
      part = 0.0;
      if (mine) {
        const double wr = p[row] - K * v[row];
        const double b = a[k * n + row] - v[row] * wk - wr * vpk;
        w[row] = wr;
        y[row] = b;
        if (row >= k + 2) part = fma(b, b, part);
      }
      part = wave_butterfly(part);
      if (lane == 0) red[4 + wave] = part;
    }
    __syncthreads();
    s = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) s += red[4 + q];
    const double alpha = y[k + 1];
    double beta = alpha, tk = 0.0, v0 = 1.0;
    if (s > 0.0) {
      const double mu = sqrt(alpha * alpha + s);
      beta = alpha <= 0.0 ? mu : -mu;
      v0 = alpha - beta;
      tk = (beta - alpha) / beta;
    }
    double c[2], vv[2], ww[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int r = k + 1 + lane + 64 * u;
      const bool ok = r < n;
      vv[u] = ok ? v[r] : 0.0;
      ww[u] = ok ? w[r] : 0.0;
      c[u] = (u == 0 && lane == 0) ? 1.0 : (tk == 0.0 || !ok ? 0.0 : y[r] / v0);
      if (ok && wave == 15) {
        vn[r] = c[u];
        A[(k0 + r) + (int64_t)(k0 + k - 1) * m] = vv[u];
      }
    }
    if (tid == 0) {
      d[k0 + k] = y[k];
      e[k0 + k] = beta;
      tau[k0 + k] = tk;
    }
    for (int j = k + 1 + wave; j < n; j += 16) {
      const double wj = w[j], vj = v[j];
      double dot = 0.0;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int r = k + 1 + lane + 64 * u;
        if (r < n) {
          const double b = a[j * n + r] - vv[u] * wj - ww[u] * vj;
          a[j * n + r] = b;
          dot = fma(b, c[u], dot);
          if (k == n - 2) d[m - 1] = b;
        }
      }
      dot = wave_butterfly(dot);
      if (lane == 0) p[j] = tk * dot;
    }
    tprev = tk;
    __syncthreads();
    double* t = v;
    v = vn;
    vn = t;
  }
}

// Number of eigenvalues of the tridiagonal matrix below x, the pairs (d_j,
// e_{j-1}^2) in LDS, padded to a multiple of kSturmB rows: negative ratios q_j =
// (d_j - x) - e_{j-1}^2 / q_{j-1}, a chain of divisions.
constexpr int kSturmB = 8;
__device__ __forceinline__ int sturm_count(int m, const double2* __restrict__ de, double x, double pivmin) {
  int c = 0;
  double q = 1.0;
  double2 cur[kSturmB], nxt[kSturmB];
#pragma unroll
  for (int u = 0; u < kSturmB; ++u) cur[u] = de[u];
  for (int j0 = 0; j0 < m; j0 += kSturmB) {
#pragma unroll
    for (int u = 0; u < kSturmB; ++u) nxt[u] = de[j0 + kSturmB + u];
#pragma unroll
    for (int u = 0; u < kSturmB; ++u) {
      // (row 0: e_{-1} = 0 over q = 1; rows past m count nothing)
      q = (cur[u].x - x) - cur[u].y / q;
      if (fabs(q) < pivmin) q = -pivmin;
      if (q < 0.0 && j0 + u < m) ++c;
    }
#pragma unroll
    for (int u = 0; u < kSturmB; ++u) cur[u] = nxt[u];
  }
  return c;
}

// The same count from the sign changes of p_j = (d_j - x) p_{j-1} -
// e_{j-1}^2 p_{j-2}, one dependent multiply-add per row; entries and x scaled by
// a power of two to at most one (`scale` for x and d, e^2 by it twice: its
// square is infinite where the entries are below 2^-512), so that in eight rows
// |p| grows at most by 3^8, and brought back by a power of two every eight rows.
// A pivot p_j / p_{j-1} of less than 2^-60 counts as -2^-60, as the ratios' pivots
// below their floor count as minus it: eight rows shrink |p| at most by 2^480,
// and a run of diagonal entries equal to x does not take it to zero.
// Rounds differently from the ratios, so it is for points many roundings
// away from the eigenvalue sought, where the counts agree.
__device__ __forceinline__ int sturm_count_far(int m, const double2* __restrict__ de, double x, double scale) {
  int cnt = 0;
  double p1 = 1.0, p2 = 0.0;
  x *= scale;
  double2 cur[kSturmB], nxt[kSturmB];
#pragma unroll
  for (int u = 0; u < kSturmB; ++u) cur[u] = de[u];
  for (int j0 = 0; j0 < m; j0 += kSturmB) {
#pragma unroll
    for (int u = 0; u < kSturmB; ++u) nxt[u] = de[j0 + kSturmB + u];
#pragma unroll
    for (int u = 0; u < kSturmB; ++u) {
      double p = fma(fma(cur[u].x, scale, -x), p1, -(cur[u].y * scale * scale) * p2);
      const double least = -0x1p-60 * p1;
      p = fabs(p) < fabs(least) ? least : p;
      if (j0 + u < m) cnt += (int)((uint32_t)(__double2hiint(p) ^ __double2hiint(p1)) >> 31);
      p2 = p1;
      p1 = p;
    }
    const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(p1), fabs(p2)));
    p1 = ldexp(p1, ex);
    p2 = ldexp(p2, ex);
#pragma unroll
    for (int u = 0; u < kSturmB; ++u) cur[u] = nxt[u];
  }
  return cnt;
}

__global__ __launch_bounds__(256) void k_tri_prep(int m, const double* __restrict__ d, const double* __restrict__ e,
                                                  double* __restrict__ bounds) {
  // bounds = {gershgorin lo, hi, pivmin, scale}
  __shared__ double red[3][4];
  double lo = INFINITY, hi = -INFINITY, emax2 = 0.0;
  for (int j = threadIdx.x; j < m; j += blockDim.x) {
    const double r = (j > 0 ? fabs(e[j - 1]) : 0.0) + (j < m - 1 ? fabs(e[j]) : 0.0);
    lo = fmin(lo, d[j] - r);
    hi = fmax(hi, d[j] + r);
    if (j < m - 1) {
      emax2 = fmax(emax2, e[j] * e[j]);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, off));
    hi = fmax(hi, __shfl_xor(hi, off));
    emax2 = fmax(emax2, __shfl_xor(emax2, off));
  }
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = lo;
    red[1][threadIdx.x >> 6] = hi;
    red[2][threadIdx.x >> 6] = emax2;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) {
      lo = fmin(red[0][0], red[0][w]);
      red[0][0] = lo;
      hi = fmax(red[1][0], red[1][w]);
      red[1][0] = hi;
      emax2 = fmax(red[2][0], red[2][w]);
      red[2][0] = emax2;
    }
    lo = red[0][0];
    hi = red[1][0];
    const double pivmin = DBL_MIN * fmax(1.0, red[2][0]);
    const double tn = fmax(fabs(lo), fabs(hi));
    bounds[0] = lo - 2.0 * DBL_EPSILON * tn - pivmin;
    bounds[1] = hi + 2.0 * DBL_EPSILON * tn + pivmin;
    bounds[2] = pivmin;
    // the power of two that scales the matrix and its bracket to at most one
    int ex = 0;
    (void)frexp(fmax(tn, DBL_MIN), &ex);
    bounds[3] = ldexp(1.0, -min(max(ex + 1, -1000), 1000));
  }
}

// Eigenvalue i by 65-section: the 64 lanes of a wavefront evaluate Sturm
// counts at 64 interior points of the bracket, which shrinks 65-fold per
// round until it is a few ulps wide.  The counts are chains of m dependent
// steps, ten times.  While the points are at least 2^-20 of the spectrum's
// scale apart, one of them lies within rounding (some 2^-45) of the eigenvalue
// only once in 2^25 rounds, and the division-free count serves; the others
// use the ratios.  440 eigenvalues: 486 us with ratios from global memory
// throughout, 286 us so.
__global__ __launch_bounds__(256) void k_bisect(int m, const double* __restrict__ d, const double* __restrict__ e,
                                                const double* __restrict__ bounds, double* __restrict__ theta) {
  extern __shared__ double2 de[];
  for (int j = threadIdx.x; j < (m + kSturmB - 1) / kSturmB * kSturmB + kSturmB; j += blockDim.x) {
    const double ej = j > 0 && j < m ? e[j - 1] : 0.0;
    de[j] = make_double2(j < m ? d[j] : 0.0, ej * ej);
  }
  __syncthreads();
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (i >= m) return;
  double lo = bounds[0], hi = bounds[1];
  const double pivmin = bounds[2], scale = bounds[3];
  for (int it = 0; it < 64; ++it) {
    if (hi - lo <= 2.0 * DBL_EPSILON * fmax(fabs(lo), fabs(hi)) + pivmin) break;
    const double h = (hi - lo) / 65.0;
    const double x = lo + (lane + 1) * h;
    const bool above = (h * scale >= 0x1p-20 ? sturm_count_far(m, de, x, scale) : sturm_count(m, de, x, pivmin)) > i;
    const unsigned long long mask = __ballot(above);
    double nlo, nhi;
    if (mask == 0ull) {
      nlo = __shfl(x, 63);
      nhi = hi;
    } else {
      const int f = __ffsll((long long)mask) - 1;
      nhi = __shfl(x, f);
      nlo = f > 0 ? __shfl(x, f - 1) : lo;
    }
    if (!(nhi - nlo < hi - lo)) break;  // no progress: bracket is at rounding level
    lo = nlo;
    hi = nhi;
  }
  if (lane == 0) theta[i] = 0.5 * (lo + hi);
}

// Inverse iteration, one selected eigenvalue per workgroup of one wavefront.
// Within a cluster of (nearly) equal values the shifts are kept 10 eps apart
// and each member starts from its own vector (its position in the cluster
// sets the phase), so the members converge to different directions of the
// eigenspace; k_cluster_orth then orthonormalises each cluster's vectors.  The
// recurrences run in one lane, their running values in registers, the LU
// factors and the iterate in LDS; what is independent along m (start vector,
// the pivots' inverses, the result) is done by all lanes.  Bound by the issue
// and latency of a single wavefront's chain: one division per row in the
// factorisation, one multiply-add per row forward and two operations backward;
// the rows are read kIvB ahead, with the normalisation of an iterate applied
// by the next sweep's reads.  Pivots are kept
// at eps times the norm at least, a swapped row's off-diagonal too.  Where the
// squares of an iterate's norm leave the range of a double (its entries are about
// 1 / (eps norm)) they are summed again, of the iterate times a power of two.
// 110 vectors of order 440: 560 us with two
// divisions per row, several lanes' arrays interleaved and separate passes for
// the norms, 232 us so.
constexpr int kIvB = 8;
constexpr int kEigMax = 2048;  // largest order
// doubles of LDS: five arrays and one flag word per kIvB rows
__host__ __device__ constexpr int invit_doubles(int m) { return 5 * m + (m / kIvB + 2) / 2 + 1; }
__global__ __launch_bounds__(64) void k_invit(int m, const double* __restrict__ d, const double* __restrict__ e,
                                              const double* __restrict__ bounds, int ncl,
                                              const int32_t* __restrict__ cstart, const double* __restrict__ sel,
                                              double* __restrict__ Z) {
  extern __shared__ double ivs[];
  const int lane = threadIdx.x, s = blockIdx.x;
  const double tn = fmax(fabs(bounds[0]), fabs(bounds[1]));
  const double tiny = DBL_EPSILON * fmax(tn, DBL_MIN);
  double* __restrict__ rinv = ivs;
  double* __restrict__ u1 = rinv + m;
  double* __restrict__ u2 = u1 + m;
  double* __restrict__ lm = u2 + m;
  double* __restrict__ z = lm + m;
  uint32_t* __restrict__ flags = reinterpret_cast<uint32_t*>(z + m);
  // the first member of s's cluster (cstart ascending, cstart[0] = 0)
  int lo = 0, hi = ncl;  // cstart[lo] <= s < cstart[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (cstart[mid] <= s) lo = mid;
    else hi = mid;
  }
  const int c0 = cstart[lo], pos = s - c0;
  // start vector: 1 + 0.5 u, u in [-1, 1) from an integer hash of (row,
  // position in the cluster), so that the members of a cluster start from
  // linearly independent vectors
  for (int i = lane; i < m; i += 64) {
    uint32_t h = (uint32_t)i * 0x9E3779B1u ^ ((uint32_t)pos + 1u) * 0x85EBCA77u;
    h ^= h >> 16;
    h *= 0x7FEB352Du;
    h ^= h >> 15;
    h *= 0x846CA68Bu;
    h ^= h >> 16;
    z[i] = 1.0 + 0.5 * ((double)h * (2.0 / 4294967296.0) - 1.0);
  }
  // Blocks of kIvB rows run without a test per row, the rest of the rows with
  // one (m - 1 eliminations, then m - 1 rows forward and m back).
  const int full = (m - 1) / kIvB * kIvB;
  if (lane == 0) {
    // shifts of the cluster's members up to s, each at least 10 eps above the last
    double lam = sel[c0];
    for (int t = c0 + 1; t <= s; ++t) lam = sel[t] - lam < 10.0 * tiny ? lam + 10.0 * tiny : sel[t];
    // LU of T - lam I with partial pivoting; row i is (a, b, c) at columns
    // (i, i+1, i+2) while it is being eliminated
    double a = d[0] - lam;
    double b = m > 1 ? e[0] : 0.0;
    uint32_t fl = 0;
    auto eliminate = [&](int i, int u, double be, double ad, double ce) {
      const bool sw = fabs(a) < fabs(be);
      // (a zero pivot has a zero below it: l = 0)
      const double piv = sw ? be : a;
      const double l = (sw ? a : be) / (piv == 0.0 ? 1.0 : piv);
      const double v1 = sw ? ad : b;
      rinv[i] = fabs(piv) < tiny ? (piv < 0.0 ? -tiny : tiny) : piv;
      lm[i] = l;
      u1[i] = v1;
      u2[i] = sw ? ce : 0.0;
      fl |= (sw ? 1u : 0u) << u;
      a = (sw ? b : ad) - l * v1;
      b = sw ? -l * ce : ce;
    };
    double eb[kIvB], dn[kIvB], en[kIvB];
    auto load = [&](int i0) {
#pragma unroll
      for (int u = 0; u < kIvB; ++u) {
        const int i = min(i0 + u, m - 2);
        eb[u] = e[i];
        dn[u] = d[i + 1];
        const double en1 = e[min(i + 1, m - 2)];
        en[u] = i + 2 < m ? en1 : 0.0;
      }
    };
    if (full > 0) load(0);
    for (int i0 = 0; i0 < full; i0 += kIvB) {
      double be[kIvB], ad[kIvB], ce[kIvB];
#pragma unroll
      for (int u = 0; u < kIvB; ++u) {
        be[u] = eb[u];
        ad[u] = dn[u] - lam;
        ce[u] = en[u];
      }
      load(i0 + kIvB);
      fl = 0;
#pragma unroll
      for (int u = 0; u < kIvB; ++u) eliminate(i0 + u, u, be[u], ad[u], ce[u]);
      flags[i0 / kIvB] = fl;
    }
    fl = 0;
    for (int i = full; i + 1 < m; ++i) eliminate(i, i - full, e[i], d[i + 1] - lam, i + 2 < m ? e[i + 1] : 0.0);
    flags[full / kIvB] = fl;
    rinv[m - 1] = fabs(a) < tiny ? (a < 0.0 ? -tiny : tiny) : a;
    u1[m - 1] = 0.0;
    u2[m - 1] = 0.0;
    if (m >= 2) u2[m - 2] = 0.0;
  }
  __syncthreads();
  for (int i = lane; i < m; i += 64) rinv[i] = 1.0 / rinv[i];
  __syncthreads();
  double rs = 1.0;  // what normalises the iterate in z
  if (lane == 0) {
    for (int it = 0; it < 3; ++it) {
      // forward: row swaps and elimination
      double y = z[0] * rs;
      {
        auto row = [&](int i, bool sw, double zn, double l) {
          const double top = sw ? zn : y, rest = sw ? y : zn;
          z[i] = top;
          y = rest - l * top;
        };
        double nz[kIvB], nl[kIvB];
        uint32_t nf = 0;
        // (rows up to full + kIvB - 1 of z and lm: inside the arrays' LDS)
        auto load = [&](int i0) {
#pragma unroll
          for (int u = 0; u < kIvB; ++u) {
            nz[u] = z[i0 + u + 1];
            nl[u] = lm[i0 + u];
          }
          nf = flags[i0 / kIvB];
        };
        if (full > 0) load(0);
        for (int i0 = 0; i0 < full; i0 += kIvB) {
          double zv[kIvB], lv[kIvB];
          const uint32_t fl = nf;
#pragma unroll
          for (int u = 0; u < kIvB; ++u) {
            zv[u] = nz[u] * rs;
            lv[u] = nl[u];
          }
          if (i0 + kIvB < full) load(i0 + kIvB);
#pragma unroll
          for (int u = 0; u < kIvB; ++u) row(i0 + u, (fl >> u) & 1u, zv[u], lv[u]);
        }
        const uint32_t fl = flags[full / kIvB];
        for (int i = full; i + 1 < m; ++i) row(i, (fl >> (i - full)) & 1u, z[i + 1] * rs, lm[i]);
      }
      z[m - 1] = y;
      // backward substitution with U (diagonal inverse, two superdiagonals)
      double x1 = 0.0, x2 = 0.0, nrm = 0.0;
      {
        auto row = [&](int i, double zi, double v1, double v2, double r) {
          const double x = (fma(-v2, x2, zi) - v1 * x1) * r;
          z[i] = x;
          nrm = fma(x, x, nrm);
          x2 = x1;
          x1 = x;
        };
        double nz[kIvB], n1[kIvB], n2[kIvB], nr[kIvB];
        auto load = [&](int i0) {
#pragma unroll
          for (int u = 0; u < kIvB; ++u) {
            nz[u] = z[i0 - u];
            n1[u] = u1[i0 - u];
            n2[u] = u2[i0 - u];
            nr[u] = rinv[i0 - u];
          }
        };
        int i0 = m - 1;
        if (i0 + 1 >= kIvB) load(i0);
        for (; i0 + 1 >= kIvB; i0 -= kIvB) {
          double zv[kIvB], v1[kIvB], v2[kIvB], rv[kIvB];
#pragma unroll
          for (int u = 0; u < kIvB; ++u) {
            zv[u] = nz[u];
            v1[u] = n1[u];
            v2[u] = n2[u];
            rv[u] = nr[u];
          }
          if (i0 + 1 >= 2 * kIvB) load(i0 - kIvB);
#pragma unroll
          for (int u = 0; u < kIvB; ++u) row(i0 - u, zv[u], v1[u], v2[u], rv[u]);
        }
        for (; i0 >= 0; --i0) row(i0, z[i0], u1[i0], u2[i0], rinv[i0]);
      }
      double unit = 1.0;
      if (!(nrm > 0x1p-900 && nrm < 0x1p1000)) {
        double mx = 0.0;
        for (int i = 0; i < m; ++i) mx = fmax(mx, fabs(z[i]));
        int ex = 0;
        (void)frexp(mx, &ex);
        unit = ldexp(1.0, min(max(-ex, -1000), 1000));
        nrm = 0.0;
        for (int i = 0; i < m; ++i) {
          const double x = z[i] * unit;
          nrm = fma(x, x, nrm);
        }
      }
      rs = nrm > 0.0 ? unit / sqrt(nrm) : 0.0;
    }
  }
  __syncthreads();
  const double r = lane_value(rs, 0);
  for (int i = lane; i < m; i += 64) Z[(int64_t)s * m + i] = z[i] * r;
}

// The vectors of each cluster with more than one member (Z columns
// cstart[c] .. cstart[c+1]-1): classical Gram-Schmidt twice against the
// cluster's earlier members, then normalisation; one workgroup per cluster.
__device__ __forceinline__ double block_sum256(double v, double* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

__global__ __launch_bounds__(256) void k_cluster_orth(int m, int ncl, const int32_t* __restrict__ cstart,
                                                      double* __restrict__ Z) {
  __shared__ double red[4];
  const int c = blockIdx.x;
  if (c >= ncl) return;
  const int c0 = cstart[c], c1 = cstart[c + 1];
  if (c1 - c0 < 2) return;
  for (int j = c0; j < c1; ++j) {
    double* zj = Z + (int64_t)j * m;
    for (int pass = 0; pass < 2; ++pass) {
      for (int q = c0; q < j; ++q) {
        const double* zq = Z + (int64_t)q * m;
        double dot = 0.0;
        for (int i = threadIdx.x; i < m; i += 256) dot = fma(zq[i], zj[i], dot);
        dot = block_sum256(dot, red);
        for (int i = threadIdx.x; i < m; i += 256) zj[i] -= dot * zq[i];
        __syncthreads();
      }
    }
    double nrm = 0.0;
    for (int i = threadIdx.x; i < m; i += 256) nrm = fma(zj[i], zj[i], nrm);
    nrm = block_sum256(nrm, red);
    const double rn = nrm > 0.0 ? 1.0 / sqrt(nrm) : 0.0;
    for (int i = threadIdx.x; i < m; i += 256) zj[i] *= rn;
    __syncthreads();
  }
}

// The reflectors' columns completed in place: column k < m - 2 gets zeros in
// rows 0 .. k and one in row k + 1.
__global__ __launch_bounds__(256) void k_reflector_heads(int m, double* __restrict__ A) {
  const int k = blockIdx.x;
  for (int i = threadIdx.x; i <= k + 1; i += 256) A[i + (int64_t)k * m] = i <= k ? 0.0 : 1.0;
}

// y = H_0 H_1 ... H_{m-3} z, H_k = I - tau_k v_k v_k^T, v_k = column k of A
// (k_reflector_heads).  One wavefront per vector; lane l keeps rows l+64t (rows
// past m read row 0, where every v_k is zero).  A chain of m - 2 wavefront
// sums, each a few tens of instructions of one wavefront; the next D reflectors
// are loaded while D are applied, since a trip to memory takes longer than one.
// 110 vectors of order 440: 394 us with sums through the LDS permute unit and
// one reflector at a time, 167 us so.
template <int MT, int D>
__global__ __launch_bounds__(256) void k_backtransform(int m, const double* __restrict__ A,
                                                       const double* __restrict__ tau, int nsel,
                                                       const double* __restrict__ Z, double* __restrict__ Y) {
  const int vec = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (vec >= nsel) return;
  double y[MT];
  int at[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    const int i = lane + 64 * t;
    y[t] = i < m ? Z[(int64_t)vec * m + i] : 0.0;
    at[t] = i < m ? i : 0;
  }
  // reflectors k, k-1, .., k-D+1 (below 0: tau 0)
  auto load = [&](int k, double (&v)[D][MT], double (&tk)[D]) {
#pragma unroll
    for (int q = 0; q < D; ++q) {
      const int kq = max(k - q, 0);
      const double* __restrict__ col = A + (int64_t)kq * m;
      const double t0 = tau[kq];
      tk[q] = k - q >= 0 ? t0 : 0.0;
#pragma unroll
      for (int t = 0; t < MT; ++t) v[q][t] = col[at[t]];
    }
  };
  auto apply = [&](const double (&v)[D][MT], const double (&tk)[D]) {
#pragma unroll
    for (int q = 0; q < D; ++q) {
      double s0 = 0.0, s1 = 0.0;
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        if (t & 1)
          s1 = fma(v[q][t], y[t], s1);
        else
          s0 = fma(v[q][t], y[t], s0);
      }
      const double dot = wave_total(s0 + s1) * tk[q];
#pragma unroll
      for (int t = 0; t < MT; ++t) y[t] -= dot * v[q][t];
    }
  };
  if (m >= 3) {
    double va[D][MT], vb[D][MT], ta[D], tb[D];
    load(m - 3, va, ta);
    for (int k = m - 3; k >= 0; k -= 2 * D) {
      load(k - D, vb, tb);
      apply(va, ta);
      load(k - 2 * D, va, ta);
      apply(vb, tb);
    }
  }
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    const int i = lane + 64 * t;
    if (i < m) Y[(int64_t)vec * m + i] = y[t];
  }
}

}  // namespace

void free_eig(EigWork& w) {
  double* ptrs[] = {w.A, w.d, w.e, w.bounds, w.tau, w.theta, w.pv, w.Z, w.Y, w.sel};
  for (double* p : ptrs)
    if (p) (void)hipFree(p);
  if (w.cl) (void)hipFree(w.cl);
  w = EigWork();
}

int eig_reserve(EigWork& w, int m, int nsel) {
  if ((size_t)m > w.cap_m) {
    double** ps[] = {&w.A, &w.d, &w.e, &w.bounds, &w.tau, &w.theta, &w.pv};
    for (double** p : ps) {
      if (*p) (void)hipFree(*p);
      *p = nullptr;
    }
    const size_t mm = (size_t)m;
    if (hipMalloc(&w.A, sizeof(double) * mm * mm) != hipSuccess || hipMalloc(&w.d, sizeof(double) * mm) != hipSuccess ||
        hipMalloc(&w.e, sizeof(double) * mm) != hipSuccess ||
        hipMalloc(&w.bounds, sizeof(double) * 4) != hipSuccess || hipMalloc(&w.tau, sizeof(double) * mm) != hipSuccess ||
        hipMalloc(&w.theta, sizeof(double) * mm) != hipSuccess || hipMalloc(&w.pv, sizeof(double) * 4 * mm) != hipSuccess) {
      set_error("eig_reserve: allocation failed");
      return KF_ENOMEM;
    }
    w.cap_m = mm;
    w.cap_sel = 0;  // Z/Y/scratch depend on m too
  }
  if ((size_t)nsel > w.cap_sel) {
    double** ps[] = {&w.Z, &w.Y, &w.sel};
    for (double** p : ps) {
      if (*p) (void)hipFree(*p);
      *p = nullptr;
    }
    if (w.cl) (void)hipFree(w.cl);
    w.cl = nullptr;
    const size_t ns = std::max<size_t>(nsel, 16);
    if (hipMalloc(&w.Z, sizeof(double) * w.cap_m * ns) != hipSuccess ||
        hipMalloc(&w.Y, sizeof(double) * w.cap_m * ns) != hipSuccess ||
        hipMalloc(&w.sel, sizeof(double) * ns) != hipSuccess ||
        hipMalloc(&w.cl, sizeof(int32_t) * (ns + 1)) != hipSuccess) {
      set_error("eig_reserve: allocation failed");
      return KF_ENOMEM;
    }
    w.cap_sel = ns;
  }
  return KF_OK;
}

int eig_values(EigWork& w, int k, const double* H, int64_t ldh, hipStream_t st) {
  if (k < 1) return KF_OK;
  if (k > kEigMax) {
    set_error("eigensolver: projected pencil larger than 2048");
    return KF_EINVAL;
  }
  KF_TRY(eig_reserve(w, k, 1));
  hipLaunchKernelGGL(k_copy_square, dim3(cdiv((int64_t)k * k, 256)), dim3(256), 0, st, k, H, ldh, w.A);
  KF_HIP(hipGetLastError());
  if (k < kTriMultiFrom) {
    const size_t lds = sizeof(double) * (4 * (size_t)k + 32);
    hipLaunchKernelGGL(k_tridiag, dim3(1), dim3(1024), lds, st, k, w.A, w.d, w.e, w.tau);
    KF_HIP(hipGetLastError());
  } else {
    // one launch per reflector; the grid shrinks with the trailing matrix
    const size_t lds = sizeof(double) * (3 * (size_t)k + 32);
    for (int j = 0; j + 2 <= k; ++j) {
      if (j >= 1 && k - j <= kTriTail) {
        const size_t tail = tri_tail_lds(k - j);
        KF_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_tri_tail),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)tri_tail_lds(kTriTail)));
        hipLaunchKernelGGL(k_tri_tail, dim3(1), dim3(1024), tail, st, k, j, w.A, w.d, w.e, w.tau, w.pv);
        KF_HIP(hipGetLastError());
        break;
      }
      const int cols = k - j - 1;
      const int mt = cdiv(k - (j & ~255), 64);
#define KF_TRI(MT) \
  hipLaunchKernelGGL(k_tri_wave<MT>, dim3(cdiv(cols, 4)), dim3(256), 0, st, k, j, w.A, w.d, w.e, w.tau, w.pv)
      if (mt <= 4)
        KF_TRI(4);
      else if (mt <= 8)
        KF_TRI(8);
      else if (mt <= 16)
        KF_TRI(16);
      else  // (beyond what the registers hold: vectors in LDS, columns strided)
        hipLaunchKernelGGL(k_tri_step, dim3(std::min(cdiv(cols, 4), 256)), dim3(256), lds, st, k, j, w.A, w.d, w.e,
                           w.tau, w.pv);
#undef KF_TRI
      KF_HIP(hipGetLastError());
    }
  }
  hipLaunchKernelGGL(k_tri_prep, dim3(1), dim3(256), 0, st, k, w.d, w.e, w.bounds);
  KF_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_bisect, dim3(cdiv(k, 4)), dim3(256), sizeof(double2) * (size_t)(k + 2 * kSturmB), st, k, w.d,
                     w.e, w.bounds, w.theta);
  KF_HIP(hipGetLastError());
  return KF_OK;
}

int eig_vectors(EigWork& w, int k, const double* theta_sel, const int32_t* cluster_start, int nclusters, int nsel,
                hipStream_t st) {
  if (nsel <= 0) return KF_OK;
  KF_TRY(eig_reserve(w, k, nsel));
  KF_HIP(hipMemcpyAsync(w.sel, theta_sel, sizeof(double) * nsel, hipMemcpyHostToDevice, st));
  KF_HIP(hipMemcpyAsync(w.cl, cluster_start, sizeof(int32_t) * (nclusters + 1), hipMemcpyHostToDevice, st));
  const size_t lds = sizeof(double) * (size_t)invit_doubles(k);
  if (lds > 65536)  // (the limit of every order: other threads launch this kernel too)
    KF_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_invit), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)(sizeof(double) * invit_doubles(kEigMax))));
  hipLaunchKernelGGL(k_invit, dim3(nsel), dim3(64), lds, st, k, w.d, w.e, w.bounds, nclusters, w.cl, w.sel, w.Z);
  KF_HIP(hipGetLastError());
  if (nclusters < nsel) {
    hipLaunchKernelGGL(k_cluster_orth, dim3(nclusters), dim3(256), 0, st, k, nclusters, w.cl, w.Z);
    KF_HIP(hipGetLastError());
  }
  if (k >= 3) {
    hipLaunchKernelGGL(k_reflector_heads, dim3(k - 2), dim3(256), 0, st, k, w.A);
    KF_HIP(hipGetLastError());
  }
  const int grid = cdiv(nsel, 4);
  const int mt = cdiv(k, 64);
  if (mt <= 1)
    hipLaunchKernelGGL((k_backtransform<1, 4>), dim3(grid), dim3(256), 0, st, k, w.A, w.tau, nsel, w.Z, w.Y);
  else if (mt <= 2)
    hipLaunchKernelGGL((k_backtransform<2, 4>), dim3(grid), dim3(256), 0, st, k, w.A, w.tau, nsel, w.Z, w.Y);
  else if (mt <= 4)
    hipLaunchKernelGGL((k_backtransform<4, 4>), dim3(grid), dim3(256), 0, st, k, w.A, w.tau, nsel, w.Z, w.Y);
  else if (mt <= 8)
    hipLaunchKernelGGL((k_backtransform<8, 4>), dim3(grid), dim3(256), 0, st, k, w.A, w.tau, nsel, w.Z, w.Y);
  else if (mt <= 16)
    hipLaunchKernelGGL((k_backtransform<16, 2>), dim3(grid), dim3(256), 0, st, k, w.A, w.tau, nsel, w.Z, w.Y);
  else
    hipLaunchKernelGGL((k_backtransform<32, 1>), dim3(grid), dim3(256), 0, st, k, w.A, w.tau, nsel, w.Z, w.Y);
  KF_HIP(hipGetLastError());
  // the host arrays must outlive the asynchronous copies
  KF_HIP(hipStreamSynchronize(st));
  return KF_OK;
}

}  // namespace kf
