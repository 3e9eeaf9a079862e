// The time step over stencil slices (StencilOp): the second-order step, the two
// launches of the fourth-order one, the batched step, and the detection and
// build of the form.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <string>
#include <vector>

#include "kf_device.h"
#include "kf_internal.h"

namespace kf {

namespace {

// ------------------------------------------------------------ stencil slices
// One wavefront per slice merges its rows' sorted columns into the ascending
// list of their offsets col - row.  FORM 0: width[slice] = the number of
// offsets (kStencilMax + 1 when there are more), negative when two rows store
// different values at one offset.  FORM 1 writes the slice's offsets, row masks
// and one value per offset at [slice * stride], FORM 2 a value per offset and
// row at [(slice * stride + offset) * 64 + row] (0 where the row has no entry).
template <typename VT, int FORM>
__global__ __launch_bounds__(256) void k_stencil(int32_t n, int32_t nslices, const int32_t* __restrict__ rowptr,
                                                 const int32_t* __restrict__ col, const double* __restrict__ val,
                                                 const double* __restrict__ rscale, int32_t* __restrict__ width,
                                                 int stride, VT* __restrict__ oval, int32_t* __restrict__ ooff,
                                                 uint64_t* __restrict__ omask) {
  const int slice = blockIdx.x * 4 + (int)(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (slice >= nslices) return;
  const int row = slice * 64 + lane;
  int a = 0, b = 0;
  double sc = 1.0;
  if (row < n) {
    a = rowptr[row];
    b = rowptr[row + 1];
    if (rscale) sc = rscale[row];
  }
  int cnt = 0;
  bool uniform = true;
  while (cnt <= kStencilMax) {
    const int mine = a < b ? col[a] - row : INT32_MAX;
    int off = mine;
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) off = min(off, __shfl_xor(off, s));
    if (off == INT32_MAX) break;
    const bool has = mine == off;
    const VT v = has ? (VT)(sc * val[a]) : (VT)0;
    const unsigned long long m = __ballot(has);
    const VT lead = __shfl(v, __ffsll(m) - 1);
    if (__ballot(has && !(v == lead)) != 0ull) uniform = false;
    if (FORM > 0) {
      const int64_t o = (int64_t)slice * stride + cnt;
      if (lane == 0) {
        if (FORM == 1) oval[o] = lead;
        ooff[o] = off;
        omask[o] = m;
      }
      if (FORM == 2) oval[o * 64 + lane] = v;
    }
    ++cnt;
    if (has) ++a;
  }
  if (FORM == 0) {
    if (lane == 0) width[slice] = uniform ? cnt : -cnt;
  } else {
    for (; cnt < stride; ++cnt) {
      const int64_t o = (int64_t)slice * stride + cnt;
      if (lane == 0) {
        if (FORM == 1) oval[o] = (VT)0;
        ooff[o] = 0;
        omask[o] = 0ull;
      }
      if (FORM == 2) oval[o * 64 + lane] = (VT)0;
    }
  }
}

// sum_j += (A x)(row, col0 + j) of a stencil slice.  The slice's entries are
// the same for the whole wavefront, so they come through the scalar cache and
// the vector loads are the gathers, which do not wait for an index load, and
// with ROWV the values of the rows.  Every load of a chunk is issued before its
// sums; rows without an entry gather their own element and multiply it by
// zero.  W: entries per slice when known (the loop is then unrolled in full),
// 0: `stride` entries, a multiple of 4, the last ones without rows where the
// list is shorter.  Where a lane has 64 bytes of a row or more those are left
// out: a batch gathered 8 rows for 5 or 7 of them, and was slower so than over
// stored entries.  Batched application, blocks of 16 in float64: 3 members 1732
// -> 1349 us (stored entries 1584), 16 members 13.98 -> 11.87 ms (14.21).  Below
// 64 bytes the branches cost what they save.
template <typename T, int B, int BL, int LPR, int W, bool ROWV>
__device__ __forceinline__ void stencil_product(const T* __restrict__ val, const int32_t* __restrict__ off,
                                                const uint64_t* __restrict__ mask, int stride, int slice, int rin,
                                                int row, const T* __restrict__ x, int col0, T (&sum)[BL]) {
  constexpr int U = W > 0 && BL * sizeof(T) <= 16 ? W : (W == 15 ? 5 : 4);
  constexpr bool leave_out = W == 0 && BL * sizeof(T) >= 64;
  const int64_t base = (int64_t)slice * (W > 0 ? W : stride);
  auto chunk = [&](int q0) {
    T a[U];
    int o[U];
    uint64_t m[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (W > 0 && q0 + u >= W) continue;
      a[u] = ROWV ? val[(base + q0 + u) * 64 + rin] : val[base + q0 + u];
      o[u] = off[base + q0 + u];
      m[u] = mask[base + q0 + u];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      // (the offsets stay in scalar registers ahead of the row tests)
      if (W > 0 && q0 + u >= W) continue;
      asm volatile("" : "+s"(o[u]));
    }
    Row<T, BL> xv[U];
    bool has[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (W > 0 && q0 + u >= W) continue;
      has[u] = LPR == 1 ? __builtin_amdgcn_inverse_ballot_w64(m[u]) : ((m[u] >> rin) & 1ull) != 0ull;
      const int c = row + (has[u] ? o[u] : 0);
      if (!leave_out || m[u] != 0) xv[u] = *reinterpret_cast<const Row<T, BL>*>(x + (int64_t)c * B + col0);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (W > 0 && q0 + u >= W) continue;
      if (leave_out && m[u] == 0) continue;
      const T au = ROWV || has[u] ? a[u] : (T)0;
#pragma unroll
      for (int j = 0; j < BL; ++j) sum[j] = fma(au, xv[u].v[j], sum[j]);
    }
  };
  if constexpr (W > 0) {
#pragma unroll
    for (int q0 = 0; q0 < W; q0 += U) chunk(q0);
  } else {
    for (int q0 = 0; q0 < stride; q0 += U) chunk(q0);
  }
}

// The fused step (k_leapfrog) over stencil slices.  With one value per offset
// there is no operator stream, a row's traffic is its vector levels alone (25 instead of 86 MB per middle
// step of the 96-cell cube in float64, whose levels then stay in the caches).
// A filter application of 38 steps there: 541 us with the stored entries,
// 266 us so (7.0 us a step, launch included); the 128-cell cube in float32,
// 51 steps: 982 and 351 us.  Bound by launch latency and by the trip of the
// levels through the Infinity Cache.  With a value per row (ROWV) the step
// saves the index stream and the wait for it: 16 vectors in float32 on the
// horn of 144,789 rows, 452 steps, 5.49 and 3.98 ms (15 entries in flight;
// five at a time 4.07).
template <typename T, int B, int MODE, int LPR, int W, bool ROWV>
__global__ __launch_bounds__(256) void k_leapfrog_st(int32_t n, int32_t nslices, const T* __restrict__ val,
                                                     const int32_t* __restrict__ soff,
                                                     const uint64_t* __restrict__ mask, int stride,
                                                     const T* __restrict__ cur, const T* prev, T* out,
                                                     T* __restrict__ acc, double* __restrict__ rout, int64_t rs,
                                                     int64_t cs, int bout, T wp, T wc, T wn, int remap) {
  constexpr int BL = B / LPR;
  constexpr int RW = 64 / LPR;
  const int wg = remap ? xcd_map(blockIdx.x, gridDim.x) : (int)blockIdx.x;
  const int gw = __builtin_amdgcn_readfirstlane(wg * 4 + (int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63;
  const int slice = (gw * RW) >> 6;
  if (slice >= nslices) return;
  const int rin = ((gw * RW) & 63) + lane / LPR;
  const int row = slice * 64 + rin;
  if (row >= n) return;
  const int col0 = (lane % LPR) * BL;
  const int64_t off = (int64_t)row * B + col0;
  Row<T, BL> yc, yp, r;
  const auto own_rows = [&]() {
    yc = *reinterpret_cast<const Row<T, BL>*>(cur + off);
    if (!(MODE & kFirst)) yp = *reinterpret_cast<const Row<T, BL>*>(prev + off);
    if (MODE == kMidAcc || MODE == kLast) r = *reinterpret_cast<const Row<T, BL>*>(acc + off);
  };
  // the row's own levels are loaded ahead of the gathers, except where a lane
  // has 64 bytes of a row: there they take the gathers' place in the first-level
  // cache (uniform grids; 63^3 rows, blocks of 16 in float64 and two lanes a row
  // 1239 us an application with them first, 1058 last, in float32 and one lane
  // 711 and 630).  With 128 bytes first is as good on 63^3 rows, and 3 to 6 %
  // faster on the 400-cell square and the horn.
  constexpr bool early = BL * sizeof(T) != 64;
  if (early) own_rows();
  T sum[BL];
#pragma unroll
  for (int j = 0; j < BL; ++j) sum[j] = (T)0;
  stencil_product<T, B, BL, LPR, W, ROWV>(val, soff, mask, stride, slice, rin, row, cur, col0, sum);
  if (!early) {
    asm volatile("" ::: "memory");
    own_rows();
  }
  if (MODE & kFirst) yp = yc;
  Row<T, BL> nx;
#pragma unroll
  for (int j = 0; j < BL; ++j) nx.v[j] = (T)2 * yc.v[j] - yp.v[j] - sum[j];
  if (!(MODE & kLast)) *reinterpret_cast<Row<T, BL>*>(out + off) = nx;
  if (MODE == kMid) return;
  if (MODE & kFirst) {
#pragma unroll
    for (int j = 0; j < BL; ++j) r.v[j] = fma(wn, nx.v[j], wc * yc.v[j]);
  } else {
#pragma unroll
    for (int j = 0; j < BL; ++j) r.v[j] = fma(wn, nx.v[j], fma(wc, yc.v[j], fma(wp, yp.v[j], r.v[j])));
  }
  if (MODE & kLast) {
#pragma unroll
    for (int j = 0; j < BL; ++j)
      if (col0 + j < bout) rout[(int64_t)row * rs + (int64_t)(col0 + j) * cs] = (double)r.v[j];
  } else {
    *reinterpret_cast<Row<T, BL>*>(acc + off) = r;
  }
}

// The two launches of a fourth-order step over stencil slices: MODE < 0 forms
// z = A cur, else the update (see stencil_product).
template <typename T, int B, int MODE, int LPR, int W, bool ROWV>
__global__ __launch_bounds__(256) void k_leapfrog4_st(int32_t n, int32_t nslices, const T* __restrict__ val,
                                                      const int32_t* __restrict__ soff,
                                                      const uint64_t* __restrict__ mask, int stride,
                                                      const T* __restrict__ cur, const T* prev, T* out,
                                                      T* __restrict__ acc, T* __restrict__ z,
                                                      double* __restrict__ rout, int64_t rs, int64_t cs, int bout, T wp,
                                                      T wc, T wn, int remap) {
  constexpr int BL = B / LPR;
  constexpr int RW = 64 / LPR;
  using V = Row<T, BL>;
  const int wg = remap ? xcd_map(blockIdx.x, gridDim.x) : (int)blockIdx.x;
  const int gw = __builtin_amdgcn_readfirstlane(wg * 4 + (int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63;
  const int slice = (gw * RW) >> 6;
  if (slice >= nslices) return;
  const int rin = ((gw * RW) & 63) + lane / LPR;
  const int row = slice * 64 + rin;
  if (row >= n) return;
  const int col0 = (lane % LPR) * BL;
  const int64_t off = (int64_t)row * B + col0;
  V yc, yp, zc, r;
  if (MODE >= 0) {
    yc = *reinterpret_cast<const V*>(cur + off);
    zc = *reinterpret_cast<const V*>(z + off);
    if (!(MODE & kFirst)) yp = *reinterpret_cast<const V*>(prev + off);
    if (MODE == kMidAcc || MODE == kLast) r = *reinterpret_cast<const V*>(acc + off);
  }
  T sum[BL];
#pragma unroll
  for (int j = 0; j < BL; ++j) sum[j] = (T)0;
  stencil_product<T, B, BL, LPR, W, ROWV>(val, soff, mask, stride, slice, rin, row, MODE < 0 ? cur : z, col0, sum);
  if (MODE < 0) {
    V o;
#pragma unroll
    for (int j = 0; j < BL; ++j) o.v[j] = sum[j];
    *reinterpret_cast<V*>(z + off) = o;
    return;
  }
  if (MODE & kFirst) yp = yc;
  constexpr T twelfth = (T)(1.0 / 12.0);
  V nx;
#pragma unroll
  for (int j = 0; j < BL; ++j) nx.v[j] = fma(twelfth, sum[j], (T)2 * yc.v[j] - yp.v[j] - zc.v[j]);
  if (!(MODE & kLast)) *reinterpret_cast<V*>(out + off) = nx;
  if (MODE == kMid) return;
  if (MODE & kFirst) {
#pragma unroll
    for (int j = 0; j < BL; ++j) r.v[j] = fma(wn, nx.v[j], wc * yc.v[j]);
  } else {
#pragma unroll
    for (int j = 0; j < BL; ++j) r.v[j] = fma(wn, nx.v[j], fma(wc, yc.v[j], fma(wp, yp.v[j], r.v[j])));
  }
  if (MODE & kLast) {
#pragma unroll
    for (int j = 0; j < BL; ++j)
      if (col0 + j < bout) rout[(int64_t)row * rs + (int64_t)(col0 + j) * cs] = (double)r.v[j];
  } else {
    *reinterpret_cast<V*>(acc + off) = r;
  }
}

// The batched step over stencil slices (see stencil_product).  The tables of
// the slice's problem are scalar loads, as the slice's entries are.
template <typename T, int B, bool ROWV>
__global__ __launch_bounds__(256) void k_leapfrog_batch_st(BatchRange rg, const T* __restrict__ val,
                                                           const int32_t* __restrict__ soff,
                                                           const uint64_t* __restrict__ mask, int stride,
                                                           const int32_t* __restrict__ sp,
                                                           const BatchTables* __restrict__ tb,
                                                           const T* __restrict__ wtab, int lmax, int ell,
                                                           const T* __restrict__ cur, const T* prev, T* out,
                                                           T* __restrict__ acc, int remap) {
  using V = Row<T, B>;
  const int wg = remap ? xcd_map(blockIdx.x, gridDim.x) : (int)blockIdx.x;
  const int at = __builtin_amdgcn_readfirstlane(wg * 4 + (int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63;
  if (at >= rg.na + rg.nm) return;
  const int slice = at < rg.na ? at : at - rg.na + rg.m0;
  const int p = sp[slice];
  const int Lp = tb->L[p];
  if (!tb->active[p] || ell > Lp - 1) return;
  const int row = slice * 64 + lane;
  const int local = row - (int)tb->row0[p];
  if (local >= tb->n[p]) return;
  const bool first = ell == 1, last = ell == Lp - 1;
  // the accumulation schedule of the single-problem steps (step_plan)
  const int u = ell >= 2 ? 1 + 3 * ((ell - 2) / 3) : 1;  // latest update before this step
  const bool sums = first || last || ell - u == 3;
  V yc, yp, r;
  const auto own_rows = [&]() {
    yc = yp = r = reinterpret_cast<const V*>(cur)[row];
    if (!first) yp = reinterpret_cast<const V*>(prev)[row];
    if (sums && !first) r = reinterpret_cast<const V*>(acc)[row];
  };
  // (as in k_leapfrog_st; 5 % on blocks of 16 in float64)
  constexpr bool early = sizeof(V) < 64;
  if (early) own_rows();
  T sum[B];
#pragma unroll
  for (int j = 0; j < B; ++j) sum[j] = (T)0;
  stencil_product<T, B, B, 1, 0, ROWV>(val, soff, mask, stride, slice, lane, row, cur, 0, sum);
  if (!early) {
    asm volatile("" ::: "memory");
    own_rows();
  }
  V nx;
#pragma unroll
  for (int j = 0; j < B; ++j) nx.v[j] = (T)2 * yc.v[j] - yp.v[j] - sum[j];
  if (!last) reinterpret_cast<V*>(out)[row] = nx;
  if (!sums) return;
  const T* __restrict__ wq = wtab + (int64_t)p * lmax;
  if (first) {
#pragma unroll
    for (int j = 0; j < B; ++j) r.v[j] = fma(wq[1], nx.v[j], wq[0] * yc.v[j]);
  } else {
    const T wp = ell - 2 > u ? wq[ell - 2] : (T)0, wc = ell - 1 > u ? wq[ell - 1] : (T)0, wn = wq[ell];
#pragma unroll
    for (int j = 0; j < B; ++j) r.v[j] = fma(wn, nx.v[j], fma(wc, yc.v[j], fma(wp, yp.v[j], r.v[j])));
  }
  if (last) {
    double* __restrict__ dst = tb->dst[p];
    const int64_t ld = tb->ld[p], drs = tb->drs[p];
    const int bout = tb->bout[p];
#pragma unroll
    for (int j = 0; j < B; ++j)
      if (j < bout) dst[local * drs + (int64_t)j * ld] = (double)r.v[j];
  } else {
    reinterpret_cast<V*>(acc)[row] = r;
  }
}

template <typename T, int B, int LPR, int W, bool ROWV>
int launch_st_w(const SellOp& A, int mode, const void* cur, const void* prev, void* out, void* acc, double* rout,
                int64_t rs, int64_t cs, int bout, double wp, double wc, double wn, int remap, hipStream_t st) {
#define KF_ST(M)                                                                                                     \
  hipLaunchKernelGGL((k_leapfrog_st<T, B, M, LPR, W, ROWV>), dim3(ceil_div64((int64_t)A.nslices * LPR, 4)), dim3(256), 0,    \
                     st, A.n, A.nslices, static_cast<const T*>(A.st.val), A.st.off, A.st.mask, A.st.stride,             \
                     static_cast<const T*>(cur), static_cast<const T*>(prev), static_cast<T*>(out),                     \
                     static_cast<T*>(acc), rout, rs, cs, bout, (T)wp, (T)wc, (T)wn, remap)
  switch (mode) {
    case kMid: KF_ST(kMid); break;
    case kFirst: KF_ST(kFirst); break;
    case kMidAcc: KF_ST(kMidAcc); break;
    case kLast: KF_ST(kLast); break;
    default: KF_ST(kFirstLast); break;
  }
#undef KF_ST
  KF_HIP(hipGetLastError());
  return KF_OK;
}

template <typename T, int B, int LPR>
int launch_st_l(const SellOp& A, int mode, const void* cur, const void* prev, void* out, void* acc, double* rout,
                int64_t rs, int64_t cs, int bout, double wp, double wc, double wn, int remap, hipStream_t st) {
  if (A.st.row_values) {
    if (A.st.stride == 15)
      return launch_st_w<T, B, LPR, 15, true>(A, mode, cur, prev, out, acc, rout, rs, cs, bout, wp, wc, wn, remap, st);
    return launch_st_w<T, B, LPR, 0, true>(A, mode, cur, prev, out, acc, rout, rs, cs, bout, wp, wc, wn, remap, st);
  }
  if (A.st.stride == 5)
    return launch_st_w<T, B, LPR, 5, false>(A, mode, cur, prev, out, acc, rout, rs, cs, bout, wp, wc, wn, remap, st);
  if (A.st.stride == 7)
    return launch_st_w<T, B, LPR, 7, false>(A, mode, cur, prev, out, acc, rout, rs, cs, bout, wp, wc, wn, remap, st);
  return launch_st_w<T, B, LPR, 0, false>(A, mode, cur, prev, out, acc, rout, rs, cs, bout, wp, wc, wn, remap, st);
}

template <typename T, int B>
int launch_st_b(const SellOp& A, int mode, const void* cur, const void* prev, void* out, void* acc, double* rout,
                int64_t rs, int64_t cs, int bout, double wp, double wc, double wn, int remap, hipStream_t st) {
  const int lpr = lanes_per_row(A, B);
  if constexpr (B >= 4)
    if (lpr == 4) return launch_st_l<T, B, 4>(A, mode, cur, prev, out, acc, rout, rs, cs, bout, wp, wc, wn, remap, st);
  if constexpr (B >= 2)
    if (lpr == 2) return launch_st_l<T, B, 2>(A, mode, cur, prev, out, acc, rout, rs, cs, bout, wp, wc, wn, remap, st);
  return launch_st_l<T, B, 1>(A, mode, cur, prev, out, acc, rout, rs, cs, bout, wp, wc, wn, remap, st);
}

// The fused step over stencil slices.
template <typename T>
int launch_st(const SellOp& A, int b, int mode, const void* cur, const void* prev, void* out, void* acc, double* rout,
              int64_t rs, int64_t cs, int bout, double wp, double wc, double wn, int remap, hipStream_t st) {
  switch (b) {
    case 1: return launch_st_b<T, 1>(A, mode, cur, prev, out, acc, rout, rs, cs, bout, wp, wc, wn, remap, st);
    case 2: return launch_st_b<T, 2>(A, mode, cur, prev, out, acc, rout, rs, cs, bout, wp, wc, wn, remap, st);
    case 4: return launch_st_b<T, 4>(A, mode, cur, prev, out, acc, rout, rs, cs, bout, wp, wc, wn, remap, st);
    case 8: return launch_st_b<T, 8>(A, mode, cur, prev, out, acc, rout, rs, cs, bout, wp, wc, wn, remap, st);
    case 16: return launch_st_b<T, 16>(A, mode, cur, prev, out, acc, rout, rs, cs, bout, wp, wc, wn, remap, st);
    default: set_error("leapfrog: block width must be 1, 2, 4, 8 or 16"); return KF_EINVAL;
  }
}

template <typename T, int B, int LPR, int W, bool ROWV>
int launch_st4_w(const SellOp& A, int mode, const void* cur, const void* prev, void* out, void* acc, void* z,
                 double* rout, int64_t rs, int64_t cs, int bout, double wp, double wc, double wn, int remap,
                 hipStream_t st) {
#define KF_ST4(M)                                                                                                   \
  hipLaunchKernelGGL((k_leapfrog4_st<T, B, M, LPR, W, ROWV>), dim3(ceil_div64((int64_t)A.nslices * LPR, 4)), dim3(256), 0,  \
                     st, A.n, A.nslices, static_cast<const T*>(A.st.val), A.st.off, A.st.mask, A.st.stride,            \
                     static_cast<const T*>(cur), static_cast<const T*>(prev), static_cast<T*>(out),                    \
                     static_cast<T*>(acc), static_cast<T*>(z), rout, rs, cs, bout, (T)wp, (T)wc, (T)wn, remap)
  KF_ST4(-1);
  switch (mode) {
    case kMid: KF_ST4(kMid); break;
    case kFirst: KF_ST4(kFirst); break;
    case kMidAcc: KF_ST4(kMidAcc); break;
    case kLast: KF_ST4(kLast); break;
    default: KF_ST4(kFirstLast); break;
  }
#undef KF_ST4
  KF_HIP(hipGetLastError());
  return KF_OK;
}

// (16 bytes of a row per lane; as many lanes share it)
template <typename T, int B>
int launch_st4_b(const SellOp& A, int mode, const void* cur, const void* prev, void* out, void* acc, void* z,
                 double* rout, int64_t rs, int64_t cs, int bout, double wp, double wc, double wn, int remap,
                 hipStream_t st) {
  constexpr int LPR = B * sizeof(T) >= 64 ? 4 : (B * sizeof(T) >= 32 ? 2 : 1);
  if (A.st.row_values) {
    if (A.st.stride == 15)
      return launch_st4_w<T, B, LPR, 15, true>(A, mode, cur, prev, out, acc, z, rout, rs, cs, bout, wp, wc, wn, remap,
                                               st);
    return launch_st4_w<T, B, LPR, 0, true>(A, mode, cur, prev, out, acc, z, rout, rs, cs, bout, wp, wc, wn, remap, st);
  }
  if (A.st.stride == 5)
    return launch_st4_w<T, B, LPR, 5, false>(A, mode, cur, prev, out, acc, z, rout, rs, cs, bout, wp, wc, wn, remap, st);
  if (A.st.stride == 7)
    return launch_st4_w<T, B, LPR, 7, false>(A, mode, cur, prev, out, acc, z, rout, rs, cs, bout, wp, wc, wn, remap, st);
  return launch_st4_w<T, B, LPR, 0, false>(A, mode, cur, prev, out, acc, z, rout, rs, cs, bout, wp, wc, wn, remap, st);
}

template <typename T>
int launch_st4(const SellOp& A, int b, int mode, const void* cur, const void* prev, void* out, void* acc, void* z,
               double* rout, int64_t rs, int64_t cs, int bout, double wp, double wc, double wn, int remap,
               hipStream_t st) {
  switch (b) {
    case 1: return launch_st4_b<T, 1>(A, mode, cur, prev, out, acc, z, rout, rs, cs, bout, wp, wc, wn, remap, st);
    case 2: return launch_st4_b<T, 2>(A, mode, cur, prev, out, acc, z, rout, rs, cs, bout, wp, wc, wn, remap, st);
    case 4: return launch_st4_b<T, 4>(A, mode, cur, prev, out, acc, z, rout, rs, cs, bout, wp, wc, wn, remap, st);
    case 8: return launch_st4_b<T, 8>(A, mode, cur, prev, out, acc, z, rout, rs, cs, bout, wp, wc, wn, remap, st);
    case 16: return launch_st4_b<T, 16>(A, mode, cur, prev, out, acc, z, rout, rs, cs, bout, wp, wc, wn, remap, st);
    default: set_error("fourth-order step: block width must be 1, 2, 4, 8 or 16"); return KF_EINVAL;
  }
}

}  // namespace

namespace {
// The stencil form of an operator's slices, when it has one and there is memory
// for it (else out.width stays 0): one value per offset where every slice is uniform, a value per row
// where that does not take more memory than the stored entries (nstored of
// them with ib bytes of index) would.
template <typename VT>
int build_stencil_t(int32_t n, int32_t ns, const int32_t* d_rowptr, const int32_t* d_col, const double* d_val,
                    const double* d_row_scale, const int32_t* w, int64_t nstored, int ib, bool exact, hipStream_t st,
                    StencilOp& out) {
  const int grid = ceil_div64(ns, 4);
  int width = 0;
  bool row_values = false;
  for (int32_t i = 0; i < ns; ++i) {
    width = std::max(width, std::abs(w[i]));
    row_values |= w[i] < 0;
  }
  if (width < 1 || width > kStencilMax) return KF_OK;
  // 5 and 7 entries (the 2D and 3D point stencils) and, with row values, 15
  // (linear tetrahedra around a vertex of a structured mesh) have kernels of
  // their own length; other lengths are padded to the loop's four entries
  const bool own = exact && (row_values ? width == 15 : width == 5 || width == 7);
  const int stride = own ? width : (width + 3) / 4 * 4;
  const size_t tot = (size_t)ns * stride;
  const size_t vals = row_values ? tot * 64 : tot;
  if (row_values && vals * sizeof(VT) + tot * 12 > (size_t)nstored * (sizeof(VT) + ib)) return KF_OK;
  // one allocation: masks, values, offsets
  char* mem = nullptr;
  if (hipMalloc(&mem, tot * sizeof(uint64_t) + vals * sizeof(VT) + tot * sizeof(int32_t)) != hipSuccess) {
    (void)hipGetLastError();
    return KF_OK;  // the stored entries do without
  }
  out.mask = reinterpret_cast<uint64_t*>(mem);
  out.val = mem + tot * sizeof(uint64_t);
  out.off = reinterpret_cast<int32_t*>(mem + tot * sizeof(uint64_t) + vals * sizeof(VT));
  out.width = width;
  out.stride = stride;
  out.row_values = row_values;
  if (row_values)
    hipLaunchKernelGGL((k_stencil<VT, 2>), dim3(grid), dim3(256), 0, st, n, ns, d_rowptr, d_col, d_val, d_row_scale,
                       (int32_t*)nullptr, stride, (VT*)out.val, out.off, out.mask);
  else
    hipLaunchKernelGGL((k_stencil<VT, 1>), dim3(grid), dim3(256), 0, st, n, ns, d_rowptr, d_col, d_val, d_row_scale,
                       (int32_t*)nullptr, stride, (VT*)out.val, out.off, out.mask);
  KF_HIP(hipGetLastError());
  return KF_OK;
}
}  // namespace

void free_stencil(StencilOp& s) {
  if (s.mask) (void)hipFree(s.mask);  // (the three arrays are one allocation)
  s = StencilOp();
}

int launch_stencil_widths(int32_t n, int32_t ns, const int32_t* d_rowptr, const int32_t* d_col, const double* d_val,
                          const double* d_row_scale, int val_bytes, int32_t* d_w, hipStream_t st) {
  if (val_bytes == 8)
    hipLaunchKernelGGL((k_stencil<double, 0>), dim3(ceil_div64(ns, 4)), dim3(256), 0, st, n, ns, d_rowptr, d_col, d_val,
                       d_row_scale, d_w, 0, (double*)nullptr, (int32_t*)nullptr, (uint64_t*)nullptr);
  else
    hipLaunchKernelGGL((k_stencil<float, 0>), dim3(ceil_div64(ns, 4)), dim3(256), 0, st, n, ns, d_rowptr, d_col, d_val,
                       d_row_scale, d_w, 0, (float*)nullptr, (int32_t*)nullptr, (uint64_t*)nullptr);
  KF_HIP(hipGetLastError());
  return KF_OK;
}

int build_stencil(int32_t n, int32_t ns, const int32_t* d_rowptr, const int32_t* d_col, const double* d_val,
                  const double* d_row_scale, const int32_t* widths, int val_bytes, int64_t nstored, int idx_bytes,
                  bool exact, hipStream_t st, StencilOp& out) {
  if (val_bytes == 8)
    return build_stencil_t<double>(n, ns, d_rowptr, d_col, d_val, d_row_scale, widths, nstored, idx_bytes, exact, st, out);
  return build_stencil_t<float>(n, ns, d_rowptr, d_col, d_val, d_row_scale, widths, nstored, idx_bytes, exact, st, out);
}

int launch_stencil_step(const SellOp& A, int b, int mode, const void* cur, const void* prev, void* out, void* acc,
                        double* rout, int64_t rs, int64_t cs, int bout, double wp, double wc, double wn, int remap,
                        hipStream_t st) {
  if (A.val_bytes == 8)
    return launch_st<double>(A, b, mode, cur, prev, out, acc, rout, rs, cs, bout, wp, wc, wn, remap, st);
  return launch_st<float>(A, b, mode, cur, prev, out, acc, rout, rs, cs, bout, wp, wc, wn, remap, st);
}

int launch_stencil_step4(const SellOp& A, int b, int mode, const void* cur, const void* prev, void* out, void* acc,
                         void* z, double* rout, int64_t rs, int64_t cs, int bout, double wp, double wc, double wn,
                         int remap, hipStream_t st) {
  if (A.val_bytes == 8)
    return launch_st4<double>(A, b, mode, cur, prev, out, acc, z, rout, rs, cs, bout, wp, wc, wn, remap, st);
  return launch_st4<float>(A, b, mode, cur, prev, out, acc, z, rout, rs, cs, bout, wp, wc, wn, remap, st);
}

namespace {
template <typename T>
int launch_lfb_st(const SellOp& A, int b, const int32_t* sp, const BatchTables* tb, const void* wtab, int lmax, int ell,
                  const void* cur, const void* prev, void* out, void* acc, const BatchRange& r, int remap, hipStream_t st) {
#define KF_LFS(B)                                                                                                  \
  hipLaunchKernelGGL((A.st.row_values ? k_leapfrog_batch_st<T, B, true> : k_leapfrog_batch_st<T, B, false>), dim3(ceil_div64(r.na + r.nm, 4)), dim3(256), 0, st, r, \
                     static_cast<const T*>(A.st.val), A.st.off, A.st.mask, A.st.stride, sp, tb,                     \
                     static_cast<const T*>(wtab), lmax, ell, static_cast<const T*>(cur), static_cast<const T*>(prev), \
                     static_cast<T*>(out), static_cast<T*>(acc), remap)
  switch (b) {
    case 1: KF_LFS(1); break;
    case 2: KF_LFS(2); break;
    case 4: KF_LFS(4); break;
    case 8: KF_LFS(8); break;
    case 16: KF_LFS(16); break;
    default: set_error("batched leapfrog: block width must be 1, 2, 4, 8 or 16"); return KF_EINVAL;
  }
#undef KF_LFS
  KF_HIP(hipGetLastError());
  return KF_OK;
}
}  // namespace

int launch_stencil_batch(const SellOp& A, int b, const int32_t* sp, const BatchTables* tb, const void* wtab, int lmax,
                         int ell, const void* cur, const void* prev, void* out, void* acc, const BatchRange& r, int remap,
                         hipStream_t st) {
  if (A.val_bytes == 8) return launch_lfb_st<double>(A, b, sp, tb, wtab, lmax, ell, cur, prev, out, acc, r, remap, st);
  return launch_lfb_st<float>(A, b, sp, tb, wtab, lmax, ell, cur, prev, out, acc, r, remap, st);
}

}  // namespace kf
