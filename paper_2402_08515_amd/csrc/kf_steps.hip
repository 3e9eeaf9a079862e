// Several time steps per launch over stencil slices: the kernel, the rule that
// chooses it and its launcher.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "kf_device.h"
#include "kf_internal.h"

namespace kf {

namespace {

// ------------------------------------- several steps per launch over stencils
// The time loop of problems too small to fill a launch: a step of one launch
// takes 3 to 4 us whatever its size (2.1 replayed from a recording), most of it
// launch and dependent-load latency.  A workgroup owns a range of row slices and advances it s steps in
// one launch; y_l of those rows, and of the hb slices a step reaches on either
// side for each later step, lie in LDS (two copies, written in turn), and each
// wavefront keeps the levels y_{l-1}, y_l and the weighted sum of its slices
// (wave, wave + 16, ...: at most R) in registers, with the places of their
// stencil neighbours in LDS; absent neighbours point at a zero.  A step then
// is W LDS reads, W products and one LDS write per row and one barrier.  Row
// values (ROWV) are read again in every step, from the caches; kept in registers
// through all steps, as four slices of 15 each would be, they spill.  The
// halo slices are computed by every workgroup that needs them; with the whole
// problem in one workgroup there are none.  The weighted sum takes one term
// per step, in the same order as three terms every third step: results are
// those of one step per launch, bit for bit.  A workgroup carries B columns
// (at most 16 bytes) of a row of `groups` times as many: wider blocks are
// independent groups of columns along the grid's y.
// Measured, us per filter application, one launched step each and so: 64-cell
// square (63 slices) fp64 257 -> 45; 128 cells 535 -> 114; 256 cells 1072 ->
// 322, its block of 4 in float32 1021 -> 463; 20-cell cube 91 -> 44.  Bound by
// a launch's latency (about 4 us) and the LDS reads of the halo slices.  The
// fourth-order step, us a step, two launches each and so (fp64, one vector):
// 20-cell square 8.4 -> 0.57, 128 cells 8.4 -> 1.7, 500 cells 8.5 -> 4.3,
// 25-cell cube 8.4 -> 4.3; 11 x 34-cell horn 8.5 -> 4.5.
//   first: y_{-1} = y_0 = x (x in ysrc), the sum starts at w_0 x; else i0, i1
//          hold y_{l0-1}, y_{l0} and acc the sum
//   last:  the sum goes to rout; otherwise y_{l0+s-1}, y_{l0+s} go to o0g,
//          o1g and the sum to acc.  o0g, o1g are not i0, i1 unless there is
//          one workgroup.
// wt(j) is the weight of y_{l0+j}; own slices are [o0, o1).
// O4: the fourth-order step, z = A y first and then y_{l+1} = 2 y_l - y_{l-1} -
// z + A z / 12; a step reaches twice as far, the second copy in LDS holds z,
// and y is written in place.
template <typename T, int B, int W, int R, bool ROWV, bool O4, class Weight>
__device__ __forceinline__ void steps_body(int32_t n, int32_t nslices, const T* __restrict__ sval,
                                           const int32_t* __restrict__ soff, const uint64_t* __restrict__ smask,
                                           int stride, const T* ysrc, const T* i0, const T* i1, T* o0g, T* o1g, T* acc,
                                           double* __restrict__ rout, int64_t rs, int64_t cs, int bout, int groups,
                                           Weight wt, int s, int o0, int o1, int hb, bool first, bool last) {
  using V = Row<T, B>;
  extern __shared__ __align__(16) unsigned char steps_raw[];
  const int reach = O4 ? 2 * hb : hb;
  const int w0 = max(0, o0 - s * reach), w1 = min(nslices, o1 + s * reach);
  const int rows = (w1 - w0) * 64;  // of one level in LDS; row `rows` is the zero
  V* lds = reinterpret_cast<V*>(steps_raw);
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int step2 = rows + 1;  // distance of the two copies
  if (threadIdx.x < 2) {
    V zero;
#pragma unroll
    for (int j = 0; j < B; ++j) zero.v[j] = (T)0;
    lds[threadIdx.x * step2 + rows] = zero;
  }
  const int grp = blockIdx.y;
  V yc[R], yp[R], ra[R];
  uint32_t at[R][(W + 1) / 2];  // two neighbours' LDS rows per register
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int sl = w0 + wave + 16 * k;
    if (sl >= w1) break;
    const int row = sl * 64 + lane;
#pragma unroll
    for (int j = 0; j < B; ++j) yc[k].v[j] = yp[k].v[j] = ra[k].v[j] = (T)0;
    if (row < n) {
      yc[k] = reinterpret_cast<const V*>(first ? ysrc : i1)[(int64_t)row * groups + grp];
      yp[k] = first ? yc[k] : reinterpret_cast<const V*>(i0)[(int64_t)row * groups + grp];
      if (sl >= o0 && sl < o1) {
        if (first) {
#pragma unroll
          for (int j = 0; j < B; ++j) ra[k].v[j] = wt(0) * yc[k].v[j];
        } else {
          ra[k] = reinterpret_cast<const V*>(acc)[(int64_t)row * groups + grp];
        }
      }
    }
#pragma unroll
    for (int q = 0; q < W; ++q) {
      const bool has = __builtin_amdgcn_inverse_ballot_w64(smask[(int64_t)sl * stride + q]);
      const int c = row - w0 * 64 + soff[(int64_t)sl * stride + q];
      const uint32_t a = has && c >= 0 && c < rows ? (uint32_t)c : (uint32_t)rows;
      at[k][q >> 1] = q & 1 ? at[k][q >> 1] | a << 16 : a;
    }
    lds[row - w0 * 64] = yc[k];
  }
  __syncthreads();
  // sum = (A x)[own row of slice sl], x a level in LDS
  const auto product = [&](int k, int sl, const V* __restrict__ src, int j, T (&sum)[B]) {
#pragma unroll
    for (int c = 0; c < B; ++c) sum[c] = (T)0;
    constexpr int U = ROWV ? (W == 15 ? 5 : 4) : W;
#pragma unroll
    for (int q0 = 0; q0 < W; q0 += U) {
      V x[U];
      T av[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int q = q0 + u;
        av[u] = ROWV ? sval[((int64_t)sl * stride + q) * 64 + lane] : sval[(int64_t)sl * stride + q];
        uint32_t pair = at[k][q >> 1];
        // (the places are unpacked here; unpacked once for all steps, which
        // the two products of a step invite, they take too many registers)
        if (O4) asm("" : "+v"(pair) : "s"(j));
        x[u] = src[q & 1 ? pair >> 16 : pair & 0xFFFFu];
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int c = 0; c < B; ++c) sum[c] = fma(av[u], x[u].v[c], sum[c]);
    }
  };
  int cur = 0;
  for (int j = 0; j < s; ++j) {
    const T wn = wt(j + 1);
    // the slices the later steps still read
    const int a0 = o0 - (s - 1 - j) * reach, a1 = o1 + (s - 1 - j) * reach;
    const V* __restrict__ src = lds + (O4 ? step2 : cur * step2);
    V* __restrict__ dst = lds + (O4 ? 0 : (cur ^ 1) * step2);
    if constexpr (O4) {
      V* __restrict__ z = lds + step2;
#pragma unroll
      for (int k = 0; k < R; ++k) {
        const int sl = w0 + wave + 16 * k;
        if (sl >= w1 || sl < a0 - hb || sl >= a1 + hb) continue;
        V o;
        product(k, sl, dst, j, o.v);
        z[sl * 64 + lane - w0 * 64] = o;
      }
      __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const int sl = w0 + wave + 16 * k;
      if (sl >= w1 || sl < a0 || sl >= a1) continue;
      V nx;
      T sum[B];
      product(k, sl, src, j, sum);
      if constexpr (O4) {
        constexpr T twelfth = (T)(1.0 / 12.0);
        const V z = src[sl * 64 + lane - w0 * 64];
#pragma unroll
        for (int c = 0; c < B; ++c) nx.v[c] = fma(twelfth, sum[c], (T)2 * yc[k].v[c] - yp[k].v[c] - z.v[c]);
      } else {
#pragma unroll
        for (int c = 0; c < B; ++c) nx.v[c] = (T)2 * yc[k].v[c] - yp[k].v[c] - sum[c];
      }
#pragma unroll
      for (int c = 0; c < B; ++c) ra[k].v[c] = fma(wn, nx.v[c], ra[k].v[c]);
      yp[k] = yc[k];
      yc[k] = nx;
      dst[sl * 64 + lane - w0 * 64] = nx;
    }
    __syncthreads();
    cur ^= 1;
  }
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int sl = w0 + wave + 16 * k;
    if (sl < o0 || sl >= o1) continue;
    const int row = sl * 64 + lane;
    if (row >= n) continue;
    if (last) {
#pragma unroll
      for (int j = 0; j < B; ++j)
        if (grp * B + j < bout) rout[(int64_t)row * rs + (int64_t)(grp * B + j) * cs] = (double)ra[k].v[j];
    } else {
      const int64_t o = (int64_t)row * groups + grp;
      reinterpret_cast<V*>(o0g)[o] = yp[k];
      reinterpret_cast<V*>(o1g)[o] = yc[k];
      reinterpret_cast<V*>(acc)[o] = ra[k];
    }
  }
}

template <typename T, int B, int W, int R, bool ROWV, bool O4>
__global__ __launch_bounds__(1024) void k_steps_st(int32_t n, int32_t nslices, const T* __restrict__ sval,
                                                   const int32_t* __restrict__ soff, const uint64_t* __restrict__ smask,
                                                   const T* ysrc, const T* i0, const T* i1, T* o0g, T* o1g, T* acc,
                                                   double* __restrict__ rout, int64_t rs, int64_t cs, int bout,
                                                   int groups, StepWeights w, int s, int own, int hb, int first,
                                                   int last) {
  const int o0 = xcd_map(blockIdx.x, gridDim.x) * own;
  steps_body<T, B, W, R, ROWV, O4>(n, nslices, sval, soff, smask, W, ysrc, i0, i1, o0g, o1g, acc, rout, rs, cs, bout,
                               groups, [&](int j) { return (T)w.w[j]; }, s, o0, min(nslices, o0 + own), hb, first != 0,
                               last != 0);
}

// The same for the members of a batch that plan_batch took: wgs[] says which
// member, slices and plan each workgroup has; launch i advances every member
// from step i * s on until its L - 1 steps are done.  i0, i1 and o0, o1 hold
// the stack's rows from ibase and obase on.
// Bound by a launch's latency, as k_steps_st is, and by the compute units it
// shares with the one-step launches beside it: 16 members of 18800 slices,
// float32 blocks of 4, of which 2148 slices of small members set the number
// of steps (199), 1180 -> 968 us an application, 1087 with the two kinds of
// launches one after another.
template <typename T, int B, int R>
__global__ __launch_bounds__(1024) void k_steps_batch(const BatchWg* __restrict__ wgs, const T* __restrict__ sval,
                                                      const int32_t* __restrict__ soff,
                                                      const uint64_t* __restrict__ smask, int stride,
                                                      const BatchTables* __restrict__ tb, const T* __restrict__ wtab,
                                                      int lmax, int i, const T* ysrc, const T* i0, const T* i1, T* o0,
                                                      T* o1, T* acc, int64_t ibase, int64_t obase, int groups) {
  const BatchWg g = wgs[xcd_map(blockIdx.x, gridDim.x)];
  const int l0 = i * g.s, left = tb->L[g.p] - 1 - l0;
  if (!tb->active[g.p] || left <= 0) return;
  const int64_t row0 = (int64_t)g.slice0 * 64, b = (int64_t)groups * B;
  const int64_t so = (int64_t)g.slice0 * stride, in = (row0 - ibase) * b, out = (row0 - obase) * b;
  const T* __restrict__ wq = wtab + (int64_t)g.p * lmax + l0;
  const auto run = [&](auto width) {
    steps_body<T, B, decltype(width)::value, R, false, false>(
        tb->n[g.p], g.nslices, sval + so, soff + so, smask + so, stride, ysrc + row0 * b, i0 + in, i1 + in, o0 + out,
        o1 + out, acc + row0 * b, tb->dst[g.p], tb->drs[g.p], tb->ld[g.p], tb->bout[g.p], groups,
        [&](int j) { return wq[j]; }, min(g.s, left), g.o0, min(g.nslices, g.o0 + g.own), g.hb, i == 0, left <= g.s);
  };
  if (g.width <= 5)
    run(std::integral_constant<int, 5>());
  else
    run(std::integral_constant<int, 7>());
}

}  // namespace

namespace {
// arguments of one k_steps_st launch that its dispatch only passes on
struct StepsArgs {
  const void *ysrc, *i0, *i1;
  void *o0, *o1, *acc;
  double* rout;
  int64_t rs, cs;
  int bout, groups, s;
  bool first, last;
};

// The dynamic LDS any launch of a form with R slices per wavefront asks for:
// its limit is set to this whatever the launch needs, as other threads launch
// the same kernels.
constexpr int steps_lds_limit(int r, size_t rb) { return (int)std::min<size_t>(160 << 10, 2 * (16 * r * 64 + 1) * rb); }

template <typename T, int B, int W, int R, bool ROWV, bool O4>
int launch_steps_r(const SellOp& A, const StepsPlan& pl, const StepsArgs& g, const StepWeights& w, hipStream_t st) {
  const int win = std::min(A.nslices, pl.own + 2 * g.s * pl.reach());
  const size_t lds = (size_t)2 * (win * 64 + 1) * B * sizeof(T);
  KF_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_steps_st<T, B, W, R, ROWV, O4>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, steps_lds_limit(R, sizeof(T) * B)));
  hipLaunchKernelGGL((k_steps_st<T, B, W, R, ROWV, O4>), dim3(ceil_div64(A.nslices, pl.own), g.groups), dim3(1024), lds, st, A.n,
                     A.nslices, static_cast<const T*>(A.st.val), A.st.off, A.st.mask, static_cast<const T*>(g.ysrc),
                     static_cast<const T*>(g.i0), static_cast<const T*>(g.i1), static_cast<T*>(g.o0),
                     static_cast<T*>(g.o1), static_cast<T*>(g.acc), g.rout, g.rs, g.cs, g.bout, g.groups, w, g.s, pl.own,
                     pl.hb, g.first ? 1 : 0, g.last ? 1 : 0);
  KF_HIP(hipGetLastError());
  return KF_OK;
}

template <typename T, int B, int W, bool ROWV, bool O4>
int launch_steps_w(const SellOp& A, const StepsPlan& pl, const StepsArgs& g, const StepWeights& w, hipStream_t st) {
  const int per = (std::min(A.nslices, pl.own + 2 * g.s * pl.reach()) + 15) / 16;  // slices of a wavefront
  if (per <= 2) return launch_steps_r<T, B, W, 2, ROWV, O4>(A, pl, g, w, st);
  constexpr int RM = steps_max_r(B * sizeof(T), ROWV ? W : 0);
  if constexpr (RM > 2) {
    if (RM == 4 || per <= 4) return launch_steps_r<T, B, W, 4, ROWV, O4>(A, pl, g, w, st);
    return launch_steps_r<T, B, W, RM, ROWV, O4>(A, pl, g, w, st);
  }
  set_error("several steps per launch: window too wide");
  return KF_EINVAL;
}

template <typename T, int B, bool O4>
int launch_steps_b(const SellOp& A, const StepsPlan& pl, const StepsArgs& g, const StepWeights& w, hipStream_t st) {
  if (A.st.row_values)
    return A.st.stride == 15 ? launch_steps_w<T, B, 15, true, O4>(A, pl, g, w, st)
                             : launch_steps_w<T, B, 8, true, O4>(A, pl, g, w, st);
  return A.st.stride == 5 ? launch_steps_w<T, B, 5, false, O4>(A, pl, g, w, st)
                          : launch_steps_w<T, B, 7, false, O4>(A, pl, g, w, st);
}

template <bool O4>
int launch_steps_o(const SellOp& A, const StepsPlan& pl, int cols, const StepsArgs& g, const StepWeights& w,
                   hipStream_t st) {
  if (A.val_bytes == 8)
    return cols == 1 ? launch_steps_b<double, 1, O4>(A, pl, g, w, st) : launch_steps_b<double, 2, O4>(A, pl, g, w, st);
  if (cols == 1) return launch_steps_b<float, 1, O4>(A, pl, g, w, st);
  return cols == 2 ? launch_steps_b<float, 2, O4>(A, pl, g, w, st) : launch_steps_b<float, 4, O4>(A, pl, g, w, st);
}
}  // namespace

namespace {
constexpr int kCus = 256;  // compute units: workgroups of a launch

// the lengths of stencils that k_steps_st is built for
bool has_steps(const StencilOp& st) {
  return st.row_values ? st.stride == 8 || st.stride == 15 : (st.stride == 5 || st.stride == 7) && st.width == st.stride;
}
}  // namespace

int launch_steps(const SellOp& A, const StepsPlan& pl, int b, int s, bool first, bool last, const void* ysrc,
                 const void* i0, const void* i1, void* o0, void* o1, void* acc, double* rout, int64_t rs, int64_t cs,
                 int bout, const StepWeights& w, hipStream_t st) {
  if (pl.s < 1 || s < 1 || s > pl.s || !has_steps(A.st)) {
    set_error("several steps per launch: no plan for this operator");
    return KF_EINVAL;
  }
  const int cols = std::min(b, 16 / A.val_bytes);
  const StepsArgs g{ysrc, i0, i1, o0, o1, acc, rout, rs, cs, bout, b / cols, s, first, last};
  return pl.order4 ? launch_steps_o<true>(A, pl, cols, g, w, st) : launch_steps_o<false>(A, pl, cols, g, w, st);
}

// The rule, for the lists the kernel is built for (5 or 7 offsets, with row
// values up to 8 stored in 8, or 15; other lists take one step per launch): the
// time of a filter application by the figures measured on
// squares of 32 to 600 and cubes of 13 to 33 cells (within 10 % of every
// measurement while a wavefront has at most four slices), in us:
//   a launch        3.7 + 0.03 per slice of the window (0.06 for 16-byte rows)
//   one of its steps  0.12 + 0.014 per slice computed (0.022), 15 % more with
//                   more than four slices per wavefront
// with at most one workgroup per compute unit, and 0.035 (0.02) more per slice of
// the window for each further group of columns, which reads a part of every
// row.  The plan is taken where it is at least 10 % below one step per launch,
// us a step (MB: of a level, n b values):
//   replayed from a recording (step_replay)  2.1 + 0.4 MB, with row values 2.75
//     in float64 and 2.45 in float32 instead of 2.1; fourth-order steps, two
//     launches each, 4.1 + 0.7 MB, with row values 5.6 and 4.85
//   else at least what the host needs: 3.8 a launch
// E.g. (taken | left, us a step so and with one step per launch) 23-cell cube
// 2.16 and 2.20 | 26 cells 2.43 and 2.22, 33 cells 3.15 and 2.25; the 400-cell
// square, one vector 2.08 and 2.62 | its block of 4 in float32 3.16 and 2.92;
// 20-cell cube, block of 4 in float32 | 2.32 and 2.28; horn of 11 x 34 cells
// 2.28 and 2.72 | 16 x 60 cells 3.02 and 2.73.
// With row values (horns of 5 to 16 cells, jittered squares and cubes, within
// 20 %) a launch takes 3.7 + 0.06 per slice of the window, whose values it
// reads, and a step per slice and entry 0.0073 in float64, 0.005 in float32,
// 0.008 with several groups of columns, which leave fewer compute units to each.
namespace {
StepsPlan plan_of(int ns, int hb, bool rv, int stride, int val_bytes, int b, int L, size_t lds_bytes, int own_min,
                  bool order4, double step_us) {
  StepsPlan best;
  best.order4 = order4;
  best.hb = hb;
  const int cols = std::min(b, 16 / val_bytes), groups = b / cols, rb = cols * val_bytes;
  const int win_max = std::min<int64_t>(16 * steps_max_r(rb, rv ? stride : 0), ((int64_t)lds_bytes / (2 * rb) - 1) / 64);
  const double load = (rv || rb > 8 ? 0.06 : 0.03) + (rv ? 0.02 : 0.035) * (groups - 1);
  const double slice = rv ? stride * (groups > 1 ? 0.008 : (val_bytes == 8 ? 0.0073 : 0.005)) : (rb > 8 ? 0.022 : 0.014);
  const int reach = best.reach();
  double t_best = step_us * (L - 1);
  if (L < 3 || own_min > win_max || groups > kCus) return best;
  for (int i = 0; i < 4; ++i) {
    const int own = i == 3 ? ns : std::min(ns, own_min << i);
    const bool whole = own >= ns;
    for (int s = 1; s <= std::min(kStepsMax, L - 1); ++s) {
      const int win = std::min(ns, own + 2 * s * reach);
      if (win > win_max) break;
      const double avg = std::min<double>(ns, own + (double)(s - 1) * reach);
      double step = (rv ? 0.0 : 0.12) + slice * avg;
      if (order4) step += (rv ? 0.0 : 0.12) + slice * std::min<double>(ns, avg + 2.0 * hb);
      if (win > 64) step *= 1.15;
      const int launches = (L - 1 + s - 1) / s;
      const double t = launches * (3.7 + load * win) + (L - 1) * step;
      if (t < t_best) {
        t_best = t;
        best.s = s;
        best.own = whole ? ns : own;
      }
    }
    if (whole) break;
  }
  return best;
}
}  // namespace

StepsPlan plan_steps(const SellOp& A, int b, int L, size_t lds_bytes, bool order4, bool replay) {
  if (!has_steps(A.st)) return StepsPlan();
  const bool rv = A.st.row_values, f64 = A.val_bytes == 8;
  const double mb = 1e-6 * A.n * b * A.val_bytes;
  double one = order4 ? (rv ? (f64 ? 5.6 : 4.85) : 4.1) + 0.7 * mb : (rv ? (f64 ? 2.75 : 2.45) : 2.1) + 0.4 * mb;
  if (!replay || !step_replay(A.n, b, A.val_bytes, L)) one = std::max(one, order4 ? 7.6 : 3.8);
  const int groups = b / std::min(b, 16 / A.val_bytes);
  return plan_of(A.nslices, (A.max_off + 63) / 64, A.st.row_values, A.st.stride, A.val_bytes, b, L, lds_bytes,
                 (int)ceil_div64((int64_t)A.nslices * groups, kCus), order4, 0.9 * one);
}

// Members of a batch side by side in one launch: each as alone, with so many
// slices a workgroup that all of them have a compute unit to themselves.
// Empty: one of them is not better off than with one step per launch (about 4
// us in a batch).
std::vector<StepsPlan> plan_batch(const std::vector<BatchMember>& m, int val_bytes, int b, size_t lds_bytes) {
  const int groups = b / std::min(b, 16 / val_bytes);
  int64_t total = 0;
  for (const BatchMember& q : m) total += q.nslices;
  std::vector<StepsPlan> plans(m.size());
  for (int own_min = std::max(1, (int)ceil_div64(total * groups, kCus));; ++own_min) {
    int64_t wgs = 0;
    for (size_t i = 0; i < m.size(); ++i) {
      plans[i] = plan_of(m[i].nslices, m[i].hb, false, 0, val_bytes, b, m[i].L, lds_bytes, own_min, false,
                         0.85 * 4.0);
      if (plans[i].s == 0) return {};
      wgs += (int64_t)ceil_div64(m[i].nslices, plans[i].own) * groups;
    }
    if (wgs <= kCus) return plans;
  }
}

namespace {
template <typename T, int B>
int launch_steps_batch_b(const SellOp& A, const BatchWg* wgs, int nwg, int win, int groups, const BatchTables* tb,
                         const void* wtab, int lmax, int i, const void* ysrc, const void* i0, const void* i1, void* o0,
                         void* o1, void* acc, int64_t ibase, int64_t obase, hipStream_t st) {
  const size_t lds = (size_t)2 * (win * 64 + 1) * B * sizeof(T);
  constexpr int RM = steps_max_r(B * sizeof(T), 0);
  if (win > 16 * RM) {
    set_error("several steps per launch: window too wide");
    return KF_EINVAL;
  }
#define KF_SB(R)                                                                                                     \
  do {                                                                                                               \
    KF_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_steps_batch<T, B, R>),                               \
                               hipFuncAttributeMaxDynamicSharedMemorySize, steps_lds_limit(R, sizeof(T) * B)));        \
    hipLaunchKernelGGL((k_steps_batch<T, B, R>), dim3(nwg, groups), dim3(1024), lds, st, wgs,                        \
                       static_cast<const T*>(A.st.val), A.st.off, A.st.mask, A.st.stride, tb,                        \
                       static_cast<const T*>(wtab), lmax, i, static_cast<const T*>(ysrc), static_cast<const T*>(i0), \
                       static_cast<const T*>(i1), static_cast<T*>(o0), static_cast<T*>(o1), static_cast<T*>(acc),    \
                       ibase, obase, groups);                                                                        \
  } while (0)
  if (win <= 32)
    KF_SB(2);
  else if (win <= 64)
    KF_SB(4);
  else
    KF_SB(RM);
#undef KF_SB
  KF_HIP(hipGetLastError());
  return KF_OK;
}
}  // namespace

int launch_steps_batch(const SellOp& A, const BatchWg* wgs, int nwg, int win, int b, const BatchTables* tb,
                       const void* wtab, int lmax, int i, const void* ysrc, const void* i0, const void* i1, void* o0,
                       void* o1, void* acc, int64_t ibase, int64_t obase, hipStream_t st) {
  const int cols = std::min(b, 16 / A.val_bytes), groups = b / cols;
#define KF_SB(T, B) \
  launch_steps_batch_b<T, B>(A, wgs, nwg, win, groups, tb, wtab, lmax, i, ysrc, i0, i1, o0, o1, acc, ibase, obase, st)
  if (A.val_bytes == 8) return cols == 1 ? KF_SB(double, 1) : KF_SB(double, 2);
  if (cols == 1) return KF_SB(float, 1);
  return cols == 2 ? KF_SB(float, 2) : KF_SB(float, 4);
#undef KF_SB
}

}  // namespace kf
