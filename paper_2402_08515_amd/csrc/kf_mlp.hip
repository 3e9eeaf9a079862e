// Learned filter weights: a small network maps the normalised problem data to
// the L filter coefficients.  Section 2.2 leaves the weight function free and
// states the design goal (|beta| large on the sought omega, small elsewhere);
// Lemma 2.3 gives the filter of any weights, beta~(omega) = sum_l w_l q_l.
//
// Normalised variables: a = tau*omega_min, c = tau*omega_max, x = tau*omega/2,
// x_max = tau*sqrt(lambda_max)/2.  In them q_l(x) = cos((l+1/2)phi)/cos(phi/2)
// with phi = 2 arcsin x, and the Fourier weights of eq. weightf are
// w_0 = 2(c-a)/pi, w_l = 4/(pi l) sin(l(c-a)/2) cos(l(c+a)/2), l < L.
//
// Network (features [a/pi, c/pi, x_max, L/512] padded to 64): three GELU
// layers of width 128, a linear layer of 512; w = w_Fourier + 0.01 * out,
// masked to l < L.  Loss on the grid x_g = 0.95 g/511: mean over the band
// [a/2, c/2] of (beta~ - 1)^2 plus the mean over x <= x_max outside the band
// widened by pi/(2L) of beta~^2.
//
// Matrix products of the network run on the matrix cores in bfloat16 with
// float32 accumulation (v_mfma_f32_16x16x16_bf16); the filter-response product
// beta~ = w Q and its adjoint run in float32 on the matrix cores
// (v_mfma_f32_16x16x4_f32), since the leakage being minimised is far below
// bfloat16 resolution.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <new>
#include <string>
#include <vector>

#include "kf_internal.h"

namespace kf {
namespace {

constexpr int kH = 128;    // hidden width
constexpr int kLM = 512;   // maximum number of weights
constexpr int kG = 512;    // frequency grid
constexpr int kNF = 64;    // padded feature count
constexpr float kOut = 0.01f;
constexpr float kXmaxGrid = 0.95f;
constexpr double kPi = 3.14159265358979323846;

// parameter layout (float32): W1[64x128] b1 W2[128x128] b2 W3[128x128] b3 W4[128x512] b4
constexpr int kOffW1 = 0;
constexpr int kOffB1 = kOffW1 + kNF * kH;
constexpr int kOffW2 = kOffB1 + kH;
constexpr int kOffB2 = kOffW2 + kH * kH;
constexpr int kOffW3 = kOffB2 + kH;
constexpr int kOffB3 = kOffW3 + kH * kH;
constexpr int kOffW4 = kOffB3 + kH;
constexpr int kOffB4 = kOffW4 + kH * kLM;
constexpr int kNParams = kOffB4 + kLM;

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ short to_bf16(float f) {
  // round to nearest even (finite inputs)
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (short)(u >> 16);
}

// A training step of 256 samples is five launches: k_forward (all layers of a
// row group in one workgroup, the Fourier weights beside them), k_response for
// beta~ and for dw, k_backward, and k_update (weight gradients, biases, losses
// and Adam).  Its products take 0.4 GFLOP: what bounds it is the latency of
// five dependent launches, 5 to 9 us each; 43 us a step against 678 us with a
// launch per product, bias, activation and reduction and a host wait per step.
// The gradient of 1024 samples: 67 us of kernels instead of 1.8 ms.  The
// float32 products alone (k_response) would take 1.7 us of matrix cores at 256
// samples and cannot be split along k without changing their rounding.

// ---- operand fragments
// A matrix instruction takes 16 x 16 tiles: lane (r16 = lane % 16, q4 =
// lane / 16) supplies four consecutive k = 4 q4 + q of row (or column) r16 and
// receives D[4 q4 + q][r16].  Everything one kernel hands to another for such
// a product is stored tile by tile in that lane order, one 8-byte run of four
// bfloat16 per lane and tile, so that an operand is one contiguous load: the
// weights in both orientations (forward: k = layer input; backward: k = layer
// output), and activations and their gradients for the weight gradients
// (k = sample).  All products take their k tiles in ascending order with one
// accumulator per output, whatever the launch shape.
constexpr int kFwd1 = 0;                                  // [128/16][64/16] tiles of 64 fragments
constexpr int kFwd2 = kFwd1 + (kH / 16) * (kNF / 16) * 64;
constexpr int kFwd3 = kFwd2 + (kH / 16) * (kH / 16) * 64;
constexpr int kFwd4 = kFwd3 + (kH / 16) * (kH / 16) * 64;
constexpr int kBwd2 = kFwd4 + (kLM / 16) * (kH / 16) * 64;
constexpr int kBwd3 = kBwd2 + (kH / 16) * (kH / 16) * 64;
constexpr int kBwd4 = kBwd3 + (kH / 16) * (kH / 16) * 64;
constexpr int kNFrag = kBwd4 + (kH / 16) * (kLM / 16) * 64;
constexpr int kPrm = 8;  // per sample: the two float4 of Band

// layer i = 0..3: parameter offset, inputs, outputs, fragment offsets
struct Layer {
  int off, bias, in, out, fwd, bwd;
};
__host__ __device__ constexpr Layer layer_of(int i) {
  return i == 0   ? Layer{kOffW1, kOffB1, kNF, kH, kFwd1, -1}
         : i == 1 ? Layer{kOffW2, kOffB2, kH, kH, kFwd2, kBwd2}
         : i == 2 ? Layer{kOffW3, kOffB3, kH, kH, kFwd3, kBwd3}
                  : Layer{kOffW4, kOffB4, kH, kLM, kFwd4, kBwd4};
}

// the weight W[row][col] of layer L into its fragments
__device__ __forceinline__ void put_fragments(const Layer L, int row, int col, float v, short* __restrict__ frag) {
  const short h = to_bf16(v);
  const int kt = row >> 4, nt = col >> 4;
  frag[((int64_t)(L.fwd + (nt * (L.in >> 4) + kt) * 64 + ((row & 15) >> 2) * 16 + (col & 15))) * 4 + (row & 3)] = h;
  if (L.bwd >= 0)
    frag[((int64_t)(L.bwd + (kt * (L.out >> 4) + nt) * 64 + ((col & 15) >> 2) * 16 + (row & 15))) * 4 + (col & 3)] = h;
}

__global__ __launch_bounds__(256) void k_pack(const float* __restrict__ theta, short* __restrict__ frag) {
  const int p = blockIdx.x * 256 + threadIdx.x;
  for (int i = 0; i < 4; ++i) {
    const Layer L = layer_of(i);
    const int t = p - L.off;
    if (t >= 0 && t < L.in * L.out) put_fragments(L, t / L.out, t % L.out, theta[p], frag);
  }
}

// Q[l][g] = q_l(x_g) for the float32 products beta~ = w Q (k = l) and dw =
// dbeta Q^T (k = g), tile by tile: lane (r16, q4) of tile (n tile, k tile)
// holds the four k = 4 sl + q4, sl < 4, of column r16 (v_mfma_f32_16x16x4
// takes one k per lane group).
__global__ void k_qmat(float* __restrict__ Qf, float* __restrict__ Qt) {
  const int l = blockIdx.x;
  for (int g = threadIdx.x; g < kG; g += blockDim.x) {
    const double x = kXmaxGrid * g / (kG - 1);
    const double phi = 2.0 * asin(x);
    const float v = (float)(cos((l + 0.5) * phi) / cos(0.5 * phi));
    auto at = [](int n, int k) { return (((n >> 4) * 32 + (k >> 4)) * 64 + (k & 3) * 16 + (n & 15)) * 4 + ((k >> 2) & 3); };
    Qf[at(g, l)] = v;
    Qt[at(l, g)] = v;
  }
}

__device__ __forceinline__ float gelu_f(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_g(float z) {
  return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

// A sample's constants: the band [a/2, c/2] of the loss grid and its edges
// widened by pi/(2L), x_max, the number of weights, and the numbers of grid
// points in the band and outside (x <= x_max, beyond the widened band).
struct Band {
  float lo, hi, wlo, whi, xm, L, ni, no;
  __device__ __forceinline__ Band(float a, float c, float Lf, float xm_) : xm(xm_), L(Lf), ni(1.f), no(1.f) {
    lo = 0.5f * a;
    hi = 0.5f * c;
    const float d = (float)(kPi / (2.0 * Lf));
    wlo = lo - d;
    whi = hi + d;
  }
  __device__ __forceinline__ Band(const float* __restrict__ prm, int64_t s) {
    const float4 u = reinterpret_cast<const float4*>(prm)[2 * s], v = reinterpret_cast<const float4*>(prm)[2 * s + 1];
    lo = u.x, hi = u.y, wlo = u.z, whi = u.w;
    xm = v.x, L = v.y, ni = v.z, no = v.w;
  }
  __device__ __forceinline__ void store(float* __restrict__ prm, int64_t s) const {
    reinterpret_cast<float4*>(prm)[2 * s] = make_float4(lo, hi, wlo, whi);
    reinterpret_cast<float4*>(prm)[2 * s + 1] = make_float4(xm, L, ni, no);
  }
  static __device__ __forceinline__ float x(int g) { return kXmaxGrid * g / (kG - 1); }
  __device__ __forceinline__ bool in(float v) const { return v >= lo && v <= hi; }
  __device__ __forceinline__ bool out(float v) const { return v <= xm && (v < wlo || v > whi); }
};

struct Sample {
  double a, c, xm;
  int L;
  __device__ __forceinline__ Sample(const double* __restrict__ r, const int32_t* __restrict__ Lover) {
    a = r[2] * r[0];
    c = r[2] * r[1];
    L = (int)ceil(2.0 * kPi / a);
    if (Lover) L = Lover[0];
    if (L > kLM) L = kLM;
    if (L < 1) L = 1;
    xm = 0.5 * r[2] * sqrt(r[3]);
  }
};

// One 16 x 16 tile: A (16 x 16 KT, bfloat16 rows in LDS, row stride ld) times
// the KT fragments of a column tile, which the caller loads long before (a
// kernel's weights do not depend on its rows, so their latency overlaps the
// staging and the layers before).
template <int KT>
__device__ __forceinline__ void load_tiles(const bf16x4* __restrict__ b, int lane, bf16x4 (&f)[KT]) {
#pragma unroll
  for (int u = 0; u < KT; ++u) f[u] = b[u * 64 + lane];
}
template <int KT>
__device__ __forceinline__ f32x4 tile_product(const short* A, int ld, const bf16x4 (&f)[KT], int lane) {
  const short* ap = A + (lane & 15) * ld + 4 * (lane >> 4);
  f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int u = 0; u < KT; ++u)
    acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(*reinterpret_cast<const bf16x4*>(ap + u * 16), f[u], acc, 0, 0, 0);
  return acc;
}

__device__ __forceinline__ bf16x4 pack4(const float (&v)[4]) {
  return bf16x4{to_bf16(v[0]), to_bf16(v[1]), to_bf16(v[2]), to_bf16(v[3])};
}

// Forward through the four layers, 16 samples per group of four workgroups
// (the hidden layers are computed by all four, the output layer's 512 columns
// are divided; one wavefront per 16 columns), and beside them one workgroup
// per sample for what does not depend on the parameters: the Fourier weights,
// the sample's constants and its grid-point counts.  The hidden rows stay in
// LDS between the layers; the first workgroup of a group stores what the
// backward pass needs.
constexpr int kHs = kH + 8;  // LDS row stride (bfloat16)
__global__ __launch_bounds__(512) void k_forward(int B, int nnet, const double* __restrict__ smp,
                                                 const int32_t* __restrict__ idx, const int32_t* __restrict__ Lover,
                                                 const float* __restrict__ theta, const bf16x4* __restrict__ frag,
                                                 bf16x4* __restrict__ xf, float* __restrict__ z,
                                                 bf16x4* __restrict__ hf, float* __restrict__ out,
                                                 float* __restrict__ prm, float* __restrict__ wF) {
  __shared__ __align__(16) short hs[2][16][kHs];
  __shared__ int cnt[2][8];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int r16 = lane & 15, q4 = lane >> 4;
  if ((int)blockIdx.x >= nnet) {
    const int s = blockIdx.x - nnet;
    const double* r = smp + 4 * (int64_t)(idx ? idx[s] : s);
    const Sample S(r, Lover);
    Band band((float)S.a, (float)S.c, (float)S.L, (float)S.xm);
    const float x = Band::x(tid);
    const bool in = band.in(x);
    const bool ou = !in && band.out(x);
    const int ni = __popcll(__ballot(in)), no = __popcll(__ballot(ou));
    if (lane == 0) {
      cnt[0][wave] = ni;
      cnt[1][wave] = no;
    }
    double w = 0.0;
    if (tid == 0)
      w = 2.0 * (S.c - S.a) / kPi;
    else if (tid < S.L)
      w = 4.0 / (kPi * tid) * sin(0.5 * tid * (S.c - S.a)) * cos(0.5 * tid * (S.c + S.a));
    wF[(int64_t)s * kLM + tid] = (float)w;
    __syncthreads();
    if (tid == 0) {
      int n0 = 0, n1 = 0;
      for (int i = 0; i < 8; ++i) {
        n0 += cnt[0][i];
        n1 += cnt[1][i];
      }
      band.ni = fmaxf((float)n0, 1.f);
      band.no = fmaxf((float)n1, 1.f);
      band.store(prm, s);
    }
    return;
  }
  const int st = blockIdx.x >> 2, part = blockIdx.x & 3, nst = B >> 4;
  const bool keep = part == 0;
  const int nt = part * 8 + wave;
  bf16x4 f1[kNF / 16], f2[kH / 16], f3[kH / 16], f4[kH / 16];
  load_tiles(frag + kFwd1 + wave * (kNF / 16) * 64, lane, f1);
  load_tiles(frag + kFwd2 + wave * (kH / 16) * 64, lane, f2);
  load_tiles(frag + kFwd3 + wave * (kH / 16) * 64, lane, f3);
  load_tiles(frag + kFwd4 + nt * (kH / 16) * 64, lane, f4);
  for (int t = tid; t < 16 * kNF; t += 512) hs[0][t / kNF][t % kNF] = 0;
  __syncthreads();
  if (tid < 16) {
    const int s = st * 16 + tid;
    const Sample S(smp + 4 * (int64_t)(idx ? idx[s] : s), Lover);
    hs[0][tid][0] = to_bf16((float)(S.a / kPi));
    hs[0][tid][1] = to_bf16((float)(S.c / kPi));
    hs[0][tid][2] = to_bf16((float)S.xm);
    hs[0][tid][3] = to_bf16((float)S.L / kLM);
  }
  __syncthreads();
  if (keep && wave < kNF / 16) {
    bf16x4 v;
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = hs[0][4 * q4 + q][wave * 16 + r16];
    xf[((int64_t)wave * nst + st) * 64 + lane] = v;
  }
  int src = 0;
  const int n = wave * 16 + r16;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const Layer L = layer_of(i);
    const float bias = theta[L.bias + n];
    const f32x4 acc = i == 0   ? tile_product(&hs[src][0][0], kHs, f1, lane)
                      : i == 1 ? tile_product(&hs[src][0][0], kHs, f2, lane)
                               : tile_product(&hs[src][0][0], kHs, f3, lane);
    float h[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float zv = acc[q] + bias;
      h[q] = gelu_f(zv);
      if (keep) z[((int64_t)i * B + st * 16 + 4 * q4 + q) * kH + n] = zv;
      hs[src ^ 1][4 * q4 + q][n] = to_bf16(h[q]);
    }
    if (keep) hf[((int64_t)(i * (kH / 16) + wave) * nst + st) * 64 + lane] = pack4(h);
    __syncthreads();
    src ^= 1;
  }
  const f32x4 acc = tile_product(&hs[src][0][0], kHs, f4, lane);
#pragma unroll
  for (int q = 0; q < 4; ++q) out[(int64_t)(st * 16 + 4 * q4 + q) * kLM + nt * 16 + r16] = acc[q];
}

// w = (wF + s (out + b4)) [l < L], the correction left out without the network
__device__ __forceinline__ float weight_of(float out, float b4, float wF, int l, float Lf, int use_net) {
#pragma clang fp contract(off)
  const float d = use_net ? kOut * (out + b4) : 0.f;
  return l < (int)Lf ? wF + d : 0.f;
}

__global__ void k_out_weights(int B, const float* __restrict__ out, const float* __restrict__ b4,
                              const float* __restrict__ wF, const float* __restrict__ prm, float* __restrict__ w,
                              int use_net) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)B * kLM) return;
  const int s = (int)(t / kLM), l = (int)(t % kLM);
  w[t] = weight_of(use_net ? out[t] : 0.f, b4[l], wF[t], l, Band(prm, s).L, use_net);
}

// The two float32 products with the response matrix, 16 rows x 64 columns
// per workgroup, one wavefront per 16 columns (the k order is fixed, so the
// work is spread over rows and columns only).  BACK = 0: beta~ = w Q with w
// formed while the rows are staged; writes w, beta~ and (grad) dJ/dbeta~.
// BACK = 1: dw = dbeta~ Q^T, and from it the output layer's gradient dz =
// s dw [l < L] as rows and as fragments.
constexpr int kRs = kG + 4;  // LDS row stride (float32)
template <int BACK>
__global__ __launch_bounds__(256) void k_response(int B, const float* __restrict__ src, const float* __restrict__ b4,
                                                  const float* __restrict__ wF, const float* __restrict__ prm,
                                                  const float4* __restrict__ Q, int use_net, float scale,
                                                  float* __restrict__ w, float* __restrict__ res,
                                                  float* __restrict__ dbeta, bf16x4* __restrict__ dzf) {
  __shared__ __align__(16) float xs[16][kRs];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int r16 = lane & 15, q4 = lane >> 4;
  const int st = blockIdx.y, nt = blockIdx.x * 4 + wave;
  const float4* __restrict__ qp = Q + (int64_t)nt * 32 * 64 + lane;
  constexpr int U = 8;
  float4 cur[U], nxt[U];
#pragma unroll
  for (int u = 0; u < U; ++u) cur[u] = qp[u * 64];
  const Band band[4] = {Band(prm, st * 16 + 4 * q4), Band(prm, st * 16 + 4 * q4 + 1), Band(prm, st * 16 + 4 * q4 + 2),
                        Band(prm, st * 16 + 4 * q4 + 3)};
  // a thread stages columns tid and tid + 256 of the 16 rows, eight rows of
  // loads at a time; k = 4 sl + q4 of a 16-block sits at 4 q4 + sl, so that a
  // lane's four are one read
#pragma unroll
  for (int r0 = 0; r0 < 16; r0 += 8) {
    float va[8][2], vf[8][2];
#pragma unroll
    for (int r = 0; r < 8; ++r)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int64_t g = (int64_t)(st * 16 + r0 + r) * kG + tid + 256 * h;
        va[r][h] = BACK || use_net ? src[g] : 0.f;
        vf[r][h] = BACK ? 0.f : wF[g];
      }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = tid + 256 * h;
      const float bias = BACK ? 0.f : b4[k];
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        float v = va[r][h];
        if (!BACK) {
          v = weight_of(v, bias, vf[r][h], k, prm[(int64_t)(st * 16 + r0 + r) * kPrm + 5], use_net);
          if (blockIdx.x == 0) w[(int64_t)(st * 16 + r0 + r) * kG + k] = v;
        }
        xs[r0 + r][(k & ~15) + (k & 3) * 4 + ((k >> 2) & 3)] = v;
      }
    }
  }
  __syncthreads();
  f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k0 = 0; k0 < 32; k0 += U) {
    if (k0 + U < 32) {
#pragma unroll
      for (int u = 0; u < U; ++u) nxt[u] = qp[(k0 + U + u) * 64];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float4 a = *reinterpret_cast<const float4*>(&xs[r16][(k0 + u) * 16 + 4 * q4]);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, cur[u].x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, cur[u].y, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, cur[u].z, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, cur[u].w, acc, 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) cur[u] = nxt[u];
  }
  const int n = nt * 16 + r16;
  if (BACK) {
    float d[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int s = st * 16 + 4 * q4 + q;
      d[q] = n < (int)band[q].L ? kOut * acc[q] : 0.f;
      res[(int64_t)s * kLM + n] = d[q];
    }
    dzf[((int64_t)nt * (B >> 4) + st) * 64 + lane] = pack4(d);
  } else {
    const float x = Band::x(n);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int s = st * 16 + 4 * q4 + q;
      const float bt = acc[q];
      res[(int64_t)s * kG + n] = bt;
      if (dbeta) {
        float gr = 0.f;
        if (band[q].in(x))
          gr = 2.f * (bt - 1.f) / band[q].ni;
        else if (band[q].out(x))
          gr = 2.f * bt / band[q].no;
        dbeta[(int64_t)s * kG + n] = gr * scale;
      }
    }
  }
}

// The loss of sample s by one wavefront: lane l takes g = 64 p + l and
// 64 p + l + 256 for p = 0..3, the four parts are summed in order.
__device__ __forceinline__ float sample_loss(const float* __restrict__ beta, const float* __restrict__ prm, int s,
                                             int lane) {
  const Band band(prm, s);
  float bt[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) bt[i] = beta[(int64_t)s * kG + 64 * (i >> 1) + lane + 256 * (i & 1)];
  float ji = 0.f, jo = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float a = 0.f, b = 0.f;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float v = bt[2 * i + h], x = Band::x(64 * i + lane + 256 * h);
      if (band.in(x))
        a = fmaf(v - 1.f, v - 1.f, a);
      else if (band.out(x))
        b = fmaf(v, v, b);
    }
    for (int off = 32; off > 0; off >>= 1) {
      a += __shfl_xor(a, off);
      b += __shfl_xor(b, off);
    }
    ji = i ? ji + a : a;
    jo = i ? jo + b : b;
  }
  return ji / band.ni + jo / band.no;
}

__global__ __launch_bounds__(256) void k_loss(int B, const float* __restrict__ beta, const float* __restrict__ prm,
                                              float* __restrict__ J) {
  const int s = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (s >= B) return;
  const float v = sample_loss(beta, prm, s, lane);
  if (lane == 0) J[s] = v;
}

// Backward through the hidden layers, 16 samples per workgroup: each of the
// eight wavefronts carries one 16-column tile through the three products
// (rows in LDS as bfloat16 between them).
__global__ __launch_bounds__(512) void k_backward(int B, const float* __restrict__ dz4, const float* __restrict__ z,
                                                  const bf16x4* __restrict__ frag, float* __restrict__ dz,
                                                  bf16x4* __restrict__ dzf) {
  __shared__ __align__(16) short d4[16][kLM + 8];
  __shared__ __align__(16) short ds[2][16][kHs];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int r16 = lane & 15, q4 = lane >> 4;
  const int st = blockIdx.x, nst = B >> 4;
  const int n = wave * 16 + r16;
  float dv[16];
#pragma unroll
  for (int u = 0; u < 16; ++u) dv[u] = dz4[(int64_t)(st * 16) * kLM + tid + 512 * u];
  bf16x4 f4[kLM / 16], f3[kH / 16], f2[kH / 16];
  load_tiles(frag + kBwd4 + wave * (kLM / 16) * 64, lane, f4);
  load_tiles(frag + kBwd3 + wave * (kH / 16) * 64, lane, f3);
  load_tiles(frag + kBwd2 + wave * (kH / 16) * 64, lane, f2);
  float zv[3][4];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) zv[i][q] = z[((int64_t)i * B + st * 16 + 4 * q4 + q) * kH + n];
#pragma unroll
  for (int u = 0; u < 16; ++u) d4[u][tid] = to_bf16(dv[u]);
  __syncthreads();
#pragma unroll
  for (int i = 2; i >= 0; --i) {
    const f32x4 acc = i == 2   ? tile_product(&d4[0][0], kLM + 8, f4, lane)
                      : i == 1 ? tile_product(&ds[i & 1][0][0], kHs, f3, lane)
                               : tile_product(&ds[i & 1][0][0], kHs, f2, lane);
    float d[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      d[q] = acc[q] * gelu_g(zv[i][q]);
      dz[((int64_t)i * B + st * 16 + 4 * q4 + q) * kH + n] = d[q];
      ds[(i & 1) ^ 1][4 * q4 + q][n] = to_bf16(d[q]);
    }
    dzf[((int64_t)(i * (kH / 16) + wave) * nst + st) * 64 + lane] = pack4(d);
    __syncthreads();
  }
}

struct AdamStep {
  float lr, c1, c2;  // c1 = 0: no update (the gradient is stored instead)
};

__device__ __forceinline__ float adam(int p, float g, float th, float* __restrict__ m1, float* __restrict__ m2,
                                      const AdamStep& o) {
  const float a = fmaf(1.f - 0.9f, g, 0.9f * m1[p]);
  const float b = fmaf(g, (1.f - 0.999f) * g, 0.999f * m2[p]);
  m1[p] = a;
  m2[p] = b;
  return th - o.lr * (a / o.c1) / (sqrtf(b / o.c2) + 1e-8f);
}

// Gradients of all parameters, and in training the Adam step on the spot (the
// gradient is never stored).  One wavefront per 16 x 16 tile of a weight
// matrix (416 tiles, both operands one contiguous run per 16 samples), then
// one workgroup per 64 biases: four wavefronts stage rows, the first sums
// them in row order; then the samples' losses, one wavefront each.
constexpr int kTiles4 = (kH / 16) * (kLM / 16), kTilesH = (kH / 16) * (kH / 16), kTiles1 = (kNF / 16) * (kH / 16);
constexpr int kTileBlocks = (kTiles4 + 2 * kTilesH + kTiles1) / 4;
constexpr int kBiasBlocks = (kLM + 3 * kH) / 64;
__global__ __launch_bounds__(256) void k_update(int B, const bf16x4* __restrict__ xf, const bf16x4* __restrict__ hf,
                                                const bf16x4* __restrict__ dzf, const bf16x4* __restrict__ dzf4,
                                                const float* __restrict__ dz, const float* __restrict__ dz4,
                                                float* __restrict__ theta, float* __restrict__ m1,
                                                float* __restrict__ m2, float* __restrict__ grad,
                                                short* __restrict__ frag, const float* __restrict__ beta,
                                                const float* __restrict__ prm, float* __restrict__ J, AdamStep o) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int nst = B >> 4;
  if ((int)blockIdx.x >= kTileBlocks + kBiasBlocks) {
    const int s = (blockIdx.x - kTileBlocks - kBiasBlocks) * 4 + wave;
    const float v = sample_loss(beta, prm, s, lane);
    if (lane == 0) J[s] = v;
    return;
  }
  if ((int)blockIdx.x >= kTileBlocks) {
    __shared__ float rows[64][64];
    int c = (blockIdx.x - kTileBlocks) * 64;  // first of this workgroup's biases, counted b4, b3, b2, b1
    int i = 3;
    const float* src = dz4;
    int ld = kLM;
    if (c >= kLM) {
      c -= kLM;
      i = 2 - c / kH;
      c %= kH;
      src = dz + (int64_t)i * B * kH;
      ld = kH;
    }
    src += c + lane;
    float s = 0.f;
    float v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = src[(int64_t)(wave + 4 * u) * ld];
    for (int r0 = 0; r0 < B; r0 += 64) {
      __syncthreads();
#pragma unroll
      for (int u = 0; u < 16; ++u) rows[wave + 4 * u][lane] = v[u];
      __syncthreads();
      if (r0 + 64 < B) {
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = src[(int64_t)(r0 + 64 + wave + 4 * u) * ld];
      }
      if (wave == 0) {
#pragma unroll
        for (int r = 0; r < 64; ++r) s += rows[r][lane];
      }
    }
    if (wave != 0) return;
    const int p = layer_of(i).bias + c + lane;
    if (o.c1 == 0.f)
      grad[p] = s;
    else
      theta[p] = adam(p, s, theta[p], m1, m2, o);
    return;
  }
  int t = blockIdx.x * 4 + wave, i = 3;
  if (t >= kTiles4) {
    t -= kTiles4;
    i = t < kTilesH ? 2 : (t < 2 * kTilesH ? 1 : 0);
    t -= (2 - i) * kTilesH;
  }
  const Layer L = layer_of(i);
  const int mt = t / (L.out >> 4), nt = t % (L.out >> 4);
  const bf16x4* __restrict__ ap = (i == 0 ? xf + (int64_t)mt * nst * 64
                                          : hf + (int64_t)((i - 1) * (kH / 16) + mt) * nst * 64) + lane;
  const bf16x4* __restrict__ bp = (i == 3 ? dzf4 + (int64_t)nt * nst * 64
                                          : dzf + (int64_t)(i * (kH / 16) + nt) * nst * 64) + lane;
  f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
  constexpr int U = 4;  // B is a multiple of 64
  bf16x4 a[U], b[U], an[U], bn[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    a[u] = ap[u * 64];
    b[u] = bp[u * 64];
  }
  for (int k = 0; k < nst; k += U) {
    if (k + U < nst) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        an[u] = ap[(k + U + u) * 64];
        bn[u] = bp[(k + U + u) * 64];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a[u], b[u], acc, 0, 0, 0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      a[u] = an[u];
      b[u] = bn[u];
    }
  }
  const int r16 = lane & 15, q4 = lane >> 4;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int row = mt * 16 + 4 * q4 + q, col = nt * 16 + r16;
    const int p = L.off + row * L.out + col;
    if (o.c1 == 0.f) {
      grad[p] = acc[q];
    } else {
      const float th = adam(p, acc[q], theta[p], m1, m2, o);
      theta[p] = th;
      put_fragments(L, row, col, th, frag);
    }
  }
}

// mean of J in double
__global__ __launch_bounds__(256) void k_mean(int B, const float* __restrict__ J, float* __restrict__ out) {
  __shared__ double red[4];
  double s = 0.0;
  for (int i = threadIdx.x; i < B; i += 256) s += J[i];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) out[0] = (float)(((red[0] + red[1]) + (red[2] + red[3])) / B);
}

inline int nblk(int64_t n, int b = 256) { return (int)((n + b - 1) / b); }

}  // namespace
}  // namespace kf

using namespace kf;

struct kf_mlp {
  hipStream_t st = nullptr;
  int cap = 0;  // batch capacity (multiple of 64)
  float* theta = nullptr;
  float* grad = nullptr;  // pinned host memory that kernels write: the gradient, then the mean loss (first use)
  float* m1 = nullptr;
  float* m2 = nullptr;
  short* frag = nullptr;  // the weights as bfloat16 fragments (kept with theta)
  float *Qf = nullptr, *Qt = nullptr;  // the response matrix and its transpose, tile by tile
  // activations (cap rows): z, dz and their fragments for the three hidden layers
  float *prm = nullptr, *wF = nullptr, *z = nullptr, *out = nullptr, *w = nullptr, *beta = nullptr, *dbeta = nullptr,
        *dz4 = nullptr, *dz = nullptr, *J = nullptr;
  bf16x4 *xf = nullptr, *hf = nullptr, *dzf4 = nullptr, *dzf = nullptr;
  double* smp = nullptr;  // device samples
  int nsmp_cap = 0;
  int32_t* idx = nullptr;
  int idx_cap = 0;
  float* Jrun = nullptr;  // the losses of a training run's steps
  int64_t Jrun_cap = 0;
  int32_t* Lover = nullptr;
  int64_t adam_t = 0;
};

namespace {

int mfail(int code, const std::string& s) {
  set_error(s);
  return code;
}

template <typename T>
int dalloc_m(T** p, size_t n) {
  if (hipMalloc((void**)p, sizeof(T) * std::max<size_t>(n, 1)) != hipSuccess) {
    *p = nullptr;
    return mfail(KF_ENOMEM, "kf_mlp: device allocation failed");
  }
  return KF_OK;
}

void mfree(void* p) {
  if (p) (void)hipFree(p);
}

int ensure_batch(kf_mlp* net, int B) {
  if (net->cap >= B) return KF_OK;
  float** bufs[] = {&net->prm, &net->wF, &net->z, &net->out, &net->w, &net->beta, &net->dbeta, &net->dz4, &net->dz, &net->J};
  bf16x4** frags[] = {&net->xf, &net->hf, &net->dzf4, &net->dzf};
  net->cap = 0;
  for (float** b : bufs) {
    mfree(*b);
    *b = nullptr;
  }
  for (bf16x4** b : frags) {
    mfree(*b);
    *b = nullptr;
  }
  const size_t Bn = (size_t)B;
  KF_TRY(dalloc_m(&net->prm, Bn * kPrm));
  KF_TRY(dalloc_m(&net->wF, Bn * kLM));
  KF_TRY(dalloc_m(&net->z, Bn * 3 * kH));
  KF_TRY(dalloc_m(&net->out, Bn * kLM));
  KF_TRY(dalloc_m(&net->w, Bn * kLM));
  KF_TRY(dalloc_m(&net->beta, Bn * kG));
  KF_TRY(dalloc_m(&net->dbeta, Bn * kG));
  KF_TRY(dalloc_m(&net->dz4, Bn * kLM));
  KF_TRY(dalloc_m(&net->dz, Bn * 3 * kH));
  KF_TRY(dalloc_m(&net->J, Bn));
  KF_TRY(dalloc_m(&net->xf, Bn * kNF / 4));
  KF_TRY(dalloc_m(&net->hf, Bn * 3 * kH / 4));
  KF_TRY(dalloc_m(&net->dzf4, Bn * kLM / 4));
  KF_TRY(dalloc_m(&net->dzf, Bn * 3 * kH / 4));
  net->cap = B;
  return KF_OK;
}

int upload_samples(kf_mlp* net, const double* samples, int n) {
  if (n > net->nsmp_cap) {
    mfree(net->smp);
    net->smp = nullptr;
    KF_TRY(dalloc_m(&net->smp, (size_t)n * 4));
    net->nsmp_cap = n;
  }
  for (int i = 0; i < n; ++i) {
    const double* r = samples + 4 * (size_t)i;
    if (!(r[0] > 0) || !(r[1] > r[0]) || !(r[2] > 0) || !(r[3] > 0) || !std::isfinite(r[1]) || !std::isfinite(r[3]))
      return mfail(KF_EINVAL, "kf_mlp: sample " + std::to_string(i) +
                                  " needs 0 < omega_min < omega_max, tau > 0, lambda_max > 0");
    if (2.0 * kPi / (r[2] * r[0]) > kLM) return mfail(KF_EINVAL, "kf_mlp: sample needs more than 512 weights");
  }
  KF_HIP(hipMemcpyAsync(net->smp, samples, sizeof(double) * 4 * n, hipMemcpyHostToDevice, net->st));
  return KF_OK;
}

// the network's output and the samples' constants (B a multiple of 64)
int forward(kf_mlp* net, int B, const int32_t* d_idx, bool use_net, const int32_t* d_Lover) {
  const int nnet = use_net ? B / 4 : 0;
  hipLaunchKernelGGL(k_forward, dim3(nnet + B), dim3(512), 0, net->st, B, nnet, net->smp, d_idx, d_Lover, net->theta,
                     reinterpret_cast<const bf16x4*>(net->frag), net->xf, net->z, net->hf, net->out, net->prm, net->wF);
  KF_HIP(hipGetLastError());
  return KF_OK;
}

// the weights of the forward pass, their filter response and, without a
// backward pass to follow, the losses into net->J
int response(kf_mlp* net, int B, bool use_net, bool grad) {
  hipLaunchKernelGGL(k_response<0>, dim3(kG / 64, B / 16), dim3(256), 0, net->st, B, net->out, net->theta + kOffB4,
                     net->wF, net->prm, reinterpret_cast<const float4*>(net->Qf), use_net ? 1 : 0, 1.0f / B, net->w,
                     net->beta, grad ? net->dbeta : nullptr, (bf16x4*)nullptr);
  KF_HIP(hipGetLastError());
  if (grad) return KF_OK;
  hipLaunchKernelGGL(k_loss, dim3(nblk(B, 4)), dim3(256), 0, net->st, B, net->beta, net->prm, net->J);
  KF_HIP(hipGetLastError());
  return KF_OK;
}

// losses into J, and the gradient into net->grad (step.c1 = 0) or an Adam step
int backward(kf_mlp* net, int B, float* J, const AdamStep& step) {
  hipStream_t st = net->st;
  hipLaunchKernelGGL(k_response<1>, dim3(kLM / 64, B / 16), dim3(256), 0, st, B, net->dbeta, (const float*)nullptr,
                     (const float*)nullptr, net->prm, reinterpret_cast<const float4*>(net->Qt), 0, 0.f,
                     (float*)nullptr, net->dz4, (float*)nullptr, net->dzf4);
  KF_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_backward, dim3(B / 16), dim3(512), 0, st, B, net->dz4, net->z,
                     reinterpret_cast<const bf16x4*>(net->frag), net->dz, net->dzf);
  KF_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_update, dim3(kTileBlocks + kBiasBlocks + B / 4), dim3(256), 0, st, B, net->xf, net->hf,
                     net->dzf, net->dzf4, net->dz, net->dz4, net->theta, net->m1, net->m2, net->grad, net->frag,
                     net->beta, net->prm, J, step);
  KF_HIP(hipGetLastError());
  return KF_OK;
}

// forward (use_net: network correction on) and loss; grad: backpropagation
int fwd_bwd(kf_mlp* net, int B, const int32_t* d_idx, bool use_net, bool grad, const int32_t* d_Lover) {
  KF_TRY(forward(net, B, d_idx, use_net, d_Lover));
  KF_TRY(response(net, B, use_net, grad));
  return grad ? backward(net, B, net->J, AdamStep{0.f, 0.f, 0.f}) : KF_OK;
}

void free_mlp(kf_mlp* net) {
  if (!net) return;
  if (net->st) (void)hipStreamSynchronize(net->st);
  if (net->grad) (void)hipHostFree(net->grad);
  void* ps[] = {net->theta, net->m1, net->m2, net->frag, net->Qf, net->Qt, net->prm, net->wF, net->z,
                net->out, net->w, net->beta, net->dbeta, net->dz4, net->dz, net->J, net->xf, net->hf,
                net->dzf4, net->dzf, net->smp, net->idx, net->Jrun, net->Lover};
  for (void* p : ps) mfree(p);
  if (net->st) (void)hipStreamDestroy(net->st);
  delete net;
}

}  // namespace

extern "C" {

int32_t kf_mlp_param_count(void) { return kNParams; }

int kf_mlp_create(const float* params, kf_mlp** out) {
  if (!out || !params) return mfail(KF_EINVAL, "kf_mlp_create: NULL argument");
  *out = nullptr;
  for (int i = 0; i < kNParams; ++i)
    if (!std::isfinite(params[i])) return mfail(KF_EINVAL, "kf_mlp_create: non-finite parameter");
  kf_mlp* net = new (std::nothrow) kf_mlp();
  if (!net) return mfail(KF_ENOMEM, "kf_mlp_create: host allocation");
  int rc = KF_OK;
  do {
    if (hipStreamCreate(&net->st) != hipSuccess) {
      rc = mfail(KF_EHIP, "kf_mlp_create: stream");
      break;
    }
    if ((rc = dalloc_m(&net->theta, kNParams)) ||
        (rc = dalloc_m(&net->m1, kNParams)) || (rc = dalloc_m(&net->m2, kNParams)) ||
        (rc = dalloc_m(&net->frag, (size_t)kNFrag * 4)) || (rc = dalloc_m(&net->Qf, (size_t)kLM * kG)) ||
        (rc = dalloc_m(&net->Qt, (size_t)kLM * kG)) || (rc = dalloc_m(&net->Lover, 1)))
      break;
    if (hipMemcpy(net->theta, params, sizeof(float) * kNParams, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemset(net->m1, 0, sizeof(float) * kNParams) != hipSuccess ||
        hipMemset(net->m2, 0, sizeof(float) * kNParams) != hipSuccess) {
      rc = mfail(KF_EHIP, "kf_mlp_create: upload");
      break;
    }
    hipLaunchKernelGGL(k_pack, dim3(nblk(kNParams)), dim3(256), 0, net->st, net->theta, net->frag);
    hipLaunchKernelGGL(k_qmat, dim3(kLM), dim3(256), 0, net->st, net->Qf, net->Qt);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(net->st) != hipSuccess) rc = mfail(KF_EHIP, "kf_mlp_create: Q");
  } while (false);
  if (rc) {
    free_mlp(net);
    return rc;
  }
  *out = net;
  return KF_OK;
}

int kf_mlp_destroy(kf_mlp* net) {
  free_mlp(net);
  return KF_OK;
}

int kf_mlp_get_params(const kf_mlp* net, float* out) {
  if (!net || !out) return mfail(KF_EINVAL, "kf_mlp_get_params: NULL argument");
  KF_HIP(hipMemcpy(out, net->theta, sizeof(float) * kNParams, hipMemcpyDeviceToHost));
  return KF_OK;
}

int kf_mlp_loss_grad(kf_mlp* net, const double* samples, int32_t n, double* loss, float* grad) {
  if (!net || !samples || !loss || n < 1) return mfail(KF_EINVAL, "kf_mlp_loss_grad: bad arguments");
  if (n % 64) return mfail(KF_EINVAL, "kf_mlp_loss_grad: n must be a multiple of 64");
  KF_TRY(ensure_batch(net, n));
  // (pinning takes 65 us, two fifths of kf_mlp_create: networks that are only
  // trained or asked for weights do without)
  if (!net->grad && hipHostMalloc((void**)&net->grad, sizeof(float) * (kNParams + 1)) != hipSuccess) {
    net->grad = nullptr;
    return mfail(KF_ENOMEM, "kf_mlp: pinned host allocation failed");
  }
  KF_TRY(upload_samples(net, samples, n));
  KF_TRY(fwd_bwd(net, n, nullptr, true, grad != nullptr, nullptr));
  // k_update and k_mean write pinned memory: copying 430 KB from the device to
  // the caller's pageable array took 55 us of a call's 149 (1024 samples), the
  // stores over the bus and a copy on the host 10
  hipLaunchKernelGGL(k_mean, dim3(1), dim3(256), 0, net->st, n, net->J, net->grad + kNParams);
  KF_HIP(hipGetLastError());
  KF_HIP(hipStreamSynchronize(net->st));
  *loss = net->grad[kNParams];
  if (grad) std::memcpy(grad, net->grad, sizeof(float) * kNParams);
  return KF_OK;
}

int kf_mlp_train(kf_mlp* net, const double* samples, int32_t n, const int32_t* order, int32_t epochs, int32_t batch,
                 double lr, double* epoch_loss) {
  if (!net || !samples || !order || n < 1 || epochs < 1) return mfail(KF_EINVAL, "kf_mlp_train: bad arguments");
  if (batch < 64 || batch % 64 || batch > n) return mfail(KF_EINVAL, "kf_mlp_train: batch must be a multiple of 64, <= n");
  if (!(lr > 0)) return mfail(KF_EINVAL, "kf_mlp_train: lr must be positive");
  for (int64_t i = 0; i < (int64_t)epochs * n; ++i)
    if (order[i] < 0 || order[i] >= n) return mfail(KF_EINVAL, "kf_mlp_train: order out of range");
  KF_TRY(ensure_batch(net, batch));
  KF_TRY(upload_samples(net, samples, n));
  const int64_t total = (int64_t)epochs * n;
  if (total > net->idx_cap) {
    mfree(net->idx);
    net->idx = nullptr;
    KF_TRY(dalloc_m(&net->idx, (size_t)total));
    net->idx_cap = (int)total;
  }
  KF_HIP(hipMemcpyAsync(net->idx, order, sizeof(int32_t) * total, hipMemcpyHostToDevice, net->st));
  const int steps = n / batch;
  const int64_t nJ = (int64_t)epochs * steps * batch;
  if (nJ > net->Jrun_cap) {
    mfree(net->Jrun);
    net->Jrun = nullptr;
    net->Jrun_cap = 0;
    KF_TRY(dalloc_m(&net->Jrun, (size_t)nJ));
    net->Jrun_cap = nJ;
  }
  for (int e = 0; e < epochs; ++e) {
    for (int s = 0; s < steps; ++s) {
      const int32_t* d_idx = net->idx + (int64_t)e * n + (int64_t)s * batch;
      KF_TRY(forward(net, batch, d_idx, true, nullptr));
      KF_TRY(response(net, batch, true, true));
      ++net->adam_t;
      // cosine decay from lr to lr/100 over the run
      const double prog = (double)(e * steps + s) / std::max(1, epochs * steps - 1);
      const double lrt = lr * (0.01 + 0.99 * 0.5 * (1.0 + std::cos(kPi * prog)));
      const float c1 = (float)(1.0 - std::pow(0.9, (double)net->adam_t));
      const float c2 = (float)(1.0 - std::pow(0.999, (double)net->adam_t));
      KF_TRY(backward(net, batch, net->Jrun + ((int64_t)e * steps + s) * batch, AdamStep{(float)lrt, c1, c2}));
    }
  }
  if (epoch_loss) {
    // (a long run's losses come back 16 MB at a time)
    const int64_t per = (int64_t)steps * batch, most = std::min<int64_t>(nJ, 1 << 22);
    float* Jh = new (std::nothrow) float[(size_t)most];
    if (!Jh) return mfail(KF_ENOMEM, "kf_mlp_train: host allocation");
    std::unique_ptr<float[]> hold(Jh);
    int64_t from = 0, to = 0;  // the losses in the block
    for (int e = 0; e < epochs; ++e) {
      double acc = 0.0;
      for (int64_t i = e * per, end = i + per; i < end;) {
        if (i == to) {
          from = to;
          to = std::min(nJ, from + most);
          KF_HIP(hipMemcpyAsync(Jh, net->Jrun + from, sizeof(float) * (size_t)(to - from), hipMemcpyDeviceToHost, net->st));
          KF_HIP(hipStreamSynchronize(net->st));
        }
        for (const int64_t stop = std::min(end, to); i < stop; ++i) acc += Jh[i - from];
      }
      epoch_loss[e] = acc / ((double)steps * batch);
    }
  }
  KF_HIP(hipStreamSynchronize(net->st));
  return KF_OK;
}

int kf_mlp_weights(kf_mlp* net, const double* samples, int32_t n, double* w_out) {
  if (!net || !samples || !w_out || n < 1) return mfail(KF_EINVAL, "kf_mlp_weights: bad arguments");
  // padded to a multiple of 64 rows by repeating the last sample
  const int np = (n + 63) / 64 * 64;
  std::vector<double> rep((size_t)4 * np);
  std::memcpy(rep.data(), samples, sizeof(double) * 4 * (size_t)n);
  for (int i = n; i < np; ++i) std::memcpy(&rep[4 * (size_t)i], samples + 4 * (size_t)(n - 1), sizeof(double) * 4);
  KF_TRY(ensure_batch(net, np));
  KF_TRY(upload_samples(net, rep.data(), np));
  KF_TRY(forward(net, np, nullptr, true, nullptr));
  hipLaunchKernelGGL(k_out_weights, dim3(nblk((int64_t)np * kLM)), dim3(256), 0, net->st, np, net->out,
                     net->theta + kOffB4, net->wF, net->prm, net->w, 1);
  KF_HIP(hipGetLastError());
  std::vector<float> wl((size_t)n * kLM);
  KF_HIP(hipMemcpyAsync(wl.data(), net->w, sizeof(float) * wl.size(), hipMemcpyDeviceToHost, net->st));
  KF_HIP(hipStreamSynchronize(net->st));
  for (size_t i = 0; i < wl.size(); ++i) w_out[i] = wl[i];
  return KF_OK;
}

int kf_weights_from_mlp(kf_mlp* net, double omega_min, double omega_max, double tau, double lambda_max, int32_t L,
                        double* w_out, int32_t* used_learned, double* j_learned, double* j_fourier) {
  if (!net || !w_out || !used_learned) return mfail(KF_EINVAL, "kf_weights_from_mlp: NULL argument");
  if (L < 1) return mfail(KF_EINVAL, "kf_weights_from_mlp: L must be >= 1");
  const double smp[4] = {omega_min, omega_max, tau, lambda_max};
  if (!(omega_min > 0) || !(omega_max > omega_min) || !(tau > 0) || !(lambda_max > 0))
    return mfail(KF_EINVAL, "kf_weights_from_mlp: need 0 < omega_min < omega_max, tau > 0, lambda_max > 0");
  const double a = tau * omega_min, c = tau * omega_max;
  std::vector<double> wf((size_t)L);
  for (int l = 0; l < L; ++l)
    wf[(size_t)l] = l == 0 ? 2.0 * (c - a) / kPi : 4.0 / (kPi * l) * std::sin(0.5 * l * (c - a)) * std::cos(0.5 * l * (c + a));
  *used_learned = 0;
  if (L > kLM) {
    std::memcpy(w_out, wf.data(), sizeof(double) * L);
    return KF_OK;
  }
  // one sample padded to a 64-row batch
  std::vector<double> rep(4 * 64);
  for (int i = 0; i < 64; ++i) std::memcpy(&rep[4 * (size_t)i], smp, sizeof(smp));
  KF_TRY(ensure_batch(net, 64));
  if (net->nsmp_cap < 64) {
    mfree(net->smp);
    net->smp = nullptr;
    KF_TRY(dalloc_m(&net->smp, 4 * 64));
    net->nsmp_cap = 64;
  }
  KF_HIP(hipMemcpyAsync(net->smp, rep.data(), sizeof(double) * 4 * 64, hipMemcpyHostToDevice, net->st));
  KF_HIP(hipMemcpyAsync(net->Lover, &L, sizeof(int32_t), hipMemcpyHostToDevice, net->st));
  float jf = 0.f, jl = 0.f;
  std::vector<float> wl((size_t)kLM);
  // the acceptance gate: Fourier weights (network off), then the network's weights
  KF_TRY(fwd_bwd(net, 64, nullptr, false, false, net->Lover));
  KF_HIP(hipMemcpyAsync(&jf, net->J, sizeof(float), hipMemcpyDeviceToHost, net->st));
  KF_HIP(hipStreamSynchronize(net->st));
  KF_TRY(fwd_bwd(net, 64, nullptr, true, false, net->Lover));
  KF_HIP(hipMemcpyAsync(&jl, net->J, sizeof(float), hipMemcpyDeviceToHost, net->st));
  KF_HIP(hipMemcpyAsync(wl.data(), net->w, sizeof(float) * kLM, hipMemcpyDeviceToHost, net->st));
  KF_HIP(hipStreamSynchronize(net->st));
  if (j_learned) *j_learned = jl;
  if (j_fourier) *j_fourier = jf;
  if (std::isfinite(jl) && jl < jf) {
    *used_learned = 1;
    for (int l = 0; l < L; ++l) w_out[l] = wl[(size_t)l];
  } else {
    std::memcpy(w_out, wf.data(), sizeof(double) * L);
  }
  return KF_OK;
}

}  // extern "C"
