// Kernels of the residual-kernel network (not part of the paper): FP32 training on the
// matrix cores (GEMMs with fused bias / GELU epilogues, GELU backward, column sums,
// loss, Adam) and fused BF16 inference.
//
// GEMM tiles: each wavefront computes a 32 x 32 tile of C with v_mfma_f32_32x32x2f32
// (lane l supplies A[l % 32][l / 32] and B[l / 32][l % 32] of a 32 x 2 x 32 step;
// accumulator element i of lane l is C[8 (i / 4) + 4 (l / 32) + i % 4][l % 32]).
//
// Inference: one workgroup of eight wavefronts carries 64 rows through the whole network
// with the activations in LDS as BF16.  The first layer (5 inputs) runs in FP32 so that
// the inputs keep their precision; the hidden and output layers use
// v_mfma_f32_32x32x16_bf16 (lane l supplies A[l % 32][8 (l / 32) .. + 7] and
// B[8 (l / 32) .. + 7][l % 32]) with FP32 accumulation, weights read from a BF16
// copy in fragment order that stays resident in L2.  Plain BF16 operands leave a relative
// output error near 1e-3; the split form (hi + lo BF16 parts, three products per step) brings
// it to the FP32 level at three times the matrix-core work.
// 200,000 rows, split: matrix cores 156 us, VALU (GELU, splits) 150 us, LDS reads 104 us and
// the output's stores 53 us, which two workgroups per compute unit overlap in part: 451 us.
// Before, 679 us: four wavefronts with two column tiles each (two waves per SIMD), weights by
// columns (a fragment touched 32 lines), activations split and stored value by value.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "mlp_defs.h"
#include "wf_internal.h"

namespace wf {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float gelu(float z) {
  return 0.5f * z * (1.0f + erff(z * 0.7071067811865475f));
}
__device__ __forceinline__ float gelu_grad(float z) {
  return 0.5f * (1.0f + erff(z * 0.7071067811865475f)) +
         z * 0.3989422804014327f * __expf(-0.5f * z * z);
}

// Round-to-nearest-even FP32 -> BF16 bits (finite inputs).
__device__ __forceinline__ uint16_t to_bf16(float f) {
  const uint32_t b = __float_as_uint(f);
  return (uint16_t)((b + 0x7fffu + ((b >> 16) & 1u)) >> 16);
}

constexpr int GT = 32;   // C tile side of one wavefront
constexpr int GD = 8;    // K groups of 8 in flight per wavefront

// C[M x N] = op(A)[M x K] op(B)[K x N]; EPI 1: Z = acc + bias, C = gelu(Z);
// 2: C = acc + bias; 3: C += acc atomically; 4: C = acc gelu'(Z).  op(A) = A^T when TA (A
// stored [K x M]), likewise for B.
//
// The products of the network are short (K = 256, 450 or a batch) and what bounds them is
// the latency of their loads, not the matrix cores (0.54 GFLOP is 3.7 us at the card's FP32
// rate): so a wavefront owns a 32 x 32 tile and keeps GD groups of eight k in flight in
// registers, straight from global memory (the other tiles' waves on the compute unit share
// its lines through L1), with no LDS staging and no barrier.  Inside a group, half-wave h
// holds k = 4 h .. 4 h + 3 (the order of a sum over k is free), so that a K-contiguous
// operand is one 16-byte load where its rows are aligned (VA, VB).
//  EPI 1/2/4: a workgroup is 2 x 2 tiles (4096 x 256 x 256: 256 workgroups).
//  EPI 3 (weight gradients, K = batch): a workgroup is one tile, its four wavefronts take a
//  quarter of the K range [z kc, (z + 1) kc) each and meet in LDS, so that one add per
//  element and z reaches memory; the tiles of m = 0 also sum B's columns into db, 32 values
//  of a half-wave at a time (a single chain over its 128 was a third worse against 64 bits).
// Batch 4096, per product: 37 / 48 / 43 us (forward / input gradient / weight gradient,
// LDS-staged 64 x 64 tiles) before, 13 / 17 / 13 us now.
template <bool TA, bool TB, int EPI, bool VA, bool VB>
__global__ __launch_bounds__(256) void k_gemm(const float* __restrict__ A, int lda,
                                              const float* __restrict__ B, int ldb,
                                              float* __restrict__ C, int ldc,
                                              float* __restrict__ Z,
                                              const float* __restrict__ bias,
                                              float* __restrict__ db, int M, int N, int K,
                                              int kc) {
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr bool SPLIT = EPI == 3;
  const int m0 = SPLIT ? blockIdx.y * GT : (blockIdx.y * 2 + (wv >> 1)) * GT;
  const int n0 = SPLIT ? blockIdx.x * GT : (blockIdx.x * 2 + (wv & 1)) * GT;
  int kb = 0, ke = K;
  if constexpr (SPLIT) {
    const int z0 = blockIdx.z * kc, z1 = min(K, z0 + kc);
    const int kq = ((z1 - z0 + 3) / 4 + 7) / 8 * 8;
    kb = min(z1, z0 + wv * kq);
    ke = min(z1, kb + kq);
  }
  const int h4 = 4 * (lane >> 5);
  // rows and columns past the matrix read the last one; they are not written
  const int m = min(m0 + (lane & 31), M - 1), n = min(n0 + (lane & 31), N - 1);
  const float* __restrict__ pa = TA ? A + (int64_t)(kb + h4) * lda + m
                                    : A + (int64_t)m * lda + kb + h4;
  const float* __restrict__ pb = TB ? B + (int64_t)n * ldb + kb + h4
                                    : B + (int64_t)(kb + h4) * ldb + n;
  const int sa = TA ? lda : 1, sb = TB ? 1 : ldb;
  f32x16 acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
  float bsum = 0.f, btot = 0.f;
  const bool sum_b = SPLIT && blockIdx.y == 0;
  const int ng = (ke - kb) >> 3;
  auto load = [&](int g, float (&a)[4], float (&b)[4]) {
    if constexpr (VA) {
      const float4 t = *reinterpret_cast<const float4*>(pa + 8 * g);
      a[0] = t.x, a[1] = t.y, a[2] = t.z, a[3] = t.w;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = pa[(8 * g + i) * sa];
    }
    if constexpr (VB) {
      const float4 t = *reinterpret_cast<const float4*>(pb + 8 * g);
      b[0] = t.x, b[1] = t.y, b[2] = t.z, b[3] = t.w;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) b[i] = pb[(8 * g + i) * sb];
    }
  };
  auto step = [&](const float (&a)[4], const float (&b)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[i], acc, 0, 0, 0);
      if constexpr (SPLIT) bsum += b[i];
    }
  };
  if (ng > 0) {
    float a[GD][4], b[GD][4];
#pragma unroll
    for (int d = 0; d < GD; ++d) load(min(d, ng - 1), a[d], b[d]);
    for (int g = 0; g < ng; g += GD) {
#pragma unroll
      for (int d = 0; d < GD; ++d) {
        if (g + d < ng) step(a[d], b[d]);
        load(min(g + d + GD, ng - 1), a[d], b[d]);   // past the end: the last group again
      }
      if constexpr (SPLIT) {
        btot += bsum;
        bsum = 0.f;
      }
    }
  }
  if (kb + 8 * ng < ke) {
    float a[4], b[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool in = kb + 8 * ng + h4 + i < ke;
      a[i] = in ? pa[(8 * ng + i) * sa] : 0.f;
      b[i] = in ? pb[(8 * ng + i) * sb] : 0.f;
    }
    step(a, b);
  }
  const int col = n0 + (lane & 31);
  if constexpr (SPLIT) {
    __shared__ float part[3][16][64];
    __shared__ float bpart[4][64];
    if (wv > 0) {
#pragma unroll
      for (int i = 0; i < 16; ++i) part[wv - 1][i][lane] = acc[i];
    }
    bpart[wv][lane] = btot + bsum;
    __syncthreads();
    if (wv > 0) return;
    if (sum_b && lane < 32 && col < N) {
      float t = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) t += bpart[w][lane] + bpart[w][lane + 32];
      atomicAdd(&db[col], t);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i)
      acc[i] = (acc[i] + part[0][i][lane]) + (part[1][i][lane] + part[2][i][lane]);
  }
  if (col >= N) return;
  const float bb = (EPI == 1 || EPI == 2) ? bias[col] : 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int row = m0 + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3);
    if (row >= M) continue;
    const float v = acc[i] + bb;
    const int64_t o = (int64_t)row * ldc + col;
    if (EPI == 1) {
      Z[o] = v;
      C[o] = gelu(v);
    } else if (EPI == 3) {
      atomicAdd(&C[o], v);
    } else if (EPI == 4) {
      C[o] = v * gelu_grad(Z[o]);
    } else {
      C[o] = v;
    }
  }
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Loss of one batch, one wavefront per example: dP = 2 (P - T) / B on the kernel
// outputs, 2 (e - log10(max(r, 1e-8))) / B on the error output with r held constant;
// loss[0] += kernel loss, loss[1] += error-output loss.  A workgroup of 16 wavefronts adds
// its examples' terms in LDS and reaches the two sums once: they are one address each, and
// two atomics per example were serialised there (batch 4096: 109 us before, 9 us now).
constexpr int LOSS_WAVES = 16;
__global__ __launch_bounds__(64 * LOSS_WAVES) void k_loss(const float* __restrict__ P,
                                                          const float* __restrict__ T,
                                                          float* __restrict__ dP, int B,
                                                          float* __restrict__ loss) {
  __shared__ float part[2][LOSS_WAVES];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int b = blockIdx.x * LOSS_WAVES + wv;
  float lk = 0.f, le = 0.f;
  if (b < B) {
    const float* p = P + (int64_t)b * MLP_OUT;
    const float* t = T + (int64_t)b * MLP_KOUT;
    float* d = dP + (int64_t)b * MLP_OUT;
    const float inv = 2.0f / (float)B;
    float s = 0.f, st = 0.f;
    for (int j = lane; j < MLP_KOUT; j += 64) {
      const float e = p[j] - t[j];
      s += e * e;
      st += t[j] * t[j];
      d[j] = inv * e;
    }
    s = wave_sum(s);
    st = wave_sum(st);
    const float r = sqrtf(s) / fmaxf(sqrtf(st), 1e-30f);
    const float tgt = log10f(fmaxf(r, 1e-8f));
    const float e = p[MLP_KOUT] - tgt;
    if (lane == 0) d[MLP_KOUT] = inv * e;
    lk = s / (float)B;
    le = e * e / (float)B;
  }
  if (lane == 0) {
    part[0][wv] = lk;
    part[1][wv] = le;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < LOSS_WAVES; ++w) t += part[threadIdx.x][w];
    atomicAdd(&loss[threadIdx.x], t);
  }
}

__global__ __launch_bounds__(256) void k_adam(float* __restrict__ p, const float* __restrict__ g,
                                              float* __restrict__ m, float* __restrict__ v,
                                              int64_t n, float lr, float b1, float b2, float eps,
                                              float c1, float c2) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  }
}

// Minibatch gather of rows idx[0..B) of X [n x cx] and T [n x ct].
__global__ __launch_bounds__(256) void k_gather(const float* __restrict__ X, int cx,
                                                const float* __restrict__ T, int ct,
                                                const int32_t* __restrict__ idx, int B,
                                                float* __restrict__ xb, float* __restrict__ tb) {
  const int b = blockIdx.x;
  const int64_t r = idx[b];
  for (int j = threadIdx.x; j < cx; j += blockDim.x) xb[(int64_t)b * cx + j] = X[r * cx + j];
  for (int j = threadIdx.x; j < ct; j += blockDim.x) tb[(int64_t)b * ct + j] = T[r * ct + j];
}

__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

constexpr int64_t WT_HALF = 3LL * MLP_HID * MLP_HID + 512LL * MLP_HID;

// BF16 copies of the hidden and output weights in the order in which the inference's
// wavefronts read them: layer l = 1..4 starts at (l - 1) * 256 * 256 (the output layer padded
// to 512 columns of zeros); per column tile of 32 and step of 16 along k, the 64 lanes' eight
// values each (lane: column n % 32, k half (k % 16) / 8), so that a fragment is one contiguous
// kilobyte.  The second half holds the residuals w - bf16(w), also in BF16 (the low parts of
// the split operands).
__global__ __launch_bounds__(256) void k_prep_bf16(const float* __restrict__ params,
                                                   uint16_t* __restrict__ wt) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < WT_HALF;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int l = i < 3LL * MLP_HID * MLP_HID ? 1 + (int)(i / (MLP_HID * MLP_HID)) : 4;
    const int64_t base = (int64_t)(l - 1) * MLP_HID * MLP_HID;
    const int j = (int)(i - base);
    const int lane = (j >> 3) & 63, step = (j >> 9) & 15, tile = j >> 13;
    const int n = tile * 32 + (lane & 31), k = step * 16 + 8 * (lane >> 5) + (j & 7);
    const int fo = mlp_fan_out(l);
    const float w = n < fo ? params[mlp_w_offset(l) + (int64_t)k * fo + n] : 0.f;
    const uint16_t hi = to_bf16(w);
    wt[i] = hi;
    wt[WT_HALF + i] = to_bf16(w - from_bf16(hi));
  }
}

// Two FP32 values as a pair of BF16 (round to nearest even) and the pair of their residuals.
__device__ __forceinline__ void split2(float a, float b, uint32_t& hi, uint32_t& lo) {
  auto pack = [](float x, float y) {
    const bf16x2 h = __builtin_convertvector((f32x2){x, y}, bf16x2);
    uint32_t r;
    __builtin_memcpy(&r, &h, 4);
    return r;
  };
  hi = pack(a, b);
  lo = pack(a - __uint_as_float(hi << 16), b - __uint_as_float(hi & 0xffff0000u));
}

constexpr int IR = 64;               // rows per inference workgroup
constexpr int IW = 8;                // its wavefronts, one column tile of 32 each
constexpr int HS = MLP_HID + 8;      // LDS row stride (bf16 elements)

// SPLIT: every operand is carried as a high BF16 part and a BF16 residual, and each
// product as hi*hi + hi*lo + lo*hi (three BF16 matrix-core steps, FP32 accumulation):
// about 16 significant bits instead of 8.
// GELU for inference: z Phi(z) with erf from Abramowitz & Stegun 7.1.26 (absolute error
// below 1.5e-7, far under the BF16 products' rounding), branch-free: one reciprocal and
// one exponential instead of the library erf's two-range evaluation.
__device__ __forceinline__ float gelu_infer(float z) {
  const float x = fabsf(z) * 0.7071067811865475f;
  const float t = __builtin_amdgcn_rcpf(1.0f + 0.3275911f * x);
  float p = 1.061405429f;
  p = fmaf(p, t, -1.453152027f);
  p = fmaf(p, t, 1.421413741f);
  p = fmaf(p, t, -0.284496736f);
  p = fmaf(p, t, 0.254829592f);
  const float e = 1.0f - p * t * __expf(-x * x);   // erf(|z| / sqrt 2)
  return 0.5f * z * (1.0f + copysignf(e, z));
}

template <bool SPLIT>
__global__ __launch_bounds__(64 * IW, 4) void k_infer_bf16(const float* __restrict__ x, int64_t n,
                                                    const float* __restrict__ params,
                                                    const uint16_t* __restrict__ wt,
                                                    float* __restrict__ out) {
  __shared__ __attribute__((aligned(16))) uint16_t H[(SPLIT ? 2 : 1) * IR * HS];
  uint16_t* Hl = H + IR * HS;
  const int64_t r0 = (int64_t)blockIdx.x * IR;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  // layer 0 in FP32: a thread owns two adjacent hidden units for a share of the rows; the
  // tile's inputs are staged in LDS once (rows past n read as zero and are never written out)
  {
    __shared__ float xs[IR * MLP_IN];
    for (int i = tid; i < IR * MLP_IN; i += 64 * IW) {
      const int64_t row = r0 + i / MLP_IN;
      xs[i] = row < n ? x[r0 * MLP_IN + i] : 0.f;
    }
    const int u = 2 * (tid & 127);
    float2 w[MLP_IN];
#pragma unroll
    for (int i = 0; i < MLP_IN; ++i)
      w[i] = make_float2(params[(int64_t)i * MLP_HID + u], params[(int64_t)i * MLP_HID + u + 1]);
    const float b0 = params[mlp_b_offset(0) + u], b1 = params[mlp_b_offset(0) + u + 1];
    __syncthreads();
    constexpr int RS = IR / (IW / 2);   // rows of a thread
    const int ra = (tid >> 7) * RS;
#pragma unroll 4
    for (int r = ra; r < ra + RS; ++r) {
      float z0 = b0, z1 = b1;
#pragma unroll
      for (int i = 0; i < MLP_IN; ++i) {
        z0 += xs[r * MLP_IN + i] * w[i].x;
        z1 += xs[r * MLP_IN + i] * w[i].y;
      }
      uint32_t hi, lo;
      split2(gelu_infer(z0), gelu_infer(z1), hi, lo);
      *reinterpret_cast<uint32_t*>(&H[r * HS + u]) = hi;
      if (SPLIT) *reinterpret_cast<uint32_t*>(&Hl[r * HS + u]) = lo;
    }
  }
  __syncthreads();
  const int am = lane & 31, ak = 8 * (lane >> 5);
  // layers 1..4: a wavefront computes column tile t0 (32 columns) of all 64 rows:
  // acc[row half].  FEAT: the products are formed as weights^T times activations^T, so that
  // a lane holds one row and groups of four adjacent columns (packed stores of the next
  // layer's input); otherwise a lane holds one column (whole lines of the output).
  auto layer = [&](const uint16_t* W, int t0, auto feat, f32x16 (&acc)[2]) {
    constexpr bool FEAT = decltype(feat)::value;
    constexpr int STEPS = MLP_HID / 16;
    const uint16_t* __restrict__ w0 = W + t0 * STEPS * 64 * 8 + lane * 8;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[a][i] = 0.f;
    auto mm = [&](bf16x8 act, bf16x8 w, f32x16 c) {
      return FEAT ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, act, c, 0, 0, 0)
                  : __builtin_amdgcn_mfma_f32_32x32x16_bf16(act, w, c, 0, 0, 0);
    };
    // the weights (L2-resident) of step st + WD are requested before the products of step
    // st, so that their latency hides behind the matrix-core work
    constexpr int WD = 2;
    bf16x8 wh[WD + 1], wl[WD + 1];
    auto load_w = [&](int st, int slot) {
      wh[slot] = *reinterpret_cast<const bf16x8*>(w0 + st * 64 * 8);
      if (SPLIT) wl[slot] = *reinterpret_cast<const bf16x8*>(w0 + st * 64 * 8 + WT_HALF);
    };
#pragma unroll
    for (int d = 0; d < WD; ++d) load_w(d, d);
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
      if (st + WD < STEPS) load_w(st + WD, (st + WD) % (WD + 1));
      const int d = st % (WD + 1);
      bf16x8 fa[2], la[2];
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        const int o = (a * 32 + am) * HS + st * 16 + ak;
        fa[a] = *reinterpret_cast<const bf16x8*>(&H[o]);
        if (SPLIT) la[a] = *reinterpret_cast<const bf16x8*>(&Hl[o]);
      }
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        acc[a] = mm(fa[a], wh[d], acc[a]);
        if (SPLIT) {
          acc[a] = mm(fa[a], wl[d], acc[a]);
          acc[a] = mm(la[a], wh[d], acc[a]);
        }
      }
    }
  };
  for (int l = 1; l < MLP_LAYERS; ++l) {
    f32x16 acc[2];
    layer(wt + (int64_t)(l - 1) * MLP_HID * MLP_HID, wv, std::true_type{}, acc);
    __syncthreads();
    const float* bias = params + mlp_b_offset(l);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      // accumulator elements 4 g .. 4 g + 3 of a lane: adjacent columns of its row
      const int col = wv * 32 + 8 * g + 4 * (lane >> 5);
      float bb[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) bb[i] = bias[col + i];
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        uint2 hi, lo;
        split2(gelu_infer(acc[a][4 * g] + bb[0]), gelu_infer(acc[a][4 * g + 1] + bb[1]), hi.x,
               lo.x);
        split2(gelu_infer(acc[a][4 * g + 2] + bb[2]), gelu_infer(acc[a][4 * g + 3] + bb[3]),
               hi.y, lo.y);
        const int o = (a * 32 + am) * HS + col;
        *reinterpret_cast<uint2*>(&H[o]) = hi;
        if (SPLIT) *reinterpret_cast<uint2*>(&Hl[o]) = lo;
      }
    }
    __syncthreads();
  }
  // output layer in two halves of 256 columns (451 real), a tile of 32 per wavefront each
  const float* bias = params + mlp_b_offset(MLP_LAYERS);
  const bool whole = r0 + IR <= n;
  for (int h = 0; h < 2; ++h) {
    const int col = 256 * h + wv * 32 + am;
    if (256 * h + wv * 32 >= MLP_OUT) continue;
    f32x16 acc[2];
    layer(wt + 3LL * MLP_HID * MLP_HID, 8 * h + wv, std::false_type{}, acc);
    if (col >= MLP_OUT) continue;
    const float bb = bias[col];
    float* __restrict__ po = out + (r0 + 4 * (lane >> 5)) * MLP_OUT + col;
    const int left = (int)min((int64_t)IR, n - r0) - 4 * (lane >> 5);
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int r = a * 32 + 8 * (i >> 2) + (i & 3);
        if (whole || r < left) po[r * MLP_OUT] = acc[a][i] + bb;
      }
  }
}

unsigned grid_for(int64_t n, int64_t cap = 8192) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, cap));
}

}  // namespace

hipError_t launch_mlp_gemm(int epi, const float* A, int lda, const float* B, int ldb, float* C,
                           int ldc, float* Z, const float* bias, float* db, int M, int N, int K,
                           hipStream_t s) {
  // 16-byte loads along K where every row starts on such a boundary
  auto aligned = [](const float* p, int ld) {
    return ld % 4 == 0 && (reinterpret_cast<uintptr_t>(p) & 15) == 0;
  };
  const bool va = aligned(A, lda), vb = aligned(B, ldb);
  dim3 grid((N + 2 * GT - 1) / (2 * GT), (M + 2 * GT - 1) / (2 * GT), 1);
  int kc = K;
  if (epi == 3) {
    // small M x N, long K: layers of workgroups along K, each adding its share of every element
    // atomically.  Up to four while a wavefront's quarter stays at 64 and more (more layers cost
    // more in adds than they hide), and as many as hold it to 256 on larger batches: its
    // products are one chain of FP32 sums (batch 65536, worst weight gradient against 64 bits:
    // 1.7e-7 with 64 layers in 2294 us, 3.5e-7 with four in 2371 us).
    const int splits = std::max({1, std::min(4, K / 256), (K + 1023) / 1024});
    kc = ((K + splits - 1) / splits + 7) / 8 * 8;
    grid = dim3((N + GT - 1) / GT, (M + GT - 1) / GT, (K + kc - 1) / kc);
  }
#define G(TA, TB, E, VA, VB)                                                             \
  {                                                                                      \
    hipLaunchKernelGGL((k_gemm<TA, TB, E, VA, VB>), grid, dim3(256), 0, s, A, lda, B,    \
                       ldb, C, ldc, Z, bias, db, M, N, K, kc);                           \
    return hipGetLastError();                                                            \
  }
  switch (epi) {
    case 1:
      if (va) G(false, false, 1, true, false)
      G(false, false, 1, false, false)
    case 2:
      if (va) G(false, false, 2, true, false)
      G(false, false, 2, false, false)
    case 3: G(true, false, 3, false, false)
    case 4:
      if (va && vb) G(false, true, 4, true, true)
      G(false, true, 4, false, false)
    default: return hipErrorInvalidValue;
  }
#undef G
}

hipError_t launch_mlp_loss(const float* P, const float* T, float* dP, int B, float* loss,
                           hipStream_t s) {
  hipLaunchKernelGGL(k_loss, dim3((B + LOSS_WAVES - 1) / LOSS_WAVES), dim3(64 * LOSS_WAVES), 0, s,
                     P, T, dP, B, loss);
  return hipGetLastError();
}

hipError_t launch_mlp_adam(float* p, const float* g, float* m, float* v, int64_t n, float lr,
                           float b1, float b2, float eps, float c1, float c2, hipStream_t s) {
  hipLaunchKernelGGL(k_adam, dim3(grid_for(n)), dim3(256), 0, s, p, g, m, v, n, lr, b1, b2, eps,
                     c1, c2);
  return hipGetLastError();
}

hipError_t launch_mlp_gather(const float* X, int cx, const float* T, int ct,
                             const int32_t* idx, int B, float* xb, float* tb, hipStream_t s) {
  hipLaunchKernelGGL(k_gather, dim3(B), dim3(256), 0, s, X, cx, T, ct, idx, B, xb, tb);
  return hipGetLastError();
}

hipError_t launch_mlp_prep_bf16(const float* params, uint16_t* wt, hipStream_t s) {
  hipLaunchKernelGGL(k_prep_bf16, dim3(1024), dim3(256), 0, s, params, wt);
  return hipGetLastError();
}

hipError_t launch_mlp_infer_bf16(const float* x, int64_t n, const float* params,
                                 const uint16_t* wt, bool split, float* out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t nb = (n + IR - 1) / IR;
  if (split)
    hipLaunchKernelGGL(k_infer_bf16<true>, dim3((unsigned)nb), dim3(64 * IW), 0, s, x, n, params, wt,
                       out);
  else
    hipLaunchKernelGGL(k_infer_bf16<false>, dim3((unsigned)nb), dim3(64 * IW), 0, s, x, n, params,
                       wt, out);
  return hipGetLastError();
}

}  // namespace wf
