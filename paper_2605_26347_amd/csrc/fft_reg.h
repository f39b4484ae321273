// Register-resident FFT passes for CDNA (wave64) of the oversampled 2-D DFT F (Sect. 3.2,
// eq. 6), for lines of 64 to 16384 points.
//
// A length-N transform runs as three Stockham passes of radices R1, R2, R3
// (N = R1 R2 R3, each at most 32).  A thread holds E = N / NT elements and performs
// E / R butterflies per pass entirely in registers; between passes the data crosses
// LDS once.  The first pass reads its inputs straight from global memory (with the
// image-domain modulation fused in) and the last pass writes its outputs, which come
// out in natural order, straight to global memory.  Pass with radix R and sub-transform
// length Ns: butterfly j in [0, N/R) reads x[j + r N/R], multiplies input r by
// W_{Ns R}^{r (j mod Ns)}, does an R-point DFT and writes output r to
// ((j / Ns) Ns R + j mod Ns) + r Ns.
// The twiddles are laid out per pass, [r][j mod Ns] for the second pass and then for the
// third, so that neighbouring lanes read neighbouring values: by the index r (j mod Ns) N /
// (Ns R) of one table of N roots, a wavefront's load touched up to 60 lines.
// R-point DFTs of 16 and 32 points are Cooley-Tukey products of the 2/4/8-point ones
// with their inner twiddles as compile-time constants (cos and sin of k pi / 16 from
// their Taylor series, evaluated in double precision by the compiler).
#pragma once

#include <hip/hip_runtime.h>

#include "fft_lds.h"
#include "wf_internal.h"

namespace wf {

namespace twc {
constexpr double PI = 3.14159265358979323846264338327950288;
// sin and cos of x in [-pi, pi] from their Taylor series (terms to x^49: below 1e-17)
constexpr double tsin(double x) {
  double term = x, sum = x;
  for (int i = 1; i < 25; ++i) {
    term *= -x * x / ((2.0 * i) * (2.0 * i + 1.0));
    sum += term;
  }
  return sum;
}
constexpr double tcos(double x) {
  double term = 1.0, sum = 1.0;
  for (int i = 1; i < 25; ++i) {
    term *= -x * x / ((2.0 * i - 1.0) * (2.0 * i));
    sum += term;
  }
  return sum;
}
// angle 2 pi m / n reduced to [-pi, pi]
constexpr double ang(int m, int n) {
  const int r = ((m % n) + n) % n;
  const double a = 2.0 * PI * (double)r / (double)n;
  return a > PI ? a - 2.0 * PI : a;
}
}  // namespace twc

// exp(-2 pi i m / n) (forward) or its conjugate (inverse), rounded to FP32
template <int M, int N, bool INV>
struct Twiddle {
  static constexpr float c = (float)twc::tcos(twc::ang(M, N));
  static constexpr float s = (float)(INV ? twc::tsin(twc::ang(M, N)) : -twc::tsin(twc::ang(M, N)));
};

template <int M, int N, bool INV>
__device__ __forceinline__ float2 twiddle_const(float2 a) {
  if constexpr (((M % N) + N) % N == 0) {
    return a;
  } else if constexpr (4 * (((M % N) + N) % N) == N) {  // -i (forward) / +i (inverse)
    return rot90<INV>(a);
  } else if constexpr (2 * (((M % N) + N) % N) == N) {
    return make_float2(-a.x, -a.y);
  } else {
    constexpr float c = Twiddle<M, N, INV>::c, s = Twiddle<M, N, INV>::s;
    return make_float2(a.x * c - a.y * s, a.x * s + a.y * c);
  }
}

template <int R, bool INV>
__device__ __forceinline__ void dft_reg(float2* v);

// Cooley-Tukey R = A B: x[B n1 + n2] -> A-point DFTs over n1, twiddles W_R^{n2 k1},
// B-point DFTs over n2 -> X[k1 + A k2].
template <int A, int B, bool INV>
struct CT {
  template <int K1, int N2>
  static __device__ __forceinline__ void tw(float2 (&t)[A * B]) {
    t[K1 * B + N2] = twiddle_const<K1 * N2, A * B, INV>(t[K1 * B + N2]);
    if constexpr (N2 + 1 < B) {
      tw<K1, N2 + 1>(t);
    } else if constexpr (K1 + 1 < A) {
      tw<K1 + 1, 0>(t);
    }
  }
  static __device__ __forceinline__ void run(float2* v) {
    float2 t[A * B];
#pragma unroll
    for (int n2 = 0; n2 < B; ++n2) {
      float2 s[A];
#pragma unroll
      for (int n1 = 0; n1 < A; ++n1) s[n1] = v[B * n1 + n2];
      dft_reg<A, INV>(s);
#pragma unroll
      for (int k1 = 0; k1 < A; ++k1) t[k1 * B + n2] = s[k1];
    }
    tw<0, 0>(t);
#pragma unroll
    for (int k1 = 0; k1 < A; ++k1) {
      float2 s[B];
#pragma unroll
      for (int n2 = 0; n2 < B; ++n2) s[n2] = t[k1 * B + n2];
      dft_reg<B, INV>(s);
#pragma unroll
      for (int k2 = 0; k2 < B; ++k2) v[k1 + A * k2] = s[k2];
    }
  }
};

template <int R, bool INV>
__device__ __forceinline__ void dft_reg(float2* v) {
  if constexpr (R == 2) dft2<INV>(v);
  else if constexpr (R == 4) dft4<INV>(v);
  else if constexpr (R == 8) dft8<INV>(v);
  else if constexpr (R == 16) CT<4, 4, INV>::run(v);
  else CT<8, 4, INV>::run(v);
}

// The three radices of a length-N transform, its threads per line, and the lines that a
// workgroup of the row passes carries (one from 512 points on; shorter lines share a
// wavefront).
template <int N>
struct RowPlan {
  static constexpr int R1 = fft_r1(N), R2 = fft_r2(N);
  static constexpr int R3 = N / (R1 * R2);
  static constexpr int E = R1 > R2 ? (R1 > R3 ? R1 : R3) : (R2 > R3 ? R2 : R3);
  static constexpr int NT = N / E;
  static constexpr int LW = NT >= 64 ? 1 : 64 / NT;
  static constexpr int WG = NT * LW;
};

// 32-bit byte offset of a lane from a wave-uniform base: the constant part of an address
// then rides in the scalar base and the lanes share one offset register.
template <typename T>
__device__ __forceinline__ T ld_off(const void* base, uint32_t off) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + off);
}
template <typename T>
__device__ __forceinline__ void st_off(void* base, uint32_t off, T v) {
  *reinterpret_cast<T*>(reinterpret_cast<char*>(base) + off) = v;
}

// LDS slot of element idx: one element of padding after every 32, so that the strided
// writes of the first pass (stride R1 elements) spread over the banks.  The padding of a sum
// is the sum of the paddings when the low five bits do not carry, which holds for every
// (thread, element) pair of the exchanges below: slots are one register per access pattern
// plus a compile-time constant (an LDS instruction's immediate offset).
__host__ __device__ constexpr int lds_slot(int idx) { return idx + (idx >> 5); }
template <int N>
constexpr int lds_elems() {
  return N + N / 32;
}

// Cross-lane exchange through LDS in two halves, the real parts and then the imaginary
// parts, so that a line occupies N floats of LDS instead of N complex values.  out[k]
// goes to slot ob + oslot(k) and in[k] comes from slot ib + islot(k), oslot and islot being
// compile-time constants of k; the block's threads pass the four barriers together (the last
// one lets the next exchange reuse the buffer).
template <int KO, int KI, typename OS, typename IS>
__device__ __forceinline__ void xchg_split(float* buf, int ob, int ib, const float2 (&out)[KO],
                                           OS&& oslot, float2 (&in)[KI], IS&& islot) {
  float* wo = buf + ob;
  const float* ri = buf + ib;
#pragma unroll
  for (int k = 0; k < KO; ++k) wo[oslot(k)] = out[k].x;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < KI; ++k) in[k].x = ri[islot(k)];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < KO; ++k) wo[oslot(k)] = out[k].y;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < KI; ++k) in[k].y = ri[islot(k)];
  __syncthreads();
}

// The same exchange with complex values in one go (N complex values of LDS per line).
template <int KO, int KI, typename OS, typename IS>
__device__ __forceinline__ void xchg_full(float2* buf, int ob, int ib, const float2 (&out)[KO],
                                          OS&& oslot, float2 (&in)[KI], IS&& islot) {
#pragma unroll
  for (int k = 0; k < KO; ++k) buf[ob + oslot(k)] = out[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < KI; ++k) in[k] = buf[ib + islot(k)];
  __syncthreads();
}

// Whether a transform of length N exchanges its lines as floats (xchg_split): from 8192
// points on, where a complex line's LDS, not its registers, limits the lines per compute
// unit; shorter lines fit by registers already and would only pay the extra barriers.
template <int N>
constexpr bool line_split() {
  return N >= 8192;
}
// LDS of one line in bytes.
template <int N>
constexpr size_t line_lds_bytes() {
  return (size_t)lds_elems<N>() * (line_split<N>() ? sizeof(float) : sizeof(float2));
}

// The middle of a transform, the line crossing LDS twice (xchg_split or xchg_full as
// line_split says; buf is the line, in floats or complex values accordingly).  v1 holds
// the first pass's outputs of the thread's butterflies j = t + b NT (output r of
// butterfly j belongs at position j R1 + r); the second pass (radix R2, sub-transform
// length R1, twiddles from tw) runs in registers between the two exchanges; v3 receives
// the third pass's inputs x[j + r R1 R2].
template <int N, bool INV>
__device__ __forceinline__ void row_middle(void* buf, const float2 (&v1)[N / RowPlan<N>::NT],
                                           float2 (&v3)[N / RowPlan<N>::NT],
                                           const float2* __restrict__ tw, int t) {
  using RP = RowPlan<N>;
  constexpr int R1 = RP::R1, R2 = RP::R2, R3 = RP::R3, NT = RP::NT, E = N / NT;
  constexpr int B2 = (N / R2) / NT;
  static_assert(((N / R1) / NT) * R1 == E && B2 * R2 == E && ((N / R3) / NT) * R3 == E,
                "every pass holds E elements per thread");
  // no carry out of the low five bits: see lds_slot
  static_assert((NT * R1) % 32 == 0 && NT % R1 == 0 && 32 % R1 == 0, "write slots");
  static_assert(NT % 32 == 0 || (NT == 16 && (N / R2) % 16 == 0 && B2 <= 2), "read slots");
  float2 v2[E];
  const int kk = t & (R1 - 1);
  const int w1 = lds_slot(t * R1);             // writes of the first exchange: t R1 + ...
  const int w2 = lds_slot((t - kk) * R2) + kk;  // of the second: (t / R1) R1 R2 + kk + ...
  const int rd = lds_slot(t);                   // reads of both: t + ...
  auto xchg = [&](int ob, const float2(&o)[E], auto&& os, float2(&in)[E], auto&& is) {
    if constexpr (line_split<N>())
      xchg_split(reinterpret_cast<float*>(buf), ob, rd, o, os, in, is);
    else
      xchg_full(reinterpret_cast<float2*>(buf), ob, rd, o, os, in, is);
  };
  xchg(
      w1, v1, [](int k) { return lds_slot((k / R1) * NT * R1) + k % R1; }, v2,
      [](int k) { return lds_slot((k / R2) * NT + (k % R2) * (N / R2)); });
#pragma unroll
  for (int r = 1; r < R2; ++r) {
    // exp(-2 pi i r kk R3 / N): the same for all of the thread's butterflies (NT is a
    // multiple of R1)
    const float2 f = ld_off<float2>(tw + r * R1, (uint32_t)kk * 8);
#pragma unroll
    for (int b = 0; b < B2; ++b)
      v2[b * R2 + r] = INV ? cmulc(v2[b * R2 + r], f) : cmul(v2[b * R2 + r], f);
  }
#pragma unroll
  for (int b = 0; b < B2; ++b) dft_reg<R2, INV>(v2 + b * R2);
  xchg(
      w2, v2,
      [](int k) { return lds_slot((k / R2) * NT * R2) + lds_slot((k % R2) * R1); }, v3,
      [](int k) { return lds_slot((k / R3) * NT + (k % R3) * (R1 * R2)); });
}

// The last pass: butterflies j = t + b NT of radix R3 with twiddles exp(-2 pi i r j / N).
template <int N, bool INV>
__device__ __forceinline__ void last_twiddle(float2* v, const float2* __restrict__ tw, int b,
                                             int t) {
  constexpr int R1 = RowPlan<N>::R1, R2 = RowPlan<N>::R2, R3 = RowPlan<N>::R3;
  constexpr int NT = RowPlan<N>::NT;
#pragma unroll
  for (int r = 1; r < R3; ++r) {
    const float2 f = ld_off<float2>(tw + R1 * R2 + r * (R1 * R2) + b * NT, (uint32_t)t * 8);
    v[r] = INV ? cmulc(v[r], f) : cmul(v[r], f);
  }
}

}  // namespace wf
