// Row and column passes of F and F^dag with the image-domain work fused in
// (Sect. 3.2, eq. 6; Sect. 3.3, eq. 8):
//   forward rows : x (.) Z_p, zero-pad to Kx, FFT of the ny image rows      -> A
//   forward cols : zero-pad to Ky, FFT of every column                     -> X
//   inverse cols : inverse FFT of every column, keep the ny image rows     -> A
//                  (and clear Y behind the read, ready for the next gridding)
//   inverse rows : inverse FFT of the ny rows, crop to nx, (.) conj(Z_p),
//                  store or accumulate the sum over w-layers (eq. 7)
// Pruning to the bin's active uv support (the discrete Fourier modes its rows touch, plus
// a one-tile halo): the forward column pass writes X only inside needed tiles, the inverse
// column pass reads (and clears) Y only there, and both row passes touch only the column
// strips that hold needed tiles; everything else is known to be unused or zero.  Null
// masks mean the full grid.
// Z_p = grid correction x w-layer: s_i s_j exp(-2 pi i w_p (n-1)) / n with the phase
// computed in FP64 (n - 1 = -(l^2+m^2)/(1+n) avoids cancellation), reduced to
// [-1/2, 1/2) cycles in FP64 and only then rounded to FP32 for sincospi.
#include <mutex>
#include <vector>

#include "fft_lds.h"
#include "fft_reg.h"
#include "wf_internal.h"

namespace wf {

// n - 1 = sqrt(1 - r2) - 1 for r2 = l^2 + m^2 in FP64.  Inside r2 < 1/20 (fields up to
// about 25 degrees across) the binomial series of sqrt(1 - x) - 1 to x^12, whose
// coefficients are exact dyadic fractions, in Horner form: the next term is below 1e-17
// of the result, so it matches -r2 / (1 + sqrt(1 - r2)) to FP64 rounding, at a dozen
// fused multiply-adds instead of a square root and a division.
__device__ __forceinline__ double nm1_of(double r2) {
  if (r2 < 0.05) {
    double p = -29393.0 / 4194304.0;
    p = fma(p, r2, -4199.0 / 524288.0);
    p = fma(p, r2, -2431.0 / 262144.0);
    p = fma(p, r2, -715.0 / 65536.0);
    p = fma(p, r2, -429.0 / 32768.0);
    p = fma(p, r2, -33.0 / 2048.0);
    p = fma(p, r2, -21.0 / 1024.0);
    p = fma(p, r2, -7.0 / 256.0);
    p = fma(p, r2, -5.0 / 128.0);
    p = fma(p, r2, -1.0 / 16.0);
    p = fma(p, r2, -1.0 / 8.0);
    p = fma(p, r2, -0.5);
    return p * r2;
  }
  return -r2 / (1.0 + sqrt(1.0 - r2));
}

__device__ __forceinline__ float2 zvalue(int i, int j, int nx, int ny, double cell, double wp,
                                         float sxi, float syj) {
  const double l = (double)(i - nx / 2) * cell;
  const double m = (double)(j - ny / 2) * cell;
  const double r2 = l * l + m * m;
  const double d = nm1_of(r2);
  const double n = 1.0 + d;
  double cyc = -wp * d;
  cyc -= rint(cyc);
  float s, c;
  sincospif((float)(2.0 * cyc), &s, &c);
  const float a = sxi * syj / (float)n;
  return make_float2(a * c, a * s);
}

// Z_p = s(l) s(m) / n exp(-2 i pi w_p (n - 1)) split by n - 1 = -(l^2 + m^2)/2 + D(r2),
// r2 = l^2 + m^2, D = -r2^2/8 - r2^3/16 - 5 r2^4/128 - 7 r2^5/256 - ...:
//   Z_p = C_p(l) R_p(m) exp(i theta) / n,  C_p(l) = s(l) exp(i pi w_p l^2) (a per-bin table
//   of the image columns, FP64 phase at build), R_p(m) = s(m) exp(i pi w_p m^2) (FP64
//   phase once per row), theta = -2 pi w_p D(r2).
// Where r2 <= 1/100 over the image and |theta| <= 1/4 (the table exists only then), D and
// 1/n = 1 + r2/2 + 3 r2^2/8 + ... are FP32 series truncated below 1e-9 relative, and
// exp(i theta) its Taylor series to theta^7 (error below 1e-9): each factor carries an
// FP32 rounding error, a few 1e-7 in all, like the FP32 sine and cosine of the direct form.
struct ChirpRow {
  float2 R;      // s(m) exp(i pi w_p m^2)
  float m2;      // m^2
  float kth;     // -2 pi w_p
  float cellf;
  int hx;        // nx / 2
};

__device__ __forceinline__ ChirpRow chirp_row(int j, int nx, int ny, double cell, double wp,
                                              float syj) {
  ChirpRow c;
  const double m = (double)(j - ny / 2) * cell;
  double cyc = 0.5 * wp * (m * m);
  cyc -= rint(cyc);
  float sn, cs;
  sincospif((float)(2.0 * cyc), &sn, &cs);
  c.R = make_float2(syj * cs, syj * sn);
  c.m2 = (float)(m * m);
  c.kth = (float)(-2.0 * M_PI * wp);
  c.cellf = (float)cell;
  c.hx = nx / 2;
  return c;
}

__device__ __forceinline__ float2 zvalue_tab(const ChirpRow& c, int i, float2 ci) {
  const float li = (float)(i - c.hx) * c.cellf;
  const float r2 = fmaf(li, li, c.m2);
  const float dl = -(r2 * r2) * fmaf(r2, fmaf(r2, fmaf(r2, 7.f / 256.f, 5.f / 128.f),
                                               1.f / 16.f), 1.f / 8.f);
  const float th = c.kth * dl;
  const float t2 = th * th;
  const float ct = fmaf(t2, fmaf(t2, fmaf(t2, -1.f / 720.f, 1.f / 24.f), -0.5f), 1.f);
  const float st = th * fmaf(t2, fmaf(t2, fmaf(t2, -1.f / 5040.f, 1.f / 120.f), -1.f / 6.f),
                             1.f);
  const float inv_n =
      fmaf(r2, fmaf(r2, fmaf(r2, fmaf(r2, 35.f / 128.f, 5.f / 16.f), 3.f / 8.f), 0.5f), 1.f);
  const float2 a = make_float2(ci.x * ct - ci.y * st, ci.x * st + ci.y * ct);
  const float2 b = make_float2(a.x * c.R.x - a.y * c.R.y, a.x * c.R.y + a.y * c.R.x);
  return make_float2(b.x * inv_n, b.y * inv_n);
}

// C_p(l_i) = s(l_i) exp(i pi w_p l_i^2), i < nx: FP64 phase reduced to one cycle, FP64 sine
// and cosine.
__global__ __launch_bounds__(256) void k_chirp_table(float2* __restrict__ ct, int nx,
                                                     double cell, double wp,
                                                     const float* __restrict__ sx) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nx) return;
  const double l = (double)(i - nx / 2) * cell;
  double cyc = 0.5 * wp * (l * l);
  cyc -= rint(cyc);
  double sn, cs;
  sincospi(2.0 * cyc, &sn, &cs);
  ct[i] = make_float2((float)(sx[i] * cs), (float)(sx[i] * sn));
}

__device__ __forceinline__ bool bit_set(const uint32_t* __restrict__ m, int i) {
  return (m[i >> 5] >> (i & 31)) & 1u;
}

// Geometry of the pruning masks: tile bitmap [Ky/tile][Kx/tile] and strip bitmap
// [Kx/MSTRIP], both as packed 32-bit words.
struct Masks {
  const uint32_t* strip;  // null: all strips needed
  const uint32_t* tile;   // null: all tiles needed
  const int32_t* groups;  // null: column groups 0..n-1
  int tiles_x;
  int tsh;                // log2(tile)
};

// Threads of a workgroup of the LDS-resident passes (lines of 16 and 32 points).
constexpr int SHORT_THREADS = 64;

template <int N, int NT>
__global__ __launch_bounds__(NT) void k_fwd_rows(const float* __restrict__ img,
                                                 float2* __restrict__ A,
                                                 const float2* __restrict__ tw,
                                                 const float* __restrict__ sx,
                                                 const float* __restrict__ sy, int nx, int ny,
                                                 double cell, double wp,
                                                 const uint32_t* __restrict__ smask) {
  extern __shared__ float2 buf[];
  const int j = blockIdx.x;
  const float syj = sy[j];
  for (int t = threadIdx.x; t < N - nx; t += NT) buf[nx / 2 + t] = make_float2(0.f, 0.f);
  const float* row = img + (int64_t)j * nx;
  for (int i = threadIdx.x; i < nx; i += NT) {
    const float v = row[i];
    const float2 z = zvalue(i, j, nx, ny, cell, wp, sx[i], syj);
    buf[(i - nx / 2) & (N - 1)] = make_float2(v * z.x, v * z.y);
  }
  __syncthreads();
  fft_lines<N, NT, 1, false>(buf, N, tw);
  for (int q = threadIdx.x; q < N; q += NT)
    if (!smask || bit_set(smask, q >> 4)) A[half_index(j, q, ny)] = buf[q];
}

template <int N, int NT>
__global__ __launch_bounds__(NT) void k_inv_rows(const float2* __restrict__ A,
                                                 void* __restrict__ out,
                                                 const float2* __restrict__ tw,
                                                 const float* __restrict__ sx,
                                                 const float* __restrict__ sy, int nx, int ny,
                                                 double cell, double wp, int mode,
                                                 const uint32_t* __restrict__ smask) {
  extern __shared__ float2 buf[];
  const int j = blockIdx.x;
  for (int q = threadIdx.x; q < N; q += NT)
    buf[q] = (!smask || bit_set(smask, q >> 4)) ? A[half_index(j, q, ny)]
                                                : make_float2(0.f, 0.f);
  __syncthreads();
  fft_lines<N, NT, 1, true>(buf, N, tw);
  const float syj = sy[j];
  for (int i = threadIdx.x; i < nx; i += NT) {
    const float2 v = buf[(i - nx / 2) & (N - 1)];
    const float2 z = zvalue(i, j, nx, ny, cell, wp, sx[i], syj);
    const float2 r = cmulc(v, z);
    const int64_t o = (int64_t)j * nx + i;
    if (mode < 2) {
      float2* po = reinterpret_cast<float2*>(out) + o;
      if (mode == 1) {
        const float2 p = *po;
        *po = make_float2(p.x + r.x, p.y + r.y);
      } else {
        *po = r;
      }
    } else {
      float* po = reinterpret_cast<float*>(out) + o;
      *po = (mode == 3) ? (*po + r.x) : r.x;
    }
  }
}

// Row passes of lines of 64 points and more: three register-resident passes (fft_reg.h).
// They are bound by instruction issue and L1 accesses rather than by HBM (217 and 281 MB per
// pass at 8192 points, half of the columns needed: 45 and 59 us at the copy rate), so that
// what counts is instructions and lines per element: constant parts of addresses in scalar
// registers and immediate offsets, twiddles in reading order, padding terms dropped by the
// compiler, masks settled by scalar branches.  Forward / inverse pass at 8192 points 109 / 121
// us before, 90 / 96 us now; 16384 points forward 524 / 362; 4096 points 38 / 37 -> 29 / 27;
// 1024 points (LDS-resident stages before) 10.5 / 13.5 -> 7.5 / 7.1.
// Since N = 2 nx, input r of a first-pass butterfly holds an image pixel exactly when r <
// R1/4 (pixel q + nx/2) or r >= 3 R1/4 (pixel q - 3 nx/2), and output r of a last-pass
// butterfly lands inside the crop under the same rule with R3: the zero half of the padded
// row and the discarded half of the inverse are skipped at compile time.
// With a sweep's layer table sl, workgroup (row, layer) takes the layer's grid, mask and
// centroid from sl[blockIdx.y] and its channel's image from img (all channels' images).
//
// Pixel (or grid column) of element (b, r) relative to the thread: a compile-time constant.
template <int N, int R>
__device__ __forceinline__ constexpr int kept_pixel(int b, int r) {
  return b * RowPlan<N>::NT + r * (N / R) + (r < R / 4 ? N / 4 : -3 * (N / 4));
}
template <int R>
__device__ __forceinline__ constexpr bool kept(int r) {
  return r < R / 4 || r >= 3 * R / 4;
}

// Calls on(k) for each of the thread's elements k whose column t + col(k) lies in a needed
// strip.  A wavefront's 64 columns are four whole mask strips (lines of 512 points and more:
// col(k) is a multiple of 64), one nibble of one mask word, which a scalar load and a scalar
// branch settle for all lanes unless the support's edge lies inside.
template <int N, int K, typename COL, typename ON>
__device__ __forceinline__ void needed_columns(const uint32_t* __restrict__ smask, int t,
                                               COL&& col, ON&& on) {
  if (!smask) {
#pragma unroll
    for (int k = 0; k < K; ++k) on(k);
  } else if constexpr (RowPlan<N>::NT % 64 == 0) {
    const int s0 = __builtin_amdgcn_readfirstlane(t >> 4);
    const int sl = (t >> 4) & 3;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int s = s0 + col(k) / MSTRIP;
      const uint32_t f = (smask[s >> 5] >> (s & 31)) & 15u;
      if (f == 15u) {
        on(k);
      } else if (f != 0u) {
        if ((f >> sl) & 1u) on(k);
      }
    }
  } else {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int s = (t + col(k)) / MSTRIP;
      if ((smask[s >> 5] >> (s & 31)) & 1u) on(k);
    }
  }
}

template <int N>
__global__ __launch_bounds__(RowPlan<N>::WG) __attribute__((amdgpu_waves_per_eu(4))) void k_fwd_rows_reg(
    const float* __restrict__ img, float2* __restrict__ A, const float2* __restrict__ tw,
    const float* __restrict__ sx, const float* __restrict__ sy, int ny, double cell, double wp,
    const uint32_t* __restrict__ smask, const SweepLayer* __restrict__ sl,
    const float2* __restrict__ ctab) {
  using RP = RowPlan<N>;
  constexpr int R1 = RP::R1, R2 = RP::R2, R3 = RP::R3, NT = RP::NT, LW = RP::LW;
  constexpr int NX = N / 2, E = N / NT;
  extern __shared__ float2 buf[];
  const int l = LW == 1 ? 0 : threadIdx.x / NT, t = LW == 1 ? threadIdx.x : threadIdx.x % NT;
  const int j0 = blockIdx.x * LW, jr = j0 + l;
  if (sl) {
    const SweepLayer& L = sl[blockIdx.y];
    img += (int64_t)L.chan * NX * ny;
    A = L.A;
    wp = L.wp;
    smask = L.smask;
    ctab = L.ctab;
  }
  const float syj = sy[jr];
  const float* __restrict__ row = img + (int64_t)j0 * NX;
  const uint32_t toff = (uint32_t)(l * NX + t) * 4;
  float2 v1[E];
  {
    // the modulation of the lane's pixels, one uniform branch for the whole row (a
    // branch per pixel would keep the loads of different pixels from overlapping)
    constexpr int B = E / R1;
    float2 zr[B][R1 / 2];
    if (N >= SERIES_N && ctab) {
      const ChirpRow cr = chirp_row(jr, NX, ny, cell, wp, syj);
#pragma unroll
      for (int b = 0; b < B; ++b)
#pragma unroll
        for (int r = 0; r < R1; ++r)
          if (kept<R1>(r)) {
            const int c = kept_pixel<N, R1>(b, r);
            zr[b][r < R1 / 4 ? r : r - R1 / 2] =
                zvalue_tab(cr, t + c, ld_off<float2>(ctab + c, (uint32_t)t * 8));
          }
    } else {
#pragma unroll
      for (int b = 0; b < B; ++b)
#pragma unroll
        for (int r = 0; r < R1; ++r)
          if (kept<R1>(r)) {
            const int i = t + kept_pixel<N, R1>(b, r);
            zr[b][r < R1 / 4 ? r : r - R1 / 2] = zvalue(i, jr, NX, ny, cell, wp, sx[i], syj);
          }
    }
#pragma unroll
    for (int b = 0; b < B; ++b) {
      float2* v = v1 + b * R1;
#pragma unroll
      for (int r = 0; r < R1; ++r) {
        if (kept<R1>(r)) {
          const float x = ld_off<float>(row + kept_pixel<N, R1>(b, r), toff);
          const float2 z = zr[b][r < R1 / 4 ? r : r - R1 / 2];
          v[r] = make_float2(x * z.x, x * z.y);
        } else {
          v[r] = make_float2(0.f, 0.f);
        }
      }
      dft_reg<R1, false>(v);
    }
  }
  float2 v3[E];
  void* line = line_split<N>() ? (void*)(reinterpret_cast<float*>(buf) + l * lds_elems<N>())
                               : (void*)(buf + l * lds_elems<N>());
  row_middle<N, false>(line, v1, v3, tw, t);
  {
    constexpr int NS = R1 * R2;
    const uint32_t off = (uint32_t)half_index(l, t, ny) * 8;
    float2* __restrict__ arow = A + ((int64_t)j0 << HALF_L);
    auto col = [](int k) { return (k / R3) * NT + (k % R3) * NS; };
#pragma unroll
    for (int b = 0; b < E / R3; ++b) {
      last_twiddle<N, false>(v3 + b * R3, tw, b, t);
      dft_reg<R3, false>(v3 + b * R3);
    }
    needed_columns<N, E>(smask, t, col, [&](int k) {
      st_off(arow + (((int64_t)(col(k) >> HALF_L) * ny) << HALF_L), off, v3[k]);
    });
  }
}

// First pass of the inverse row transform: the needed columns of row j0 + l of A.
template <int N>
__device__ __forceinline__ void inv_rows_first(const float2* __restrict__ A,
                                               const uint32_t* __restrict__ smask, int ny,
                                               int j0, int l, int t,
                                               float2 (&v1)[N / RowPlan<N>::NT]) {
  constexpr int R1 = RowPlan<N>::R1, NT = RowPlan<N>::NT, E = N / NT;
  const uint32_t off = (uint32_t)half_index(l, t, ny) * 8;
  const float2* __restrict__ arow = A + ((int64_t)j0 << HALF_L);
  auto col = [](int k) { return (k / R1) * NT + (k % R1) * (N / R1); };
#pragma unroll
  for (int k = 0; k < E; ++k) v1[k] = make_float2(0.f, 0.f);
  needed_columns<N, E>(smask, t, col, [&](int k) {
    v1[k] = ld_off<float2>(arow + (((int64_t)(col(k) >> HALF_L) * ny) << HALF_L), off);
  });
#pragma unroll
  for (int b = 0; b < E / R1; ++b) dft_reg<R1, true>(v1 + b * R1);
}

template <int N>
__global__ __launch_bounds__(RowPlan<N>::WG) __attribute__((amdgpu_waves_per_eu(N >= 8192 ? 3 : 4))) void k_inv_rows_reg(
    const float2* __restrict__ A, void* __restrict__ out, const float2* __restrict__ tw,
    const float* __restrict__ sx, const float* __restrict__ sy, int ny, double cell, double wp,
    int mode, const uint32_t* __restrict__ smask, const float2* __restrict__ ctab) {
  using RP = RowPlan<N>;
  constexpr int R3 = RP::R3, NT = RP::NT, LW = RP::LW, NX = N / 2, E = N / NT;
  extern __shared__ float2 buf[];
  const int l = LW == 1 ? 0 : threadIdx.x / NT, t = LW == 1 ? threadIdx.x : threadIdx.x % NT;
  const int j0 = blockIdx.x * LW, jr = j0 + l;
  float2 v1[E], v3[E];
  inv_rows_first<N>(A, smask, ny, j0, l, t, v1);
  void* line = line_split<N>() ? (void*)(reinterpret_cast<float*>(buf) + l * lds_elems<N>())
                               : (void*)(buf + l * lds_elems<N>());
  row_middle<N, true>(line, v1, v3, tw, t);
  const float syj = sy[jr];
  const ChirpRow cr = chirp_row(jr, NX, ny, cell, wp, syj);
  const uint32_t pix = (uint32_t)(l * NX + t);   // the lane's pixel 0 from row j0 on
#pragma unroll
  for (int b = 0; b < E / R3; ++b) {
    // one group's modulations at a time (registers), one uniform branch per group
    float2 zr[R3 / 2];
    if (N >= SERIES_N && ctab) {
#pragma unroll
      for (int r = 0; r < R3; ++r)
        if (kept<R3>(r)) {
          const int c = kept_pixel<N, R3>(b, r);
          zr[r < R3 / 4 ? r : r - R3 / 2] =
              zvalue_tab(cr, t + c, ld_off<float2>(ctab + c, (uint32_t)t * 8));
        }
    } else {
#pragma unroll
      for (int r = 0; r < R3; ++r)
        if (kept<R3>(r)) {
          const int i = t + kept_pixel<N, R3>(b, r);
          zr[r < R3 / 4 ? r : r - R3 / 2] = zvalue(i, jr, NX, ny, cell, wp, sx[i], syj);
        }
    }
    // the previous image sum of the real-part accumulate mode, requested before this
    // group's transform so that its latency hides behind it (per group: registers)
    float prev[R3 / 2];
    if (mode == 3) {
      const float* row = reinterpret_cast<const float*>(out) + (int64_t)j0 * NX;
#pragma unroll
      for (int r = 0; r < R3; ++r)
        if (kept<R3>(r))
          prev[r < R3 / 4 ? r : r - R3 / 2] =
              ld_off<float>(row + kept_pixel<N, R3>(b, r), pix * 4);
    }
    float2* v = v3 + b * R3;
    last_twiddle<N, true>(v, tw, b, t);
    dft_reg<R3, true>(v);
#pragma unroll
    for (int r = 0; r < R3; ++r) {
      if (kept<R3>(r)) {
        const float2 c = cmulc(v[r], zr[r < R3 / 4 ? r : r - R3 / 2]);
        const int64_t o = (int64_t)j0 * NX + kept_pixel<N, R3>(b, r);
        if (mode < 2) {
          float2* row = reinterpret_cast<float2*>(out) + o;
          if (mode == 1) {
            const float2 p = ld_off<float2>(row, pix * 8);
            st_off(row, pix * 8, make_float2(p.x + c.x, p.y + c.y));
          } else {
            st_off(row, pix * 8, c);
          }
        } else {
          float* row = reinterpret_cast<float*>(out) + o;
          st_off(row, pix * 4, mode == 3 ? prev[r < R3 / 4 ? r : r - R3 / 2] + c.x : c.x);
        }
      }
    }
  }
}

// Inverse row pass of a sweep: workgroup (row jr, channel c = c0 + y) transforms row jr of every
// layer of channel c in turn (chan_layers[c] = first layer, count) and accumulates
// conj(Z_p) F^dag ... in registers, then writes the channel's image row once (complex, or
// its real part): the sum over w-layers (eq. 7) needs no read-modify-write and no
// atomics.  With stamps, the channel's last workgroup records the device clock.
template <int N>
__global__ __launch_bounds__(RowPlan<N>::NT) void k_inv_rows_sweep(
    const SweepLayer* __restrict__ sl, const int2* __restrict__ chan_layers, int c0,
    void* __restrict__ out, const float2* __restrict__ tw, const float* __restrict__ sx,
    const float* __restrict__ sy, int ny, double cell, int real_out,
    unsigned long long* __restrict__ stamps, int* __restrict__ done) {
  using RP = RowPlan<N>;
  constexpr int R3 = RP::R3, NT = RP::NT, NX = N / 2, E = N / NT;
  static_assert(RP::LW == 1, "one row per workgroup");
  constexpr int B3 = E / R3;
  extern __shared__ float2 buf[];
  const int t = threadIdx.x;
  const int jr = blockIdx.x, c = c0 + (int)blockIdx.y;
  const int2 cl = chan_layers[c];
  const float syj = sy[jr];
  float2 acc[B3][R3 / 2];
#pragma unroll
  for (int b = 0; b < B3; ++b)
#pragma unroll
    for (int r = 0; r < R3 / 2; ++r) acc[b][r] = make_float2(0.f, 0.f);
  for (int li = cl.x; li < cl.x + cl.y; ++li) {
    const SweepLayer& L = sl[li];
    float2 v1[E], v3[E];
    inv_rows_first<N>(L.A, L.smask, ny, jr, 0, t, v1);
    row_middle<N, true>(buf, v1, v3, tw, t);
#pragma unroll
    for (int b = 0; b < B3; ++b) {
      float2* v = v3 + b * R3;
      last_twiddle<N, true>(v, tw, b, t);
      dft_reg<R3, true>(v);
#pragma unroll
      for (int r = 0; r < R3; ++r) {
        if (kept<R3>(r)) {
          const int i = t + kept_pixel<N, R3>(b, r);
          const float2 z = zvalue(i, jr, NX, ny, cell, L.wp, sx[i], syj);
          const float2 m = cmulc(v[r], z);
          float2& a = acc[b][r < R3 / 4 ? r : r - R3 / 2];
          a = make_float2(a.x + m.x, a.y + m.y);
        }
      }
    }
  }
  const int64_t base = (int64_t)c * NX * ny + (int64_t)jr * NX;
#pragma unroll
  for (int b = 0; b < B3; ++b) {
#pragma unroll
    for (int r = 0; r < R3; ++r) {
      if (kept<R3>(r)) {
        const int i = t + kept_pixel<N, R3>(b, r);
        const float2 a = acc[b][r < R3 / 4 ? r : r - R3 / 2];
        if (real_out) reinterpret_cast<float*>(out)[base + i] = a.x;
        else reinterpret_cast<float2*>(out)[base + i] = a;
      }
    }
  }
  if (stamps) {
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0 && atomicAdd(done + c, 1) == (int)gridDim.x - 1) {
      stamps[c] = wall_clock64();
      atomicExch(done + c, 0);
    }
  }
}

// Column passes of 64 points and more, register-resident like the row passes: CW columns
// per workgroup (col_width_for), NT threads per column, interleaved so that the columns of
// one strip are read and written by neighbouring lanes.  Bound by the lines that their narrow
// accesses touch, then by HBM (at 4096 points the inverse pass moves 335 MB in 63 us).
// Forward / inverse at 8192 points 115 / 163 us before, 88 / 119 now; 4096 points 52 / 84 ->
// 48 / 63; 1024 points 24 / 25 -> 8 / 10 (64 workgroups of 16 columns before, 256 of 4 now).
// Since N = 2 ny, the zero half of
// each forward column and the discarded half of each inverse column follow the same
// compile-time rule as rows.
template <int N>
struct ColPlan {
  static constexpr int CW = col_width_for(N);
  static constexpr int NTC = RowPlan<N>::NT;   // threads per column
  static constexpr int NT = CW * NTC;
  // The CW columns of one grid row sit on neighbouring lanes.  An LDS access of 64 lanes
  // is served in halves of 32 lanes, i.e. 32 / CW consecutive elements of each of CW
  // lines: lines 32 / CW elements apart beyond their padded length (which is a multiple
  // of 32) put those CW runs on disjoint banks.
  static constexpr int LS = lds_elems<N>() + 32 / CW;
  static constexpr size_t line_bytes() {
    return (size_t)CW * LS * (line_split<N>() ? sizeof(float) : sizeof(float2));
  }
  // CW lines of LS complex values, or of LS floats where lines cross LDS in halves
  // (xchg_split, line_split), then the tile bits
  static size_t lds_bytes(int nbits) { return line_bytes() + 4 * (size_t)nbits; }
};

// Needed-tile bits of a column pass's elements: element (b, r) of thread t is grid row
// j + r S, j = t + b NTC < S = N / R, r < R <= 32.  Entry t0 = j >> tsh holds bit r for each r
// (the tile row of j + r S is that of (t0 << tsh) + r S: below a tile's side nothing carries),
// so that a butterfly reads one word.  Without a mask (tsh beyond the line) the one entry has
// every bit set.
template <int N, int R>
__host__ __device__ __forceinline__ int tile_bit_entries(int tsh) {
  const int n = (N / R) >> tsh;
  return n > 0 ? n : 1;
}
template <int N, int R>
__device__ __forceinline__ void load_tile_bits(uint32_t* bits, const Masks& mk, int ct,
                                               int nthreads) {
  const int n = tile_bit_entries<N, R>(mk.tsh);
  for (int t0 = threadIdx.x; t0 < n; t0 += nthreads) {
    uint32_t m = 0xffffffffu;
    if (mk.tile) {
      m = 0;
      for (int r = 0; r < R; ++r)
        m |= (uint32_t)bit_set(mk.tile, (((t0 << mk.tsh) + r * (N / R)) >> mk.tsh) * mk.tiles_x + ct)
             << r;
    }
    bits[t0] = m;
  }
}
// Calls on(r) for the elements r of a butterfly whose bit is set in need: by scalar branches
// where all lanes of the wavefront share the word (their rows lie in one row of tiles).
template <int R, typename ON>
__device__ __forceinline__ void needed_rows(uint32_t need, ON&& on) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane(need);
  if (__all(need == lo)) {
#pragma unroll
    for (int r = 0; r < R; ++r)
      if ((lo >> r) & 1u) on(r);
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r)
      if ((need >> r) & 1u) on(r);
  }
}

// Byte offset of row t of column q0 + c of an R-row grid from column q0's strip (CW columns
// never straddle a strip unless they are whole strips).
template <int L>
__device__ __forceinline__ uint32_t col_offset(int q0, int c, int t, int R) {
  return (uint32_t)strip_index<L>(t, (q0 & ((1 << L) - 1)) + c, R) * 8;
}
template <int L>
__device__ __forceinline__ int64_t col_base(int q0, int R) {
  return ((int64_t)(q0 >> L) * R) << L;
}

// With a sweep's layer table sl, workgroup i takes (layer, column group) pairs[i].
template <int N>
__global__ __launch_bounds__(ColPlan<N>::NT) __attribute__((amdgpu_waves_per_eu(4))) void k_fwd_cols_reg(const float2* __restrict__ A,
                                                                 float2* __restrict__ X,
                                                                 const float2* __restrict__ tw,
                                                                 Masks mk,
                                                                 const SweepLayer* __restrict__ sl,
                                                                 const int2* __restrict__ pairs) {
  using RP = RowPlan<N>;
  constexpr int R1 = RP::R1, R3 = RP::R3, NY = N / 2;
  constexpr int CW = ColPlan<N>::CW, NTC = ColPlan<N>::NTC, NT = ColPlan<N>::NT;
  constexpr int LS = ColPlan<N>::LS, E = N / NTC;
  extern __shared__ float2 buf[];
  uint32_t* omask = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(buf) +
                                                ColPlan<N>::line_bytes());
  const int gi = xcd_remap(blockIdx.x, gridDim.x);
  int g;
  if (sl) {
    const int2 pr = pairs[gi];
    const SweepLayer& L = sl[pr.x];
    A = L.A;
    X = L.X;
    mk.tile = L.tile;
    g = pr.y;
  } else {
    g = mk.groups ? mk.groups[gi] : gi;
  }
  const int q0 = g * CW;
  const int c = threadIdx.x % CW, t = threadIdx.x / CW;
  void* line = line_split<N>() ? (void*)(reinterpret_cast<float*>(buf) + c * LS)
                               : (void*)(buf + c * LS);
  // the bits are read after the exchanges' barriers only
  load_tile_bits<N, R3>(omask, mk, q0 >> mk.tsh, NT);
  const float2* __restrict__ src = A + col_base<HALF_L>(q0, NY);
  const uint32_t so = col_offset<HALF_L>(q0, c, t, NY);
  float2 v1[E];
#pragma unroll
  for (int b = 0; b < E / R1; ++b) {
    float2* v = v1 + b * R1;
#pragma unroll
    for (int r = 0; r < R1; ++r)
      v[r] = kept<R1>(r) ? ld_off<float2>(src + kept_pixel<N, R1>(b, r) * (1 << HALF_L), so)
                         : make_float2(0.f, 0.f);
    dft_reg<R1, false>(v);
  }
  float2 v3[E];
  row_middle<N, false>(line, v1, v3, tw, t);
  float2* __restrict__ dst = X + col_base<GRID_L>(q0, N);
  {
    // the lane's column and butterfly index are taken afresh from the thread index (the
    // empty asm hides that it is unchanged) rather than held through the exchanges
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int cl = tid % CW, tl = tid / CW;
    const uint32_t off = col_offset<GRID_L>(q0, cl, tl, N);
#pragma unroll
    for (int b = 0; b < E / R3; ++b) {
      float2* v = v3 + b * R3;
      last_twiddle<N, false>(v, tw, b, tl);
      dft_reg<R3, false>(v);
      needed_rows<R3>(omask[(tl + b * NTC) >> mk.tsh], [&](int r) {
        st_off(dst + ((b * NTC + r * (N / R3)) << GRID_L), off, v[r]);
      });
    }
  }
}

template <int N>
__global__ __launch_bounds__(ColPlan<N>::NT) __attribute__((amdgpu_waves_per_eu(4))) void k_inv_cols_reg(float2* __restrict__ Y,
                                                                 float2* __restrict__ A,
                                                                 const float2* __restrict__ tw,
                                                                 Masks mk,
                                                                 const SweepLayer* __restrict__ sl,
                                                                 const int2* __restrict__ pairs) {
  using RP = RowPlan<N>;
  constexpr int R1 = RP::R1, R3 = RP::R3, NY = N / 2;
  constexpr int CW = ColPlan<N>::CW, NTC = ColPlan<N>::NTC, NT = ColPlan<N>::NT;
  constexpr int LS = ColPlan<N>::LS, E = N / NTC;
  extern __shared__ float2 buf[];
  uint32_t* imask = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(buf) +
                                                ColPlan<N>::line_bytes());
  const int gi = xcd_remap(blockIdx.x, gridDim.x);
  int g;
  if (sl) {
    const int2 pr = pairs[gi];
    const SweepLayer& L = sl[pr.x];
    Y = L.Y;
    A = L.A;
    mk.tile = L.tile;
    g = pr.y;
  } else {
    g = mk.groups ? mk.groups[gi] : gi;
  }
  const int q0 = g * CW;
  const int c = threadIdx.x % CW, t = threadIdx.x / CW;
  void* line = line_split<N>() ? (void*)(reinterpret_cast<float*>(buf) + c * LS)
                               : (void*)(buf + c * LS);
  load_tile_bits<N, R1>(imask, mk, q0 >> mk.tsh, NT);
  __syncthreads();
  // Y is read only inside needed tiles and cleared there, ready for the next gridding;
  // elsewhere it is zero already
  float2* __restrict__ src = Y + col_base<GRID_L>(q0, N);
  const uint32_t so = col_offset<GRID_L>(q0, c, t, N);
  float2 v1[E];
#pragma unroll
  for (int k = 0; k < E; ++k) v1[k] = make_float2(0.f, 0.f);
#pragma unroll
  for (int b = 0; b < E / R1; ++b) {
    float2* v = v1 + b * R1;
    needed_rows<R1>(imask[(t + b * NTC) >> mk.tsh], [&](int r) {
      v[r] = ld_off<float2>(src + ((b * NTC + r * (N / R1)) << GRID_L), so);
    });
    dft_reg<R1, true>(v);
  }
  float2 v3[E];
  row_middle<N, true>(line, v1, v3, tw, t);
  float2* __restrict__ dst = A + col_base<HALF_L>(q0, NY);
  // the lane's column and butterfly index taken afresh (see the forward pass)
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int cl = tid % CW, tl = tid / CW;
  const uint32_t off = col_offset<HALF_L>(q0, cl, tl, NY);
#pragma unroll
  for (int b = 0; b < E / R3; ++b) {
    float2* v = v3 + b * R3;
    last_twiddle<N, true>(v, tw, b, tl);
    dft_reg<R3, true>(v);
#pragma unroll
    for (int r = 0; r < R3; ++r)
      if (kept<R3>(r)) st_off(dst + kept_pixel<N, R3>(b, r) * (1 << HALF_L), off, v[r]);
  }
  // the clearing comes last: between the loads it held them up, and before the exchanges its
  // addresses cost registers
  const uint32_t zo = col_offset<GRID_L>(q0, cl, tl, N);
#pragma unroll
  for (int b = 0; b < E / R1; ++b)
    needed_rows<R1>(imask[(tl + b * NTC) >> mk.tsh], [&](int r) {
      st_off(src + ((b * NTC + r * (N / R1)) << GRID_L), zo, make_float2(0.f, 0.f));
    });
}

// Column passes of 16 and 32 points: CW adjacent columns per workgroup, lines padded by one
// element in LDS so that the strip-order global accesses (column index fastest) hit
// distinct banks.
template <int N, int NT, int CW>
__global__ __launch_bounds__(NT) void k_fwd_cols(const float2* __restrict__ A,
                                                 float2* __restrict__ X,
                                                 const float2* __restrict__ tw, int ny,
                                                 Masks mk) {
  extern __shared__ float2 buf[];
  constexpr int S = N + 1;
  const int gi = xcd_remap(blockIdx.x, gridDim.x);
  const int g = mk.groups ? mk.groups[gi] : gi;
  const int q0 = g * CW;
  const int nz = N - ny;
  for (int t = threadIdx.x; t < CW * nz; t += NT) {
    const int c = t / nz, r = t - c * nz;
    buf[c * S + ny / 2 + r] = make_float2(0.f, 0.f);
  }
  for (int t = threadIdx.x; t < CW * ny; t += NT) {
    const int jr = t / CW, c = t - jr * CW;
    buf[c * S + ((jr - ny / 2) & (N - 1))] = A[half_index(jr, q0 + c, ny)];
  }
  __syncthreads();
  fft_lines<N, NT, CW, false>(buf, S, tw);
  for (int t = threadIdx.x; t < CW * N; t += NT) {
    const int qv = t / CW, c = t - qv * CW;
    if (!mk.tile || bit_set(mk.tile, (qv >> mk.tsh) * mk.tiles_x + ((q0 + c) >> mk.tsh)))
      X[grid_index(qv, q0 + c, N)] = buf[c * S + qv];
  }
}

template <int N, int NT, int CW>
__global__ __launch_bounds__(NT) void k_inv_cols(float2* __restrict__ Y, float2* __restrict__ A,
                                                 const float2* __restrict__ tw, int ny,
                                                 Masks mk) {
  extern __shared__ float2 buf[];
  constexpr int S = N + 1;
  const int gi = xcd_remap(blockIdx.x, gridDim.x);
  const int g = mk.groups ? mk.groups[gi] : gi;
  const int q0 = g * CW;
  for (int t = threadIdx.x; t < CW * N; t += NT) {
    const int qv = t / CW, c = t - qv * CW;
    float2* p = Y + grid_index(qv, q0 + c, N);
    if (!mk.tile || bit_set(mk.tile, (qv >> mk.tsh) * mk.tiles_x + ((q0 + c) >> mk.tsh))) {
      buf[c * S + qv] = *p;
      *p = make_float2(0.f, 0.f);
    } else {
      buf[c * S + qv] = make_float2(0.f, 0.f);
    }
  }
  __syncthreads();
  fft_lines<N, NT, CW, true>(buf, S, tw);
  for (int t = threadIdx.x; t < CW * ny; t += NT) {
    const int jr = t / CW, c = t - jr * CW;
    A[half_index(jr, q0 + c, ny)] = buf[c * S + ((jr - ny / 2) & (N - 1))];
  }
}

__global__ void k_strip_to_rowmajor(const float2* __restrict__ src, float2* __restrict__ dst,
                                    int R, int Q) {
  const int64_t n = (int64_t)R * Q;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int r = (int)(t / Q), q = (int)(t - (int64_t)r * Q);
    dst[t] = src[grid_index(r, q, R)];
  }
}

// ------------------------------------------------------------------ launchers

// Raise a kernel's dynamic LDS limit once per (kernel, device, size), so that launches
// issued later (also inside a stream capture) make no attribute call.
template <typename K>
static hipError_t set_lds(K kern, size_t bytes) {
  if (bytes <= 65536) return hipSuccess;
  struct Done {
    const void* k;
    int dev;
    size_t bytes;
  };
  static std::mutex mu;
  static std::vector<Done> done;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const void* k = reinterpret_cast<const void*>(kern);
  std::lock_guard<std::mutex> lock(mu);
  for (const Done& d : done)
    if (d.k == k && d.dev == dev && d.bytes >= bytes) return hipSuccess;
  e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e == hipSuccess) done.push_back(Done{k, dev, bytes});
  return e;
}

#define WF_FOR_SIZES(X) \
  X(64) X(128) X(256) X(512) X(1024) X(2048) X(4096) X(8192) X(16384)
#define WF_FOR_SHORT(X) X(16) X(32)

template <int N>
static constexpr size_t row_lds() {
  return RowPlan<N>::LW * line_lds_bytes<N>();
}

hipError_t launch_chirp_table(float2* ct, int nx, double cell, double wp, const float* sx,
                              hipStream_t s) {
  hipLaunchKernelGGL(k_chirp_table, dim3((nx + 255) / 256), dim3(256), 0, s, ct, nx, cell, wp,
                     sx);
  return hipGetLastError();
}

hipError_t launch_fwd_rows(const float* img, float2* A, const float2* tw, const float* sx,
                           const float* sy, int nx, int ny, int Kx, double cell, double wp,
                           const uint32_t* smask, const float2* ctab, hipStream_t s) {
  if (Kx != 2 * nx || ny % 8 != 0) return hipErrorInvalidValue;
  switch (Kx) {
#define C(N)                                                                              \
  case N: {                                                                               \
    hipError_t e = set_lds(k_fwd_rows_reg<N>, row_lds<N>());                              \
    if (e != hipSuccess) return e;                                                        \
    hipLaunchKernelGGL((k_fwd_rows_reg<N>), dim3(ny / RowPlan<N>::LW),                    \
                       dim3(RowPlan<N>::WG), row_lds<N>(), s, img, A, tw, sx, sy, ny,     \
                       cell, wp, smask, nullptr, ctab);                                   \
    return hipGetLastError();                                                             \
  }
    WF_FOR_SIZES(C)
#undef C
#define C(N)                                                                              \
  case N: {                                                                               \
    constexpr int NT = SHORT_THREADS;                                                     \
    hipLaunchKernelGGL((k_fwd_rows<N, NT>), dim3(ny), dim3(NT), N * sizeof(float2), s,    \
                       img, A, tw, sx, sy, nx, ny, cell, wp, smask);                      \
    return hipGetLastError();                                                             \
  }
    WF_FOR_SHORT(C)
#undef C
    default:
      return hipErrorInvalidValue;
  }
}

hipError_t launch_inv_rows(const float2* A, void* out, const float2* tw, const float* sx,
                           const float* sy, int nx, int ny, int Kx, double cell, double wp,
                           int mode, const uint32_t* smask, const float2* ctab,
                           hipStream_t s) {
  if (Kx != 2 * nx || ny % 8 != 0) return hipErrorInvalidValue;
  switch (Kx) {
#define C(N)                                                                              \
  case N: {                                                                               \
    hipError_t e = set_lds(k_inv_rows_reg<N>, row_lds<N>());                              \
    if (e != hipSuccess) return e;                                                        \
    hipLaunchKernelGGL((k_inv_rows_reg<N>), dim3(ny / RowPlan<N>::LW),                    \
                       dim3(RowPlan<N>::WG), row_lds<N>(), s, A, out, tw, sx, sy, ny,     \
                       cell, wp, mode, smask, ctab);                                      \
    return hipGetLastError();                                                             \
  }
    WF_FOR_SIZES(C)
#undef C
#define C(N)                                                                              \
  case N: {                                                                               \
    constexpr int NT = SHORT_THREADS;                                                     \
    hipLaunchKernelGGL((k_inv_rows<N, NT>), dim3(ny), dim3(NT), N * sizeof(float2), s, A, \
                       out, tw, sx, sy, nx, ny, cell, wp, mode, smask);                   \
    return hipGetLastError();                                                             \
  }
    WF_FOR_SHORT(C)
#undef C
    default:
      return hipErrorInvalidValue;
  }
}

// Masks and workgroup count of a column pass of CW columns per workgroup.
template <int CW>
static Masks col_masks(const ColPrune* pr, int Kx, int* ng) {
  Masks mk{nullptr, nullptr, nullptr, 1, 0};
  *ng = Kx / CW;
  if (pr) {
    mk = Masks{pr->strip, pr->tile, pr->groups, pr->tiles_x, pr->tsh};
    *ng = pr->ngroups;
  }
  if (!pr || !pr->tile) mk.tsh = 30;   // no mask: one row of tiles of any side
  return mk;
}

template <int N, bool INV>
static hipError_t launch_cols_reg(float2* in, float2* out, const float2* tw, int Kx,
                                  const ColPrune* pr, hipStream_t s) {
  using CP = ColPlan<N>;
  if (Kx % CP::CW != 0) return hipErrorInvalidValue;
  int ng;
  const Masks mk = col_masks<CP::CW>(pr, Kx, &ng);
  if (ng == 0) return hipSuccess;
  hipError_t e;
  if constexpr (INV) {
    const size_t lds = CP::lds_bytes(tile_bit_entries<N, RowPlan<N>::R1>(mk.tsh));
    e = set_lds(k_inv_cols_reg<N>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_inv_cols_reg<N>), dim3(ng), dim3(CP::NT), lds, s, in, out, tw, mk,
                       nullptr, nullptr);
  } else {
    const size_t lds = CP::lds_bytes(tile_bit_entries<N, RowPlan<N>::R3>(mk.tsh));
    e = set_lds(k_fwd_cols_reg<N>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_fwd_cols_reg<N>), dim3(ng), dim3(CP::NT), lds, s, (const float2*)in,
                       out, tw, mk, nullptr, nullptr);
  }
  return hipGetLastError();
}

hipError_t launch_fwd_cols(const float2* A, float2* X, const float2* tw, int ny, int Kx,
                           int Ky, const ColPrune* pr, hipStream_t s) {
  if (Ky != 2 * ny) return hipErrorInvalidValue;
  switch (Ky) {
#define C(N) \
  case N: return launch_cols_reg<N, false>(const_cast<float2*>(A), X, tw, Kx, pr, s);
    WF_FOR_SIZES(C)
#undef C
#define C(N)                                                                              \
  case N: {                                                                               \
    constexpr int CW = col_width_for(N), NT = SHORT_THREADS;                              \
    if (Kx % CW != 0) return hipErrorInvalidValue;                                        \
    int ng;                                                                               \
    const Masks mk = col_masks<CW>(pr, Kx, &ng);                                          \
    if (ng == 0) return hipSuccess;                                                       \
    hipLaunchKernelGGL((k_fwd_cols<N, NT, CW>), dim3(ng), dim3(NT),                       \
                       CW * (N + 1) * sizeof(float2), s, A, X, tw, ny, mk);               \
    return hipGetLastError();                                                             \
  }
    WF_FOR_SHORT(C)
#undef C
    default:
      return hipErrorInvalidValue;
  }
}

hipError_t launch_inv_cols(float2* Y, float2* A, const float2* tw, int ny, int Kx, int Ky,
                           const ColPrune* pr, hipStream_t s) {
  if (Ky != 2 * ny) return hipErrorInvalidValue;
  switch (Ky) {
#define C(N) \
  case N: return launch_cols_reg<N, true>(Y, A, tw, Kx, pr, s);
    WF_FOR_SIZES(C)
#undef C
#define C(N)                                                                              \
  case N: {                                                                               \
    constexpr int CW = col_width_for(N), NT = SHORT_THREADS;                              \
    if (Kx % CW != 0) return hipErrorInvalidValue;                                        \
    int ng;                                                                               \
    const Masks mk = col_masks<CW>(pr, Kx, &ng);                                          \
    if (ng == 0) return hipSuccess;                                                       \
    hipLaunchKernelGGL((k_inv_cols<N, NT, CW>), dim3(ng), dim3(NT),                       \
                       CW * (N + 1) * sizeof(float2), s, Y, A, tw, ny, mk);               \
    return hipGetLastError();                                                             \
  }
    WF_FOR_SHORT(C)
#undef C
    default:
      return hipErrorInvalidValue;
  }
}

hipError_t launch_strip_to_rowmajor(const float2* src, float2* dst, int R, int Q,
                                    hipStream_t s) {
  const int64_t n = (int64_t)R * Q;
  const int blocks = (int)((n + 255) / 256 > 65536 ? 65536 : (n + 255) / 256);
  hipLaunchKernelGGL(k_strip_to_rowmajor, dim3(blocks), dim3(256), 0, s, src, dst, R, Q);
  return hipGetLastError();
}

// ------------------------------------------------------------------ sweep stages
// One launch per stage over every layer of a sweep (grid sides 2048 .. 16384, Kx = 2 nx,
// Ky = 2 ny).  Layer tables and pairs are device arrays built by the host.

hipError_t launch_sweep_fwd_rows(const float* img, const SweepLayer* sl, int nlayers,
                                 const float2* tw, const float* sx, const float* sy, int nx,
                                 int ny, int Kx, double cell, hipStream_t s) {
  if (nlayers <= 0) return hipSuccess;
  if (Kx != 2 * nx) return hipErrorInvalidValue;
  switch (Kx) {
#define C(NN)                                                                               \
  case NN: {                                                                                \
    const size_t lds = line_lds_bytes<NN>();                                            \
    hipError_t e = set_lds(k_fwd_rows_reg<NN>, lds);                                        \
    if (e != hipSuccess) return e;                                                          \
    hipLaunchKernelGGL((k_fwd_rows_reg<NN>), dim3(ny, nlayers), dim3(RowPlan<NN>::NT), lds, \
                       s, img, nullptr, tw, sx, sy, ny, cell, 0.0, nullptr, sl, nullptr);   \
    return hipGetLastError();                                                               \
  }
    C(2048) C(4096) C(8192) C(16384)
#undef C
    default:
      return hipErrorInvalidValue;
  }
}

hipError_t launch_sweep_cols(bool inverse, const SweepLayer* sl, const int2* pairs, int npairs,
                             const float2* tw, int ny, int Ky, int tsh, int tiles_x,
                             hipStream_t s) {
  if (npairs <= 0) return hipSuccess;
  if (Ky != 2 * ny) return hipErrorInvalidValue;
  Masks mk{nullptr, nullptr, nullptr, tiles_x, tsh};
  switch (Ky) {
#define C(NN)                                                                                 \
  case NN: {                                                                                  \
    using CP = ColPlan<NN>;                                                                   \
    using RP = RowPlan<NN>;                                                                   \
    const size_t lds = CP::lds_bytes(inverse ? tile_bit_entries<NN, RP::R1>(tsh)              \
                                             : tile_bit_entries<NN, RP::R3>(tsh));            \
    hipError_t e;                                                                             \
    if (inverse) {                                                                            \
      e = set_lds(k_inv_cols_reg<NN>, lds);                                                   \
      if (e != hipSuccess) return e;                                                          \
      hipLaunchKernelGGL((k_inv_cols_reg<NN>), dim3(npairs), dim3(ColPlan<NN>::NT), lds, s,   \
                         nullptr, nullptr, tw, mk, sl, pairs);                                \
    } else {                                                                                  \
      e = set_lds(k_fwd_cols_reg<NN>, lds);                                                   \
      if (e != hipSuccess) return e;                                                          \
      hipLaunchKernelGGL((k_fwd_cols_reg<NN>), dim3(npairs), dim3(ColPlan<NN>::NT), lds, s,   \
                         nullptr, nullptr, tw, mk, sl, pairs);                                \
    }                                                                                         \
    return hipGetLastError();                                                                 \
  }
    C(2048) C(4096) C(8192) C(16384)
#undef C
    default:
      return hipErrorInvalidValue;
  }
}

hipError_t launch_sweep_inv_rows(const SweepLayer* sl, const int2* chan_layers, int c0,
                                 int nchan, void* out, bool real_out, const float2* tw,
                                 const float* sx,
                                 const float* sy, int nx, int ny, int Kx, double cell,
                                 unsigned long long* stamps, int* done, hipStream_t s) {
  if (nchan <= 0) return hipSuccess;
  if (Kx != 2 * nx) return hipErrorInvalidValue;
  switch (Kx) {
#define C(NN)                                                                                \
  case NN: {                                                                                 \
    const size_t lds = line_lds_bytes<NN>();                                            \
    hipError_t e = set_lds(k_inv_rows_sweep<NN>, lds);                                       \
    if (e != hipSuccess) return e;                                                           \
    hipLaunchKernelGGL((k_inv_rows_sweep<NN>), dim3(ny, nchan), dim3(RowPlan<NN>::NT), lds,  \
                       s, sl, chan_layers, c0, out, tw, sx, sy, ny, cell,                  \
                       real_out ? 1 : 0, stamps, done);                                      \
    return hipGetLastError();                                                                \
  }
    C(2048) C(4096) C(8192) C(16384)
#undef C
    default:
      return hipErrorInvalidValue;
  }
}

}  // namespace wf
