// Sparse products with the de-gridding matrix G_p (Sect. 3.2, eq. 6) and its adjoint
// (Sect. 3.3, eq. 8).
//
// Rows are sorted by (bin, grid tile, patch side, patch origin) and cut into work
// items that hold one patch-size class; a workgroup owns one work item and each of its
// wavefronts walks a contiguous segment of the item's rows.  The 64 lanes of a
// wavefront hold a row's T x T patch in MK slots each, slot k of lane l being tap
// t = l + 64 k of the row (patch row t / T, column t % T): a row's stored values are
// read as they lie in memory, one coalesced pass, with no per-row index arithmetic.
// The values are read through a buffer resource sized to the row, so that the slots
// past its T^2 taps read zero from the hardware's range check instead of being masked.
// Consecutive rows with the same patch origin and side form a "run" (visibilities
// falling in one grid cell).  Per run
//   * the grid values X of the run's patch are gathered once,
//   * conj(g_k) y_k is accumulated in registers over the run and added into the LDS
//     window of the tile (plus halo) once (wide patches: row by row),
// and the stored values of G are streamed from HBM exactly once.  A row's sum
// y_k = sum_t g_k[t] X[t] is reduced across the wavefront by a half swap and DPP, which
// leaves y_k wave-uniform.  At the end the
// window is added into Y with global atomics (untouched cells skipped).
//   fused G^dag G : gather + reduce + accumulate (Phi^dag Phi);
//   de-gridding   : gather + reduce, y written to the caller's visibility order (Phi);
//   gridding      : y read from the caller's order, accumulate (Phi^dag).
// Values are stored as complex FP32, FP16 or BF16; all arithmetic is FP32.
//
// Bound by instruction issue and latency, not by the G stream: dense rows (4096^2, 30M rows,
// FP16 fused) read G at 3.6 TB/s with the VALUs half busy, sparse rows (2048^2, 10 rows per
// item) at 0.9 TB/s, where an item's chain of loads and its accumulator's clearing and
// flushing are most of its time.  So a run's addresses are words formed once per patch side
// plus scalars, both sums of a row share one reduction, the accumulator is cleared behind the
// first loads, the flush goes by grid lines, and each class is held to the registers that let
// two or three workgroups share a compute unit (row_form).  Per w-layer, fused: 452 -> 365 us
// (dense), 326 -> 205 us (sparse, channels of 1 to 3M rows).
#include <hip/hip_fp16.h>

#include <algorithm>

#include "fft_lds.h"
#include "wf_internal.h"

namespace wf {

constexpr int GWAVES = 8;          // wavefronts per workgroup
constexpr int GNT = GWAVES * 64;

// Word 3 of a raw (untyped, unswizzled) buffer resource on CDNA: 32-bit data format,
// so that a load whose byte offset lies at or past the resource's size returns zero.
constexpr int RSRC_WORD3 = 0x00020000;

// Stored values are loaded in their raw form (two 32-bit words for FP32, one word
// holding two 16-bit halves otherwise) and widened to FP32 only where they are used,
// so that the loads of a row can all be in flight together.
template <int STORE>
struct RawT {
  using type = uint32_t;
};
template <>
struct RawT<WF_STORE_F32> {
  using type = uint2;
};

template <int STORE>
constexpr int value_bytes() {
  return STORE == WF_STORE_F32 ? 8 : 4;
}

template <int STORE>
__device__ __forceinline__ typename RawT<STORE>::type load_tap(__amdgpu_buffer_rsrc_t r,
                                                               int byte_off) {
  if constexpr (STORE == WF_STORE_F32) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, byte_off, 0, 0);
    return make_uint2(v[0], v[1]);
  } else {
    return __builtin_amdgcn_raw_buffer_load_b32(r, byte_off, 0, 0);
  }
}

template <int STORE>
__device__ __forceinline__ float2 widen(typename RawT<STORE>::type r) {
  if constexpr (STORE == WF_STORE_F32) {
    return make_float2(__uint_as_float(r.x), __uint_as_float(r.y));
  } else if constexpr (STORE == WF_STORE_F16) {
    __half2 h;
    __builtin_memcpy(&h, &r, 4);
    return __half22float2(h);
  } else {
    return make_float2(__uint_as_float(r << 16), __uint_as_float(r & 0xffff0000u));
  }
}

// Sums of x and of y over the wavefront, returned wave-uniform.  Swapping the upper half of
// x with the lower half of y leaves one register that holds x's partial sums in lanes 0..31
// and y's in lanes 32..63 after a single addition; DPP butterflies inside each row of 16
// lanes (quad xor 1, quad xor 2, half-row mirror, row mirror) leave every lane with its row's
// sum, and broadcasting lane 15 into row 1 (47 into row 3) leaves x's total in lane 31 and
// y's in lane 63: seven instructions for both (twelve for two separate reductions).
__device__ __forceinline__ void wave_sums_uniform(float x, float y, float& sx, float& sy) {
  const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false,
                                                  false);
  float v = __uint_as_float(p[0]) + __uint_as_float(p[1]);
  v += __builtin_amdgcn_update_dpp(0.f, v, 0xb1, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0.f, v, 0x4e, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0.f, v, 0x141, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0.f, v, 0x140, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0.f, v, 0x142, 0xa, 0xf, false);
  sx = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 31));
  sy = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// A row's word: window-local patch origin lu0 | lv0 << 8 | patch side T << 16.
struct Run {
  int T, TT, lu0, lv0;
};
__device__ __forceinline__ Run decode(uint32_t m) {
  Run r;
  r.lu0 = m & 0xff;
  r.lv0 = (m >> 8) & 0xff;
  r.T = (m >> 16) & 0xff;
  r.TT = r.T * r.T;
  return r;
}

// Patch coordinates (a = row, b = column) of tap t, invT ~ 1/T to within 2 ulp: exact for
// t < 2^13, T <= 64, since (t + 1/2)/T stays at least 1/(2T) away from an integer.
__device__ __forceinline__ void tap_ab(int t, int T, float invT, int& a, int& b) {
  a = (int)(((float)t + 0.5f) * invT);
  b = t - a * T;
}

// Buffer resource over the T^2 stored values of one row starting at value index vi.
template <int STORE>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const void* vals, int64_t vi,
                                                           int TT) {
  const char* p = reinterpret_cast<const char*>(vals) + vi * value_bytes<STORE>();
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(p), (short)0,
                                           TT * value_bytes<STORE>(), RSRC_WORD3);
}

// The work item's bounding box of patch cells in its window (packed by the host as
// origin u, origin v, width, height, 8 bits each).  The LDS accumulator holds exactly
// this box, as two planes of FP64 (real parts, then imaginary parts): LDS float atomics
// in FP64 issue an order of magnitude faster than in FP32 on CDNA4, and the wider sums
// cost no precision.  Only these cells are cleared and flushed.
struct Box {
  int u0, v0, w, h;
};
__device__ __forceinline__ Box box_of(int32_t packed) {
  const uint32_t b = (uint32_t)packed;
  return Box{(int)(b & 0xff), (int)((b >> 8) & 0xff), (int)((b >> 16) & 0xff), (int)(b >> 24)};
}

// Where the lane's taps of a T x T patch sit, one word per slot: byte offset of the cell in
// a plane of the box accumulator (16 bits: 36 rows of 101 cells at most), patch row a << 16,
// patch column b << 24.  It depends on T and the box alone, so it is formed when T changes
// (an item's rows are sorted by T) and a run only adds its origin.  Slots past the patch hold
// its last cell: they read X there (their stored value is zero) and never scatter.
template <int MK>
struct Slots {
  uint32_t w[MK];
  int T = 0;
  __device__ __forceinline__ void set(int side, int box_w, int lane) {
    if (side == T) return;
    T = side;
    const float invT = __builtin_amdgcn_rcpf((float)side);
    const int last = side * side - 1;
#pragma unroll
    for (int k = 0; k < MK; ++k) {
      int a, b;
      tap_ab(min(lane + 64 * k, last), side, invT, a, b);
      w[k] = (uint32_t)((a * box_w + b) * 8) | ((uint32_t)a << 16) | ((uint32_t)b << 24);
    }
  }
};

// Load the grid values of a run's patch (one per lane and slot).  Away from the grid's edge
// the patch's origin rides in a scalar base.
template <int MK>
__device__ __forceinline__ void load_patch_x(const Run& r, const Slots<MK>& sl, int u0, int v0,
                                             int Kx, int Ky, int ksh,
                                             const float2* __restrict__ X, float2 (&xr)[MK]) {
  constexpr uint32_t M = (1u << GRID_L) - 1;
  const int U = u0 + r.lu0, V = v0 + r.lv0;
  if (U >= 0 && V >= 0 && U + r.T <= Kx && V + r.T <= Ky) {
    const char* __restrict__ base =
        reinterpret_cast<const char*>(X + ((((int64_t)(U >> GRID_L) << ksh) + V) << GRID_L));
    const uint32_t f = (uint32_t)U & M;
#pragma unroll
    for (int k = 0; k < MK; ++k) {
      const uint32_t e = (sl.w[k] >> 24) + f, a = (sl.w[k] >> 16) & 0xffu;
      const uint32_t off =
          ((e >> GRID_L) << (ksh + GRID_L + 3)) + ((a << (GRID_L + 3)) + ((e & M) << 3));
      xr[k] = *reinterpret_cast<const float2*>(base + off);
    }
  } else {
#pragma unroll
    for (int k = 0; k < MK; ++k) {
      const int gu = (U + (int)(sl.w[k] >> 24)) & (Kx - 1);
      const int gv = (V + (int)((sl.w[k] >> 16) & 0xffu)) & (Ky - 1);
      xr[k] = X[grid_index(gv, gu, Ky)];
    }
  }
}

// Add a patch of values (value(k): slot k's) into the box accumulator (planes of plane bytes).
template <int MK, typename V>
__device__ __forceinline__ void scatter_patch(const Run& r, const Slots<MK>& sl, const Box& bx,
                                              int lane, V&& value, double* acc, int plane) {
  const int base = ((r.lv0 - bx.v0) * bx.w + (r.lu0 - bx.u0)) * 8;
  char* p = reinterpret_cast<char*>(acc);
#pragma unroll
  for (int k = 0; k < MK; ++k) {
    auto add = [&] {
      const int li = base + (int)(sl.w[k] & 0xffffu);
      const float2 v = value(k);
      atomicAdd(reinterpret_cast<double*>(p + li), (double)v.x);
      atomicAdd(reinterpret_cast<double*>(p + li + plane), (double)v.y);
    };
    // whole slots by scalar branches; the patch's last, partial one by lane
    if (64 * (k + 1) <= r.TT) add();
    else if (lane + 64 * k < r.TT) add();
  }
}

__device__ __forceinline__ void window_zero(double* acc, const Box& bx, int tid) {
  const int n = bx.w * bx.h;
  for (int c = tid; c < 2 * n; c += GNT) acc[c] = 0.0;
}

// Goes over the cells of a box line by line of the grid's layout: 32 lanes on the 32 floats of
// one 128-byte line (2^GRID_L columns x 2^(4 - GRID_L) rows of complex cells), lines first, first
// + step, ..., calling on(a, b, part, at) for cell (row a, column b) of the box, part 0 the real
// and 1 the imaginary float, at() its address.  An atomic costs by the 64-byte segments that it
// touches, so a line is sent whole: real parts and imaginary parts in instructions of their own
// touched every segment twice.
template <typename ON>
__device__ __forceinline__ void each_line(const Box& bx, int u0, int v0, int Kx, int Ky,
                                          float2* __restrict__ Y, int tid, int first, int step,
                                          ON&& on) {
  constexpr int L = GRID_L, H = 4 - GRID_L;
  const int ub = u0 + bx.u0, vb = v0 + bx.v0;          // grid origin of the box (unwrapped)
  const int fu = ub & ((1 << L) - 1), fv = vb & ((1 << H) - 1);
  const int nx = (fu + bx.w + (1 << L) - 1) >> L, ny = (fv + bx.h + (1 << H) - 1) >> H;
  const float inv = __builtin_amdgcn_rcpf((float)nx);
  const int part = tid & 1, cell = (tid >> 1) & 15;
  const int cu = (cell & ((1 << L) - 1)) - fu, cv = (cell >> L) - fv;
  float* __restrict__ Yp = reinterpret_cast<float*>(Y) + part;
  for (int c = first + (tid >> 5); c < nx * ny; c += step) {
    int ly, lx;
    tap_ab(c, nx, inv, ly, lx);
    const int a = (ly << H) + cv, b = (lx << L) + cu;
    if ((unsigned)a < (unsigned)bx.h && (unsigned)b < (unsigned)bx.w)
      on(a, b, part,
         [&] { return Yp + 2 * grid_index((vb + a) & (Ky - 1), (ub + b) & (Kx - 1), Ky); });
  }
}

// Add the box into Y (untouched cells skipped).
__device__ __forceinline__ void window_flush(const double* acc, const Box& bx, int u0, int v0,
                                             int Kx, int Ky, float2* __restrict__ Y, int tid) {
  const double* __restrict__ plane = acc + (tid & 1) * (bx.w * bx.h);
  each_line(bx, u0, v0, Kx, Ky, Y, tid, 0, GNT / 32, [&](int a, int b, int, auto&& at) {
    const float v = (float)plane[a * bx.w + b];
    if (v != 0.f) unsafeAtomicAdd(at(), v);
  });
}

// Store the box where the pieces of its item meet.
__device__ __forceinline__ void window_store(const double* acc, const Box& bx,
                                             double2* __restrict__ sums, int tid) {
  const int n = bx.w * bx.h;
  for (int c = tid; c < n; c += GNT) sums[c] = make_double2(acc[c], acc[n + c]);
}

// The cut items' sums into Y: a workgroup adds up the pieces of eight of an item's lines in
// FP64, a cell's values of MERGE_P pieces requested at once (their latency is what the pass
// costs), and adds each cell once.
constexpr int MERGE_LINES = 8, MERGE_P = 8;
__global__ __launch_bounds__(32 * MERGE_LINES) void k_merge(const CutItem* __restrict__ cuts,
                                                            const CutPart* __restrict__ parts,
                                                            const double2* __restrict__ sums,
                                                            float2* __restrict__ Y, int Kx,
                                                            int Ky) {
  const CutItem it = cuts[blockIdx.x];
  const Box bx = box_of(it.box);
  each_line(bx, it.u0, it.v0, Kx, Ky, Y, threadIdx.x, blockIdx.y * MERGE_LINES,
            gridDim.y * MERGE_LINES, [&](int a, int b, int part, auto&& at) {
              const double* __restrict__ src = reinterpret_cast<const double*>(sums) + part;
              double s = 0.0;
              for (int j0 = 0; j0 < it.nparts; j0 += MERGE_P) {
                double v[MERGE_P];
#pragma unroll
                for (int j = 0; j < MERGE_P; ++j) {
                  const CutPart p = parts[it.part0 + min(j0 + j, it.nparts - 1)];
                  const Box pb = box_of(p.box);
                  const int pa = a + bx.v0 - pb.v0, pu = b + bx.u0 - pb.u0;
                  v[j] = j0 + j < it.nparts && (unsigned)pa < (unsigned)pb.h &&
                                 (unsigned)pu < (unsigned)pb.w
                             ? src[2 * (int64_t)(p.slot + pa * pb.w + pu)]
                             : 0.0;
                }
#pragma unroll
                for (int j = 0; j < MERGE_P; ++j) s += v[j];
              }
              const float f = (float)s;
              if (f != 0.f) unsafeAtomicAdd(at(), f);
            });
}

// How a row kernel is held to the registers that let its workgroups (two wavefronts per SIMD
// each) share a compute unit: 64 registers for four, 80 for three, 128 for two, 256 for one.  A
// sparse row is a chain of loads, sums and LDS atomics that only other wavefronts hide.
//   direct: a row's products go straight into the box accumulator instead of a run
//           accumulator in registers (2 MK of them), and its buffer is loaded again only once
//           they have, which saves a copy of it (MK to 2 MK).
//   depth:  rows of values in flight.
//   waves:  wavefronts per SIMD that the compiler has to allow.
//   ahead:  the next run's grid values are gathered while the current run is reduced.
// Each form is the one with the most workgroups that needs no scratch memory (one that does
// runs two to three times slower), and among those the faster.  Fused, FP16, us per launch
// (2048^2 with four channels of 1 to 3M rows; 4096^2 with 30M rows), before with one workgroup
// (a run accumulator, the next run's grid values a run ahead) and now: MK 7 43 -> 38 and
// 94 -> 86, MK 12 69 -> 47 and 108 -> 76, MK 16 49 -> 33 and 72 -> 57, MK 22 120 -> 77 and
// 120 -> 96.  MK 12 keeps its run accumulator in FP16, where it fits: without it 83 for 76.
// Fused MK 22 of FP32 and BF16 needs 164 registers.  De-gridding MK 22 in FP32 fits 128 by its
// late loads, which cost more than the second workgroup gives (37 us for 33).
// The persistent kernels of a sweep need a few registers more for their queue, so three of FP16
// fused take one workgroup less than above (MK 4, 7) or no run accumulator (MK 12).  A sweep of
// four channels (2048^2, 8M rows; fused / de-gridding / gridding), with these forms but no
// bound on the registers and now: FP16 24.4 / 14.2 / 15.5 -> 20.8 / 13.6 / 15.5 ms, FP32 24.9 /
// 16.5 / 17.7 -> 23.3 / 15.9 / 17.1, BF16 23.3 / 14.5 / 15.7 -> 22.4 / 14.6 / 15.6.
struct RowForm {
  bool direct;
  int depth, waves;
  bool ahead = false;
};
constexpr RowForm row_form(int store, int mk, int mode, bool sweep = false) {
  const bool f16 = store == WF_STORE_F16, f32 = store == WF_STORE_F32;
  const bool thin = f16 || (!f32 && mode != 0);   // the classes below fit one workgroup more
  if (sweep && f16 && mode == 0 && mk > 2 && mk <= 12)
    return {mk == 12, mk == 4 ? 4 : 2, mk == 4 ? 6 : 4, mk != 12};
  if (mk <= 4) return {false, 4, f32 && mode == 0 ? 4 : !f32 && thin && mode != 2 ? 8 : 6, true};
  if (mk == 7) return {false, 2, thin ? 6 : 4};
  if (mk == 12) return {!f16, 2, 4};
  if (mk == 16) return {true, 1, 4};
  if (mode == 1 && f32) return {false, 1, 2};
  return {true, 1, f16 || mode == 2 ? 4 : 2};
}

// A table entry (an item, a sweep's layer) in scalar registers.  The tables do not change during
// a launch, but beside plain stores or a loop's atomics the compiler does not know that and loads
// them per lane, each time with a wait (the fused kernels 10% slower): so they are read as
// constant memory.
template <typename T>
__device__ __forceinline__ T read_entry(const T* p) {
  static_assert(sizeof(T) % 4 == 0 && alignof(T) >= 4, "whole words");
  const auto* w = (const __attribute__((address_space(4))) uint32_t*)(uintptr_t)p;
  uint32_t r[sizeof(T) / 4];
#pragma unroll
  for (size_t i = 0; i < sizeof(T) / 4; ++i) r[i] = w[i];
  T t;
  __builtin_memcpy(&t, r, sizeof(T));
  return t;
}

// One work item on one workgroup.  Its box is added into Y; that of a piece of a cut item (sums
// given, slot in wi.bin) is stored for k_merge.  MODE 0: fused G^dag G; 1: de-gridding; 2:
// gridding.
// Every thread passes the same two barriers (scattering modes), whatever its rows.
template <int STORE, int MK, int MODE, bool SWEEP>
__device__ __forceinline__ void row_item(const WorkItem wi, const uint32_t* __restrict__ meta,
                                         const uint32_t* __restrict__ voff,
                                         const int32_t* __restrict__ perm,
                                         const void* __restrict__ vals,
                                         const float2* __restrict__ X, float2* __restrict__ Y,
                                         float2* __restrict__ vis, int Kx, int Ky,
                                         double* acc, double2* __restrict__ sums, int tid) {
  constexpr bool GATHER = MODE != 2;
  constexpr bool SCATTER = MODE != 1;
  constexpr int VB = value_bytes<STORE>();
  const Box bx = box_of(wi.box);
  const int plane = bx.w * bx.h * 8;
  const int slot = sums ? wi.bin : -1;
  auto finish = [&] {
    if (slot >= 0)
      window_store(acc, bx, sums + slot, tid);
    else
      window_flush(acc, bx, wi.u0, wi.v0, Kx, Ky, Y, tid);
  };
  const int ksh = 31 - __builtin_clz(Ky);
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int seg = (wi.nrows + GWAVES - 1) / GWAVES;
  const int r0 = wave * seg;
  const int r1 = min(wi.nrows, r0 + seg);
  float2 xr[MK], ac[MK];
  Run rg{};
  uint32_t cur = 0xffffffffu;
  using Raw = typename RawT<STORE>::type;
  if (r0 >= r1) {
    if constexpr (SCATTER) {
      window_zero(acc, bx, tid);
      __syncthreads();
      __syncthreads();
      finish();
    }
    return;
  }
  // Software pipeline, D rows deep.  The metadata of the wavefront's whole segment (at
  // most 128 rows: items hold at most 1024 rows) sits in two VGPRs, lane i holding rows
  // r0 + i and r0 + 64 + i, and is read back with readlane, so the loop never waits on
  // the LDS/scalar counter that the window atomics use.  Value offsets are the running
  // sum of T^2 inside the item; the values of row r + D are requested (after a new run's
  // grid values) before row r is reduced.
  constexpr RowForm F = row_form(STORE, MK, MODE, SWEEP);
  constexpr int D = F.depth;
  constexpr bool PREFETCH = GATHER && F.ahead;
  const int nseg = r1 - r0;
  const uint32_t* __restrict__ mrow = meta + wi.row0 + r0;
  const uint32_t mv0 = mrow[min(lane, nseg - 1)];
  const uint32_t mv1 = mrow[min(64 + lane, nseg - 1)];
  auto meta_of = [&](int r) -> uint32_t {
    const int i = r - r0;
    return (uint32_t)__builtin_amdgcn_readlane((int)(i < 64 ? mv0 : mv1), i & 63);
  };
  // gridding: the segment's visibilities are fetched once, like its metadata (lane i
  // holds rows r0 + i and r0 + 64 + i), so that no row waits on its own y
  float2 yv0 = make_float2(0.f, 0.f), yv1 = make_float2(0.f, 0.f);
  if constexpr (MODE == 2) {
    yv0 = vis[perm[wi.row0 + r0 + min(lane, nseg - 1)]];
    yv1 = vis[perm[wi.row0 + r0 + min(64 + lane, nseg - 1)]];
  }
  Raw buf[D][MK];
  float2 xn[PREFETCH ? MK : 1];                       // grid values of the next run
  uint32_t nm = 0xffffffffu;                          // ... and its row word
  uint32_t mb[D];                                     // row words of the rows in flight
  int rp = r0;                                        // next row to request
  int64_t vbp = wi.voff + (int64_t)voff[wi.row0 + r0];  // its first value
  uint32_t mp = meta_of(r0);                          // its word
  auto request = [&](int d) {
    const int Tn = (int)((mp >> 16) & 0xff);
    const __amdgpu_buffer_rsrc_t rs = row_rsrc<STORE>(vals, vbp, Tn * Tn);
#pragma unroll
    for (int k = 0; k < MK; ++k) buf[d][k] = load_tap<STORE>(rs, (lane + 64 * k) * VB);
    mb[d] = mp;
    vbp += (int64_t)Tn * Tn;
    ++rp;
    mp = rp < r1 ? meta_of(rp) : 0u;
  };
#pragma unroll
  for (int d = 0; d < D; ++d) {
    mb[d] = 0u;
    if (rp < r1) request(d);
  }
  // the accumulator is cleared while the first rows' values are on their way
  if constexpr (SCATTER) {
    window_zero(acc, bx, tid);
    __syncthreads();
  }
  Slots<MK> sl;
  for (int rb = r0; rb < r1; rb += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int r = rb + d;
      if (r >= r1) break;
      const int row = wi.row0 + r;
      const uint32_t m = mb[d];
      Raw graw[F.direct ? 1 : MK];
      if constexpr (!F.direct) {
#pragma unroll
        for (int k = 0; k < MK; ++k) graw[k] = buf[d][k];
      }
      if (m != cur) {
        if constexpr (SCATTER) {
          if (!F.direct && cur != 0xffffffffu)
            scatter_patch<MK>(rg, sl, bx, lane, [&](int k) { return ac[k]; }, acc, plane);
        }
        cur = m;
        rg = decode(m);
        sl.set(rg.T, bx.w, lane);
        if constexpr (PREFETCH) {
          if (nm == m) {
#pragma unroll
            for (int k = 0; k < MK; ++k) xr[k] = xn[k];
          } else {
            load_patch_x<MK>(rg, sl, wi.u0, wi.v0, Kx, Ky, ksh, X, xr);
          }
          int q = r + 1;
          while (q < r1 && meta_of(q) == m) ++q;
          nm = 0xffffffffu;
          // one run ahead, where its patch has the same side (the slots' words)
          if (q < r1) {
            const uint32_t mq = meta_of(q);
            const Run rq = decode(mq);
            if (rq.T == rg.T) {
              nm = mq;
              load_patch_x<MK>(rq, sl, wi.u0, wi.v0, Kx, Ky, ksh, X, xn);
            }
          }
        } else if constexpr (GATHER) {
          load_patch_x<MK>(rg, sl, wi.u0, wi.v0, Kx, Ky, ksh, X, xr);
        }
#pragma unroll
        for (int k = 0; k < MK; ++k) ac[k] = make_float2(0.f, 0.f);
      }
      // row r + D (in-bounds: past a row's taps reads zero)
      if (!F.direct && rp < r1) request(d);
      float2 g[MK];
#pragma unroll
      for (int k = 0; k < MK; ++k)
        g[k] = widen<STORE>(F.direct ? buf[d][k] : graw[F.direct ? 0 : k]);
      float yx, yy;
      if constexpr (GATHER) {
        float sx = 0.f, sy = 0.f;
#pragma unroll
        for (int k = 0; k < MK; ++k) {  // y += g X, one fused multiply-add per term
          sx = fmaf(g[k].x, xr[k].x, sx);
          sx = fmaf(-g[k].y, xr[k].y, sx);
          sy = fmaf(g[k].x, xr[k].y, sy);
          sy = fmaf(g[k].y, xr[k].x, sy);
        }
        wave_sums_uniform(sx, sy, yx, yy);
        if constexpr (MODE == 1) {
          if (lane == 0) vis[perm[row]] = make_float2(yx, yy);
        }
      } else {
        const int i = r - r0;
        const float2 yv = i < 64 ? yv0 : yv1;
        yx = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(yv.x), i & 63));
        yy = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(yv.y), i & 63));
      }
      if constexpr (SCATTER && F.direct) {
        scatter_patch<MK>(rg, sl, bx, lane, [&](int k) {  // conj(g) y
          return make_float2(fmaf(g[k].y, yy, g[k].x * yx), fmaf(-g[k].y, yx, g[k].x * yy));
        }, acc, plane);
      } else if constexpr (SCATTER) {
#pragma unroll
        for (int k = 0; k < MK; ++k) {  // += conj(g) y
          ac[k].x = fmaf(g[k].x, yx, ac[k].x);
          ac[k].x = fmaf(g[k].y, yy, ac[k].x);
          ac[k].y = fmaf(g[k].x, yy, ac[k].y);
          ac[k].y = fmaf(-g[k].y, yx, ac[k].y);
        }
      }
      if (F.direct && rp < r1) request(d);
    }
  }
  if constexpr (SCATTER) {
    if (!F.direct && cur != 0xffffffffu)
      scatter_patch<MK>(rg, sl, bx, lane, [&](int k) { return ac[k]; }, acc, plane);
    __syncthreads();
    finish();
  }
}

// The classes that share a launch, from c0 on: those whose forms ask for the same number of
// wavefronts, except where four workgroups share a compute unit (4096^2 psf 16.21 -> 16.37 ms with
// those two merged).
constexpr int group_end(int store, int mode, int c0) {
  const int w = row_form(store, class_mk(c0), mode).waves;
  int c = c0 + 1;
  while (w < 8 && c < NCLS && row_form(store, class_mk(c), mode).waves == w) ++c;
  return c;
}

// Rows from which class 0 is launched apart from the group that it is part of (-1: never).  The
// group's kernel has the registers of its largest class, and class 0 compiled alone holds more
// workgroups (FP32 fused: 45 registers and four for 122 and two).  The lines lie where the
// launch costs less than that gives: 512^2, 4M rows of class 0, us an apply in the group and
// apart: FP32 fused 741 / 569 (300,000 rows 129 / 126, 100,000 75 / 80), de-gridding 800 / 727 (94
// / 89, 52 / 54), BF16 fused 519 / 450 (1.5M rows 243 / 237, 700,000 158 / 163), FP16 and BF16
// gridding 431 / 380 (1.5M rows 186 / 188).  FP32 gridding gains at no size, nor do the other
// classes that would hold more workgroups alone (1 and 4, and 3 of BF16, in gridding).
constexpr int64_t alone_rows(int store, int mode) {
  const bool f16 = store == WF_STORE_F16, f32 = store == WF_STORE_F32;
  if (mode == 0) return f32 ? 300'000 : f16 ? -1 : 1'200'000;
  if (mode == 1) return f32 ? 300'000 : -1;
  return f32 ? -1 : 2'000'000;
}

// One launch over the pieces of the classes [C0, C1), the widest patches first: the workgroups
// of one class run beside the last ones of another instead of behind them.  (All classes at 128
// registers in one launch, those that need fewer losing workgroups: 4096^2 psf 16.1 -> 17.5 ms.)
// Measured against a launch per class: 512^2 iteration (FP32, 460 pieces in all) 172 -> 142 us,
// 1024^2 adjoint 940 -> 881 us, 2048^2 wideband 16.82 -> 16.66 ms.
template <int STORE, int MODE, int C0, int C1>
__device__ __forceinline__ void row_block(int b, const RowPieces& pc,
                                          const uint32_t* __restrict__ meta,
                                          const uint32_t* __restrict__ voff,
                                          const int32_t* __restrict__ perm,
                                          const void* __restrict__ vals,
                                          const float2* __restrict__ X, float2* __restrict__ Y,
                                          float2* __restrict__ vis, int Kx, int Ky,
                                          double* acc) {
  if constexpr (C1 > C0) {
    constexpr int C = C1 - 1;
    if (b < pc.n[C])
      row_item<STORE, class_mk(C), MODE, false>(read_entry(pc.items + pc.first[C] + b), meta,
                                                voff, perm, vals, X, Y, vis, Kx, Ky, acc,
                                                pc.sums, (int)threadIdx.x);
    else
      row_block<STORE, MODE, C0, C>(b - pc.n[C], pc, meta, voff, perm, vals, X, Y, vis, Kx, Ky,
                                    acc);
  }
}

template <int STORE, int MODE, int C0, int C1>
__global__ __launch_bounds__(GNT)
__attribute__((amdgpu_waves_per_eu(row_form(STORE, class_mk(C0), MODE).waves))) void k_rows(
    RowPieces pc, const uint32_t* __restrict__ meta, const uint32_t* __restrict__ voff,
    const int32_t* __restrict__ perm, const void* __restrict__ vals,
    const float2* __restrict__ X, float2* __restrict__ Y, float2* __restrict__ vis, int Kx,
    int Ky) {
  extern __shared__ double acc[];
  // A class's pieces are ordered largest first and dealt round-robin over the XCDs by the
  // hardware, which spreads the dense uv core (many items) evenly and schedules longest first.
  row_block<STORE, MODE, C0, C1>(blockIdx.x, pc, meta, voff, perm, vals, X, Y, vis, Kx, Ky,
                                 acc);
}

// Persistent form over the items of every layer of a sweep (one patch class): resident
// workgroups take items from a queue (queue[0]) until it is drained; each item's layer
// (its bin field) selects its grids, its row data and its visibilities (vis_base plus
// the layer's offset).  The last workgroup to leave clears the queue and the exit count
// (queue[1]), so that the next launch, or the next replay of a captured graph, starts
// from zero without a separate clearing step.
template <int STORE, int MK, int MODE>
__global__ __launch_bounds__(GNT)
__attribute__((amdgpu_waves_per_eu(row_form(STORE, MK, MODE, true).waves))) void k_rows_sweep(
    const WorkItem* __restrict__ wis, int nitems, const SweepLayer* __restrict__ layers,
    float2* __restrict__ vis_base, int* __restrict__ queue, int Kx, int Ky) {
  extern __shared__ double acc[];
  __shared__ int slot;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // An item's words in scalar registers, except for 16-bit gridding of the two widest classes:
  // there the compiler's code is slower for it (FP16 MK 22 2.45 ms a sweep for 2.09).
  constexpr bool SCALAR = MODE != 2 || MK < 16 || STORE == WF_STORE_F32;
  // the thread's index, formed afresh for every item (the empty asm hides that it is unchanged):
  // it and what follows from it would otherwise be held in registers over the loop
  auto thread = [&] {
    if constexpr (!SCALAR) return (int)threadIdx.x;
    uint32_t none = 0;
    asm volatile("" : "+v"(none));
    const int t =
        64 * wave + (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, none));
    __builtin_assume(t >= 0 && t < GNT);
    return t;
  };
  for (;;) {
    if (thread() == 0) slot = atomicAdd(queue, 1);
    __syncthreads();
    int i = slot;
    if constexpr (SCALAR) i = __builtin_amdgcn_readfirstlane(i);
    __syncthreads();
    if (i >= nitems) break;
    const WorkItem wi = SCALAR ? read_entry(wis + i) : wis[i];
    const SweepLayer L = SCALAR ? read_entry(layers + wi.bin) : layers[wi.bin];
    row_item<STORE, MK, MODE, true>(wi, L.meta, L.voff, L.perm, L.vals, L.X, L.Y,
                              vis_base ? vis_base + L.vis_off : nullptr, Kx, Ky, acc,
                              nullptr, thread());
  }
  if (thread() == 0) {
    __threadfence();
    if (atomicAdd(queue + 1, 1) == (int)gridDim.x - 1) {
      atomicExch(queue, 0);
      atomicExch(queue + 1, 0);
    }
  }
}

// ------------------------------------------------------------------ launchers

template <typename K>
static hipError_t set_lds(K kern, size_t bytes) {
  if (bytes <= 65536) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// Largest (odd) patch side of a class of MK taps per lane.
constexpr int class_tmax(int mk) {
  int t = 1;
  while ((t + 2) * (t + 2) <= 64 * mk) t += 2;
  return t;
}

// Bytes of the box accumulator of a class's items: rows' cells lie in one tile and their
// patches of side <= class_tmax reach tile + side - 1 cells per axis; two FP64 planes.
constexpr size_t box_bytes(int mk, int mode, int tile) {
  const size_t side = (size_t)tile + class_tmax(mk) - 1;
  return mode == 1 ? 0 : side * side * 2 * sizeof(double);
}

// One launch over the classes [C0, C1).
template <int STORE, int MODE, int C0, int C1>
static hipError_t launch_classes(const RowPieces& pc, const uint32_t* meta, const uint32_t* voff,
                                 const int32_t* perm, const void* vals, const float2* X,
                                 float2* Y, float2* vis, int Kx, int Ky, int tile,
                                 hipStream_t s) {
  int blocks = 0;
  size_t lds = 0;
  for (int c = C0; c < C1; ++c) {
    blocks += pc.n[c];
    if (pc.n[c] > 0) lds = box_bytes(class_mk(c), MODE, tile);
  }
  if (blocks == 0) return hipSuccess;
  hipError_t e = set_lds(k_rows<STORE, MODE, C0, C1>, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_rows<STORE, MODE, C0, C1>), dim3(blocks), dim3(GNT), lds, s, pc, meta,
                     voff, perm, vals, X, Y, vis, Kx, Ky);
  return hipGetLastError();
}

template <int STORE, int MODE, int C0 = 0>
static hipError_t launch_groups(RowPieces pc, const uint32_t* meta, const uint32_t* voff,
                                const int32_t* perm, const void* vals, const float2* X,
                                float2* Y, float2* vis, int Kx, int Ky, int tile,
                                hipStream_t s) {
  if constexpr (C0 < NCLS) {
    constexpr int C1 = group_end(STORE, MODE, C0);
    hipError_t e;
    if constexpr (C0 == 0 && alone_rows(STORE, MODE) >= 0) {
      if (pc.rows0 >= alone_rows(STORE, MODE)) {
        e = launch_classes<STORE, MODE, 0, 1>(pc, meta, voff, perm, vals, X, Y, vis, Kx, Ky, tile,
                                              s);
        if (e != hipSuccess) return e;
        pc.n[0] = 0;
      }
    }
    e = launch_classes<STORE, MODE, C0, C1>(pc, meta, voff, perm, vals, X, Y, vis, Kx, Ky, tile,
                                            s);
    if (e != hipSuccess) return e;
    return launch_groups<STORE, MODE, C1>(pc, meta, voff, perm, vals, X, Y, vis, Kx, Ky, tile,
                                          s);
  }
  return hipSuccess;
}

template <int MODE>
static hipError_t launch_mode(const RowPieces& pc, const uint32_t* meta, const uint32_t* voff,
                              const int32_t* perm, const void* vals, wf_store store,
                              const float2* X, float2* Y, float2* vis, int Kx, int Ky, int tile,
                              hipStream_t s) {
  hipError_t e;
  switch (store) {
    case WF_STORE_F32:
      e = launch_groups<WF_STORE_F32, MODE>(pc, meta, voff, perm, vals, X, Y, vis, Kx, Ky, tile,
                                            s);
      break;
    case WF_STORE_F16:
      e = launch_groups<WF_STORE_F16, MODE>(pc, meta, voff, perm, vals, X, Y, vis, Kx, Ky, tile,
                                            s);
      break;
    default:
      e = launch_groups<WF_STORE_BF16, MODE>(pc, meta, voff, perm, vals, X, Y, vis, Kx, Ky, tile,
                                             s);
      break;
  }
  if (e != hipSuccess || MODE == 1 || pc.ncuts == 0) return e;
  hipLaunchKernelGGL(k_merge, dim3(pc.ncuts, (pc.cut_lines + MERGE_LINES - 1) / MERGE_LINES),
                     dim3(32 * MERGE_LINES), 0, s, pc.cuts, pc.parts, pc.sums, Y, Kx, Ky);
  return hipGetLastError();
}

template <int STORE, int MK, int MODE>
static hipError_t launch_sweep_one(const WorkItem* wi, int nwi, const SweepLayer* layers,
                                   float2* vis_base, int* queue, int Kx, int Ky, int tile,
                                   int grid_cap, hipStream_t s) {
  const size_t lds = box_bytes(MK, MODE, tile);
  hipError_t e = set_lds(k_rows_sweep<STORE, MK, MODE>, lds);
  if (e != hipSuccess) return e;
  // resident workgroups only: as many as the device holds at once, capped by the items
  int per_cu = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_rows_sweep<STORE, MK, MODE>,
                                                   GNT, lds);
  if (e != hipSuccess) return e;
  const int grid = std::max(1, std::min(nwi, std::max(1, per_cu) * grid_cap));
  hipLaunchKernelGGL((k_rows_sweep<STORE, MK, MODE>), dim3(grid), dim3(GNT), lds, s, wi, nwi,
                     layers, vis_base, queue, Kx, Ky);
  return hipGetLastError();
}

template <int MODE>
static hipError_t launch_sweep_mode(int cls, const WorkItem* wi, int nwi,
                                    const SweepLayer* layers, wf_store store, float2* vis_base,
                                    int* queue, int Kx, int Ky, int tile, int ncu,
                                    hipStream_t s) {
  if (nwi <= 0) return hipSuccess;
#define WF_SW(ST, MK) \
  launch_sweep_one<ST, MK, MODE>(wi, nwi, layers, vis_base, queue, Kx, Ky, tile, ncu, s)
#define WF_SWC(ST)                 \
  switch (cls) {                   \
    case 0: return WF_SW(ST, 2);   \
    case 1: return WF_SW(ST, 4);   \
    case 2: return WF_SW(ST, 7);   \
    case 3: return WF_SW(ST, 12);  \
    case 4: return WF_SW(ST, 16);  \
    default: return WF_SW(ST, 22); \
  }
  switch (store) {
    case WF_STORE_F32: WF_SWC(WF_STORE_F32)
    case WF_STORE_F16: WF_SWC(WF_STORE_F16)
    default: WF_SWC(WF_STORE_BF16)
  }
#undef WF_SWC
#undef WF_SW
}

hipError_t launch_rows_sweep(int mode, int cls, const WorkItem* wi, int nwi,
                             const SweepLayer* layers, wf_store store, float2* vis_base,
                             int* queue, int Kx, int Ky, int tile, int ncu, hipStream_t s) {
  switch (mode) {
    case 0: return launch_sweep_mode<0>(cls, wi, nwi, layers, store, vis_base, queue, Kx, Ky,
                                        tile, ncu, s);
    case 1: return launch_sweep_mode<1>(cls, wi, nwi, layers, store, vis_base, queue, Kx, Ky,
                                        tile, ncu, s);
    default: return launch_sweep_mode<2>(cls, wi, nwi, layers, store, vis_base, queue, Kx, Ky,
                                         tile, ncu, s);
  }
}

hipError_t launch_gtg(const RowPieces& pc, const uint32_t* meta, const uint32_t* voff,
                      const void* vals, wf_store store, const float2* X, float2* Y, int Kx,
                      int Ky, int tile, hipStream_t s) {
  return launch_mode<0>(pc, meta, voff, nullptr, vals, store, X, Y, nullptr, Kx, Ky, tile, s);
}

hipError_t launch_degrid(const RowPieces& pc, const uint32_t* meta, const uint32_t* voff,
                         const int32_t* perm, const void* vals, wf_store store, const float2* X,
                         float2* vis, int Kx, int Ky, hipStream_t s) {
  return launch_mode<1>(pc, meta, voff, perm, vals, store, X, nullptr, vis, Kx, Ky, 0, s);
}

hipError_t launch_grid(const RowPieces& pc, const uint32_t* meta, const uint32_t* voff,
                       const int32_t* perm, const void* vals, wf_store store, const float2* vis,
                       float2* Y, int Kx, int Ky, int tile, hipStream_t s) {
  return launch_mode<2>(pc, meta, voff, perm, vals, store, nullptr, Y,
                        const_cast<float2*>(vis), Kx, Ky, tile, s);
}

}  // namespace wf
