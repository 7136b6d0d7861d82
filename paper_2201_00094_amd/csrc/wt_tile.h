// Device code shared by the per-tile kernels over a binned fragment stream (build, evaluate, render, one-pass render).
//
// One workgroup owns one screen tile. Its coefficient tile lives in LDS, pixels innermost ([channel * rows + row][pixel]:
// the updates of a wavefront go to random pixels, hence random banks), and every fragment of the tile is applied with
// LDS atomics, so no per-fragment update leaves the compute unit. Global memory sees the streaming read of the binned
// records plus one load and/or store of each coefficient and accumulation tile.
//
//   build     (section 2.3.1): chi += a (1 - x); for n = 0..N: d[2^n + k] -= a tau(2^n x - k),
//             k = min(floor(2^n x), 2^n - 1), tau(t) = t on [0, 1/2), 1 - t on [1/2, 1]; a = -ln(1 - alpha).
//             d = 2^(n/2) X_{n,k}, so the N + 2 updates of a fragment are plain products.
//   cells     (section 2.3): the Haar expansion is constant on the M cells of width 1/M; the inverse of the
//             level-scaled transform gives the cell values with one add and one subtract per coefficient.
//   evaluate  (sections 2.2, 2.3.2): u = M x, j = min(floor(u), M - 1), t = u - j,
//             A~ = (1 - t) Abar_{j-1} + t Abar_j (Abar_{-1} = 0), v = exp(-A~);
//             accumulate alpha rgb v and a per pixel.
//   resolve   (section 2.1 step 4): out = colour + bg exp(-sum a).
#pragma once

#include <type_traits>

#include "wt_common.h"

namespace wt {

// ------------------------------------------------------------------------------------------- tile addressing

struct TileRef {
  uint32_t x0, y0;   // origin in the frame
  uint32_t beg, end; // binned record range
};

__device__ __forceinline__ TileRef tile_ref(const Geom& g, const Binned& b, uint32_t t) {
  TileRef r;
  r.x0 = (t % g.tilesX) * g.TW;
  r.y0 = (t / g.tilesX) * g.TH;
  r.beg = b.offsets[t * g.NX];
  r.end = b.offsets[(t + 1) * g.NX];
  return r;
}

// Frame pixel of tile-local pixel lp, or false when it lies outside the frame. The row is tested inside the tile: the last
// tile of a frame nearly 2^32 rows high has rows past 2^32, whose 32-bit frame row would be one of the first.
__host__ __device__ __forceinline__ bool tile_pixel(const Geom& g, const TileRef& r, uint32_t lp, uint64_t& p) {
  p = 0;
  const uint32_t px = r.x0 + (lp & (g.TW - 1)), row = lp >> g.lTW;
  if (px >= g.W || row >= g.H - r.y0) return false;
  p = (uint64_t)(r.y0 + row) * g.W + px;
  return true;
}

__device__ __forceinline__ float clamp01(float x) { return fminf(fmaxf(x, 0.f), 1.f); }

// ------------------------------------------------------------------------------------------- records

// Head of a forward record: pixel, depth and per channel the absorbance step a = -ln(1 - alpha) (NaN for a dropped
// fragment). Its tail holds the colour weighted with the coverage, alpha rgb.
template <int C>
struct Head {
  uint32_t lp;
  float x;
  float al[C];
};

template <bool NT>
__device__ __forceinline__ uint32_t load_word(const uint32_t* p) {
  if constexpr (NT)
    return __builtin_nontemporal_load(p);
  else
    return *p;
}

// Head of record i; false for a NaN fragment (skipped, already counted as dropped).
template <int C, bool NT = false>
__device__ __forceinline__ bool load_head(const Binned& b, uint32_t i, Head<C>& f) {
  const uint32_t* r = b.head + (uint64_t)i * b.DH;
  f.lp = load_word<NT>(r);
  f.x = __uint_as_float(load_word<NT>(r + 1));
  bool bad = isnan(f.x);
#pragma unroll
  for (int c = 0; c < C; ++c) {
    f.al[c] = __uint_as_float(load_word<NT>(r + 2 + c));
    bad |= isnan(f.al[c]);
  }
  return !bad;
}

constexpr uint32_t kNoRecord = 0xffffffffu;

template <bool NT>
__device__ __forceinline__ void load_tail(const Binned& b, uint32_t i, float (&w)[3]) {
  const uint32_t* r = b.tail + (uint64_t)i * b.DT;
#pragma unroll
  for (int q = 0; q < 3; ++q) w[q] = __uint_as_float(load_word<NT>(r + q));
}

// Records are read non-temporally by their last reader at one channel, so that the lines of the tiles still being
// built stay in the caches for their second read (smoke frame: tile kernel 0.96 -> 0.89 ms; non-temporal loads in the
// build as well: 1.02 ms). At three channels a tile's records are few and the same loads made the glass frame's tile
// kernel slower (3.02 -> 3.11 ms), so there they stay ordinary.
template <int C>
constexpr bool last_read_nt() { return C == 1; }

// Binned records each thread keeps in flight in the build and evaluate loops (memory-level parallelism of one
// workgroup per compute unit).
constexpr int kBuildUnroll = 8;
constexpr int kEvalUnroll = 4;

// Records [beg, end) dealt to the workgroup's threads in batches of U per thread, all of a batch's loads in flight before
// its first use: load(i, u) reads record i into the batch's slot u and says whether it counts, use(u) applies it. Whole
// batches run without a test; the last, partial one takes U or U / 2 slots at once (record indices clamped to the last),
// because records left to be loaded one by one cost a memory latency each (smoke frame, 65 records per thread: the
// five that remain beside whole batches took 5% of the tile kernel). One slot is enough where no thread has a second
// record, as in the tiles of a pixel or two at rank 10, where clamped loads are most of the batch (three channels with
// depth bounds 6.40 -> 6.21 ms).
template <int U, bool BACK = false, typename Load, typename Use>
__device__ __forceinline__ void for_records(uint32_t beg, uint32_t end, Load&& load, Use&& use) {
  const uint32_t T = blockDim.x;
  uint32_t base = beg;
  for (; end - base >= U * T;) {
    const uint32_t from = BACK ? end - U * T : base;
    bool ok[U];
#pragma unroll
    for (int u = 0; u < U; ++u) ok[u] = load(from + u * T + threadIdx.x, u);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (ok[u]) use(u);
    if (BACK)
      end -= U * T;
    else
      base += U * T;
  }
  auto last = [&](auto n) {
    constexpr int N = decltype(n)::value;
    bool ok[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const uint32_t i = base + u * T + threadIdx.x;
      ok[u] = load(min(i, end - 1), u) && i < end;
    }
#pragma unroll
    for (int u = 0; u < N; ++u)
      if (ok[u]) use(u);
  };
  if (end - base > U / 2 * T)
    last(std::integral_constant<int, U>{});
  else if (end - base > T)
    last(std::integral_constant<int, U / 2>{});
  else if (end > base)
    last(std::integral_constant<int, 1>{});
}

// ------------------------------------------------------------------------------------------- depth bounds

// Per-pixel depth bounds of the tile (section 2.1, step 1): lb[lp] = lo, lb[TP + lp] = hi as FP32 bit patterns,
// over the clamped depths of the tile's valid fragments (non-negative floats order like their bit patterns, so
// LDS u32 min/max atomics take them). Ends with a barrier.
__device__ __forceinline__ void bounds_add(uint32_t* lb, uint32_t TP, uint32_t lp, float x) {
  const uint32_t xb = __float_as_uint(fminf(fmaxf(x, 0.f), 1.f));
  atomicMin(lb + lp, xb);
  atomicMax(lb + TP + lp, xb);
}

__device__ __forceinline__ void bounds_clear(uint32_t* lb, uint32_t TP) {
  for (uint32_t lp = threadIdx.x; lp < TP; lp += blockDim.x) {
    lb[lp] = __float_as_uint(1.f);
    lb[TP + lp] = 0u;
  }
}

template <int C>
__device__ __forceinline__ void bounds_range(const Binned& b, uint32_t beg, uint32_t end, uint32_t* lb, uint32_t TP) {
  Head<C> f[kBuildUnroll];
  for_records<kBuildUnroll>(
      beg, end, [&](uint32_t i, int u) { return load_head<C>(b, i, f[u]); },
      [&](int u) { bounds_add(lb, TP, f[u].lp, f[u].x); });
}

template <int C>
__device__ __forceinline__ void bounds_tile(const Binned& b, const Geom& g, const TileRef& r, uint32_t* lb) {
  bounds_clear(lb, g.tile_px);
  __syncthreads();
  bounds_range<C>(b, r.beg, r.end, lb, g.tile_px);
  __syncthreads();
}

// ------------------------------------------------------------------------------------------- build

// On-chip sums are FP64: on gfx950 an LDS FP64 atomic add sustains about nine times the rate of an FP32 one,
// and every FP32 term then rounds once while the sum rounds nowhere.
using acc_t = double;

// A fragment's contribution to every coefficient depends on its depth only through its finest cell j and the
// offset t = M x - j in it: 1 - x and every tent tau(2^n x - k) are linear on a finest cell (their kinks lie on
// cell boundaries for n <= N). So the N + 2 closed-form updates of section 2.3.1 factor exactly through two
// endpoint masses, e_j += a (1 - t) and e_{j+1} += a t, per fragment and channel:
//   chi     = sum_m e_m (1 - m/M),   d_{n,k} = -sum_m e_m tau(2^n m / M - k),   sum a = sum_m e_m,
// with exact dyadic weights and all terms of one sign (no cancellation). Two LDS atomics per fragment instead
// of N + 2, and the absorbance total comes for free.
template <int C>
__device__ __forceinline__ void ep_add(acc_t* le, uint32_t TP, uint32_t M1, uint32_t lp, uint32_t j, float t, float omt,
                                       const float (&al)[C]) {
#pragma unroll
  for (int c = 0; c < C; ++c) {
    acc_t* e = le + (c * M1 + j) * TP + lp;
    atomicAdd(e, (acc_t)(al[c] * omt));
    atomicAdd(e + TP, (acc_t)(al[c] * t));
  }
}

template <int C>
__device__ __forceinline__ void build_ep_add(acc_t* le, const Geom& g, const Head<C>& f, const uint32_t* lb) {
  uint32_t j;
  float t, omt;
  cell_coord(f.x, lb, g.tile_px, f.lp, g.M, j, t, omt);
  ep_add<C>(le, g.tile_px, g.M + 1, f.lp, j, t, omt, f.al);
}

// Applies records [beg, end) to the endpoint masses.
template <int C>
__device__ __forceinline__ void build_ep_range(const Binned& b, const Geom& g, uint32_t beg, uint32_t end, acc_t* le,
                                               const uint32_t* lb) {
  Head<C> f[kBuildUnroll];
  for_records<kBuildUnroll>(
      beg, end, [&](uint32_t i, int u) { return load_head<C>(b, i, f[u]); },
      [&](int u) { build_ep_add<C>(le, g, f[u], lb); });
}

template <int C>
__device__ __forceinline__ void build_ep_tile(const Binned& b, const Geom& g, const TileRef& r, acc_t* le,
                                              const uint32_t* lb) {
  if (serial_records(g, r.beg, r.end, [&](uint32_t i) {
        Head<C> f;
        if (load_head<C>(b, i, f)) build_ep_add<C>(le, g, f, lb);
      }))
    return;
  build_ep_range<C>(b, g, r.beg, r.end, le, lb);
}

// Sums over the inner endpoint masses of an interval of N finest cells: weighted with a ramp up and a ramp down over the
// interval, and plain.
struct Ramps {
  acc_t up, down, sum;
};

// The interval of N cells at `lo` whose wavelet coefficient is stored at idx (its halves' at 2 idx and 2 idx + 1): emits
// its coefficients, minus the tent-weighted sums, and returns its ramps. Each interval's tent and ramps follow from its
// halves' and the mass between them with a factor of one half, so the whole column takes O(M) operations, each mass is
// used once, and no weight has to be held in a register (FP64 operands have no 64-bit literals). All terms have one sign.
template <int N, typename Mass, typename Emit>
__device__ __forceinline__ Ramps interval_coeffs(int idx, int lo, Mass&& mass, Emit&& emit) {
  if constexpr (N == 2) {
    const acc_t e = mass(lo + 1), h = 0.5 * e;
    emit(idx, -h);
    return {h, h, e};
  } else {
    const Ramps l = interval_coeffs<N / 2>(2 * idx, lo, mass, emit);
    const acc_t e = mass(lo + N / 2);
    const Ramps r = interval_coeffs<N / 2>(2 * idx + 1, lo + N / 2, mass, emit);
    // eight cells at a time: scheduled all at once, the masses of 32 cells alone take more than half the registers
    if constexpr (N == 8) __builtin_amdgcn_sched_barrier(0);
    emit(idx, -0.5 * (l.up + e + r.down));
    return {0.5 * (l.up + (e + r.sum) + r.up), 0.5 * (l.down + (l.sum + e) + r.down), l.sum + e + r.sum};
  }
}

// Coefficients (stored layout) of one pixel and channel from its M + 1 endpoint masses mass(0..M): emit(m, coefficient).
// Returns the absorbance total.
template <int M, typename Mass, typename Emit>
__device__ __forceinline__ acc_t column_coeffs(Mass&& mass, Emit&& emit) {
  const acc_t first = mass(0);
  const Ramps r = interval_coeffs<M>(1, 0, mass, emit);
  emit(0, first + r.down);
  return first + r.sum + mass(M);
}

// ------------------------------------------------------------------------------------------- cells

// Inverse of the level-scaled Haar transform on M values held in registers: coefficients -> cell values.
template <int M>
__device__ __forceinline__ void synth_regs(float (&v)[M]) {
  float w[M];
  w[0] = v[0];
#pragma unroll
  for (int s = 1; s < M; s <<= 1) {
#pragma unroll
    for (int k = s - 1; k >= 0; --k) {
      const float d = v[s + k];
      const float a = w[k];
      w[2 * k] = a + d;
      w[2 * k + 1] = a - d;
    }
  }
#pragma unroll
  for (int j = 0; j < M; ++j) v[j] = w[j];
}
// Writes M values of TS for one pixel/channel, 16 bytes at a time where the layout allows.
template <typename TS, int M>
__device__ __forceinline__ void store_row(TS* dst, const TS (&s)[M]) {
  if ((M * sizeof(TS)) % 16 == 0) {
#pragma unroll
    for (int k = 0; k < (int)(M * sizeof(TS) / 16); ++k) {
      uint4 u;
      __builtin_memcpy(&u, (const char*)s + 16 * k, 16);
      ((uint4*)dst)[k] = u;
    }
  } else {
#pragma unroll
    for (int m = 0; m < M; ++m) dst[m] = s[m];
  }
}

// The same from values that the storage type holds exactly (read back from narrow_d), two to a word for the narrow types.
template <typename TS, int M>
__device__ __forceinline__ void store_exact_row(TS* dst, const float (&v)[M]) {
  if constexpr (std::is_same<TS, float>::value) {
    store_row<float, M>(dst, v);
  } else {
    uint32_t w[M / 2];
#pragma unroll
    for (int k = 0; k < M / 2; ++k) {
      if constexpr (std::is_same<TS, __half>::value)
        w[k] = __half_as_ushort(__float2half(v[2 * k])) | (uint32_t)__half_as_ushort(__float2half(v[2 * k + 1])) << 16;
      else
        w[k] = __float_as_uint(v[2 * k]) >> 16 | (__float_as_uint(v[2 * k + 1]) & 0xffff0000u);
    }
    store_row<uint32_t, M / 2>((uint32_t*)dst, w);
  }
}

// Row of M storage values of one pixel/channel, 16 bytes at a time where the layout allows.
template <typename TS, int M>
__device__ __forceinline__ void load_row(const TS* src, TS (&s)[M]) {
  if ((M * sizeof(TS)) % 16 == 0) {
#pragma unroll
    for (int k = 0; k < (int)(M * sizeof(TS) / 16); ++k) {
      const uint4 u = ((const uint4*)src)[k];
      __builtin_memcpy((char*)s + 16 * k, &u, 16);
    }
  } else {
#pragma unroll
    for (int m = 0; m < M; ++m) s[m] = src[m];
  }
}

// ------------------------------------------------------------------------------------------- E5B9G9R9 storage
//
// Three channels share one word per coefficient index (wt.h). Coefficient 0 (chi) is >= 0 and every wavelet
// coefficient <= 0 (section 2.3.1), so the words hold magnitudes and the sign is restored from the index.

__device__ __forceinline__ float e5_sign(uint32_t m) { return m ? -1.f : 1.f; }

template <typename F>
__device__ __forceinline__ void with_m(const Geom& g, F&& f) {
  switch (g.M) {
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 8: f(std::integral_constant<int, 8>{}); break;
    case 16: f(std::integral_constant<int, 16>{}); break;
    default: f(std::integral_constant<int, 32>{}); break;
  }
}

// ------------------------------------------------------------------------------------------- shading

// Adds one fragment's visible colour to the colour rows la ([3][TP]); w is its coverage-weighted colour and
// cell(c, j) the average absorbance of cell j of channel c of its pixel.
template <int C, typename Cell>
__device__ __forceinline__ void shade_add(acc_t* la, uint32_t TP, uint32_t lp, uint32_t j, float t, float omt,
                                          const float (&w)[3], Cell&& cell) {
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const float hi = cell(c, j);
    const float below = cell(c, j ? j - 1 : 0u);
    const float lo = j ? below : 0.f;
    const float v = __expf(-fmaf(t, hi, omt * lo));
    if (C == 1) {
#pragma unroll
      for (int q = 0; q < 3; ++q) atomicAdd(la + q * TP + lp, (acc_t)(w[q] * v));
    } else {
      atomicAdd(la + c * TP + lp, (acc_t)(w[c] * v));
    }
  }
}

// ------------------------------------------------------------------------------------------- direct build (M > 32)

// The N + 2 coefficient updates of one fragment, per channel. lc is [C*M][TP] of acc_t.
template <int C>
__device__ __forceinline__ void build_add(acc_t* lc, const Geom& g, const Head<C>& f, const uint32_t* lb) {
  const uint32_t TP = g.tile_px;
  const double xd = unit_depth_d(f.x, lb, TP, f.lp);
  float a[C];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    a[c] = f.al[c];  // binned records hold the absorbance
    atomicAdd(lc + (c * g.M) * TP + f.lp, (acc_t)(a[c] * (float)(1.0 - xd)));
  }
  for (uint32_t n = 0; n <= g.rank; ++n) {
    const uint32_t s = 1u << n;
    const double u = xd * (double)s;
    const uint32_t k = min((uint32_t)u, s - 1);
    const double t = u - (double)k;
    const float tau = (float)(t < 0.5 ? t : 1.0 - t);
#pragma unroll
    for (int c = 0; c < C; ++c) atomicAdd(lc + (c * g.M + s + k) * TP + f.lp, (acc_t)(-a[c] * tau));
  }
}

template <int C>
__device__ __forceinline__ void build_tile(const Binned& b, const Geom& g, const TileRef& r, acc_t* lc,
                                           const uint32_t* lb) {
  if (serial_records(g, r.beg, r.end, [&](uint32_t i) {
        Head<C> f;
        if (load_head<C>(b, i, f)) build_add<C>(lc, g, f, lb);
      }))
    return;
  uint32_t i = r.beg + threadIdx.x;
  // two records per thread per step keep more loads in flight
  for (; i + blockDim.x < r.end; i += 2 * blockDim.x) {
    Head<C> f0, f1;
    const bool ok0 = load_head<C>(b, i, f0);
    const bool ok1 = load_head<C>(b, i + blockDim.x, f1);
    if (ok0) build_add<C>(lc, g, f0, lb);
    if (ok1) build_add<C>(lc, g, f1, lb);
  }
  if (i < r.end) {
    Head<C> f0;
    if (load_head<C>(b, i, f0)) build_add<C>(lc, g, f0, lb);
  }
}

// Cell value Abar_j straight from the stored coefficients of one pixel/channel (column stride TP).
template <typename T>
__device__ __forceinline__ float cell_from_coeffs(const T* cf, uint32_t TP, const Geom& g, uint32_t j) {
  T A = cf[0];
  for (uint32_t n = 0; n <= g.rank; ++n) {
    const uint32_t k = j >> (g.L - n);
    const T d = cf[((1u << n) + k) * TP];
    A += ((j >> (g.L - 1 - n)) & 1u) ? -d : d;
  }
  return (float)A;
}
// ------------------------------------------------------------------------------------------- tile <-> global

// Load: words -> signed values of T in LDS [3*M][TP] (zero off-frame).
template <typename T>
__device__ __forceinline__ void e5_load_tile(const Geom& g, const TileRef& r, T* lc, const uint32_t* coeffs) {
  const uint32_t TP = g.tile_px, M = g.M;
  for (uint32_t q = threadIdx.x; q < TP * M; q += blockDim.x) {
    const uint32_t lp = q / M, m = q - lp * M;
    uint64_t p;
    const uint32_t w = tile_pixel(g, r, lp, p) ? coeffs[p * M + m] : 0u;
    const float sg = e5_sign(m);
#pragma unroll
    for (uint32_t c = 0; c < 3; ++c) lc[(c * M + m) * TP + lp] = (T)(sg * e5_unpack(w, c));
  }
}


// Coefficient tile between LDS ([C*M][TP] of T) and global memory ([P][C][M] of TS). Work item q covers VW
// consecutive elements of one pixel, so consecutive lanes touch consecutive global addresses.
// MODE 0: load (zero off-frame), 1: store, 2: round to TS in place and store when coeffs is not null.
template <int C, typename TS, int MODE, typename T>
__device__ __forceinline__ void coeff_tile_io(const Geom& g, const TileRef& r, T* lc, TS* coeffs) {
  if constexpr (is_e5<TS>::value) {
    // packed storage: loads only (stores run on the endpoint path, make_geom)
    if (MODE == 0) e5_load_tile<T>(g, r, lc, (const uint32_t*)coeffs);
  } else {
  const uint32_t TP = g.tile_px, per = C * g.M;
  const uint32_t VW = g.M < 4 ? g.M : 4;
  const uint32_t groups = per / VW;
  for (uint32_t q = threadIdx.x; q < TP * groups; q += blockDim.x) {
    const uint32_t lp = q / groups, e0 = (q - lp * groups) * VW;
    uint64_t p;
    const bool in = tile_pixel(g, r, lp, p);
    TS* gp = coeffs ? coeffs + p * per + e0 : nullptr;
    for (uint32_t e = 0; e < VW; ++e) {
      T* l = lc + (e0 + e) * TP + lp;  // row (c * M + m) = e0 + e
      if (MODE == 0) {
        *l = in ? (T)widen<TS>(gp[e]) : (T)0;
      } else if (MODE == 1) {
        if (in) gp[e] = narrow_d<TS>((double)*l);
      } else {
        const TS s = narrow_d<TS>((double)*l);
        *l = (T)widen<TS>(s);
        if (in && gp) gp[e] = s;
      }
    }
  }
  }
}
// ------------------------------------------------------------------------------------------- launching

template <typename K>
static hipError_t prep(K kernel, size_t lds) {
  if (lds > 65536)
    return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  return hipSuccess;
}

// Dispatch on channels and storage type: f(std::integral_constant<int, C>, TS* tag) for the frame's values.
template <typename F>
static hipError_t dispatch(const Geom& g, F&& f) {
  if (g.C == 1) {
    if (g.dtype == WT_F32) return f(std::integral_constant<int, 1>{}, (float*)nullptr);
    if (g.dtype == WT_F16) return f(std::integral_constant<int, 1>{}, (__half*)nullptr);
    return f(std::integral_constant<int, 1>{}, (bf16_t*)nullptr);
  }
  if (g.dtype == WT_F32) return f(std::integral_constant<int, 3>{}, (float*)nullptr);
  if (g.dtype == WT_F16) return f(std::integral_constant<int, 3>{}, (__half*)nullptr);
  if (g.dtype == WT_E5B9G9R9) {
    return f(std::integral_constant<int, 3>{}, (e5_t*)nullptr);
  }
  return f(std::integral_constant<int, 3>{}, (bf16_t*)nullptr);
}

}  // namespace wt
