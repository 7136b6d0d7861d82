// Build and evaluate kernels of the accumulating passes over a binned stream, and the composites over a finished
// accumulation.
#include <algorithm>

#include "wt_tile.h"

namespace wt {

// ------------------------------------------------------------------------------------------- build

// Build (accumulating): words += the coefficients of the endpoint masses (decoded, added in FP64, rounded to
// FP32 and packed again). Each thread turns the endpoint column of a pixel and channel into coefficients in place.
template <int M>
__device__ __forceinline__ void e5_build_store(const Geom& g, const TileRef& r, acc_t* le, uint32_t* coeffs) {
  constexpr uint32_t C = 3;
  const uint32_t TP = g.tile_px;
  for (uint32_t q = threadIdx.x; q < TP * C; q += blockDim.x) {
    const uint32_t c = q / TP;
    acc_t* col = le + (size_t)c * (M + 1) * TP + (q - c * TP);
    acc_t cf[M];
    column_coeffs<M>([&](int m) { return col[m * TP]; }, [&](int m, acc_t v) { cf[m] = v; });
#pragma unroll
    for (int m = 0; m < M; ++m) col[m * TP] = cf[m];
  }
  __syncthreads();
  for (uint32_t q = threadIdx.x; q < TP * M; q += blockDim.x) {  // consecutive lanes on consecutive words
    const uint32_t px = q / M, m = q & (M - 1);
    uint64_t p;
    if (!tile_pixel(g, r, px, p)) continue;
    const uint32_t old = coeffs[p * M + m];
    const double sg = e5_sign(m);
    float v[C];
#pragma unroll
    for (uint32_t c = 0; c < C; ++c)
      v[c] = (float)(sg * le[(size_t)(c * (M + 1) + m) * TP + px] + (double)e5_unpack(old, c));
    coeffs[p * M + m] = e5_pack(v[0], v[1], v[2]);
  }
}

// Build (accumulating): coeffs += coefficients of the endpoint masses, one pixel/channel per thread.
template <int C, typename TS, int M>
__device__ __forceinline__ void ep_build_store(const Geom& g, const TileRef& r, const acc_t* le, TS* coeffs) {
  const uint32_t TP = g.tile_px;
  for (uint32_t q = threadIdx.x; q < TP * C; q += blockDim.x) {
    const uint32_t c = q / TP, lp = q - c * TP;
    uint64_t p;
    if (!tile_pixel(g, r, lp, p)) continue;
    const acc_t* col = le + (size_t)c * (M + 1) * TP + lp;
    TS* gp = coeffs + (p * C + c) * M;
    TS s[M];
    load_row<TS, M>(gp, s);
    float v[M];
#pragma unroll
    for (int m = 0; m < M; ++m) v[m] = widen<TS>(s[m]);
    column_coeffs<M>([&](int m) { return col[m * TP]; },
                     [&](int m, acc_t x) { v[m] = widen<TS>(narrow_d<TS>(x + (acc_t)v[m])); });
    store_exact_row<TS, M>(gp, v);
  }
}

// LDS: endpoint masses [C * (M + 1)][TP] FP64, or coefficients [C * M][TP] FP64 (M > 32), then the depth bounds.
template <int C, typename TS>
__global__ __launch_bounds__(kTileThreads) void k_build(Binned b, Geom g, TS* __restrict__ coeffs) {
  extern __shared__ acc_t smem_d[];
  acc_t* lc = smem_d;
  uint32_t tile;
  if (!binned_ok(b, g, tile)) return;
  const TileRef r = tile_ref(g, b, tile);
  // per-pixel depth bounds after the coefficient region
  uint32_t* lb = g.tight ? (uint32_t*)(smem_d + (g.ep ? C * (g.M + 1) : C * g.M) * g.tile_px) : nullptr;
  if (lb) bounds_tile<C>(b, g, r, lb);
  if (g.ep) {
    for (uint32_t e = threadIdx.x; e < C * (g.M + 1) * g.tile_px; e += blockDim.x) lc[e] = 0.0;
    __syncthreads();
    build_ep_tile<C>(b, g, r, lc, lb);
    __syncthreads();
    if constexpr (is_e5<TS>::value)
      with_m(g, [&](auto mm) { e5_build_store<decltype(mm)::value>(g, r, lc, (uint32_t*)coeffs); });
    else
      with_m(g, [&](auto mm) { ep_build_store<C, TS, decltype(mm)::value>(g, r, lc, coeffs); });
    return;
  }
  coeff_tile_io<C, TS, 0>(g, r, lc, coeffs);
  __syncthreads();
  build_tile<C>(b, g, r, lc, lb);
  __syncthreads();
  coeff_tile_io<C, TS, 1>(g, r, lc, coeffs);
}

// ------------------------------------------------------------------------------------------- evaluate

// One fragment of the evaluate pass. la is [AL][TP] of acc_t: rows 0..2 colour, then sum a (C = 1) or sum a_r, a_g,
// a_b (C = 3). lc holds FP32 cells (CELLS) or coefficients (otherwise), [C*M][TP].
template <int C, bool CELLS>
__device__ __forceinline__ void eval_add(const float* lc, acc_t* la, const Geom& g, const Head<C>& f,
                                         const float (&w)[3], const uint32_t* lb) {
  const uint32_t TP = g.tile_px;
  uint32_t j;
  float t, omt;
  cell_coord(f.x, lb, TP, f.lp, g.M, j, t, omt);
  shade_add<C>(la, TP, f.lp, j, t, omt, w, [&](int c, uint32_t jj) {
    const float* cf = lc + (c * g.M) * TP + f.lp;
    return CELLS ? cf[jj * TP] : cell_from_coeffs(cf, TP, g, jj);
  });
#pragma unroll
  for (int c = 0; c < C; ++c) atomicAdd(la + (3 + c) * TP + f.lp, (acc_t)f.al[c]);
}

template <int C, bool CELLS>
__device__ __forceinline__ void eval_tile(const Binned& b, const Geom& g, const TileRef& r, const float* lc, acc_t* la,
                                          const uint32_t* lb) {
  constexpr bool kNT = last_read_nt<C>();
  if (serial_records(g, r.beg, r.end, [&](uint32_t i) {
        Head<C> f;
        float w[3];
        load_tail<kNT>(b, i, w);
        if (load_head<C, kNT>(b, i, f)) eval_add<C, CELLS>(lc, la, g, f, w, lb);
      }))
    return;
  // U whole records per thread in flight per step (six at three channels, where a tile holds a few thousand records:
  // glass 3840x2160 3.03 -> 2.96 ms; at one channel six were slower, 0.89 -> 0.93 ms)
  constexpr int U = C == 1 ? kEvalUnroll : 6;
  Head<C> f[U];
  float w[U][3];
  for_records<U>(
      r.beg, r.end,
      [&](uint32_t i, int u) {
        load_tail<kNT>(b, i, w[u]);
        return load_head<C, kNT>(b, i, f[u]);
      },
      [&](int u) { eval_add<C, CELLS>(lc, la, g, f[u], w[u], lb); });
}

// Cells of an FP32 coefficient tile, in place (one pixel/channel per thread).
template <int C, int M>
__device__ __forceinline__ void synth_tile_f32(float* lc, uint32_t TP) {
  for (uint32_t q = threadIdx.x; q < TP * C; q += blockDim.x) {
    const uint32_t c = q / TP, lp = q - c * TP;
    float* cf = lc + (c * M) * TP + lp;
    float v[M];
#pragma unroll
    for (int m = 0; m < M; ++m) v[m] = cf[m * TP];
    synth_regs<M>(v);
#pragma unroll
    for (int m = 0; m < M; ++m) cf[m * TP] = v[m];
  }
}

// LDS: accumulation rows [AL][TP] FP64, FP32 cells or coefficients [C * M][TP], then the depth bounds.
template <int C, typename TS, bool CELLS>
__global__ __launch_bounds__(kTileThreads) void k_evaluate(Binned b, Geom g, const TS* __restrict__ coeffs,
                                                           float* __restrict__ accum) {
  extern __shared__ acc_t smem_d[];
  const uint32_t TP = g.tile_px;
  acc_t* la = smem_d;                              // [AL][TP] FP64
  float* lc = (float*)(smem_d + g.AL * TP);        // [C*M][TP] FP32
  uint32_t* lb = g.tight ? (uint32_t*)(lc + C * g.M * TP) : nullptr;  // per-pixel depth bounds
  uint32_t tile;
  if (!binned_ok(b, g, tile)) return;
  const TileRef r = tile_ref(g, b, tile);
  if (lb) bounds_tile<C>(b, g, r, lb);
  coeff_tile_io<C, TS, 0>(g, r, lc, const_cast<TS*>(coeffs));
  for (uint32_t lp = threadIdx.x; lp < TP; lp += blockDim.x) {
    uint64_t p;
    const bool in = tile_pixel(g, r, lp, p);
    for (uint32_t k = 0; k < 3; ++k) la[k * TP + lp] = in ? accum[p * g.AW + k] : 0.0;
    for (uint32_t c = 0; c < C; ++c)
      la[(3 + c) * TP + lp] = in ? accum[p * g.AW + (C == 1 ? 3 : 4 + c)] : 0.0;
  }
  __syncthreads();
  if (CELLS) with_m(g, [&](auto mm) { synth_tile_f32<C, decltype(mm)::value>(lc, TP); });
  __syncthreads();
  eval_tile<C, CELLS>(b, g, r, lc, la, lb);
  __syncthreads();
  for (uint32_t lp = threadIdx.x; lp < TP; lp += blockDim.x) {
    uint64_t p;
    if (!tile_pixel(g, r, lp, p)) continue;
    for (uint32_t k = 0; k < 3; ++k) accum[p * g.AW + k] = (float)la[k * TP + lp];
    for (uint32_t c = 0; c < C; ++c) accum[p * g.AW + (C == 1 ? 3 : 4 + c)] = (float)la[(3 + c) * TP + lp];
  }
}
__global__ __launch_bounds__(256) void k_resolve(const float* __restrict__ accum, Geom g, float bg0, float bg1,
                                                 float bg2, float* __restrict__ out) {
  const float bg[3] = {bg0, bg1, bg2};
  const uint64_t n = (uint64_t)g.P * 3;
  for (uint64_t e = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; e < n; e += (uint64_t)gridDim.x * blockDim.x) {
    const uint64_t p = e / 3;
    const uint32_t q = (uint32_t)(e - p * 3);
    const float colour = accum[p * g.AW + q];
    const float suma = (g.AW == 4) ? accum[p * 4 + 3] : accum[p * 8 + 4 + q];
    out[e] = colour + bg[q] * __expf(-suma);
  }
}

// ------------------------------------------------------------------------------------------- chromatic composite
//
// Composite over a background image sampled through each pixel's screen-space refraction offset, with the
// chromatic-aberration gather of section 3: k taps along the offset, tap i at parameter t = i / (k - 1) displaced
// by s = 1 + dispersion (t - 1/2) times the offset, each a bilinear sample of the background (clamp to edge),
// weighted per channel by the spectral weights (red: the smoothstep formula falling from 1 at t = 1/3 to 0 at
// t = 1/2; blue: rising from 0 at t = 1/2 to 1 at t = 2/3; green: the remainder) and normalised per channel.

__device__ __forceinline__ float smoothstep_formula(float e0, float e1, float x) {
  const float u = fminf(fmaxf((x - e0) / (e1 - e0), 0.f), 1.f);
  return u * u * (3.f - 2.f * u);
}

// Images of two columns or more whose texels have 32-bit byte offsets, and row pitches and coordinates below 2^24: a texel's
// address is one 24-bit multiply and an add on a base that stays in scalar registers, and a row's two texels of a tap, which
// are neighbours, come with one 16-byte load (channel q of the left one in its first word, of the right one in its last).
// The gather is bound by its requests and their cache lines: with a load per texel the scheduler drew a row's two loads
// apart, and offsets without a common direction found the line gone at the second. 64-bit addresses and a load per texel,
// 24-bit addresses, and with pairs, 1920x1080, smooth offsets and independent ones: 5 taps 37.5 and 87, 36.0 and 88, 30.1
// and 68 us; 7 taps 54 and 107, 47 and 112, 38 and 76; 9 taps 71 and 152, 65 and 129, 56 and 105. (A band of the image per
// XCD changed little.)
// Three taps over a large three-channel accumulation wait on that accumulation: 3840x2160 147 us with 64-bit addresses, 153
// with pairs. They keep the former.
static bool chromatic_small(const Geom& g, uint32_t taps) {
  if (taps == 3 && g.AW == 8 && g.P > (4u << 20)) return false;
  return g.W >= 2 && (uint64_t)g.P * 12 < (1ull << 32) && g.H < (1u << 24) && g.W * 12ull < (1u << 24);
}

typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

// Tap i of k for one pixel: the bilinear sample of every channel with a non-zero spectral weight, accumulated
// into num/den. The tap position is split into the pixel's integer coordinate and the offset's own integer and
// fractional parts, so the bilinear fractions keep the offset's precision at any frame size.
template <bool SMALL>
__device__ __forceinline__ void chromatic_tap(const Geom& g, const float* __restrict__ bgimg, uint32_t x, uint32_t y,
                                              float dx, float dy, float dispersion, uint32_t i, uint32_t k,
                                              float (&num)[3], float (&den)[3]) {
  using coord_t = std::conditional_t<SMALL, int, long>;
  const float t = (float)i / (float)(k - 1);
  float w[3];
  w[0] = smoothstep_formula(0.5f, 1.f / 3.f, t);
  w[2] = smoothstep_formula(0.5f, 2.f / 3.f, t);
  w[1] = 1.f - w[0] - w[2];
  const float sc = 1.f + dispersion * (t - 0.5f);
  const float ox = sc * dx, oy = sc * dy;
  const float fox = floorf(ox), foy = floorf(oy);
  const float fx = ox - fox, fy = oy - foy;  // exact
  // sample position minus the half-texel shift: (x + ox, y + oy); the left/top texel and the clamped pair (the
  // integer parts are bounded before conversion, so a NaN or huge offset still addresses the image's edge)
  const coord_t lx = (coord_t)x + (coord_t)fminf(fmaxf(fox, -1e9f), 1e9f);
  const coord_t ly = (coord_t)y + (coord_t)fminf(fmaxf(foy, -1e9f), 1e9f);
  const coord_t Wm = (coord_t)g.W - 1, Hm = (coord_t)g.H - 1;
  const uint32_t x0 = (uint32_t)min(max(lx, (coord_t)0), Wm), x1 = (uint32_t)min(max(lx + 1, (coord_t)0), Wm);
  const uint32_t y0 = (uint32_t)min(max(ly, (coord_t)0), Hm), y1 = (uint32_t)min(max(ly + 1, (coord_t)0), Hm);
  const uint32_t xb = SMALL ? min(x0, (uint32_t)Wm - 1) : 0;  // a row's two texels are xb and xb + 1, or one of them
  const char* base = (const char*)bgimg;
  const uint32_t pitch = g.W * 12, at0 = __umul24(y0, pitch) + xb * 12, at1 = __umul24(y1, pitch) + xb * 12;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    if (w[q] == 0.f) continue;  // depends on the tap only (a constant when k is)
    float ta, tb, tc, td;
    if constexpr (SMALL) {
      const f32x4_any r0 = *(const f32x4_any*)(base + (at0 + 4 * q)), r1 = *(const f32x4_any*)(base + (at1 + 4 * q));
      ta = x0 == xb ? r0.x : r0.w;
      tb = x1 == xb ? r0.x : r0.w;
      tc = x0 == xb ? r1.x : r1.w;
      td = x1 == xb ? r1.x : r1.w;
    } else {
      ta = bgimg[((uint64_t)y0 * g.W + x0) * 3 + q];
      tb = bgimg[((uint64_t)y0 * g.W + x1) * 3 + q];
      tc = bgimg[((uint64_t)y1 * g.W + x0) * 3 + q];
      td = bgimg[((uint64_t)y1 * g.W + x1) * 3 + q];
    }
    const float v = (1.f - fy) * ((1.f - fx) * ta + fx * tb) + fy * ((1.f - fx) * tc + fx * td);
    num[q] += w[q] * v;
    den[q] += w[q];
  }
}

// One pixel per thread. K > 0 fixes the tap count at compile time (the weights fold to constants and the taps'
// loads issue together); K = 0 takes it from `taps`.
template <int K, bool SMALL>
__global__ __launch_bounds__(256) void k_resolve_chromatic(const float* __restrict__ accum, Geom g,
                                                           const float* __restrict__ bgimg,
                                                           const float* __restrict__ offset, float dispersion,
                                                           uint32_t taps, float* __restrict__ out) {
  const uint32_t p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= g.P) return;
  const uint32_t y = fastdiv(p, g.divW);
  const uint32_t x = p - y * g.W;
  const float2 o = ((const float2*)offset)[p];
  float num[3] = {0.f, 0.f, 0.f}, den[3] = {0.f, 0.f, 0.f};
  if constexpr (K > 0) {
#pragma unroll
    for (uint32_t i = 0; i < (uint32_t)K; ++i)
      chromatic_tap<SMALL>(g, bgimg, x, y, o.x, o.y, dispersion, i, K, num, den);
  } else {
    for (uint32_t i = 0; i < taps; ++i)
      chromatic_tap<SMALL>(g, bgimg, x, y, o.x, o.y, dispersion, i, taps, num, den);
  }
  float colour[3], suma[3];
  if (g.AW == 4) {
    const float4 a = ((const float4*)accum)[p];
    colour[0] = a.x; colour[1] = a.y; colour[2] = a.z;
    suma[0] = suma[1] = suma[2] = a.w;
  } else {
    const float4 a = ((const float4*)accum)[2 * (uint64_t)p];
    const float4 b = ((const float4*)accum)[2 * (uint64_t)p + 1];
    colour[0] = a.x; colour[1] = a.y; colour[2] = a.z;
    suma[0] = b.x; suma[1] = b.y; suma[2] = b.z;
  }
#pragma unroll
  for (int q = 0; q < 3; ++q) out[(uint64_t)p * 3 + q] = colour[q] + __expf(-suma[q]) * (num[q] / den[q]);
}
// ------------------------------------------------------------------------------------------- launchers

static size_t lds_eval_bytes(const Geom& g) {
  return (size_t)g.tile_px * (4 * g.C * g.M + 8 * g.AL + (g.tight ? 8 : 0));
}

hipError_t launch_build(const Geom& g, const Binned& b, void* coeffs, hipStream_t s) {
  const size_t lds = lds_tile_bytes(g, false);
  return dispatch(g, [&](auto cc, auto* tag) {
    constexpr int C = decltype(cc)::value;
    using TS = std::remove_pointer_t<decltype(tag)>;
    auto k = k_build<C, TS>;
    hipError_t err = prep(k, lds);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(k, dim3(g.ntiles), dim3(g.tthreads), lds, s, b, g, (TS*)coeffs);
    return hipGetLastError();
  });
}

hipError_t launch_evaluate(const Geom& g, const Binned& b, const void* coeffs, float* accum, hipStream_t s) {
  const size_t lds = lds_eval_bytes(g);
  // M > 32: FP32 coefficients are half the LDS that the tile was sized for, and two workgroups share a compute unit where
  // registers allow it: at one channel of 1024 threads, at three of 512 (512x512 at 8 per pixel, rank 8: one channel 391 us
  // with 512 threads and 354 with 1024, three channels 966 and 1417), when there are tiles enough to share (5x30, rank 7,
  // 885,000 fragments: 462 us with 512 threads, 380 with 1024). A single tile with all fragments of a large frame pays for
  // it (300x200, rank 5, 300,000 fragments on 64 pixels: 1.52 ms with 512 threads, 1.03 with 1024, 2.75 with 256).
  const uint32_t threads = g.M > 32 && g.C == 3 && g.ntiles > kComputeUnits ? kTileThreads / 2 : g.tthreads;
  return dispatch(g, [&](auto cc, auto* tag) {
    constexpr int C = decltype(cc)::value;
    using TS = std::remove_pointer_t<decltype(tag)>;
    auto k = (g.M <= 32) ? k_evaluate<C, TS, true> : k_evaluate<C, TS, false>;
    hipError_t err = prep(k, lds);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(k, dim3(g.ntiles), dim3(threads), lds, s, b, g, (const TS*)coeffs, accum);
    return hipGetLastError();
  });
}

hipError_t launch_resolve_chromatic(const Geom& g, const float* accum, const float* bgimg, const float* offset,
                                   float dispersion, uint32_t taps, float* out, hipStream_t s) {
  const unsigned grid = (unsigned)(((uint64_t)g.P + 255) / 256);
  auto pick = [&](auto small) {
    constexpr bool S = decltype(small)::value;
    return taps == 3   ? k_resolve_chromatic<3, S>
           : taps == 5 ? k_resolve_chromatic<5, S>
           : taps == 7 ? k_resolve_chromatic<7, S>
           : taps == 9 ? k_resolve_chromatic<9, S>
                       : k_resolve_chromatic<0, S>;
  };
  auto k = chromatic_small(g, taps) ? pick(std::true_type{}) : pick(std::false_type{});
  hipLaunchKernelGGL(k, dim3(grid), dim3(256), 0, s, accum, g, bgimg, offset, dispersion, taps, out);
  return hipGetLastError();
}

hipError_t launch_resolve(const Geom& g, const float* accum, const float* bg, float* out, hipStream_t s) {
  const uint64_t n = (uint64_t)g.P * 3;
  const unsigned grid = (unsigned)std::min<uint64_t>((n + 255) / 256, 65536);
  hipLaunchKernelGGL(k_resolve, dim3(grid), dim3(256), 0, s, accum, g, bg[0], bg[1], bg[2], out);
  return hipGetLastError();
}

}  // namespace wt
