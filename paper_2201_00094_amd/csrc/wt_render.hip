// Whole-frame kernels over a binned stream: build, evaluate and resolve fused per tile, and the one-pass render against
// the previous frame's coefficients.
#include <algorithm>

#include "wt_tile.h"

namespace wt {

// ------------------------------------------------------------------------------------------- conversion in place
//
// After the build each pixel and channel is a column of M + 1 FP64 endpoint masses in LDS (rows TP apart). One thread
// turns a column into the coefficients at storage precision (stored when dst is not null), their FP32 cells and the
// absorbance total, written over the same column: cells 2k and 2k + 1 in slot k < M/2, the total in slot M/2. A thread
// writes only the column it has read, so no barrier separates the two, no column waits in registers for the others,
// and a tile may hold more columns than the workgroup has threads.

// Cell j of the column at col (its pixel's slot in row 0 of the channel).
__device__ __forceinline__ float* cell_at(acc_t* col, uint32_t TP, uint32_t j) {
  return (float*)(col + (j >> 1) * TP) + (j & 1u);
}

template <int N>
__device__ __forceinline__ void put_cells(acc_t* col, uint32_t TP, const float (&v)[N]) {
#pragma unroll
  for (int k = 0; k < N / 2; ++k) *(float2*)(col + k * TP) = make_float2(v[2 * k], v[2 * k + 1]);
}

template <typename TS, int M>
__device__ __forceinline__ void column_to_cells(acc_t* col, uint32_t TP, TS* dst) {
  float v[M];
  const acc_t total = column_coeffs<M>([&](int m) { return col[m * TP]; },
                                       [&](int m, acc_t x) { v[m] = widen<TS>(narrow_d<TS>(x)); });
  if (dst) store_exact_row<TS, M>(dst, v);
  synth_regs<M>(v);
  put_cells<M>(col, TP, v);
  *(float*)(col + (M / 2) * TP) = (float)total;
}

template <int C, typename TS, int M>
__device__ __forceinline__ void tile_to_cells(const Geom& g, const TileRef& r, acc_t* le, TS* coeffs) {
  const uint32_t TP = g.tile_px;
  for (uint32_t q = threadIdx.x; q < TP * C; q += blockDim.x) {
    const uint32_t c = C == 1 ? 0 : q / TP, lp = q - c * TP;
    uint64_t p;
    TS* dst = coeffs && tile_pixel(g, r, lp, p) ? coeffs + (p * C + c) * M : nullptr;
    column_to_cells<TS, M>(le + (size_t)c * (M + 1) * TP + lp, TP, dst);
  }
}

// Packed storage: the coefficients as FP32 in place, then each pixel's words packed from its three channels, two at a time
// (a pixel's pairs are shared by the three threads of its columns), and decoded in place, then the cells in place.
// Consecutive lanes take consecutive pixels throughout, so the columns are read without bank conflicts; the words go
// through the rows of the first channel that the columns no longer use (M / 2 of them: just the tile's words; a pixel's
// pairs permuted by its low bits to spread over the banks) to be stored with consecutive lanes on consecutive words.
// (With consecutive lanes on consecutive words of a pixel in the packing, its six LDS accesses per word met in the same
// banks: glass 1366x768 render 368 us, 356 now, at rank 4 572 and 477, with depth bounds 550 and 521; 344 for FP32
// storage, 329 for FP16.)
template <int M>
__device__ __forceinline__ void e5_tile_to_cells(const Geom& g, const TileRef& r, acc_t* le, uint32_t* words) {
  constexpr uint32_t C = 3, K = M / 2;
  const uint32_t TP = g.tile_px, rows = (M + 1) * TP;
  for (uint32_t q = threadIdx.x; q < TP * C; q += blockDim.x) {
    const uint32_t c = q / TP;
    acc_t* col = le + (size_t)c * rows + (q - c * TP);
    float v[M];
    const acc_t total = column_coeffs<M>([&](int m) { return col[m * TP]; }, [&](int m, acc_t x) { v[m] = (float)x; });
    put_cells<M>(col, TP, v);
    *(float*)(col + K * TP) = (float)total;
  }
  __syncthreads();
  uint2* const stage = (uint2*)(le + (K + 1) * TP);
  for (uint32_t q = threadIdx.x; q < TP * C; q += blockDim.x) {
    const uint32_t c = q / TP, lp = q - c * TP;
    for (uint32_t k = c; k < K; k += C) {
      const float s0 = e5_sign(2 * k), s1 = e5_sign(2 * k + 1);
      float2* const f = (float2*)(le + lp + k * TP);
      const float2 a = f[0], b = f[rows], d = f[2 * rows];
      const uint2 w = make_uint2(e5_pack(s0 * a.x, s0 * b.x, s0 * d.x), e5_pack(s1 * a.y, s1 * b.y, s1 * d.y));
#pragma unroll
      for (uint32_t i = 0; i < C; ++i) f[i * rows] = make_float2(s0 * e5_unpack(w.x, i), s1 * e5_unpack(w.y, i));
      stage[lp * K + (k ^ (lp & (K - 1)))] = w;
    }
  }
  __syncthreads();
  if (words) {
    typedef unsigned int u32x2_any __attribute__((ext_vector_type(2), aligned(4)));
    for (uint32_t q = threadIdx.x; q < TP * K; q += blockDim.x) {
      const uint32_t lp = q / K, k = q & (K - 1);
      uint64_t p;
      if (!tile_pixel(g, r, lp, p)) continue;
      const uint2 w = stage[lp * K + (k ^ (lp & (K - 1)))];
      *(u32x2_any*)(words + p * M + 2 * k) = u32x2_any{w.x, w.y};
    }
  }
  for (uint32_t q = threadIdx.x; q < TP * C; q += blockDim.x) {
    const uint32_t c = q / TP;
    acc_t* col = le + (size_t)c * rows + (q - c * TP);
    float v[M];
#pragma unroll
    for (uint32_t k = 0; k < K; ++k) {
      const float2 pair = *(const float2*)(col + k * TP);
      v[2 * k] = pair.x;
      v[2 * k + 1] = pair.y;
    }
    synth_regs<M>(v);
    put_cells<M>(col, TP, v);
  }
}

template <int C, typename TS>
__device__ __forceinline__ void render_convert(const Geom& g, const TileRef& r, acc_t* le, TS* coeffs) {
  with_m(g, [&](auto mm) {
    if constexpr (is_e5<TS>::value)
      e5_tile_to_cells<decltype(mm)::value>(g, r, le, (uint32_t*)coeffs);
    else
      tile_to_cells<C, TS, decltype(mm)::value>(g, r, le, coeffs);
  });
}

// One pixel's results: out = colour + bg exp(-sum a), and its accumulation where accum is not null.
template <int C>
__device__ __forceinline__ void put_pixel(uint64_t p, const float (&colour)[3], const float (&suma)[C],
                                          const float (&bg)[3], float* __restrict__ accum, float* __restrict__ out) {
#pragma unroll
  for (int q = 0; q < 3; ++q) out[p * 3 + q] = colour[q] + bg[q] * __expf(-suma[C == 1 ? 0 : q]);
  if (!accum) return;
  float* a = accum + p * (C == 1 ? 4 : 8);
#pragma unroll
  for (int q = 0; q < 3; ++q) a[q] = colour[q];
  if constexpr (C == 3) a[3] = a[7] = 0.f;
#pragma unroll
  for (int c = 0; c < C; ++c) a[(C == 1 ? 3 : 4) + c] = suma[c];
}

// The results of the tile's pixels, from the colour rows and the totals the conversion left.
template <int C>
__device__ __forceinline__ void resolve_tile(const Geom& g, const TileRef& r, const acc_t* le, const acc_t* la,
                                             const float (&bg)[3], float* __restrict__ accum,
                                             float* __restrict__ out) {
  const uint32_t TP = g.tile_px;
  for (uint32_t lp = threadIdx.x; lp < TP; lp += blockDim.x) {
    uint64_t p;
    if (!tile_pixel(g, r, lp, p)) continue;
    float suma[C];
#pragma unroll
    for (int c = 0; c < C; ++c) suma[c] = *(const float*)(le + (size_t)(c * (g.M + 1) + g.M / 2) * TP + lp);
    const float colour[3] = {(float)la[lp], (float)la[TP + lp], (float)la[2 * TP + lp]};
    put_pixel<C>(p, colour, suma, bg, accum, out);
  }
}

// ------------------------------------------------------------------------------------------- render, M <= 32

// Records whose pixel, cell and offset a thread keeps in registers from the build to the evaluation, which then reads
// only their colours: a tile of up to kKept * blockDim.x records has its heads read from memory once instead of twice
// (three times with depth bounds); a deeper one re-reads the others, the latest built first.
// As many as the conversion between the two leaves registers for (128 per thread at 1024 threads).
template <int C, bool TIGHT>
constexpr int kept() { return C == 1 && !TIGHT ? 16 : 12; }

// One kept record: pixel | cell << 16, the offset in the cell, and with depth bounds 1 - t (rounded from FP64 on its
// own; otherwise 1 - t is exact or rounds the same way again).
template <bool TIGHT>
struct Kept {
  uint32_t key;
  float t, omt;
};
template <>
struct Kept<false> {
  uint32_t key;
  float t;
};

template <int C>
__device__ __forceinline__ void shade_cells(acc_t* le, acc_t* la, const Geom& g, uint32_t lp, uint32_t j, float t,
                                            float omt, const float (&w)[3]) {
  shade_add<C>(la, g.tile_px, lp, j, t, omt, w, [&](int c, uint32_t jj) {
    return *cell_at(le + (size_t)c * (g.M + 1) * g.tile_px + lp, g.tile_px, jj);
  });
}

template <int C>
__device__ __forceinline__ void shade_record(const Binned& b, const Geom& g, uint32_t i, acc_t* le, acc_t* la,
                                             const uint32_t* lb) {
  Head<C> f;
  float w[3];
  load_tail<false>(b, i, w);
  if (!load_head<C>(b, i, f)) return;
  uint32_t j;
  float t, omt;
  cell_coord(f.x, lb, g.tile_px, f.lp, g.M, j, t, omt);
  shade_cells<C>(le, la, g, f.lp, j, t, omt, w);
}

// LDS: endpoint masses [C * (M + 1)][TP] FP64 (then cells and totals in their place), colour sums [3][TP] FP64, depth
// bounds [2][TP] (TIGHT).
template <int C, typename TS, bool TIGHT>
__global__ __launch_bounds__(kTileThreads) void k_render(Binned b, Geom g, TS* __restrict__ coeffs, float bg0,
                                                         float bg1, float bg2, float* __restrict__ accum,
                                                         float* __restrict__ out) {
  extern __shared__ acc_t smem_d[];
  constexpr int K = kept<C, TIGHT>(), U = 4;
  constexpr bool kNT = last_read_nt<C>();
  const uint32_t TP = g.tile_px, T = blockDim.x;
  uint32_t tile;
  if (!binned_ok(b, g, tile)) return;
  const TileRef r = tile_ref(g, b, tile);
  const float bg[3] = {bg0, bg1, bg2};
  acc_t* le = smem_d;
  acc_t* la = smem_d + C * (g.M + 1) * TP;
  uint32_t* lb = TIGHT ? (uint32_t*)(la + 3 * TP) : nullptr;
  const uint32_t rest = r.end - min(r.end - r.beg, (uint32_t)K * T);  // the records from here on are kept
  const uint32_t i0 = rest + threadIdx.x;
  Kept<TIGHT> kept[K];
  for (uint32_t e = threadIdx.x; e < (C * (g.M + 1) + 3) * TP; e += T) smem_d[e] = 0.0;
  if (g.serial) {
    if constexpr (TIGHT) bounds_tile<C>(b, g, r, lb);
    __syncthreads();
    build_ep_tile<C>(b, g, r, le, lb);
  } else if constexpr (TIGHT) {
    // bounds, then masses, of the kept records from one read
    Head<C> f[K];
    bounds_clear(lb, TP);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
      kept[k].key = kNoRecord;
      if (i0 + k * T < r.end && load_head<C, kNT>(b, i0 + k * T, f[k])) kept[k].key = f[k].lp;
    }
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (kept[k].key != kNoRecord) bounds_add(lb, TP, f[k].lp, f[k].x);
    bounds_range<C>(b, r.beg, rest, lb, TP);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (kept[k].key == kNoRecord) continue;
      uint32_t j;
      cell_coord(f[k].x, lb, TP, f[k].lp, g.M, j, kept[k].t, kept[k].omt);
      kept[k].key |= j << 16;
      ep_add<C>(le, TP, g.M + 1, f[k].lp, j, kept[k].t, kept[k].omt, f[k].al);
    }
    build_ep_range<C>(b, g, r.beg, rest, le, lb);
  } else {
    __syncthreads();
    build_ep_range<C>(b, g, r.beg, rest, le, nullptr);
#pragma unroll
    for (int k = 0; k < K; ++k) kept[k].key = kNoRecord;
#pragma unroll
    for (int k0 = 0; k0 < K; k0 += U) {
      if (rest + k0 * T >= r.end) break;
      Head<C> f[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t i = i0 + (k0 + u) * T;
        if (load_head<C, kNT>(b, min(i, r.end - 1), f[u]) && i < r.end) kept[k0 + u].key = f[u].lp;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        Kept<TIGHT>& kr = kept[k0 + u];
        if (kr.key == kNoRecord) continue;
        uint32_t j;
        float omt;
        cell_coord(f[u].x, nullptr, TP, f[u].lp, g.M, j, kr.t, omt);
        kr.key |= j << 16;
        ep_add<C>(le, TP, g.M + 1, f[u].lp, j, kr.t, omt, f[u].al);
      }
    }
  }
  __syncthreads();
  render_convert<C, TS>(g, r, le, coeffs);
  __syncthreads();
  if (!serial_records(g, r.beg, r.end, [&](uint32_t i) { shade_record<C>(b, g, i, le, la, lb); })) {
#pragma unroll
    for (int k0 = 0; k0 < K; k0 += U) {
      if (rest + k0 * T >= r.end) break;
      float w[U][3];
#pragma unroll
      for (int u = 0; u < U; ++u) load_tail<kNT>(b, min(i0 + (k0 + u) * T, r.end - 1), w[u]);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const Kept<TIGHT>& kr = kept[k0 + u];
        if (kr.key == kNoRecord) continue;
        float omt;
        if constexpr (TIGHT)
          omt = kr.omt;
        else
          omt = 1.f - kr.t;
        shade_cells<C>(le, la, g, kr.key & 0xffffu, kr.key >> 16, kr.t, omt, w[u]);
      }
    }
    Head<C> f[U];
    float w[U][3];
    for_records<U, true>(
        r.beg, rest,
        [&](uint32_t i, int u) {
          load_tail<kNT>(b, i, w[u]);
          return load_head<C, kNT>(b, i, f[u]);
        },
        [&](int u) {
          uint32_t j;
          float t, omt;
          cell_coord(f[u].x, lb, TP, f[u].lp, g.M, j, t, omt);
          shade_cells<C>(le, la, g, f[u].lp, j, t, omt, w[u]);
        });
  }
  __syncthreads();
  resolve_tile<C>(g, r, le, la, bg, accum, out);
}

// ------------------------------------------------------------------------------------------- render, M > 32

// The direct N + 2 updates: coefficients [C * M][TP] FP64, rounded to storage precision in place (and stored when
// coeffs is not null), accumulation rows [AL][TP] FP64, depth bounds. Bound by its LDS atomics and reads (2 (N + 2) of a
// fragment) and by the clearing and rounding of M sums per pixel. (512x512 at 8 per pixel: rank 8 with 256 threads and one
// record in flight 0.77 ms, with 1024 and four 0.72; rank 10, three channels, 7.2 and 5.8.)
template <int C, typename TS>
__global__ __launch_bounds__(kTileThreads) void k_render_direct(Binned b, Geom g, TS* __restrict__ coeffs, float bg0,
                                                                float bg1, float bg2, float* __restrict__ accum,
                                                                float* __restrict__ out) {
  extern __shared__ acc_t smem_d[];
  const uint32_t TP = g.tile_px;
  uint32_t tile;
  if (!binned_ok(b, g, tile)) return;
  const TileRef r = tile_ref(g, b, tile);
  const float bg[3] = {bg0, bg1, bg2};
  acc_t* lc = smem_d;
  acc_t* la = smem_d + C * g.M * TP;
  uint32_t* lb = g.tight ? (uint32_t*)(la + g.AL * TP) : nullptr;
  if (lb) bounds_tile<C>(b, g, r, lb);
  for (uint32_t e = threadIdx.x; e < (C * g.M + g.AL) * TP; e += blockDim.x) smem_d[e] = 0.0;
  __syncthreads();
  build_tile<C>(b, g, r, lc, lb);
  __syncthreads();
  coeff_tile_io<C, TS, 2>(g, r, lc, coeffs);
  __syncthreads();
  auto shade = [&](const Head<C>& f, const float (&w)[3]) {
    uint32_t j;
    float t, omt;
    cell_coord(f.x, lb, TP, f.lp, g.M, j, t, omt);
    shade_add<C>(la, TP, f.lp, j, t, omt, w,
                 [&](int c, uint32_t jj) { return cell_from_coeffs(lc + (c * g.M) * TP + f.lp, TP, g, jj); });
#pragma unroll
    for (int c = 0; c < C; ++c) atomicAdd(la + (3 + c) * TP + f.lp, (acc_t)f.al[c]);
  };
  if (!serial_records(g, r.beg, r.end, [&](uint32_t i) {
        Head<C> f;
        float w[3];
        load_tail<false>(b, i, w);
        if (load_head<C>(b, i, f)) shade(f, w);
      })) {
    constexpr int U = kEvalUnroll;
    constexpr bool kNT = last_read_nt<C>();
    Head<C> f[U];
    float w[U][3];
    for_records<U>(
        r.beg, r.end,
        [&](uint32_t i, int u) {
          load_tail<kNT>(b, i, w[u]);
          return load_head<C, kNT>(b, i, f[u]);
        },
        [&](int u) { shade(f[u], w[u]); });
  }
  __syncthreads();
  for (uint32_t lp = threadIdx.x; lp < TP; lp += blockDim.x) {
    uint64_t p;
    if (!tile_pixel(g, r, lp, p)) continue;
    float suma[C];
#pragma unroll
    for (int c = 0; c < C; ++c) suma[c] = (float)la[(3 + c) * TP + lp];
    const float colour[3] = {(float)la[lp], (float)la[TP + lp], (float)la[2 * TP + lp]};
    put_pixel<C>(p, colour, suma, bg, accum, out);
  }
}

// ------------------------------------------------------------------------------------------- one pass, previous frame
//
// The single-pass variant the paper proposes as future work: the frame's coefficients are built in the same pass
// that shades its fragments, so the shading reconstructs visibility from the PREVIOUS frame's coefficients, read
// at each pixel's reprojected position (an integer pixel map supplied by the caller; identity without one). Each
// binned record is read once instead of twice.

// FP32 cells [C*M][TP] of the previous frame for the tile's pixels: pixel p reads the previous buffer at
// map[p] (p without a map). Zero (no history: visibility 1) without a previous buffer, for a map entry >= P and
// for pixels outside the frame.
template <int C, typename TS, int M>
__device__ __forceinline__ void prev_cells(const Geom& g, const TileRef& r, const TS* prev, const uint32_t* map,
                                           float* lc) {
  const uint32_t TP = g.tile_px;
  for (uint32_t q = threadIdx.x; q < TP * C; q += blockDim.x) {
    const uint32_t c = q / TP, lp = q - c * TP;
    uint64_t p;
    uint32_t src = 0xffffffffu;
    if (prev && tile_pixel(g, r, lp, p)) src = map ? map[p] : (uint32_t)p;
    float v[M];
    if (src < g.P) {
      if constexpr (is_e5<TS>::value) {
        uint32_t w[M];
        load_row<uint32_t, M>((const uint32_t*)prev + (uint64_t)src * M, w);
#pragma unroll
        for (int m = 0; m < M; ++m) v[m] = e5_sign(m) * e5_unpack(w[m], c);
      } else {
        TS s[M];
        load_row<TS, M>(prev + ((uint64_t)src * C + c) * M, s);
#pragma unroll
        for (int m = 0; m < M; ++m) v[m] = widen<TS>(s[m]);
      }
      synth_regs<M>(v);
    } else {
#pragma unroll
      for (int m = 0; m < M; ++m) v[m] = 0.f;
    }
#pragma unroll
    for (int m = 0; m < M; ++m) lc[(c * M + m) * TP + lp] = v[m];
  }
}

// One fragment of the single pass: its two endpoint masses into this frame's build (le, [C*(M+1)][TP] FP64) and
// its colour, weighted by the previous frame's visibility (lc), into the colour sums (la, [3][TP] FP64).
template <int C>
__device__ __forceinline__ void temporal_add(acc_t* le, const float* lc, acc_t* la, const Geom& g,
                                             const Head<C>& f, const float (&w)[3]) {
  const uint32_t TP = g.tile_px;
  uint32_t j;
  float t, omt;
  cell_coord(f.x, nullptr, TP, f.lp, g.M, j, t, omt);
  ep_add<C>(le, TP, g.M + 1, f.lp, j, t, omt, f.al);
  shade_add<C>(la, TP, f.lp, j, t, omt, w,
               [&](int c, uint32_t jj) { return lc[(c * g.M + jj) * TP + f.lp]; });
}

// LDS: endpoint masses [C*(M+1)][TP] FP64 (then this frame's cells and totals in their place), colour sums
// [3][TP] FP64, previous cells [C*M][TP] FP32. prev and coeffs may be the same buffer when map is null: a tile
// reads the previous coefficients of its own pixels before it writes theirs.
template <int C, typename TS>
__global__ __launch_bounds__(kTileThreads) void k_render_temporal(Binned b, Geom g, const TS* prev,
                                                                  const uint32_t* __restrict__ map, TS* coeffs,
                                                                  float bg0, float bg1, float bg2,
                                                                  float* __restrict__ out) {
  extern __shared__ acc_t smem_d[];
  const uint32_t TP = g.tile_px;
  uint32_t tile;
  if (!binned_ok(b, g, tile)) return;
  const TileRef r = tile_ref(g, b, tile);
  const float bg[3] = {bg0, bg1, bg2};
  acc_t* le = smem_d;
  acc_t* la = smem_d + C * (g.M + 1) * TP;
  float* lc = (float*)(la + 3 * TP);
  for (uint32_t e = threadIdx.x; e < (C * (g.M + 1) + 3) * TP; e += blockDim.x) smem_d[e] = 0.0;
  with_m(g, [&](auto mm) { prev_cells<C, TS, decltype(mm)::value>(g, r, prev, map, lc); });
  __syncthreads();
  constexpr bool kNT = last_read_nt<C>();
  auto one = [&](uint32_t i) {
    Head<C> f;
    float w[3];
    load_tail<kNT>(b, i, w);
    if (load_head<C, kNT>(b, i, f)) temporal_add<C>(le, lc, la, g, f, w);
  };
  const bool serial = serial_records(g, r.beg, r.end, one);
  Head<C> f[kEvalUnroll];
  float w[kEvalUnroll][3];
  if (!serial)
    for_records<kEvalUnroll>(
        r.beg, r.end,
        [&](uint32_t i, int u) {
          load_tail<kNT>(b, i, w[u]);
          return load_head<C, kNT>(b, i, f[u]);
        },
        [&](int u) { temporal_add<C>(le, lc, la, g, f[u], w[u]); });
  __syncthreads();
  render_convert<C, TS>(g, r, le, coeffs);
  __syncthreads();
  resolve_tile<C>(g, r, le, la, bg, nullptr, out);
}

// ------------------------------------------------------------------------------------------- launchers

// LDS of the render (with_accum) and build kernels: endpoint masses (+ three colour sums), or coefficient
// sums (+ AL accumulations).
size_t lds_tile_bytes(const Geom& g, bool with_accum) {
  const size_t bounds = g.tight ? 8ull * g.tile_px : 0;
  if (g.ep) return (size_t)g.tile_px * (g.C * (g.M + 1) + (with_accum ? 3 : 0)) * sizeof(acc_t) + bounds;
  return (size_t)g.tile_px * (g.C * g.M + (with_accum ? g.AL : 0)) * sizeof(acc_t) + bounds;
}

size_t lds_temporal_bytes(const Geom& g) {
  return (size_t)g.tile_px * ((g.C * (g.M + 1) + 3) * sizeof(acc_t) + g.C * g.M * sizeof(float));
}

hipError_t launch_render(const Geom& g, const Binned& b, const float* bg, void* coeffs, float* accum, float* out,
                         hipStream_t s) {
  const size_t lds = lds_tile_bytes(g, true);
  return dispatch(g, [&](auto cc, auto* tag) {
    constexpr int C = decltype(cc)::value;
    using TS = std::remove_pointer_t<decltype(tag)>;
    auto k = g.tight ? k_render<C, TS, true> : k_render<C, TS, false>;
    if constexpr (!is_e5<TS>::value) {
      if (!g.ep) k = k_render_direct<C, TS>;
    }
    hipError_t err = prep(k, lds);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(k, dim3(g.ntiles), dim3(g.tthreads), lds, s, b, g, (TS*)coeffs, bg[0], bg[1], bg[2], accum, out);
    return hipGetLastError();
  });
}

hipError_t launch_render_temporal(const Geom& g, const Binned& b, const float* bg, const void* prev,
                                  const uint32_t* map, void* coeffs, float* out, hipStream_t s) {
  if (!g.ep) return hipErrorNotSupported;  // the API limits the one-pass render to the endpoint path
  const size_t lds = lds_temporal_bytes(g);
  return dispatch(g, [&](auto cc, auto* tag) {
    constexpr int C = decltype(cc)::value;
    using TS = std::remove_pointer_t<decltype(tag)>;
    auto k = k_render_temporal<C, TS>;
    hipError_t err = prep(k, lds);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(k, dim3(g.ntiles), dim3(g.tthreads), lds, s, b, g, (const TS*)prev, map, (TS*)coeffs,
                       bg[0], bg[1], bg[2], out);
    return hipGetLastError();
  });
}

}  // namespace wt
