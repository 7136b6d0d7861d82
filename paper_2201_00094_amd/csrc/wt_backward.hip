// Gradient of the resolve with respect to alpha and colour, one workgroup per screen tile.
//
// Forward, per pixel and visibility channel c (colour channels q with c(q) = c):
//   out_q = sum_i alpha_i c_{i,q} v_i + bg_q exp(-sum_i a_i),  v_i = exp(-A~(x_i)),  a_i = -ln(1 - alpha_i),
//   A~(z) = (1 - t) Abar_{j-1} + t Abar_j  (u = M z, j = min(floor(u), M-1), t = u - j).
// With g = dL/dout:
//   dL/dc_{i,q}  = g_q alpha_i v_i
//   dL/dA~(x_i)  = -s_i,  s_i = alpha_i v_i sum_q g_q c_{i,q}
//   cell adjoint  Abar'_m = sum_i -s_i dA~(x_i)/dAbar_m   (two cells per fragment: (1 - t), t)
//   dL/da_i      = sum_m Abar'_m dAbar_m/da_i - exp(-sum a) sum_q g_q bg_q
//   dL/dalpha_i  = v_i sum_q g_q c_{i,q} + dL/da_i / (1 - alpha_i)
// The map a_i -> Abar_m is the build (section 2.3.1) followed by the Haar synthesis; composed, it is the
// average of the fragment's step over cell m, dAbar_m/da_i = clamp((m + 1) - M x_i, 0, 1). Its adjoint is
// therefore a suffix sum of the cell adjoints: with S_m = sum_{m' >= m} Abar'_{m'} and j = floor(M x_i),
//   sum_m Abar'_m dAbar_m/da_i = (j + 1 - M x_i) Abar'_j + S_{j+1},
// which needs O(M) work per pixel and O(1) per fragment for any rank.
#include <algorithm>

#include "wt_tile.h"

namespace wt {

// Record i of a binning made with stream indices (alpha and plain colour).
template <int C>
struct GradRecord {
  Head<C> h;  // al: alpha
  float rgb[3];
  uint32_t src;
};

template <int C, bool NT>
__device__ __forceinline__ bool load_grad(const Binned& b, uint32_t i, GradRecord<C>& f) {
  const uint32_t* t = b.tail + (uint64_t)i * b.DT;
#pragma unroll
  for (int q = 0; q < 3; ++q) f.rgb[q] = __uint_as_float(load_word<NT>(t + q));
  f.src = load_word<NT>(t + 3);
  return load_head<C, NT>(b, i, f.h);
}

// What the second pass needs of a fragment: where it is (pixel, cell, offsets), its alpha, and per channel
// v sum_q g_q c_q and alpha v.
template <int C>
struct GradKept {
  uint32_t key, src;  // pixel | cell << 16; the stream index
  float t, omt, al[C], vg[C], av[C];
};

// Fragments whose GradKept a thread holds in registers between the passes: the second pass reads nothing for them and
// takes no exponential. (512x512, 32 fragments per pixel: gradient with its binning 436 us at four, 416 at eight, 388 at
// sixteen, all that 128 registers hold; the kernel before, 512 threads and one record in flight per thread, with the
// gradients cleared first, 537. Writing the gradients at their scattered stream positions is 140 of the kernel's 265 us;
// as non-temporal stores three channels take 4.5 ms instead of 2.1, 1024x768.)
template <int C>
constexpr int grad_kept() { return C == 1 ? 16 : 8; }

struct GradTile {
  double* adj;        // [C * M][TP] cell adjoints, then their suffix sums
  const float* cell;  // [C * M][TP] cell values, or coefficients where M > 32
  const float* grad;  // [3][TP] dL/dout
  const float* back;  // [C][TP] background transmittance
  const uint32_t* lb; // [2][TP] depth bounds, or null
};

// First pass, one fragment: its visibility, its terms of the cell adjoints, and what the second pass needs.
template <int C, bool CELLS>
__device__ __forceinline__ void grad_first(const GradTile& s, const Geom& g, const GradRecord<C>& f, bool add,
                                           GradKept<C>& k) {
  const uint32_t TP = g.tile_px, lp = f.h.lp;
  uint32_t j;
  cell_coord(f.h.x, s.lb, TP, lp, g.M, j, k.t, k.omt);
  k.key = lp | j << 16;
  k.src = f.src;
  const float gq[3] = {s.grad[lp], s.grad[TP + lp], s.grad[2 * TP + lp]};
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const float* cf = s.cell + (c * g.M) * TP + lp;
    const float hi = CELLS ? cf[j * TP] : cell_from_coeffs(cf, TP, g, j);
    const uint32_t jb = j ? j - 1 : 0u;
    const float below = CELLS ? cf[jb * TP] : cell_from_coeffs(cf, TP, g, jb);
    const float v = __expf(-fmaf(k.t, hi, k.omt * (j ? below : 0.f)));
    const float alc = alpha_clamped(f.h.al[c]);
    const float gc = (C == 1) ? (gq[0] * f.rgb[0] + gq[1] * f.rgb[1] + gq[2] * f.rgb[2]) : gq[c] * f.rgb[c];
    k.al[c] = f.h.al[c];
    k.vg[c] = v * gc;
    k.av[c] = alc * v;
    if (add) {
      const float sg = alc * v * gc;
      double* a = s.adj + (c * g.M) * TP + lp;
      if (j) atomicAdd(a + (j - 1) * TP, (double)(-sg * k.omt));
      atomicAdd(a + j * TP, (double)(-sg * k.t));
    }
  }
}

// Second pass, one fragment: its gradients, written at its stream position.
template <int C>
__device__ __forceinline__ void grad_second(const GradTile& s, const Geom& g, const float (&bg)[3],
                                            const GradKept<C>& k, float* __restrict__ grad_alpha,
                                            float* __restrict__ grad_rgb) {
  const uint32_t TP = g.tile_px, lp = k.key & 0xffffu, j = k.key >> 16;
  const uint64_t src = k.src;
  const float gq[3] = {s.grad[lp], s.grad[TP + lp], s.grad[2 * TP + lp]};
  float out[3];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const double* S = s.adj + (c * g.M) * TP + lp;
    const double Sj = S[j * TP];
    const double Sj1 = (j + 1 < g.M) ? S[(j + 1) * TP] : 0.0;
    const float through_cells = (float)((double)k.omt * (Sj - Sj1) + Sj1);
    const float gbg = (C == 1) ? (gq[0] * bg[0] + gq[1] * bg[1] + gq[2] * bg[2]) : gq[c] * bg[c];
    const float dLda = through_cells - gbg * s.back[c * TP + lp];
    const bool inside = k.al[c] > 0.f && k.al[c] < kAlphaMax;
    grad_alpha[src * C + c] = inside ? k.vg[c] + dLda / (1.f - alpha_clamped(k.al[c])) : 0.f;
    if (C == 1) {
#pragma unroll
      for (int q = 0; q < 3; ++q) out[q] = gq[q] * k.av[c];
    } else {
      out[c] = gq[c] * k.av[c];
    }
  }
#pragma unroll
  for (int q = 0; q < 3; ++q) grad_rgb[src * 3 + q] = out[q];
}

// Cells of one pixel and channel from its stored row, or its coefficients as they are (M > 32), into column lc.
template <typename TS, int M>
__device__ __forceinline__ void grad_cells(const TS* row, uint32_t c, float* lc, uint32_t TP) {
  float v[M];
#pragma unroll
  for (int m = 0; m < M; ++m) v[m] = 0.f;
  if (row) {
    if constexpr (is_e5<TS>::value) {
      uint32_t w[M];
      load_row<uint32_t, M>((const uint32_t*)row, w);
#pragma unroll
      for (int m = 0; m < M; ++m) v[m] = e5_sign(m) * e5_unpack(w[m], c);
    } else {
      TS s[M];
      load_row<TS, M>(row, s);
#pragma unroll
      for (int m = 0; m < M; ++m) v[m] = widen<TS>(s[m]);
    }
    synth_regs<M>(v);
  }
#pragma unroll
  for (int m = 0; m < M; ++m) lc[m * TP] = v[m];
}

// LDS rows of TP values: cell adjoints [C*M] FP64, cell values [C*M] FP32, dL/dout [3], background transmittance [C],
// depth bounds [2].
template <int C, typename TS, bool CELLS>
__global__ __launch_bounds__(kTileThreads) void k_backward(Binned b, Geom g, const TS* __restrict__ coeffs,
                                                           const float* __restrict__ accum, float bg0, float bg1,
                                                           float bg2, const float* __restrict__ grad_out,
                                                           float* __restrict__ grad_alpha,
                                                           float* __restrict__ grad_rgb) {
  extern __shared__ double smem_b[];
  constexpr int K = grad_kept<C>(), U = 4;
  constexpr bool kNT = last_read_nt<C>();
  const uint32_t TP = g.tile_px, per = C * g.M, T = blockDim.x;
  double* ladj = smem_b;
  float* lc = (float*)(ladj + per * TP);
  float* lg = lc + per * TP;
  float* lT = lg + 3 * TP;
  uint32_t* lb = g.tight ? (uint32_t*)(lT + C * TP) : nullptr;
  uint32_t tile;
  if (!binned_ok(b, g, tile)) return;
  const TileRef r = tile_ref(g, b, tile);
  const float bg[3] = {bg0, bg1, bg2};
  for (uint32_t e = threadIdx.x; e < per * TP; e += T) ladj[e] = 0.0;
  for (uint32_t lp = threadIdx.x; lp < TP; lp += T) {
    uint64_t p;
    const bool in = tile_pixel(g, r, lp, p);
    for (uint32_t q = 0; q < 3; ++q) lg[q * TP + lp] = in ? grad_out[p * 3 + q] : 0.f;
    for (uint32_t c = 0; c < C; ++c)
      lT[c * TP + lp] = in ? __expf(-accum[p * g.AW + (C == 1 ? 3 : 4 + c)]) : 0.f;
  }
  if constexpr (CELLS) {
    with_m(g, [&](auto mm) {
      constexpr int M = decltype(mm)::value;
      for (uint32_t q = threadIdx.x; q < TP * C; q += T) {
        const uint32_t c = C == 1 ? 0 : q / TP, lp = q - c * TP;
        uint64_t p;
        const bool in = tile_pixel(g, r, lp, p);
        // packed storage: the three channels share the pixel's row of words
        const TS* row = in ? coeffs + (is_e5<TS>::value ? p * M : (p * C + c) * M) : nullptr;
        grad_cells<TS, M>(row, c, lc + (c * M) * TP + lp, TP);
      }
    });
  } else {
    coeff_tile_io<C, TS, 0>(g, r, lc, const_cast<TS*>(coeffs));
  }
  __syncthreads();
  if (lb) bounds_tile<C>(b, g, r, lb);
  const GradTile s{ladj, lc, lg, lT, lb};
  const uint32_t rest = g.serial ? r.end : r.end - min(r.end - r.beg, (uint32_t)K * T);  // kept from here on
  const uint32_t i0 = rest + threadIdx.x;
  // pass 1: cell adjoints
  GradKept<C> kept[K];
  bool ok[K];
  GradRecord<C> f[U];
  if (serial_records(g, r.beg, r.end, [&](uint32_t i) {
        GradRecord<C> one;
        GradKept<C> k;
        if (load_grad<C, false>(b, i, one)) grad_first<C, CELLS>(s, g, one, true, k);
      })) {
  } else {
    for_records<U>(
        r.beg, rest, [&](uint32_t i, int u) { return load_grad<C, false>(b, i, f[u]); },
        [&](int u) {
          GradKept<C> k;
          grad_first<C, CELLS>(s, g, f[u], true, k);
        });
  }
#pragma unroll
  for (int k = 0; k < K; ++k) {
    ok[k] = false;
    kept[k].src = kNoRecord;
  }
#pragma unroll
  for (int k0 = 0; k0 < K; k0 += U) {
    if (rest + k0 * T >= r.end) break;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t i = i0 + (k0 + u) * T;
      ok[k0 + u] = load_grad<C, kNT>(b, min(i, r.end - 1), f[u]) && i < r.end;
      if (i < r.end) kept[k0 + u].src = f[u].src;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (ok[k0 + u]) grad_first<C, CELLS>(s, g, f[u], true, kept[k0 + u]);
  }
  __syncthreads();
  // suffix sums of the cell adjoints
  for (uint32_t q = threadIdx.x; q < TP * C; q += T) {
    const uint32_t c = C == 1 ? 0 : q / TP, lp = q - c * TP;
    double* adj = ladj + (c * g.M) * TP + lp;
    double run = 0.0;
#pragma unroll 8
    for (int m = (int)g.M - 1; m >= 0; --m) {
      run += adj[m * TP];
      adj[m * TP] = run;
    }
  }
  __syncthreads();
  // pass 2: per-fragment gradients; a dropped fragment's are zero
  auto dropped = [&](uint32_t at) {
    const uint64_t src = at;
#pragma unroll
    for (int c = 0; c < C; ++c) grad_alpha[src * C + c] = 0.f;
#pragma unroll
    for (int q = 0; q < 3; ++q) grad_rgb[src * 3 + q] = 0.f;
  };
#pragma unroll
  for (int k = 0; k < K; ++k) {
    if (ok[k])
      grad_second<C>(s, g, bg, kept[k], grad_alpha, grad_rgb);
    else if (kept[k].src != kNoRecord)
      dropped(kept[k].src);
  }
  for_records<U, true>(
      r.beg, rest,
      [&](uint32_t i, int u) {
        if (!load_grad<C, kNT>(b, i, f[u])) f[u].h.lp = kNoRecord;
        return true;
      },
      [&](int u) {
        if (f[u].h.lp == kNoRecord) {
          dropped(f[u].src);
          return;
        }
        GradKept<C> k;
        grad_first<C, CELLS>(s, g, f[u], false, k);
        grad_second<C>(s, g, bg, k, grad_alpha, grad_rgb);
      });
}

size_t lds_backward_bytes(const Geom& g) {
  return (size_t)g.tile_px * (12 * g.C * g.M + 4 * (3 + g.C) + (g.tight ? 8 : 0));
}

hipError_t launch_backward(const Geom& g, const Binned& b, const void* coeffs, const float* accum, const float* bg,
                           const float* grad_out, float* grad_alpha, float* grad_rgb, hipStream_t s) {
  const size_t lds = lds_backward_bytes(g);
  if (lds > kLdsBytes) return hipErrorNotSupported;
  return dispatch(g, [&](auto cc, auto* tag) {
    constexpr int C = decltype(cc)::value;
    using TS = std::remove_pointer_t<decltype(tag)>;
    auto k = g.M <= 32 ? k_backward<C, TS, true> : k_backward<C, TS, false>;
    hipError_t err = prep(k, lds);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(k, dim3(g.ntiles), dim3(g.tthreads), lds, s, b, g, (const TS*)coeffs, accum, bg[0], bg[1], bg[2],
                       grad_out, grad_alpha, grad_rgb);
    return hipGetLastError();
  });
}

}  // namespace wt
