// Ingest and screen-tile binning of an unordered fragment stream.
//
// The paper builds and evaluates inside a raster pipeline, where the fragments of one screen region arrive on
// the same shader core (section 2.1). A stored stream carries no such locality, and on this GPU per-fragment
// random atomics into a frame-sized coefficient buffer run at a few billion fragments per second. So the
// stream is first regrouped by screen tile with a counting sort (histogram, scan, scatter), after which every
// per-pixel update of the build and evaluate passes happens in the LDS of the compute unit that owns the tile.
//
// Kernels:
//   k_hist_lds        pixel ids (4 B/fragment) -> per-(class, tile) counts in an LDS table (in passes of tile
//                     ranges for very large frames); range drops counted.
//   k_scan            exclusive scan of the counts, tile-major over (tile, class), into segment offsets and write
//                     cursors; tile order for the tile kernels (heaviest first).
//   k_scatter_staged  one chunk (8 fragments per thread) per workgroup: vector loads into registers, LDS
//                     rank per tile, records placed in LDS in tile order in rounds, one cursor reservation per tile
//                     present in a round just before the round is written record by record with consecutive lanes
//                     on consecutive records (head array, then tail array), so each tile's run is written
//                     coalesced.
//   k_scatter_stream  the same with the whole chunk staged and one workgroup per compute unit that takes chunk after
//                     chunk, the next one's loads in flight while it writes (wherever the tables fit).
//   Frames with more than kTwoLevelTiles tiles: a chunk would touch most tiles about once, so the stream is
//   binned into super-tiles of SW x SH tiles first (k_super_counts, k_scan and k_scatter_stream or k_scatter_staged
//   over the super-tile geometry), then k_split moves each super-tile's records into its tiles without atomics.
//   k_hist_global,    one global atomic per fragment (beyond kMaxLdsBins super-tiles).
//   k_scatter_global
// A chunk's class is chunk % NX in both the histogram and the scatter; a scatter workgroup takes chunks of one class,
// which is also the XCD the workgroup runs on, so each (bin, class) run is written from a single L2.
// NaN fragments are counted as dropped and still binned; the tile kernels skip them.

#include <algorithm>

#include "wt_common.h"

namespace wt {

// Super-tiles of a frame of tx x ty tiles that is binned in two levels: SW (a power of two) x SH tiles, at most kMaxSub,
// at most kMaxSupers of them (as many as it takes when that cannot be), chosen so that the split, which gives a compute
// unit one super-tile at a time, ends with full rounds. Returns the tiles on the fullest unit.
static uint64_t pick_supers(uint32_t tx, uint32_t ty, uint32_t& lSW, uint32_t& SH) {
  uint64_t best = ~0ull, fewest = ~0ull;
  for (uint32_t l = 1; l <= 3; ++l) {
    for (uint32_t sh = 2; (sh << l) <= kMaxSub; ++sh) {
      const uint64_t n = (uint64_t)(((tx - 1) >> l) + 1) * ((ty - 1) / sh + 1);
      const uint64_t cost = n <= kMaxSupers ? (n + kComputeUnits - 1) / kComputeUnits * (sh << l) : ~0ull;
      if (cost < best || (best == ~0ull && n < fewest)) {
        best = cost;
        fewest = n;
        lSW = l;
        SH = sh;
      }
    }
  }
  return best == ~0ull ? (fewest + kComputeUnits - 1) / kComputeUnits * (SH << lSW) : best;
}

// LDS of a tile's pixel. Forward: FP64 endpoint masses (M + 1 per channel) and three FP64 colour sums, or, for M > 32, FP64
// coefficient sums plus FP64 accumulations; the one-pass render adds the previous frame's FP32 cells (M <= 32 and no depth
// bounds are checked by the API). Backward: FP32 cells, FP64 cell adjoints and per-pixel gradient data. Depth bounds are
// two FP32.
static uint32_t tile_px_bytes(const Geom& g, bool backward) {
  return (backward ? 12 * g.C * g.M + 4 * (3 + g.C)
          : g.ep   ? 8 * g.C * (g.M + 1) + 24 + (g.temporal ? 4 * g.C * g.M : 0)
                   : 8 * (g.C * g.M + g.AL)) + (g.tight ? 8 : 0);
}

// The multiplier of row_tile for tiles TH rows high, or 0 where its conditions do not hold.
static uint32_t row_multiplier(uint32_t H, uint32_t TH) {
  const uint32_t m = ((1u << 20) + TH - 1) / TH;
  return H <= (1u << 14) && TH <= 64 && (uint64_t)(H - 1) * m >> 32 == 0 ? m : 0;
}

static uint32_t log2_floor(uint32_t v) { return 31 - __builtin_clz(v); }

// Tile of a frame, from the LDS bytes per pixel: TW a power of two, TH any height in [TW/2, 2 TW), and the workgroup size
// of the tile kernels.
//
// A compute unit takes its tiles one after the other (its LDS holds one large tile, or several small ones that share its
// lanes), so a frame costs about (tiles on the fullest unit) x (pixels per tile + what a tile costs by itself), the
// latter worth about kTileFixedPx pixels of a frame with 24 fragments per pixel; a frame binned in two levels costs its
// fullest unit's super-tiles in the split besides. The shape that makes this least is taken, the larger one where it
// changes nothing: as large as the LDS allows for a large frame (few tiles also make the binning's runs long), a divisor
// of the frame that leaves no nearly empty last round for a middle one, and tiles small enough to reach every compute
// unit for a small one. M > 32 keeps power-of-two tiles: there the tile is a few dozen pixels or less.
static void pick_tile(Geom& g, uint32_t per_px) {
  uint32_t most = std::min<uint32_t>(std::max<uint32_t>(1, kLdsBytes / per_px), kMaxTilePx);
  const uint32_t e = log2_floor(most);  // the largest power-of-two tile
  g.lTW = (e + 1) / 2;
  g.TH = 1u << (e / 2);
  g.ntiles_large = (((g.W - 1) >> g.lTW) + 1) * ((g.H - 1) / g.TH + 1);
  if (g.M <= 32) {
    // a column of coefficients per thread where the columns are long (one more pass over the threads for a few columns
    // costs as much as a full one)
    if (g.M >= 16) most = std::min<uint32_t>(most, kTileThreads / g.C);
    // Widest first: the shapes that are near the best come early, and the frame's pixels alone, in tiles of px, bound the
    // cost of the others from below (the search took 3 us of every call on a full HD frame and 10 on 8K without the bounds).
    uint64_t best = ~0ull;
    for (uint32_t l = 6; l >= 3; --l) {
      const uint32_t tw = 1u << l, tx = ((g.W - 1) >> l) + 1;
      for (uint32_t th = std::min(2 * tw - 1, most / tw); th >= tw / 2 && tw * th >= kMinTilePx; --th) {
        const uint32_t px = tw * th, ty = (g.H - 1) / th + 1;
        if (best >> 40 == 0 && (uint64_t)g.P * (px + kTileFixedPx) > best * px * kComputeUnits) break;
        const uint64_t nt = (uint64_t)tx * ty, fullest = (nt + kComputeUnits - 1) / kComputeUnits;
        uint64_t cost = fullest * (px + kTileFixedPx);
        if (nt > kMaxLdsBins * kMaxSub) {
          cost = nt << 24;  // past the tables of two levels: as few tiles as can be
        } else if (nt > kTwoLevelTiles) {
          if (cost + fullest * px > best) continue;  // (a compute unit's super-tiles hold no fewer tiles)
          uint32_t lsw, sh;
          cost += pick_supers(tx, ty, lsw, sh) * px;
        }
        if (cost < best || (cost == best && px >= g.TH << g.lTW)) {  // the larger one of equals, the narrower of those
          best = cost;
          g.lTW = l;
          g.TH = th;
        }
      }
    }
  }
  g.TW = 1u << g.lTW;
  g.divTH = make_fastdiv(g.TH);
  g.mulTH = row_multiplier(g.H, g.TH);
  g.tile_px = g.TW * g.TH;
  g.tilesX = (g.W - 1) / g.TW + 1;
  g.tilesY = (g.H - 1) / g.TH + 1;
  g.ntiles = g.tilesX * g.tilesY;
  // as many threads as fill a compute unit together with the other tiles it holds, at least four per pixel of a tile
  // that is alone on it
  const uint32_t together =
      std::min<uint32_t>(kLdsBytes / (g.tile_px * per_px), (g.ntiles - 1) / kComputeUnits + 1);
  g.tthreads = together >= 4 ? kTileThreads / 4 : together >= 2 ? kTileThreads / 2 : kTileThreads;
  while (g.tthreads > kTileThreads / 4 && g.tthreads >= 8 * g.tile_px) g.tthreads /= 2;
  // No more tiles than compute units: the fullest tile has its unit to itself, and all threads for what may be most of the
  // stream (149x101 with 300,000 fragments on 64 pixels, 64-pixel tiles, 256 threads and 1024: render 526 and 348 us, with
  // depth bounds 858 and 448, build 410 and 212; fragments spread evenly: the same within 1%).
  // M > 32: a pixel's hundreds of coefficients are work for all threads of a unit, however few the pixels (build, 512x512 at
  // 8 per pixel, 256 threads and 1024: rank 8 1.01 and 0.72 ms; rank 10, three channels, 10.1 and 5.9; gradients 2.1 and
  // 1.8 ms at rank 8, 0.51 and 0.36 at rank 5 with three channels)
  if (g.M > 32 || g.ntiles <= kComputeUnits) g.tthreads = kTileThreads;
}

Geom make_geom(const wt_frame_desc& d, bool backward) {
  Geom g{};
  g.W = d.width;
  g.H = d.height;
  g.P = d.width * d.height;
  g.C = d.channels;
  g.rank = d.rank;
  g.L = d.rank + 1;
  g.M = 1u << g.L;
  g.AW = (d.channels == 3) ? 8 : 4;
  g.AL = (d.channels == 3) ? 6 : 4;
  g.dtype = d.coeff_dtype;
  g.tight = (d.flags & WT_TIGHT_DEPTH) ? 1 : 0;
  g.serial = (d.flags & WT_DETERMINISTIC) ? 1 : 0;
  g.temporal = !backward && (d.flags & WT_TEMPORAL) ? 1 : 0;
  g.ep = !backward && g.M <= 32 ? 1 : 0;
  pick_tile(g, tile_px_bytes(g, backward));
  g.divW = make_fastdiv(g.W);
  // One LDS tile table for the scatter (up to kTwoLevelTiles tiles; beyond, two levels below)
  g.lds_bins = g.ntiles <= kTwoLevelTiles ? 1 : 0;
  g.rb = g.ntiles;
  const uint32_t hnr = (g.ntiles - 1) / kMaxHistBins + 1;
  g.hrb = (g.ntiles - 1) / hnr + 1;
  // Many tiles: a chunk of the stream touches each tile about chunk / ntiles times, too few for whole runs. Bin
  // into at most kMaxSupers super-tiles of SW x SH tiles first (runs as long as for a small frame), then split
  // each super-tile's records into its tiles (runs of hundreds of records, no atomics).
  g.two = 0;
  g.SW = g.SH = 1;
  g.lSW = 0;
  if (g.ntiles > kTwoLevelTiles) {
    pick_supers(g.tilesX, g.tilesY, g.lSW, g.SH);
    g.SW = 1u << g.lSW;
    // super-tile tables must fit the scatter's LDS; beyond that (about half a million tiles) the stream is
    // binned with one global atomic per fragment
    g.two = (uint64_t)((g.tilesX - 1) / g.SW + 1) * ((g.tilesY - 1) / g.SH + 1) <= kMaxLdsBins ? 1 : 0;
    g.lds_bins = g.two;
  }
  g.sX = (g.tilesX - 1) / g.SW + 1;
  g.sY = (g.tilesY - 1) / g.SH + 1;
  g.nsuper = g.sX * g.sY;
  g.NX = g.lds_bins ? kClasses : 1;
  // Scatter chunks (powers of two): 4096 fragments up to kShortBins bins (of the binning level that scatters), where a chunk
  // still holds more than one record per bin, else 8192. k_scatter_stream takes the former (see stream_scatter); what it
  // leaves of three channels, k_scatter_staged takes in two workgroups of 512 threads per compute unit, so that one loads
  // while the other ranks, stages and writes (glass 3840x2160, scatter phases: 7.86 ms with one workgroup of 1024 threads,
  // 7.22 with two); a round of 1024 records of at most 40 bytes and the tables of kShortBins bins fit half the LDS.
  // (One channel, 50 M fragments, 4096 against 8192: 2,280 bins 0.678 ms and 0.718; 3,000 bins 0.692 and 0.725; at 4,080
  // the longer chunk is faster, smoke frame 2.07 ms and 2.10.)
  const uint32_t bins = g.two ? g.nsuper : g.rb;
  static_assert(8 * kShortBins + 1024 * 40 <= kLdsBytes / 2 - 1024, "a round and the tables fit half the LDS");
  const bool short_chunk = g.lds_bins && bins <= kShortBins;
  g.sthreads = short_chunk && g.C == 3 ? 512 : 1024;
  g.chunk = short_chunk ? 4096 : 1024 * kPer;
  return g;
}

Geom super_geom(const Geom& g) {
  Geom s = g;
  s.lTW = g.lTW + g.lSW;
  s.TW = 1u << s.lTW;
  s.TH = g.TH * g.SH;
  s.divTH = make_fastdiv(s.TH);
  s.mulTH = row_multiplier(s.H, s.TH);
  s.tile_px = s.TW * s.TH;
  s.tilesX = g.sX;
  s.tilesY = g.sY;
  s.ntiles = g.nsuper;
  s.rb = s.hrb = g.nsuper;
  s.two = 0;
  s.SW = s.SH = 1;
  s.lSW = 0;
  s.sX = s.tilesX;
  s.sY = s.tilesY;
  return s;  // NX and chunk stay those of g: the first level uses the classes the histogram counted
}

static size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

Layout make_layout(const Geom& g, uint64_t cap) {
  Layout l{};
  size_t o = 0;
  l.header = o;
  o += 256;
  l.counts = o;
  o = align256(o + 4ull * g.NX * g.ntiles);
  l.offsets = o;
  o = align256(o + 4ull * (g.NX * (uint64_t)g.ntiles + 1));
  l.cursors = o;
  o = align256(o + 4ull * g.NX * g.ntiles * kCursorPad);
  l.order = o;
  o = align256(o + 4ull * g.ntiles);
  l.scan = o;
  o = align256(o + 4ull * 257 * ((g.NX * (uint64_t)g.ntiles + kScanRange - 1) / kScanRange));
  l.heads = o;
  o = align256(o + 4ull * head_dwords(g.C) * cap);
  l.tails = o;
  o = align256(o + 4ull * tail_dwords(true) * cap);
  l.counts1 = l.offsets1 = l.cursors1 = l.order1 = l.heads1 = l.tails1 = o;
  if (g.two) {
    l.counts1 = o;
    o = align256(o + 4ull * g.NX * g.nsuper);
    l.offsets1 = o;
    o = align256(o + 4ull * (g.NX * (uint64_t)g.nsuper + 1));
    l.cursors1 = o;
    o = align256(o + 4ull * g.NX * g.nsuper * kCursorPad);
    l.order1 = o;
    o = align256(o + 4ull * g.nsuper);
    l.heads1 = o;
    o = align256(o + 4ull * head_dwords(g.C) * cap);
    l.tails1 = o;
    o = align256(o + 4ull * tail_dwords(true) * cap);
  }
  l.total = o;
  l.cap = cap;
  return l;
}

uint64_t capacity_for(const Geom& g, size_t ws_bytes) {
  const size_t fixed = make_layout(g, 0).total;
  if (ws_bytes < fixed) return 0;
  const uint64_t per = 4ull * record_dwords(g.C, true) * (g.two ? 2 : 1);
  uint64_t cap = (ws_bytes - fixed) / per;
  while (cap > 0 && make_layout(g, cap).total > ws_bytes) --cap;
  return cap;
}

// Whether a frame in the largest power-of-two tiles (no more of them than hold a column per thread, for packed storage and
// the one-pass render) has more super-tiles of 8 x 8 of them than two levels bin.
static bool past_two_levels(const Geom& g) {
  uint32_t e = log2_floor(std::min(kLdsBytes / tile_px_bytes(g, false), kMaxTilePx));
  if (g.dtype == WT_E5B9G9R9 || g.temporal) e = std::min(e, log2_floor(kTileThreads / g.C));
  const uint32_t lw = (e + 1) / 2 + 3, lh = e / 2 + 3;
  return (uint64_t)(((g.W - 1) >> lw) + 1) * (((g.H - 1) >> lh) + 1) > kMaxLdsBins;
}

bool scratch_geom(const wt_frame_desc& d, uint64_t count, Geom& g, size_t& need, size_t& limit) {
  auto fits = [&] {
    need = make_layout(g, count).total;
    Geom few = g;
    few.ntiles = std::min(g.ntiles, g.ntiles_large);
    few.nsuper = 1;
    limit = std::min(kScratchBytes, WT_SCRATCH_BYTES + make_layout(g, 0).total - make_layout(few, 0).total);
    return need <= limit;
  };
  g = make_geom(d);
  if (fits()) return true;
  if (!g.two || !past_two_levels(g)) return false;
  g.two = g.lds_bins = 0;
  g.NX = 1;
  g.SW = g.SH = 1;
  g.lSW = 0;
  g.sX = g.tilesX;
  g.sY = g.tilesY;
  g.nsuper = g.ntiles;
  g.sthreads = 1024;
  g.chunk = 1024 * kPer;
  return fits();
}

Binned binned_view(const Geom& g, const Layout& l, const void* ws, bool with_index) {
  const char* b = (const char*)ws;
  Binned v;
  v.offsets = (const uint32_t*)(b + l.offsets);
  v.order = (const uint32_t*)(b + l.order);
  v.head = (const uint32_t*)(b + l.heads);
  v.tail = (const uint32_t*)(b + l.tails);
  v.DH = head_dwords(g.C);
  v.DT = tail_dwords(with_index);
  v.hdr = (WsHeader*)(b + l.header);
  v.stamp = layout_stamp(g, l, with_index);
  v.cap = l.cap;
  return v;
}

// The stamp covers everything the tile kernels index by: frame, channels, rank, tile and super-tile geometry, write
// classes, record capacity and format, and the layout's size.
unsigned long long layout_stamp(const Geom& g, const Layout& l, bool with_index) {
  const uint32_t w[] = {0x57544c31u, g.W, g.H, g.C, g.rank, g.TW, g.TH, g.NX, g.two, g.SW, g.SH, g.lds_bins, g.serial,
                        (uint32_t)l.cap, (uint32_t)(l.cap >> 32), (uint32_t)l.total, (uint32_t)(l.total >> 32),
                        with_index ? 1u : 0u};
  return stamp_words(w, (int)(sizeof w / sizeof w[0]));
}

// A count is stamped with the layout and the stream it counted (size and the four array addresses), so that a
// scatter of another stream, or under another layout, refuses to write.
unsigned long long count_stamp(const Geom& g, const Layout& l, const wt_fragments& f) {
  const unsigned long long ls = layout_stamp(g, l, false);
  const uintptr_t a[4] = {(uintptr_t)f.pixel, (uintptr_t)f.depth, (uintptr_t)f.alpha, (uintptr_t)f.rgb};
  uint32_t w[12] = {(uint32_t)ls, (uint32_t)(ls >> 32), (uint32_t)f.count, (uint32_t)(f.count >> 32)};
  for (int i = 0; i < 4; ++i) {
    w[4 + 2 * i] = (uint32_t)a[i];
    w[5 + 2 * i] = (uint32_t)((uint64_t)a[i] >> 32);
  }
  return stamp_words(w, 12);
}

// Start of a count: the tile counts start from zero; no complete binning and no count in the workspace any more; the
// drop counter and the scatter's progress restart. The sticky error bits stay until wt_dropped_count reports them.
__global__ __launch_bounds__(256) void k_count_reset(WsHeader* h, uint32_t* __restrict__ counts, uint64_t n) {
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    counts[i] = 0u;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (h->magic != kWsMagic) {  // a workspace the device has not written yet: no errors to keep
      h->errors = 0;
      h->magic = kWsMagic;
    }
    h->dropped = 0;
    h->fault = 0;
    h->counted = 0;
    h->binned = 0;
  }
}

// End of a scatter: the binning is complete when the count before it was this stream's under this layout, the
// scatter did not refuse, and every write cursor reached the end of its segment (so each segment holds exactly the
// records counted for it). Then the header gets `stamp`, else 0.
// One workgroup. cursors are [NX][nt] (row stride kCursorPad words), offsets [nt * NX + 1]. A thread has a tile's
// cursors and segment ends in flight together (one at a time, with a division each, the check was a chain of memory
// latencies: 2,280 tiles 17 us). (Checked by the scatter's last workgroup instead, after a ticket per workgroup, it cost
// the smoke frame's scatter 28 us against 10 for this launch.)
template <uint32_t NX>
__global__ __launch_bounds__(1024) void k_seal(WsHeader* h, const uint32_t* __restrict__ cursors,
                                                const uint32_t* __restrict__ offsets, uint32_t nt,
                                                unsigned long long cstamp, unsigned long long stamp) {
  __shared__ int bad;
  if (threadIdx.x == 0) bad = 0;
  __syncthreads();
  int mine = 0;
  for (uint32_t t = threadIdx.x; t < nt; t += 1024) {
    uint32_t c[NX], end[NX];
#pragma unroll
    for (uint32_t x = 0; x < NX; ++x) {
      c[x] = cursors[(x * nt + t) * kCursorPad];
      end[x] = offsets[(uint64_t)t * NX + x + 1];
    }
#pragma unroll
    for (uint32_t x = 0; x < NX; ++x) mine |= c[x] != end[x];
  }
  if (mine) bad = 1;
  __syncthreads();
  if (threadIdx.x == 0) {
    const bool ok = !bad && h->fault == 0 && h->counted == cstamp;
    h->binned = ok ? stamp : 0ull;
    // a scatter that did not belong to its count (another stream, arrays changed since the count, run twice)
    if (!ok) ws_raise(h, kWsErrScatter);
  }
}

static void launch_seal(WsHeader* h, const uint32_t* cursors, const uint32_t* offsets, uint32_t NX, uint32_t nt,
                        unsigned long long cstamp, unsigned long long stamp, hipStream_t s) {
  auto k = NX == 1 ? k_seal<1> : k_seal<kClasses>;
  hipLaunchKernelGGL(k, dim3(1), dim3(1024), 0, s, h, cursors, offsets, nt, cstamp, stamp);
}

// After the split of a two-level binning: complete when the first level was (the split only moves its records).
__global__ void k_seal_split(WsHeader* h, unsigned long long level1, unsigned long long stamp) {
  h->binned = h->binned == level1 ? stamp : 0ull;
}

// A first-level binning of a two-level layout carries this stamp until its split has run.
static unsigned long long level1_stamp(unsigned long long s) { return s ^ 0x9e3779b97f4a7c15ull; }

__global__ void k_fill_u32(uint32_t* __restrict__ p, uint64_t n, uint32_t v) {
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

hipError_t launch_fill_u32(uint32_t* p, uint64_t n, uint32_t v, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)std::min<uint64_t>((n + 255) / 256, 4096)), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

// Sixteen bytes of the stream, non-temporal (the histogram reads each pixel id once).
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 load_stream_u4(const uint32_t* p) {
  const u32x4_t v = __builtin_nontemporal_load((const u32x4_t*)p);
  return make_uint4(v.x, v.y, v.z, v.w);
}

// ------------------------------------------------------------------------------------------------ histogram

// Workgroups of 256 threads, or of 1024 when the tile table is large (up to 144 KB of LDS leaves one workgroup per
// compute unit, which then still has sixteen waves of loads in flight). The pixel ids are read with non-temporal
// loads (smoke frame: 0.132 -> 0.121 ms for the count).

template <int kHistThreads>
__global__ __launch_bounds__(kHistThreads) void k_hist_lds(const uint32_t* __restrict__ pixel, uint32_t F, Geom g,
                                                           int vec, uint32_t* __restrict__ counts,
                                                           unsigned long long* __restrict__ dropped) {
  extern __shared__ uint32_t lh[];
  const uint32_t cls = blockIdx.x % g.NX;
  const uint32_t nchunks = (uint32_t)(((uint64_t)F + g.chunk - 1) / g.chunk);
  uint32_t nd = 0;
  // one pass per range of g.hrb tiles (a single pass unless the frame has more tiles than the table holds)
  for (uint32_t t0 = 0; t0 < g.ntiles; t0 += g.hrb) {
  const uint32_t nt = std::min(g.hrb, g.ntiles - t0);
  const bool first = t0 == 0;
  for (uint32_t t = threadIdx.x; t < nt; t += blockDim.x) lh[t] = 0;
  __syncthreads();
  // The workgroup's whole chunks (chunk k of the workgroup is c = blockIdx.x + k gridDim.x, all of its class) as one
  // flat range of 16-byte units, so that every thread has four loads in flight whatever the chunk size; chunk sizes
  // are powers of two (threads per scatter workgroup times fragments per thread).
  const uint32_t nfull = vec ? F / g.chunk : 0;
  const uint32_t kfull = blockIdx.x < nfull ? (nfull - 1 - blockIdx.x) / gridDim.x + 1 : 0;
  const uint32_t nv = g.chunk / 4, lnv = __builtin_ctz(nv);
  const uint32_t units = kfull * nv;
  for (uint32_t u0 = 0; u0 < units; u0 += 4 * kHistThreads) {
    uint4 q[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const uint32_t u = u0 + v * kHistThreads + threadIdx.x;
      const uint32_t c = blockIdx.x + (u >> lnv) * gridDim.x;
      q[v] = u < units ? load_stream_u4(pixel + (uint64_t)c * g.chunk + 4 * (u & (nv - 1)))
                       : make_uint4(0u, 0u, 0u, 0u);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      if (u0 + v * kHistThreads + threadIdx.x >= units) continue;
      const uint32_t ps[4] = {q[v].x, q[v].y, q[v].z, q[v].w};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (ps[k] < g.P) {
          const uint32_t t = tile_of(g, ps[k]) - t0;
          if (t < nt) atomicAdd(&lh[t], 1u);
        } else if (first) {
          ++nd;
        }
      }
    }
  }
  // the rest: the partial last chunk, or every chunk of an unaligned stream
  for (uint32_t c = blockIdx.x + kfull * gridDim.x; c < nchunks; c += gridDim.x) {
    const uint32_t base = c * g.chunk;
    const uint32_t n = std::min<uint32_t>(g.chunk, F - base);
    for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) {
      const uint32_t p = pixel[base + i];
      if (p < g.P) {
        const uint32_t t = tile_of(g, p) - t0;
        if (t < nt) atomicAdd(&lh[t], 1u);
      } else if (first) {
        ++nd;
      }
    }
  }
  __syncthreads();
  for (uint32_t t = threadIdx.x; t < nt; t += blockDim.x) {
    const uint32_t v = lh[t];
    if (v) atomicAdd(&counts[cls * g.ntiles + t0 + t], v);
  }
  __syncthreads();
  }
  nd = wave_sum(nd);
  if ((threadIdx.x & 63) == 0 && nd) atomicAdd(dropped, (unsigned long long)nd);
}

// Fallback for very many tiles: one global atomic per fragment, one class.
__global__ __launch_bounds__(256) void k_hist_global(const uint32_t* __restrict__ pixel, uint32_t F, Geom g,
                                                     uint32_t* __restrict__ counts,
                                                     unsigned long long* __restrict__ dropped) {
  uint32_t nd = 0;
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < F; i += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t p = pixel[i];
    if (p < g.P)
      atomicAdd(&counts[tile_of(g, p)], 1u);
    else
      ++nd;
  }
  nd = wave_sum(nd);
  if ((threadIdx.x & 63) == 0 && nd) atomicAdd(dropped, (unsigned long long)nd);
}

// ------------------------------------------------------------------------------------------------ scan

constexpr int kScanThreads = 1024;
constexpr int kScanItems = 16;
constexpr uint32_t kOrderBuckets = 256;  // size classes of the heaviest-first tile order
static_assert(kScanRange == (uint32_t)kScanThreads * kScanItems, "a scan workgroup covers one pass of k_scan");
static_assert(kScanRange % kClasses == 0, "scan ranges hold whole tiles");

// Exclusive prefix of s over the workgroup (wavefront shuffles, then the wave totals); *total receives the sum.
// wsum holds kScanThreads / 64 + 1 entries. Ends with a barrier.
__device__ __forceinline__ uint32_t block_exclusive(uint32_t s, uint32_t* wsum, uint32_t* total) {
  const uint32_t lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint32_t inc = s;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t v = __shfl_up(inc, o, 64);
    if (lane >= (uint32_t)o) inc += v;
  }
  if (lane == 63) wsum[wv] = inc;
  __syncthreads();
  if (wv == 0) {
    constexpr uint32_t NW = kScanThreads / 64;
    const uint32_t w = lane < NW ? wsum[lane] : 0u;
    uint32_t wi = w;
#pragma unroll
    for (int o = 1; o < (int)NW; o <<= 1) {
      const uint32_t v = __shfl_up(wi, o, 64);
      if (lane >= (uint32_t)o) wi += v;
    }
    if (lane < NW) wsum[lane] = wi - w;
    if (lane == NW - 1) wsum[NW] = wi;
  }
  __syncthreads();
  *total = wsum[kScanThreads / 64];
  const uint32_t r = wsum[wv] + inc - s;
  __syncthreads();  // wsum may be reused
  return r;
}

// Size class of a tile for the heaviest-first order: log-linear in the count (the leading bit's position and the
// three bits below it), monotone, 256 classes.
__device__ __forceinline__ uint32_t size_class(uint32_t c) {
  const uint32_t v = c + 1;
  const uint32_t e = 31 - __clz(v);
  const uint32_t m = e >= 3 ? (v >> (e - 3)) & 7u : (v << (3 - e)) & 7u;
  return e * 8 + m;
}

// Scan of the tiles [t0, t0 + kScanThreads * TPT): a thread holds the class counts of its TPT tiles in registers (loaded
// together, consecutive lanes on consecutive tiles), so the scan is one memory latency, one block prefix per TPT and the
// stores. counts and cursors are class-major [NX][ntiles], offsets tile-major; cnt receives each tile's records.
template <uint32_t NX, uint32_t TPT>
__device__ __forceinline__ void scan_tiles(const uint32_t* __restrict__ counts, const Geom& g, uint32_t t0,
                                           uint32_t* __restrict__ offsets, uint32_t* __restrict__ cursors,
                                           uint32_t* wsum, uint32_t& carry, uint32_t (&cnt)[TPT]) {
  uint32_t c[TPT][NX];
#pragma unroll
  for (uint32_t k = 0; k < TPT; ++k) {
    const uint32_t t = t0 + k * kScanThreads + threadIdx.x;
    cnt[k] = 0;
    if (t0 + k * kScanThreads >= g.ntiles) continue;
#pragma unroll
    for (uint32_t x = 0; x < NX; ++x) {
      c[k][x] = t < g.ntiles ? counts[x * g.ntiles + t] : 0u;
      cnt[k] += c[k][x];
    }
  }
#pragma unroll
  for (uint32_t k = 0; k < TPT; ++k) {
    if (t0 + k * kScanThreads >= g.ntiles) break;
    const uint32_t t = t0 + k * kScanThreads + threadIdx.x;
    uint32_t total;
    uint32_t run = carry + block_exclusive(cnt[k], wsum, &total);
    carry += total;
    if (t >= g.ntiles) continue;
#pragma unroll
    for (uint32_t x = 0; x < NX; ++x) {
      offsets[(uint64_t)t * NX + x] = run;
      cursors[(x * g.ntiles + t) * kCursorPad] = run;
      run += c[k][x];
    }
  }
}

// Exclusive scan over segments in (tile, class) order by one workgroup, then the tile order for the tile kernels:
// heaviest first by size class (a bucket sort; ties in any order), so the last workgroups to start are the light ones.
constexpr uint32_t kScanTiles = 8;  // tiles per thread
static_assert(kTwoLevelTiles <= kScanTiles * kScanThreads && kMaxLdsBins <= kScanTiles * kScanThreads,
              "one pass holds the tiles of a binning level");

__global__ __launch_bounds__(kScanThreads) void k_scan(const uint32_t* __restrict__ counts, Geom g,
                                                       uint32_t* __restrict__ offsets,
                                                       uint32_t* __restrict__ cursors,
                                                       uint32_t* __restrict__ order, int with_order,
                                                       WsHeader* hdr, unsigned long long stamp) {
  if (hdr && threadIdx.x == 0) hdr->counted = stamp;  // the last scan of a count (seen by later kernels)
  __shared__ uint32_t wsum[kScanThreads / 64 + 1];
  __shared__ uint32_t bucket[kOrderBuckets];
  const uint32_t tid = threadIdx.x;
  for (uint32_t b = tid; b < kOrderBuckets; b += kScanThreads) bucket[b] = 0;
  uint32_t carry = 0, cnt[kScanTiles];
  scan_tiles<kClasses, kScanTiles>(counts, g, 0, offsets, cursors, wsum, carry, cnt);
  if (tid == 0) offsets[(uint64_t)g.ntiles * kClasses] = carry;
  if (!with_order) return;
  __syncthreads();
#pragma unroll
  for (uint32_t k = 0; k < kScanTiles; ++k)
    if (k * kScanThreads + tid < g.ntiles) atomicAdd(&bucket[kOrderBuckets - 1 - size_class(cnt[k])], 1u);
  __syncthreads();
  uint32_t total;
  const uint32_t bc = tid < kOrderBuckets ? bucket[tid] : 0u;
  const uint32_t start = block_exclusive(bc, wsum, &total);
  if (tid < kOrderBuckets) bucket[tid] = start;
  __syncthreads();
#pragma unroll
  for (uint32_t k = 0; k < kScanTiles; ++k) {
    const uint32_t t = k * kScanThreads + tid;
    if (t < g.ntiles) order[atomicAdd(&bucket[kOrderBuckets - 1 - size_class(cnt[k])], 1u)] = t;
  }
}

// The same scan and tile order for frames with many tiles, over several workgroups: workgroup w owns the
// segments [w R, (w + 1) R) (R = kScanRange, whole tiles since R is a multiple of NX). Pass one: each workgroup's
// segment total and the size classes of its tiles (part[w][0], part[w][1 + k] for reversed class k). Pass two:
// each workgroup adds the totals of the workgroups before it, scans its range, and places its tiles in the
// heaviest-first order after every heavier class and after its class's tiles of earlier workgroups.
template <uint32_t NX>
__global__ __launch_bounds__(kScanThreads) void k_scan_part(const uint32_t* __restrict__ counts, Geom g,
                                                            uint32_t* __restrict__ part) {
  __shared__ uint32_t wsum[kScanThreads / 64 + 1];
  __shared__ uint32_t bucket[kOrderBuckets];
  constexpr uint32_t TPT = kScanItems / NX;
  const uint32_t tid = threadIdx.x, t0 = blockIdx.x * (kScanRange / NX);
  for (uint32_t b = tid; b < kOrderBuckets; b += kScanThreads) bucket[b] = 0;
  uint32_t cnt[TPT], s = 0;
#pragma unroll
  for (uint32_t k = 0; k < TPT; ++k) {
    const uint32_t t = t0 + k * kScanThreads + tid;
    cnt[k] = 0;
#pragma unroll
    for (uint32_t x = 0; x < NX; ++x) cnt[k] += t < g.ntiles ? counts[x * g.ntiles + t] : 0u;
    s += cnt[k];
  }
  uint32_t total;
  block_exclusive(s, wsum, &total);  // its barriers also order the bucket clears before the adds
#pragma unroll
  for (uint32_t k = 0; k < TPT; ++k)
    if (t0 + k * kScanThreads + tid < g.ntiles) atomicAdd(&bucket[kOrderBuckets - 1 - size_class(cnt[k])], 1u);
  __syncthreads();
  uint32_t* mine = part + (size_t)blockIdx.x * (1 + kOrderBuckets);
  if (tid == 0) mine[0] = total;
  for (uint32_t b = tid; b < kOrderBuckets; b += kScanThreads) mine[1 + b] = bucket[b];
}

template <uint32_t NX>
__global__ __launch_bounds__(kScanThreads) void k_scan_apply(const uint32_t* __restrict__ counts, Geom g,
                                                             const uint32_t* __restrict__ part,
                                                             uint32_t* __restrict__ offsets,
                                                             uint32_t* __restrict__ cursors,
                                                             uint32_t* __restrict__ order, WsHeader* hdr,
                                                             unsigned long long stamp) {
  __shared__ uint32_t wsum[kScanThreads / 64 + 1];
  __shared__ uint32_t start[kOrderBuckets];
  constexpr uint32_t TPT = kScanItems / NX;
  const uint32_t G = gridDim.x, w = blockIdx.x, tid = threadIdx.x, t0 = w * (kScanRange / NX);
  if (hdr && w == 0 && tid == 0) hdr->counted = stamp;
  // segments of the workgroups before this one
  uint32_t before = 0;
  for (uint32_t v = tid; v < w; v += kScanThreads) before += part[(size_t)v * (1 + kOrderBuckets)];
  uint32_t carry, cnt[TPT];
  block_exclusive(before, wsum, &carry);
  scan_tiles<NX, TPT>(counts, g, t0, offsets, cursors, wsum, carry, cnt);
  if (w == G - 1 && tid == 0) offsets[(uint64_t)g.ntiles * NX] = carry;
  // start of this workgroup's tiles in each size class: all heavier classes, then earlier workgroups' tiles of
  // the same class
  uint32_t tot = 0, pre = 0;
  if (tid < kOrderBuckets) {
    for (uint32_t u = 0; u < G; ++u) {
      const uint32_t b = part[(size_t)u * (1 + kOrderBuckets) + 1 + tid];
      tot += b;
      if (u < w) pre += b;
    }
  }
  uint32_t all;
  const uint32_t base = block_exclusive(tid < kOrderBuckets ? tot : 0u, wsum, &all);
  if (tid < kOrderBuckets) start[tid] = base + pre;
  __syncthreads();
#pragma unroll
  for (uint32_t k = 0; k < TPT; ++k) {
    const uint32_t t = t0 + k * kScanThreads + tid;
    if (t < g.ntiles) order[atomicAdd(&start[kOrderBuckets - 1 - size_class(cnt[k])], 1u)] = t;
  }
}

// Per-class counts of the super-tiles (first level of two-level binning) from the per-class tile counts.
__global__ __launch_bounds__(256) void k_super_counts(const uint32_t* __restrict__ counts, Geom g,
                                                      uint32_t* __restrict__ counts1) {
  const uint32_t id = blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= g.NX * g.nsuper) return;
  const uint32_t x = id / g.nsuper, sidx = id - x * g.nsuper;
  const uint32_t sx = sidx % g.sX, sy = sidx / g.sX;
  uint32_t sum = 0;
  for (uint32_t j = 0; j < g.SW * g.SH; ++j) {
    const uint32_t tx = (sx << g.lSW) + (j & (g.SW - 1)), ty = sy * g.SH + (j >> g.lSW);
    if (tx < g.tilesX && ty < g.tilesY) sum += counts[x * g.ntiles + ty * g.tilesX + tx];
  }
  counts1[id] = sum;
}

// ------------------------------------------------------------------------------------------------ scatter

// One chunk's fragments, held in registers by the thread that loaded them.
template <int C>
struct ChunkRegs {
  static_assert(kPer % 4 == 0, "vector loads take fragments four at a time");
  uint32_t p[kPer];
  float x[kPer];
  float a[C * kPer];
  float c[3 * kPer];
};

// Loads fragments [i0, i0 + kPer) of the chunk at base; out-of-range slots get pixel id 0xffffffff. (Ordinary loads: with
// one workgroup of this kernel per compute unit non-temporal ones took the smoke frame's scatter from 2.05 to 2.41 ms.)
template <int C>
__device__ __forceinline__ void load_chunk(const wt_fragments& f, uint32_t base, uint32_t i0, uint32_t n, int vec,
                                           ChunkRegs<C>& r) {
  if (vec && i0 + kPer <= n) {
    // pixel ids first: the tile count needs only them, and the other loads stay in flight meanwhile
#pragma unroll
    for (uint32_t v = 0; v < kPer / 4; ++v) {
      const uint4 p4 = *(const uint4*)(f.pixel + (uint64_t)base + i0 + 4 * v);
      r.p[4 * v + 0] = p4.x; r.p[4 * v + 1] = p4.y; r.p[4 * v + 2] = p4.z; r.p[4 * v + 3] = p4.w;
    }
#pragma unroll
    for (uint32_t v = 0; v < kPer / 4; ++v) {
      const uint64_t i = (uint64_t)base + i0 + 4 * v;
      const float4 x4 = *(const float4*)(f.depth + i);
      r.x[4 * v + 0] = x4.x; r.x[4 * v + 1] = x4.y; r.x[4 * v + 2] = x4.z; r.x[4 * v + 3] = x4.w;
#pragma unroll
      for (int q = 0; q < C; ++q) {
        const float4 a4 = *(const float4*)(f.alpha + C * i + 4 * q);
        r.a[4 * C * v + 4 * q + 0] = a4.x; r.a[4 * C * v + 4 * q + 1] = a4.y;
        r.a[4 * C * v + 4 * q + 2] = a4.z; r.a[4 * C * v + 4 * q + 3] = a4.w;
      }
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const float4 c4 = *(const float4*)(f.rgb + 3 * i + 4 * q);
        r.c[12 * v + 4 * q + 0] = c4.x; r.c[12 * v + 4 * q + 1] = c4.y;
        r.c[12 * v + 4 * q + 2] = c4.z; r.c[12 * v + 4 * q + 3] = c4.w;
      }
    }
  } else {
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
      const uint32_t li = i0 + k;
      r.p[k] = 0xffffffffu;
      if (li < n) {
        const uint64_t i = (uint64_t)base + li;
        r.p[k] = f.pixel[i];
        r.x[k] = f.depth[i];
#pragma unroll
        for (int q = 0; q < C; ++q) r.a[C * k + q] = f.alpha[C * i + q];
#pragma unroll
        for (int q = 0; q < 3; ++q) r.c[3 * k + q] = f.rgb[3 * i + q];
      }
    }
  }
}

template <int C>
__device__ __forceinline__ bool has_nan(const ChunkRegs<C>& r, uint32_t k) {
  bool bad = isnan(r.x[k]);
#pragma unroll
  for (int q = 0; q < C; ++q) bad |= isnan(r.a[C * k + q]);
  return bad;
}

// A record's words after the pixel and depth (alphas `a`, colours `c`) from the fragment's to the forward binning's: each
// alpha as its absorbance step (binned_absorbance) and the colour times the clamped alpha, the two forms in which the
// tile kernels use them. Records binned for the gradient keep alpha and the plain colour.
template <int C>
__device__ __forceinline__ void to_forward(uint32_t* a, uint32_t* c) {
#pragma unroll
  for (int q = 0; q < 3; ++q)
    c[q] = __float_as_uint(__uint_as_float(c[q]) * alpha_clamped(__uint_as_float(a[C == 1 ? 0 : q])));
#pragma unroll
  for (int q = 0; q < C; ++q) a[q] = __float_as_uint(binned_absorbance(__uint_as_float(a[q])));
}

// Record dword j of fragment k (tile-local pixel `local`, stream index `src`), with the fragment's own alpha and colour.
template <int C>
__device__ __forceinline__ uint32_t record_word(const ChunkRegs<C>& r, uint32_t k, uint32_t local, uint32_t src,
                                                uint32_t j) {
  if (j == 0) return local;
  if (j == 1) return __float_as_uint(r.x[k]);
  if (j < 2 + C) return __float_as_uint(r.a[C * k + (j - 2)]);
  if (j < 5 + C) return __float_as_uint(r.c[3 * k + (j - 2 - C)]);
  return src;
}

// Block-wide exclusive scan of cnt[0, nt) in place; wsum holds THREADS / 64 partial sums.
template <int THREADS>
__device__ __forceinline__ void block_scan_inplace(uint32_t* cnt, uint32_t nt, uint32_t* wsum) {
  const uint32_t per = (nt + THREADS - 1) / THREADS;
  const uint32_t t0 = threadIdx.x * per, t1 = std::min(t0 + per, nt);
  uint32_t s = 0;
  for (uint32_t t = t0; t < t1; ++t) s += cnt[t];
  const uint32_t lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint32_t inc = s;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t v = __shfl_up(inc, o, 64);
    if (lane >= (uint32_t)o) inc += v;
  }
  if (lane == 63) wsum[wv] = inc;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t a = 0;
    for (uint32_t w = 0; w < THREADS / 64; ++w) {
      const uint32_t v = wsum[w];
      wsum[w] = a;
      a += v;
    }
  }
  __syncthreads();
  uint32_t run = wsum[wv] + inc - s;
  for (uint32_t t = t0; t < t1; ++t) {
    const uint32_t v = cnt[t];
    cnt[t] = run;
    run += v;
  }
}

// The same over 16-bit counts, returning the total to every thread. Ends with a barrier.
template <int THREADS>
__device__ __forceinline__ uint32_t block_scan_total(uint16_t* cnt, uint32_t nt, uint32_t* wsum) {
  constexpr uint32_t NW = THREADS / 64;
  const uint32_t per = (nt + THREADS - 1) / THREADS;
  const uint32_t t0 = std::min(threadIdx.x * per, nt), t1 = std::min(t0 + per, nt);
  uint32_t s = 0;
  for (uint32_t t = t0; t < t1; ++t) s += cnt[t];
  const uint32_t lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint32_t inc = s;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t v = __shfl_up(inc, o, 64);
    if (lane >= (uint32_t)o) inc += v;
  }
  if (lane == 63) wsum[wv] = inc;
  __syncthreads();
  uint32_t before = 0, total = 0;
#pragma unroll
  for (uint32_t w = 0; w < NW; ++w) {
    const uint32_t v = wsum[w];
    before += w < wv ? v : 0u;
    total += v;
  }
  uint32_t run = before + inc - s;
  for (uint32_t t = t0; t < t1; ++t) {
    const uint32_t v = cnt[t];
    cnt[t] = (uint16_t)run;
    run += v;
  }
  __syncthreads();
  return total;
}

constexpr uint32_t kNoTile = 0xffffffffu;

// A record as it is stored: N dwords, 4-byte aligned, so that one lane writes one record with one wide store and
// consecutive lanes write consecutive records.
template <uint32_t N>
struct Words {
  uint32_t w[N];
};

// Bytes of one record staged in LDS by the chunk scatter (its head words plus the tile, and its tail words) or by
// the split (head words plus the record's slot, and tail words), unpadded.
constexpr uint32_t staged_record_bytes(uint32_t C, bool idx) { return 4 * (head_dwords(C) + 1 + tail_dwords(idx)); }

// N words to or from LDS with the widest accesses the address allows (d holds N-word records back to back, at a
// 16-byte aligned base).
template <uint32_t N>
__device__ __forceinline__ void lds_put(uint32_t* d, const uint32_t* w) {
  if constexpr (N % 4 == 0) {
#pragma unroll
    for (uint32_t u = 0; u < N / 4; ++u) ((uint4*)d)[u] = make_uint4(w[4 * u], w[4 * u + 1], w[4 * u + 2], w[4 * u + 3]);
  } else if constexpr (N % 2 == 0) {
#pragma unroll
    for (uint32_t u = 0; u < N / 2; ++u) ((uint2*)d)[u] = make_uint2(w[2 * u], w[2 * u + 1]);
  } else {
#pragma unroll
    for (uint32_t u = 0; u < N; ++u) d[u] = w[u];
  }
}

template <uint32_t N>
__device__ __forceinline__ void lds_get(const uint32_t* d, uint32_t* w) {
  if constexpr (N % 4 == 0) {
#pragma unroll
    for (uint32_t u = 0; u < N / 4; ++u) {
      const uint4 v = ((const uint4*)d)[u];
      w[4 * u] = v.x; w[4 * u + 1] = v.y; w[4 * u + 2] = v.z; w[4 * u + 3] = v.w;
    }
  } else if constexpr (N % 2 == 0) {
#pragma unroll
    for (uint32_t u = 0; u < N / 2; ++u) {
      const uint2 v = ((const uint2*)d)[u];
      w[2 * u] = v.x; w[2 * u + 1] = v.y;
    }
  } else {
#pragma unroll
    for (uint32_t u = 0; u < N; ++u) w[u] = d[u];
  }
}

// The gradient of a fragment that is in no tile (its pixel is out of range) is written where the binning leaves it out;
// every other gradient is written by the tile kernel.
template <int C>
__device__ __forceinline__ void zero_gradient(const GradOut& go, uint64_t i) {
#pragma unroll
  for (int q = 0; q < C; ++q) go.alpha[C * i + q] = 0.f;
#pragma unroll
  for (int q = 0; q < 3; ++q) go.rgb[3 * i + q] = 0.f;
}

// Refusal of a scatter that does not belong to the count before it, or whose stream puts more records in a segment
// than were counted: nothing more is written and the binning is not sealed.
__device__ __forceinline__ void scatter_refuse(WsHeader* hdr) {
  atomicOr(&hdr->fault, 1u);
  ws_raise(hdr, kWsErrScatter);
}

// LDS: sh[stage][HW] and st[stage][DT] one round of records in tile order (head words and the tile, tail words), cnt[ntiles]
// (the chunk's counts, then first staged positions), gb[ntiles] (reserved base - run start, per round). The chunk's order is
// written in rounds of `stage` records, a power of two chosen by the host to fit the LDS. With 512 threads (three channels)
// two workgroups share a compute unit (LDS <= 80 KB, four waves per SIMD): one's loads and stores overlap the other's
// ranking and staging.
template <int C, bool IDX, int THREADS>
__global__ __launch_bounds__(THREADS, THREADS == 512 ? 4 : 1) void k_scatter_staged(wt_fragments f, Geom g, int vec,
                                                                    uint32_t stage,
                                                                    uint32_t* __restrict__ cursors,
                                                                    uint32_t* __restrict__ head,
                                                                    uint32_t* __restrict__ tail,
                                                                    WsHeader* hdr, unsigned long long cstamp,
                                                                    uint32_t cap, GradOut go) {
  constexpr uint32_t DH = head_dwords(C), DT = tail_dwords(IDX), HW = DH + 1;
  extern __shared__ uint4 sm4[];
  uint32_t* sh = (uint32_t*)sm4;               // [stage][HW]: head words, then the tile
  uint32_t* st = sh + (size_t)stage * HW;      // [stage][DT]: tail words
  uint32_t* cnt = st + (size_t)stage * DT;
  uint32_t* gb = cnt + g.ntiles;
  __shared__ uint32_t wsum[THREADS / 64];
  __shared__ uint32_t nvalid, refused;
  const uint32_t F = (uint32_t)f.count;
  const uint32_t cls = blockIdx.x % g.NX;
  const uint32_t base = blockIdx.x * g.chunk;
  const uint32_t n = std::min<uint32_t>(g.chunk, F - base);
  for (uint32_t t = threadIdx.x; t < g.ntiles; t += blockDim.x) cnt[t] = 0;
  if (threadIdx.x == 0) nvalid = refused = 0;
  ChunkRegs<C> r;
  const uint32_t i0 = threadIdx.x * kPer;
  load_chunk<C>(f, base, i0, n, vec, r);
  // only the stream the preceding count counted, under the same layout, is scattered into its segments (the
  // stamp is loaded behind the chunk, so the check adds no wait of its own)
  if (hdr->counted != cstamp) {
    if (threadIdx.x == 0) scatter_refuse(hdr);
    return;
  }
  __syncthreads();
  uint32_t tile[kPer], rank[kPer], local[kPer];
  uint32_t nan_count = 0, mine = 0;
#pragma unroll
  for (uint32_t k = 0; k < kPer; ++k) {
    tile[k] = 0xffffffffu;
    if (r.p[k] < g.P) {
      tile_locate(g, r.p[k], tile[k], local[k]);
      rank[k] = atomicAdd(&cnt[tile[k]], 1u);
      nan_count += has_nan<C>(r, k) ? 1u : 0u;
      ++mine;
    } else if constexpr (IDX) {
      if (i0 + k < n) zero_gradient<C>(go, (uint64_t)base + i0 + k);
    }
  }
  mine = wave_sum(mine);
  if ((threadIdx.x & 63) == 0 && mine) atomicAdd(&nvalid, mine);
  __syncthreads();
  block_scan_inplace<THREADS>(cnt, g.ntiles, wsum);
  __syncthreads();
  // cnt[t] is now the chunk's first staged position of tile t (tile-major order)
  uint32_t sp[kPer];
#pragma unroll
  for (uint32_t k = 0; k < kPer; ++k) sp[k] = (tile[k] == 0xffffffffu) ? 0xffffffffu : cnt[tile[k]] + rank[k];
  const uint32_t total = nvalid;
  for (uint32_t r0 = 0; r0 < total; r0 += stage) {
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
      if (sp[k] < r0 || sp[k] >= r0 + stage) continue;  // also skips invalid slots (0xffffffff)
      uint32_t hw[HW], tw[DT];
#pragma unroll
      for (uint32_t j = 0; j < HW; ++j) hw[j] = j < DH ? record_word<C>(r, k, local[k], base + i0 + k, j) : tile[k];
#pragma unroll
      for (uint32_t j = 0; j < DT; ++j) tw[j] = record_word<C>(r, k, local[k], base + i0 + k, DH + j);
      lds_put<HW>(sh + (size_t)(sp[k] - r0) * HW, hw);
      lds_put<DT>(st + (size_t)(sp[k] - r0) * DT, tw);
    }
    // Reserve this round's run of every tile it holds (one returning atomic per tile on the XCD's shared cursor)
    // just before the round is written: slots stay reserved but unwritten for one round only, so fewer partly
    // written lines wait at the frontier and more of them complete in L2 before write-back. The run of tile t is
    // [max(first_t, r0), min(end_t, r1)); gb[t] = reserved base - run start, so a record's slot is gb[t] plus its
    // staged position. (Issuing the next round's reservations during this round's writes was slower: the
    // registers that hold them push the kernel past its two-workgroup budget.)
    const uint32_t r1 = std::min(r0 + stage, total);
    for (uint32_t t = threadIdx.x; t < g.ntiles; t += THREADS) {
      const uint32_t p0 = cnt[t], p1 = t + 1 < g.ntiles ? cnt[t + 1] : total;
      const uint32_t lo = std::max(p0, r0), hi = std::min(p1, r1);
      if (hi > lo) {
        const uint32_t got = atomicAdd(&cursors[(cls * g.ntiles + t) * kCursorPad], hi - lo);
        gb[t] = got - lo;
        // writes stay inside the record arrays whatever the cursors hold; a stream that changed since its count
        // and overruns a segment into its neighbour leaves cursors off their segment ends, which the seal sees
        if (got > cap || cap - got < hi - lo) refused = 1;
      }
    }
    __syncthreads();
    if (refused) {
      if (threadIdx.x == 0) scatter_refuse(hdr);
      return;
    }
    const uint32_t ns = std::min(stage, total - r0);
    for (uint32_t sidx = threadIdx.x; sidx < ns; sidx += blockDim.x) {
      uint32_t hw[HW], tw[DT];
      lds_get<HW>(sh + (size_t)sidx * HW, hw);
      lds_get<DT>(st + (size_t)sidx * DT, tw);
      const uint64_t slot = (uint32_t)(gb[hw[DH]] + r0 + sidx);
      // converted here, where every lane has a record and little else is live (before the ranking, the products and
      // logarithms cost the 64-register kernel spills: smoke scatter 1.66 -> 2.6 ms)
      if constexpr (!IDX) to_forward<C>(hw + 2, tw);
      Words<DH> h;
#pragma unroll
      for (uint32_t j = 0; j < DH; ++j) h.w[j] = hw[j];
      Words<DT> t;
#pragma unroll
      for (uint32_t j = 0; j < DT; ++j) t.w[j] = tw[j];
      *(Words<DH>*)(head + slot * DH) = h;
      *(Words<DT>*)(tail + slot * DT) = t;
    }
    __syncthreads();
  }
  nan_count = wave_sum(nan_count);
  if ((threadIdx.x & 63) == 0 && nan_count) atomicAdd(&hdr->dropped, (unsigned long long)nan_count);
}

// Four consecutive fragments of each array from fragment i on, as they lie in memory (any 4-byte alignment), non-temporal
// (each fragment is read once). No branch and no copy: the loads of one chunk stay in flight while another is written.
typedef unsigned int u32x4_any __attribute__((ext_vector_type(4), aligned(4)));
template <int C>
struct Quad {
  u32x4_any p, x, a[C], c[3];
  __device__ __forceinline__ void load(const wt_fragments& f, uint64_t i) {
    p = __builtin_nontemporal_load((const u32x4_any*)(f.pixel + i));
    x = __builtin_nontemporal_load((const u32x4_any*)(f.depth + i));
#pragma unroll
    for (int q = 0; q < C; ++q) a[q] = __builtin_nontemporal_load((const u32x4_any*)(f.alpha + C * i) + q);
#pragma unroll
    for (int q = 0; q < 3; ++q) c[q] = __builtin_nontemporal_load((const u32x4_any*)(f.rgb + 3 * i) + q);
  }
  __device__ __forceinline__ uint32_t alpha(int k, int q) const { return a[(C * k + q) / 4][(C * k + q) % 4]; }
  __device__ __forceinline__ uint32_t colour(int k, int q) const { return c[(3 * k + q) / 4][(3 * k + q) % 4]; }
};

// The same with a workgroup that stays on its compute unit and takes every gridDim.x-th chunk (a multiple of the classes,
// so its class is its XCD's). What bounds k_scatter_staged up to about a thousand bins is not memory but the chain of
// each workgroup: load, rank, scan, then per round stage, reserve, write. Here the chunk is staged whole (every lane has a
// record to stage, where a round stages with a quarter of the lanes); its runs are reserved as soon as it is ranked, and
// the reservations come back while it is scanned and staged; the next chunk's loads are in flight while it is written; and
// a wave that has written its records goes on to rank the next chunk. Slots are open from the ranking to the write-out.
// Measured against k_scatter_staged (one channel; 48 bytes per fragment, a copy at 4.7 TB/s in brackets):
// 1024x768 at 16 per pixel, 768 bins: 150 -> 130 us (127); 1280x720, 1000 bins: 180 -> 158 (149); 1280x720 rank 4,
// 1,720 bins: 280 -> 249; smoke frame, 2,040 bins: 1.675 -> 1.66 ms; 1920x1080 at 24, 3,000 bins: 687 -> 667 us; glass
// 3840x2160 (960 super-tiles, with its split): 6.94 -> 6.83 ms. Writing the last records with the wait for the next
// chunk's loads counted apart from the stores (an unrolled write) gave 40 us on the glass frame and cost 8 on smoke.
// Reservations awaited before the scan instead: 3% to 6% slower. Streams of at least four fragments.
// Three channels stage a record in eight words (the tile above the pixel's 18 bits: a super-tile has at most 64 x 2048
// pixels, and there are at most kShortBins bins), and the counts are 16-bit (a chunk's), so that a chunk and the tables
// of kShortBins bins fit: glass 1366x768, 3,182 bins: 594 us staged in rounds, 542 here; 1024x768 at 27, 2,496 bins, 426
// and 388; 1920x1080 rank 2, 3,240 bins, 1.20 ms and 1.12. At few bins neither changes the time.
template <int C, bool IDX, int THREADS>
__global__ __launch_bounds__(THREADS) void k_scatter_stream(wt_fragments f, Geom g, uint32_t nchunks,
                                                            uint32_t* __restrict__ cursors, uint32_t* __restrict__ head,
                                                            uint32_t* __restrict__ tail, WsHeader* hdr,
                                                            unsigned long long cstamp, uint32_t cap, GradOut go) {
  constexpr uint32_t PER = 4, DH = head_dwords(C), DT = tail_dwords(IDX), HW = DH + 1, CH = THREADS * PER;
  constexpr uint32_t R = THREADS == 1024 ? 4 : 1;  // tiles per thread at most (kShortBins, 512)
  constexpr bool kPacked = C == 3;  // eight words: pixel | tile << 18, depth, absorbances, colour
  extern __shared__ uint4 sm4[];
  const uint32_t half = (g.ntiles + 1) / 2;
  uint32_t* sh = (uint32_t*)sm4;  // [CH][HW]: head words, then the tile; [CH][8] packed
  uint32_t* st = sh + CH * HW;    // [CH][DT]: tail words
  uint32_t* gb = kPacked ? sh + CH * 8 : st + CH * DT;  // [ntiles]: reserved base - first staged position
  uint32_t* cnt = gb + g.ntiles;  // [ntiles] 16-bit counts, then first staged positions
  uint32_t* cnt2 = cnt + half;    // the same of the next chunk
  __shared__ uint32_t wsum[THREADS / 64];
  __shared__ uint32_t refused;
  const uint32_t F = (uint32_t)f.count, cls = blockIdx.x % g.NX;
  if (threadIdx.x == 0) refused = 0;
  uint32_t nan_count = 0, c = blockIdx.x;
  // A thread's fragments are [first, first + 4) of the chunk; past the end of the stream it loads the last four, of
  // which it takes those from `first` on.
  uint32_t first = c * CH + threadIdx.x * PER;
  Quad<C> r;
  r.load(f, std::min(first, F - PER));
  if (hdr->counted != cstamp) {
    if (threadIdx.x == 0) scatter_refuse(hdr);
    return;
  }
  for (uint32_t t = threadIdx.x; t < half; t += THREADS) cnt[t] = cnt2[t] = 0;
  __syncthreads();
  while (true) {
    const uint32_t from = std::min(first, F - PER);
    uint32_t tile[PER], rank[PER], local[PER];
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
      tile[k] = kNoTile;
      if (from + k < first) continue;
      if (r.p[k] < g.P) {
        tile_locate(g, r.p[k], tile[k], local[k]);
        const uint32_t sh16 = 16 * (tile[k] & 1);  // (a count is at most the chunk: no carry into the other half)
        rank[k] = atomicAdd(&cnt[tile[k] >> 1], 1u << sh16) >> sh16 & 0xffffu;
      } else if constexpr (IDX) {
        zero_gradient<C>(go, from + k);
      }
    }
    __syncthreads();
    uint16_t* const pos = (uint16_t*)cnt;
    uint32_t got[R], n[R];
#pragma unroll
    for (uint32_t u = 0; u < R; ++u) {
      const uint32_t t = threadIdx.x + u * THREADS;
      n[u] = t < g.ntiles ? pos[t] : 0u;
      if (n[u]) got[u] = atomicAdd(&cursors[(cls * g.ntiles + t) * kCursorPad], n[u]);
    }
    const uint32_t total = block_scan_total<THREADS>(pos, g.ntiles, wsum);
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
      if (tile[k] == kNoTile) continue;
      uint32_t hw[HW], tw[DT];
      hw[0] = local[k];
      hw[1] = r.x[k];
      bool bad = isnan(__uint_as_float(hw[1]));
#pragma unroll
      for (int q = 0; q < C; ++q) {
        hw[2 + q] = r.alpha(k, q);
        bad |= isnan(__uint_as_float(hw[2 + q]));
      }
      hw[DH] = tile[k];
      if constexpr (kPacked) hw[0] |= tile[k] << 18;
#pragma unroll
      for (int q = 0; q < 3; ++q) tw[q] = r.colour(k, q);
      if constexpr (IDX) tw[3] = from + k;
      nan_count += bad ? 1u : 0u;
      const uint32_t sp = pos[tile[k]] + rank[k];
      if constexpr (kPacked) {
        sm4[2 * sp] = make_uint4(hw[0], hw[1], hw[2], hw[3]);
        sm4[2 * sp + 1] = make_uint4(hw[4], tw[0], tw[1], tw[2]);
      } else {
        lds_put<HW>(sh + sp * HW, hw);
        lds_put<DT>(st + sp * DT, tw);
      }
    }
#pragma unroll
    for (uint32_t u = 0; u < R; ++u) {
      const uint32_t t = threadIdx.x + u * THREADS;
      if (t < half) cnt2[t] = 0;
      if (!n[u]) continue;
      gb[t] = got[u] - pos[t];
      // writes stay inside the record arrays whatever the cursors hold
      if (got[u] > cap || cap - got[u] < n[u]) refused = 1;
    }
    c += gridDim.x;
    const bool more = c < nchunks;
    first = c * CH + threadIdx.x * PER;
    if (more) r.load(f, std::min(first, F - PER));
    __syncthreads();
    if (refused) {
      if (threadIdx.x == 0) scatter_refuse(hdr);
      return;
    }
    for (uint32_t s = threadIdx.x; s < total; s += THREADS) {
      uint32_t hw[HW], tw[DT];
      if constexpr (kPacked) {
        const uint4 a = sm4[2 * s], b = sm4[2 * s + 1];
        hw[0] = a.x & 0x3ffffu; hw[1] = a.y; hw[2] = a.z; hw[3] = a.w; hw[4] = b.x;
        tw[0] = b.y; tw[1] = b.z; tw[2] = b.w;
        hw[DH] = a.x >> 18;
      } else {
        lds_get<HW>(sh + s * HW, hw);
        lds_get<DT>(st + s * DT, tw);
      }
      const uint64_t slot = (uint32_t)(gb[hw[DH]] + s);
      if constexpr (!IDX) to_forward<C>(hw + 2, tw);
      Words<DH> h;
#pragma unroll
      for (uint32_t j = 0; j < DH; ++j) h.w[j] = hw[j];
      Words<DT> t;
#pragma unroll
      for (uint32_t j = 0; j < DT; ++j) t.w[j] = tw[j];
      *(Words<DH>*)(head + slot * DH) = h;
      *(Words<DT>*)(tail + slot * DT) = t;
    }
    if (!more) break;
    // A wave goes on to rank the next chunk while others still write: the tables it counts in were cleared before the
    // last barrier, and the barriers after its ranking keep the stage until all have written.
    uint32_t* const x = cnt;
    cnt = cnt2;
    cnt2 = x;
  }
  nan_count = wave_sum(nan_count);
  if ((threadIdx.x & 63) == 0 && nan_count) atomicAdd(&hdr->dropped, (unsigned long long)nan_count);
}

template <int C, bool IDX>
__global__ __launch_bounds__(1024) void k_scatter_global(wt_fragments f, Geom g, int vec, uint32_t* __restrict__ cursors,
                                                         uint32_t* __restrict__ head, uint32_t* __restrict__ tail,
                                                         WsHeader* hdr, unsigned long long cstamp, uint32_t cap,
                                                         GradOut go) {
  constexpr uint32_t DH = head_dwords(C), DT = tail_dwords(IDX);
  if (hdr->counted != cstamp) {
    if (threadIdx.x == 0) scatter_refuse(hdr);
    return;
  }
  const uint32_t F = (uint32_t)f.count;
  const uint32_t base = blockIdx.x * g.chunk;
  const uint32_t n = std::min<uint32_t>(g.chunk, F - base);
  ChunkRegs<C> r;
  const uint32_t i0 = threadIdx.x * kPer;
  load_chunk<C>(f, base, i0, n, vec, r);
  uint32_t nan_count = 0;
#pragma unroll
  for (uint32_t k = 0; k < kPer; ++k) {
    if (r.p[k] >= g.P) {
      if constexpr (IDX)
        if (i0 + k < n) zero_gradient<C>(go, (uint64_t)base + i0 + k);
      continue;
    }
    uint32_t tile, local;
    tile_locate(g, r.p[k], tile, local);
    nan_count += has_nan<C>(r, k) ? 1u : 0u;
    const uint64_t pos = atomicAdd(&cursors[tile * kCursorPad], 1u);
    if (pos >= cap) {  // inside the record arrays whatever the cursors hold (the seal checks the segments)
      scatter_refuse(hdr);
      continue;
    }
    uint32_t w[DH + DT];
#pragma unroll
    for (uint32_t j = 0; j < DH + DT; ++j) w[j] = record_word<C>(r, k, local, base + i0 + k, j);
    if constexpr (!IDX) to_forward<C>(w + 2, w + DH);
#pragma unroll
    for (uint32_t j = 0; j < DH; ++j) head[pos * DH + j] = w[j];
#pragma unroll
    for (uint32_t j = 0; j < DT; ++j) tail[pos * DT + j] = w[DH + j];
  }
  nan_count = wave_sum(nan_count);
  if ((threadIdx.x & 63) == 0 && nan_count) atomicAdd(&hdr->dropped, (unsigned long long)nan_count);
}

// WT_DETERMINISTIC binning: one thread copies the stream in stream order straight into the tile segments (the
// class of fragment i is that of its chunk, as in the count), so every segment holds its records in stream order.
template <int C, bool IDX>
__global__ void k_scatter_serial(wt_fragments f, Geom g, uint32_t* __restrict__ cursors,
                                 const uint32_t* __restrict__ offsets, uint32_t* __restrict__ head,
                                 uint32_t* __restrict__ tail, WsHeader* hdr, unsigned long long cstamp, GradOut go) {
  constexpr uint32_t DH = head_dwords(C), DT = tail_dwords(IDX);
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  if (hdr->counted != cstamp) {
    scatter_refuse(hdr);
    return;
  }
  unsigned long long nan_count = 0;
  for (uint64_t i = 0; i < f.count; ++i) {
    const uint32_t p = f.pixel[i];
    if (p >= g.P) {
      if (IDX) zero_gradient<C>(go, i);
      continue;
    }
    uint32_t tile, local;
    tile_locate(g, p, tile, local);
    const uint32_t cls = (uint32_t)((i / g.chunk) % g.NX);
    uint32_t* cur = &cursors[(cls * g.ntiles + tile) * kCursorPad];
    const uint32_t pos = *cur;
    if (pos >= offsets[tile * g.NX + cls + 1]) {
      scatter_refuse(hdr);
      return;
    }
    *cur = pos + 1;
    const float x = f.depth[i];
    bool bad = isnan(x);
    uint32_t w[DH + 3] = {local, __float_as_uint(x)};
    for (int c = 0; c < C; ++c) {
      bad |= isnan(f.alpha[i * C + c]);
      w[2 + c] = __float_as_uint(f.alpha[i * C + c]);
    }
    for (int q = 0; q < 3; ++q) w[DH + q] = __float_as_uint(f.rgb[i * 3 + q]);
    if (!IDX) to_forward<C>(w + 2, w + DH);
    uint32_t* h = head + (uint64_t)pos * DH;
    for (uint32_t q = 0; q < DH; ++q) h[q] = w[q];
    uint32_t* t = tail + (uint64_t)pos * DT;
    for (uint32_t q = 0; q < 3; ++q) t[q] = w[DH + q];
    if (IDX) t[3] = (uint32_t)i;
    nan_count += bad ? 1 : 0;
  }
  if (nan_count) atomicAdd(&hdr->dropped, nan_count);
}

// Second level of two-level binning: one workgroup per super-tile moves its records (all classes, contiguous in
// the first-level arrays) into the tiles' segments of the final arrays. Rounds of split_per(C, IDX) records per
// thread: rank by tile in LDS, place in tile order in LDS (head words plus the record's slot, then the tail words,
// unpadded), write with consecutive lanes on consecutive records. The workgroup owns its tiles, so their write
// cursors live in LDS; runs are about kSplitThreads * split_per / (SW SH) records long, so each round takes as many
// records as the LDS holds (glass 3840x2160, 32 tiles per super-tile: two records per thread 3.35 ms, three 3.28,
// four 3.18).
constexpr uint32_t kSplitThreads = 1024;
constexpr uint32_t split_per(uint32_t C, bool idx) {
  return (kLdsBytes - 2048) / (kSplitThreads * staged_record_bytes(C, idx));
}

template <int C, bool IDX>
__global__ __launch_bounds__(kSplitThreads) void k_split(Geom g, const uint32_t* __restrict__ offsets1,
                                                         const uint32_t* __restrict__ offsets,
                                                         const uint32_t* __restrict__ head1,
                                                         const uint32_t* __restrict__ tail1,
                                                         uint32_t* __restrict__ head, uint32_t* __restrict__ tail,
                                                         const WsHeader* hdr, unsigned long long level1) {
  constexpr uint32_t DH = head_dwords(C), DT = tail_dwords(IDX), HW = DH + 1;
  constexpr uint32_t PER = split_per(C, IDX), RECS = kSplitThreads * PER;
  // only a complete first level is split (its records then hold valid super-tile-local pixels)
  if (hdr->binned != level1) return;
  extern __shared__ uint4 sm4[];
  uint32_t* sh = (uint32_t*)sm4;  // [RECS][HW]: head words, then the record's slot
  uint32_t* st = sh + RECS * HW;  // [RECS][DT]: tail words
  __shared__ uint32_t cur[kMaxSub], cnt[kMaxSub], pre[kMaxSub];
  const uint32_t sidx = blockIdx.x;
  const uint32_t sx = sidx % g.sX, sy = sidx / g.sX;
  const uint32_t nsub = g.SW * g.SH;
  const uint32_t beg = offsets1[sidx * g.NX], end = offsets1[(sidx + 1) * g.NX];
  const uint32_t lTWs = g.lTW + g.lSW;  // super-tile width in pixels is 2^lTWs
  if (threadIdx.x < nsub) {
    const uint32_t j = threadIdx.x;
    const uint32_t tx = (sx << g.lSW) + (j & (g.SW - 1)), ty = sy * g.SH + (j >> g.lSW);
    cur[j] = (tx < g.tilesX && ty < g.tilesY) ? offsets[(ty * g.tilesX + tx) * g.NX] : 0u;
  }
  for (uint32_t c0 = beg; c0 < end; c0 += RECS) {
    if (threadIdx.x < nsub) cnt[threadIdx.x] = 0;
    __syncthreads();
    uint32_t hw[PER][HW], tw[PER][DT], sub[PER], rank[PER];
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
      const uint32_t i = c0 + k * kSplitThreads + threadIdx.x;
      sub[k] = 0xffffffffu;
      if (i < end) {
#pragma unroll
        for (uint32_t w = 0; w < DH; ++w) hw[k][w] = head1[(uint64_t)i * DH + w];
#pragma unroll
        for (uint32_t w = 0; w < DT; ++w) tw[k][w] = tail1[(uint64_t)i * DT + w];
        const uint32_t loc = hw[k][0];  // pixel within the super-tile
        const uint32_t lx = loc & ((1u << lTWs) - 1), ly = loc >> lTWs;
        const uint32_t ty = fastdiv(ly, g.divTH);
        sub[k] = (ty << g.lSW) + (lx >> g.lTW);
        hw[k][0] = ((ly - ty * g.TH) << g.lTW) + (lx & (g.TW - 1));  // pixel within the tile
        rank[k] = atomicAdd(&cnt[sub[k]], 1u);
      }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t run = 0;
      for (uint32_t j = 0; j < nsub; ++j) {
        pre[j] = run;
        run += cnt[j];
      }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
      if (sub[k] == 0xffffffffu) continue;
      hw[k][DH] = cur[sub[k]] + rank[k];
      const uint32_t pos = pre[sub[k]] + rank[k];
      lds_put<HW>(sh + (size_t)pos * HW, hw[k]);
      lds_put<DT>(st + (size_t)pos * DT, tw[k]);
    }
    __syncthreads();
    const uint32_t ns = std::min(RECS, end - c0);
    for (uint32_t q = threadIdx.x; q < ns; q += kSplitThreads) {
      uint32_t h[HW], t[DT];
      lds_get<HW>(sh + (size_t)q * HW, h);
      lds_get<DT>(st + (size_t)q * DT, t);
      const uint64_t slot = h[DH];
      Words<DH> hh;
#pragma unroll
      for (uint32_t w = 0; w < DH; ++w) hh.w[w] = h[w];
      Words<DT> tt;
#pragma unroll
      for (uint32_t w = 0; w < DT; ++w) tt.w[w] = t[w];
      *(Words<DH>*)(head + slot * DH) = hh;
      *(Words<DT>*)(tail + slot * DT) = tt;
    }
    __syncthreads();
    if (threadIdx.x < nsub) cur[threadIdx.x] += cnt[threadIdx.x];
  }
}

// Small streams: the whole binning in one launch (after the header's reset), P workgroups for every P tiles. Each reads every
// pixel id, lists in LDS the fragments of its tiles that are in its part of the stream (one P-th) and counts those that come
// before them (of the tiles below, and of its tiles in other parts), which is where its records start, and writes them
// there, consecutive lanes on consecutive records. The ids are read once per tile, from L2, which costs less than the
// count, scan, scatter and seal one after the other (five launches that each wait for the one before) up to kSmallReads ids
// in all; lists of 16-bit indices take kSmallStream fragments at most. 64x64 with 33,000 fragments: 29 -> 18 us a frame.
// Parts bound what one compute unit moves (1.1 ns a record) when a tile holds most of the stream, and cost reductions and
// compares when it does not (binning alone, one channel; all fragments in one tile, or spread over 256; the general way 30
// us and 28): 24,000 fragments whole 32 us and 13.3, in two parts 21 and 13; 32,768 whole 41 and 13.4, in two 26.5 and 13.4
// (64x64 frame 18.9 whole, 19.8); 40,000 whole 50 and 13.4, in two 31.7 and 13.7, in four 23.2 and 15.4; 65,536 whole 78
// and 16.7, in two 48 and 18.3, in four 34 and 21.
constexpr uint32_t kSmallStream = 65536;
constexpr uint64_t kSmallReads = 16u << 20;

static uint32_t small_parts(uint64_t F) { return F <= 32768 ? 1 : F <= 40960 ? 2 : 4; }
__host__ __device__ inline uint32_t small_quads(uint32_t F, uint32_t P) { return (F / 4 + P - 1) / P; }  // of a part
// Entries of one tile's list: its part's whole groups of four, and the last part's rest.
__host__ __device__ inline uint32_t small_list(uint32_t F, uint32_t P) { return 4 * small_quads(F, P) + 4; }
static_assert(2 * (kSmallStream + 8 * 4) <= kLdsBytes - 1024, "the lists of all parts fit the LDS");

template <int C, bool IDX, uint32_t P>
__global__ __launch_bounds__(1024) void k_bin_small(wt_fragments f, Geom g, int vec, uint32_t* __restrict__ offsets,
                                                    uint32_t* __restrict__ order, uint32_t* __restrict__ head,
                                                    uint32_t* __restrict__ tail, WsHeader* hdr,
                                                    unsigned long long stamp, GradOut go) {
  constexpr uint32_t DH = head_dwords(C), DT = tail_dwords(IDX);
  extern __shared__ uint16_t list[];  // [P][small_list]
  __shared__ uint32_t mine[P], earlier[P], later[P], before, lost;
  const uint32_t F = (uint32_t)f.count, t0 = blockIdx.x / P * P, part = blockIdx.x - t0;
  const uint32_t quads = vec ? F / 4 : 0, per = small_quads(F, P), stride = small_list(F, P);
  const uint32_t lo = std::min(part * per, quads), hi = part == P - 1 ? quads : std::min(lo + per, quads);
  if (threadIdx.x < P) mine[threadIdx.x] = earlier[threadIdx.x] = later[threadIdx.x] = 0;
  if (threadIdx.x == 0) before = lost = 0;
  __syncthreads();
  uint32_t below = 0, drops = 0, early[P], late[P];
#pragma unroll
  for (uint32_t j = 0; j < P; ++j) early[j] = late[j] = 0;
  // an id of its part: listed when it is in one of its tiles; fragments in no tile are the first workgroups' to account for
  auto take = [&](uint32_t i, uint32_t p) {
    if (p >= g.P) {
      if (t0 == 0) {
        ++drops;
        if constexpr (IDX) zero_gradient<C>(go, i);
      }
      return;
    }
    const uint32_t t = tile_of(g, p);
    if (t < t0) ++below;
#pragma unroll
    for (uint32_t j = 0; j < P; ++j)
      if (t == t0 + j) list[j * stride + atomicAdd(&mine[j], 1u)] = (uint16_t)i;
  };
  // an id of another part
  auto count = [&](uint32_t p, uint32_t (&of)[P]) {
    if (p >= g.P) return;
    const uint32_t t = tile_of(g, p);
    below += t < t0 ? 1u : 0u;
#pragma unroll
    for (uint32_t j = 0; j < P; ++j) of[j] += t == t0 + j ? 1u : 0u;
  };
  // groups of four ids [q0, q1), two in flight
  auto each = [&](uint32_t q0, uint32_t q1, auto&& fn) {
    for (uint32_t q = q0 + threadIdx.x; q < q1; q += 2048) {
      const bool two = q + 1024 < q1;
      const uint4 a = ((const uint4*)f.pixel)[q], b = ((const uint4*)f.pixel)[two ? q + 1024 : q];
      const uint32_t pa[4] = {a.x, a.y, a.z, a.w}, pb[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k) fn(4 * q + k, pa[k]);
      if (two) {
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) fn(4 * (q + 1024) + k, pb[k]);
      }
    }
  };
  if constexpr (P > 1) each(0, lo, [&](uint32_t, uint32_t p) { count(p, early); });
  each(lo, hi, take);
  if constexpr (P > 1) each(hi, quads, [&](uint32_t, uint32_t p) { count(p, late); });
  for (uint32_t i = 4 * quads + threadIdx.x; i < F; i += 1024) {  // an unaligned stream, or the last ids
    const uint32_t at = P == 1 ? 0u : std::min(i / (4 * per), P - 1), p = f.pixel[i];
    if (at == part)
      take(i, p);
    else if (at < part)
      count(p, early);
    else
      count(p, late);
  }
  below = wave_sum(below);
  if ((threadIdx.x & 63) == 0 && below) atomicAdd(&before, below);
  if constexpr (P > 1) {
#pragma unroll
    for (uint32_t j = 0; j < P; ++j) {
      const uint32_t e = wave_sum(early[j]), l = wave_sum(late[j]);
      if ((threadIdx.x & 63) == 0 && e) atomicAdd(&earlier[j], e);
      if ((threadIdx.x & 63) == 0 && l) atomicAdd(&later[j], l);
    }
  }
  __syncthreads();
  // its records of tile t0 + j are number[j] .. number[j + 1] - 1 of the lists and start at base[j]; the tile starts at first[j]
  uint32_t number[P + 1], base[P], first[P + 1];
  number[0] = 0;
  first[0] = before;
#pragma unroll
  for (uint32_t j = 0; j < P; ++j) {
    base[j] = first[j] + earlier[j];
    first[j + 1] = base[j] + mine[j] + later[j];
    number[j + 1] = number[j] + mine[j];
  }
  for (uint32_t k = threadIdx.x; k < number[P]; k += 1024) {
    uint32_t at = k, slot = base[0] + k;  // its entry, its record
#pragma unroll
    for (uint32_t j = 1; j < P; ++j) {
      if (k >= number[j]) {
        at = j * stride + (k - number[j]);
        slot = base[j] + (k - number[j]);
      }
    }
    const uint32_t i = list[at];
    uint32_t w[DH + DT], tile;
    tile_locate(g, f.pixel[i], tile, w[0]);
    w[1] = __float_as_uint(f.depth[i]);
    bool bad = isnan(f.depth[i]);
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const float al = f.alpha[C * i + c];
      bad |= isnan(al);
      w[2 + c] = __float_as_uint(al);
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) w[DH + q] = __float_as_uint(f.rgb[3 * i + q]);
    if constexpr (IDX) w[DH + 3] = i;
    if constexpr (!IDX) to_forward<C>(w + 2, w + DH);
    drops += bad ? 1u : 0u;
    Words<DH> h;
#pragma unroll
    for (uint32_t j = 0; j < DH; ++j) h.w[j] = w[j];
    Words<DT> t;
#pragma unroll
    for (uint32_t j = 0; j < DT; ++j) t.w[j] = w[DH + j];
    *(Words<DH>*)(head + (uint64_t)slot * DH) = h;
    *(Words<DT>*)(tail + (uint64_t)slot * DT) = t;
  }
  drops = wave_sum(drops);
  if ((threadIdx.x & 63) == 0 && drops) atomicAdd(&lost, drops);
  if (part == 0) {
    // all of a tile's records are in its first class
#pragma unroll
    for (uint32_t j = 0; j < P; ++j) {
      if (t0 + j >= g.ntiles) break;
      if (threadIdx.x < g.NX) offsets[(t0 + j) * g.NX + threadIdx.x] = threadIdx.x ? first[j + 1] : first[j];
      if (threadIdx.x == 0) order[t0 + j] = t0 + j;
      if (threadIdx.x == 0 && t0 + j == g.ntiles - 1) offsets[g.ntiles * g.NX] = first[j + 1];
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    if (lost) atomicAdd(&hdr->dropped, (unsigned long long)lost);
    if (blockIdx.x == 0) hdr->binned = stamp;
  }
}

static bool small_stream(const Geom& g, uint64_t F) {
  return F > 0 && F <= kSmallStream && F * g.ntiles <= kSmallReads && g.lds_bins && !g.two && !g.serial;
}

static bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

// Largest staging round with two workgroups per compute unit. A round's slots are reserved when it is staged and
// stay partly written until it is, so longer rounds leave more partial lines at the frontier: on the smoke frame
// rounds of 2048 records took 1.93 ms against 1.69 ms for 1024 (and shorter rounds expose the reservations' latency
// more often: 512, 2.07 ms).
constexpr uint32_t kStageTwoWg = 1024;

template <int C, bool IDX, int THREADS>
static hipError_t launch_scatter_staged(const Geom& g, const wt_fragments& f, int vec, uint32_t* cursors,
                                        uint32_t* head, uint32_t* tail, WsHeader* hdr, unsigned long long cstamp,
                                        uint32_t cap, const GradOut& go, uint32_t nchunks, hipStream_t s) {
  constexpr uint32_t RB = staged_record_bytes(C, IDX);
  // largest power-of-two round beside the tile tables (1 KB left for static LDS), within half the LDS when two
  // workgroups share a compute unit
  constexpr bool kTwoWg = THREADS == 512;
  const size_t budget = (kTwoWg ? kLdsBytes / 2 : kLdsBytes) - 1024;
  uint32_t stage = std::min<uint32_t>(g.chunk, kTwoWg ? kStageTwoWg : g.chunk);
  while (stage > 256 && (size_t)stage * RB + 8ull * g.rb > budget) stage >>= 1;
  const size_t lds = (size_t)stage * RB + 8ull * g.rb;
  auto k = k_scatter_staged<C, IDX, THREADS>;
  if (lds > 65536) {
    hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k, dim3(nchunks), dim3(THREADS), lds, s, f, g, vec, stage, cursors, head, tail, hdr, cstamp,
                     cap, go);
  return hipGetLastError();
}

// k_scatter_stream takes every stream in short chunks that has at least four fragments; the tables of kShortBins bins fit
// beside a chunk. Three channels need six chunks for each compute unit to pay for themselves: k_scatter_staged has as many
// lanes to stage with there (512x512 at 16 per pixel 75 us staged, 79 as a stream; at 32 per pixel 151 and 137). With
// their indexes they do not fit. With more bins than kShortBins runs are one record long and writing is what counts
// (3,840 bins, 1920x1080 rank 4: 1.51 ms staged, 1.53 as a stream).
static size_t stream_lds(uint32_t chunk, uint32_t C, bool idx, uint32_t bins) {
  return (size_t)chunk * (C == 3 ? 32 : staged_record_bytes(C, idx)) + 4 * (bins + 2 * (size_t)((bins + 1) / 2));
}

static bool stream_scatter(const Geom& g, uint64_t F, bool idx) {
  if (!g.lds_bins || F < 4 || g.chunk > 4096) return false;
  return g.C == 1 || (!idx && F >= 6ull * kComputeUnits * 4096);
}
static_assert(4096 * 32 + 4 * (kShortBins + 2 * ((kShortBins + 1) / 2)) <= kLdsBytes - 1024 && kShortBins < 4096 &&
                  kMaxSub * kMaxTilePx <= 1u << 18 && staged_record_bytes(1, true) <= 32,
              "a short chunk and the tables of its bins fit the LDS, and a packed word its tile and pixel");


// The chunk a stream of F fragments is counted and scattered in: that of the geometry, or half of it, with two workgroups
// of k_scatter_stream per compute unit, for a one-channel stream of few chunks and bins whose last round of chunks would
// leave a tenth of the compute units or more idle. (240 bins: 300 chunks 26.4 us whole, 21.4 halved; 900, 67 and 62; 1,800,
// 82 and 79; 3,600, 144 and 151. 480 bins: 900 chunks 50.4 and 47.3, 1,800 chunks 83.3 and 85.3. With full rounds it loses:
// 256 bins, 512 chunks, 27.2 and 28.6. With many more bins the halved chunk's runs are short: 800x600 at 64 per pixel,
// 500 bins, 333 us staged, 301 whole, 416 halved.)
constexpr uint32_t kSmallChunk = 2048;

static Geom chunked(Geom g, uint64_t F) {
  const uint64_t n = (F + 4095) / 4096, rounds = (n + kComputeUnits - 1) / kComputeUnits;
  const uint32_t bins = g.two ? g.nsuper : g.ntiles;
  if (g.C == 1 && g.lds_bins && g.chunk == 4096 && F >= 4 && bins <= 512 && rounds * bins <= 2048 &&
      10 * n <= 9 * rounds * kComputeUnits)
    g.chunk = kSmallChunk;
  return g;
}

template <int C, bool IDX>
static hipError_t launch_scatter(const Geom& g, const wt_fragments& f, int vec, uint32_t* cursors,
                                 uint32_t* head, uint32_t* tail, WsHeader* hdr,
                                 unsigned long long cstamp, uint32_t cap, const GradOut& go, uint32_t nchunks, hipStream_t s) {
  if constexpr (C == 1 || !IDX) {  // (a chunk of three-channel records with their indexes is all of the LDS)
    if (stream_scatter(g, f.count, IDX)) {
      auto k = k_scatter_stream<C, IDX, 1024>;
      if constexpr (C == 1)
        if (g.chunk == kSmallChunk) k = k_scatter_stream<C, IDX, kSmallChunk / 4>;
      const size_t lds = stream_lds(g.chunk, C, IDX, g.ntiles);
      hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
      // one workgroup per compute unit, two of the small ones (multiples of the classes)
      const uint32_t grid = std::min<uint32_t>(nchunks, g.chunk == kSmallChunk ? 2 * kComputeUnits : kComputeUnits);
      hipLaunchKernelGGL(k, dim3(grid), dim3(g.chunk / 4), lds, s, f, g, nchunks, cursors, head, tail, hdr, cstamp, cap, go);
      return hipGetLastError();
    }
  }
  if (!g.lds_bins) {
    hipLaunchKernelGGL((k_scatter_global<C, IDX>), dim3(nchunks), dim3(1024), 0, s, f, g, vec, cursors, head, tail, hdr,
                       cstamp, cap, go);
    return hipGetLastError();
  }
  // (a one-channel stream in short chunks comes here only with fewer than four fragments)
  auto run = launch_scatter_staged<C, IDX, 1024>;
  if constexpr (C == 3)
    if (g.sthreads == 512) run = launch_scatter_staged<C, IDX, 512>;
  return run(g, f, vec, cursors, head, tail, hdr, cstamp, cap, go, nchunks, s);
}

hipError_t launch_bin_count(const Geom& geom, const wt_fragments& f, void* ws, const Layout& l, hipStream_t s) {
  const Geom g = chunked(geom, f.count);
  char* b = (char*)ws;
  uint32_t* counts = (uint32_t*)(b + l.counts);
  uint32_t* offsets = (uint32_t*)(b + l.offsets);
  uint32_t* cursors = (uint32_t*)(b + l.cursors);
  WsHeader* hdr = (WsHeader*)(b + l.header);
  unsigned long long* dropped = &hdr->dropped;
  const uint64_t ncount = (uint64_t)g.NX * g.ntiles;
  // reset the header and zero the tile counts (kernels, not memsets: safe inside captured graphs)
  hipLaunchKernelGGL(k_count_reset, dim3((unsigned)std::min<uint64_t>((ncount + 255) / 256, 4096)), dim3(256), 0, s,
                     hdr, counts, ncount);
  const uint32_t F = (uint32_t)f.count;
  const uint32_t nchunks = (uint32_t)(((uint64_t)F + g.chunk - 1) / g.chunk);
  const int vec = aligned16(f.pixel);
  if (F > 0) {
    if (g.lds_bins) {
      // at most 1024 workgroups (four per compute unit with 256 threads): each counts about 32 chunks of its class
      // and then adds its table to the global counts once (half the global adds of 2048 workgroups; the smoke
      // frame's histogram measured 0.111 -> 0.101 ms)
      const uint32_t grid = std::min<uint32_t>(((nchunks + g.NX - 1) / g.NX) * g.NX, 1024);
      const size_t lds = 4ull * g.hrb;
      if (lds <= 32768) {
        hipLaunchKernelGGL(k_hist_lds<256>, dim3(grid), dim3(256), lds, s, f.pixel, F, g, vec, counts, dropped);
      } else {
        auto k = k_hist_lds<1024>;
        if (lds > 65536) {
          hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
          if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(k, dim3(grid), dim3(1024), lds, s, f.pixel, F, g, vec, counts, dropped);
      }
    } else {
      hipLaunchKernelGGL(k_hist_global, dim3(2048), dim3(256), 0, s, f.pixel, F, g, counts, dropped);
    }
  }
  const unsigned long long cstamp = count_stamp(g, l, f);
  const uint64_t nseg = (uint64_t)g.NX * g.ntiles;
  if (g.NX == kClasses && g.ntiles <= kScanTiles * kScanThreads) {
    hipLaunchKernelGGL(k_scan, dim3(1), dim3(kScanThreads), 0, s, counts, g, offsets, cursors,
                       (uint32_t*)(b + l.order), 1, g.two ? nullptr : hdr, cstamp);
  } else {
    // many tiles (two-level and global-atomic binnings): the scan over several workgroups
    uint32_t* part = (uint32_t*)(b + l.scan);
    const uint32_t G = (uint32_t)((nseg + kScanRange - 1) / kScanRange);
    auto sum = g.NX == 1 ? k_scan_part<1> : k_scan_part<kClasses>;
    auto apply = g.NX == 1 ? k_scan_apply<1> : k_scan_apply<kClasses>;
    hipLaunchKernelGGL(sum, dim3(G), dim3(kScanThreads), 0, s, counts, g, part);
    hipLaunchKernelGGL(apply, dim3(G), dim3(kScanThreads), 0, s, counts, g, part, offsets, cursors,
                       (uint32_t*)(b + l.order), g.two ? nullptr : hdr, cstamp);
  }
  if (g.two) {
    // first level: per-class super-tile counts, and their segments and cursors
    const Geom gs = super_geom(g);
    uint32_t* counts1 = (uint32_t*)(b + l.counts1);
    const uint32_t n1 = g.NX * g.nsuper;
    hipLaunchKernelGGL(k_super_counts, dim3((n1 + 255) / 256), dim3(256), 0, s, counts, g, counts1);
    hipLaunchKernelGGL(k_scan, dim3(1), dim3(kScanThreads), 0, s, counts1, gs, (uint32_t*)(b + l.offsets1),
                       (uint32_t*)(b + l.cursors1), (uint32_t*)(b + l.order1), 0, hdr, cstamp);
  }
  return hipGetLastError();
}

hipError_t launch_bin_scatter(const Geom& geom, const wt_fragments& f, void* ws, const Layout& l, const GradOut& go,
                              hipStream_t s) {
  const Geom g = chunked(geom, f.count);
  const bool record_index = go.on;
  char* b = (char*)ws;
  uint32_t* cursors = (uint32_t*)(b + l.cursors);
  const uint32_t* offsets = (const uint32_t*)(b + l.offsets);
  uint32_t* head = (uint32_t*)(b + l.heads);
  uint32_t* tail = (uint32_t*)(b + l.tails);
  WsHeader* hdr = (WsHeader*)(b + l.header);
  const unsigned long long cstamp = count_stamp(g, l, f);
  const unsigned long long stamp = layout_stamp(g, l, record_index);
  const uint32_t cap = (uint32_t)std::min<uint64_t>(l.cap, 0xffffffffull);  // records each array holds
  const uint32_t F = (uint32_t)f.count;
  const uint32_t nchunks = (uint32_t)(((uint64_t)F + g.chunk - 1) / g.chunk);
  const int vec = aligned16(f.pixel) && aligned16(f.depth) && aligned16(f.alpha) && aligned16(f.rgb);
  hipError_t e = hipSuccess;
  if (g.serial) {
    // deterministic: straight into the tile segments, whatever the number of levels
    auto k = g.C == 1 ? (record_index ? k_scatter_serial<1, true> : k_scatter_serial<1, false>)
                      : (record_index ? k_scatter_serial<3, true> : k_scatter_serial<3, false>);
    hipLaunchKernelGGL(k, dim3(1), dim3(64), 0, s, f, g, cursors, offsets, head, tail, hdr, cstamp, go);
    launch_seal(hdr, cursors, offsets, g.NX, g.ntiles, cstamp, stamp, s);
    return hipGetLastError();
  }
  // two levels: the stream into super-tiles (first-level arrays), then each super-tile into its tiles
  const Geom gs = g.two ? super_geom(g) : g;
  uint32_t* cursors1 = g.two ? (uint32_t*)(b + l.cursors1) : cursors;
  uint32_t* head1 = g.two ? (uint32_t*)(b + l.heads1) : head;
  uint32_t* tail1 = g.two ? (uint32_t*)(b + l.tails1) : tail;
  const uint32_t* offsets1 = g.two ? (const uint32_t*)(b + l.offsets1) : offsets;
  const unsigned long long stamp1 = g.two ? level1_stamp(stamp) : stamp;
  if (F > 0) {
    auto scatter = g.C == 1 ? (record_index ? launch_scatter<1, true> : launch_scatter<1, false>)
                            : (record_index ? launch_scatter<3, true> : launch_scatter<3, false>);
    e = scatter(gs, f, vec, cursors1, head1, tail1, hdr, cstamp, cap, go, nchunks, s);
    if (e != hipSuccess) return e;
  }
  launch_seal(hdr, cursors1, offsets1, gs.NX, gs.ntiles, cstamp, stamp1, s);
  if (!g.two) return hipGetLastError();
  auto split = [&](auto kern, uint32_t rb, uint32_t per) -> hipError_t {
    const size_t lds = (size_t)kSplitThreads * per * rb;
    if (lds > 65536) {
      hipError_t e2 = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e2 != hipSuccess) return e2;
    }
    hipLaunchKernelGGL(kern, dim3(g.nsuper), dim3(kSplitThreads), lds, s, g, offsets1, offsets, head1, tail1, head,
                       tail, hdr, stamp1);
    return hipGetLastError();
  };
  if (g.C == 1)
    e = record_index ? split(k_split<1, true>, staged_record_bytes(1, true), split_per(1, true))
                     : split(k_split<1, false>, staged_record_bytes(1, false), split_per(1, false));
  else
    e = record_index ? split(k_split<3, true>, staged_record_bytes(3, true), split_per(3, true))
                     : split(k_split<3, false>, staged_record_bytes(3, false), split_per(3, false));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_seal_split, dim3(1), dim3(1), 0, s, hdr, stamp1, stamp);
  return hipGetLastError();
}

hipError_t launch_bin(const Geom& g, const wt_fragments& f, void* ws, const Layout& l, const GradOut& go,
                      hipStream_t s) {
  if (small_stream(g, f.count)) {
    char* b = (char*)ws;
    WsHeader* hdr = (WsHeader*)(b + l.header);
    hipLaunchKernelGGL(k_count_reset, dim3(1), dim3(256), 0, s, hdr, nullptr, (uint64_t)0);
    const uint32_t P = small_parts(f.count);
    auto form = [&](auto parts) {
      constexpr uint32_t N = decltype(parts)::value;
      return g.C == 1 ? (go.on ? k_bin_small<1, true, N> : k_bin_small<1, false, N>)
                      : (go.on ? k_bin_small<3, true, N> : k_bin_small<3, false, N>);
    };
    auto k = P == 1   ? form(std::integral_constant<uint32_t, 1>{})
             : P == 2 ? form(std::integral_constant<uint32_t, 2>{})
                      : form(std::integral_constant<uint32_t, 4>{});
    const size_t lds = (2ull * P * small_list((uint32_t)f.count, P) + 3) & ~(size_t)3;
    if (lds > 65536 - 1024) {
      hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k, dim3((g.ntiles + P - 1) / P * P), dim3(1024), lds, s, f, g, aligned16(f.pixel) ? 1 : 0,
                       (uint32_t*)(b + l.offsets), (uint32_t*)(b + l.order), (uint32_t*)(b + l.heads),
                       (uint32_t*)(b + l.tails), hdr, layout_stamp(g, l, go.on), go);
    return hipGetLastError();
  }
  hipError_t e = launch_bin_count(g, f, ws, l, s);
  if (e != hipSuccess) return e;
  return launch_bin_scatter(g, f, ws, l, go, s);
}

}  // namespace wt
