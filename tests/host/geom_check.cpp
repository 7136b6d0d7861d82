// Host checks of the frame geometry (wt_bin.hip: make_geom, make_layout; wt_tile.h: tile addressing). One check per
// argument; prints "bad 0" when it holds.
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "wt_bin.hip"
#include "wt_tile.h"

static int bad = 0;

static void expect(bool ok, const char* what, const wt_frame_desc& d, bool bwd) {
  if (ok) return;
  if (++bad <= 20)
    printf("FAIL %s: %ux%u rank %u channels %u dtype %u flags %u %s\n", what, d.width, d.height, d.rank, d.channels,
           d.coeff_dtype, d.flags, bwd ? "gradient" : "forward");
}

// Every valid combination of rank, channels, storage that changes the tile, flags and direction.
template <typename F>
static void each_form(uint32_t w, uint32_t h, F&& f) {
  for (uint32_t rank = 0; rank <= 10; ++rank)
    for (uint32_t ch : {1u, 3u})
      for (uint32_t fl : {0u, WT_TIGHT_DEPTH, WT_TEMPORAL})
        for (int bwd = 0; bwd < 2; ++bwd) {
          if (fl == WT_TEMPORAL && rank > 4) continue;
          f(wt_frame_desc{w, h, rank, ch, WT_F32, fl}, bwd != 0);
        }
}

// The last tile's pixels are those of the frame and no others, also where its rows end at 2^32.
static void last_tile() {
  const uint32_t top = 0xffffffffu;
  std::vector<std::pair<uint32_t, uint32_t>> sizes = {{top, 1}, {top - 7, 1}, {1920, 1080}, {65535, 65537}, {3, 1431655765}};
  for (uint32_t k : {0u, 1u, 4u, 5u, 31u, 58u, 59u, 60u, 63u, 64u, 1000u}) sizes.push_back({1, top - k});
  for (auto [w, h] : sizes)
    each_form(w, h, [&](const wt_frame_desc& d, bool bwd) {
      const wt::Geom g = wt::make_geom(d, bwd);
      const wt::TileRef r{(g.tilesX - 1) * g.TW, (g.tilesY - 1) * g.TH, 0, 0};
      bool ok = g.W - r.x0 <= g.TW && g.H - r.y0 <= g.TH;
      for (uint32_t lp = 0; lp < g.tile_px; ++lp) {
        const uint64_t x = (uint64_t)r.x0 + (lp & (g.TW - 1)), y = (uint64_t)r.y0 + (lp >> g.lTW);
        const bool want = x < g.W && y < g.H;
        uint64_t p;
        ok &= wt::tile_pixel(g, r, lp, p) == want && (!want || p == y * g.W + x);
      }
      expect(ok, "pixels of the last tile", d, bwd);
    });
}

// Frames at the limits of every size still get tables that cover all their tiles.
static void limits() {
  const uint32_t top = 0xffffffffu;
  const std::pair<uint32_t, uint32_t> sizes[] = {{1, 1}, {top, 1}, {1, top}, {2, 0x7fffffff}, {3, 1431655765}, {65535, 65537}};
  for (auto [w, h] : sizes)
    each_form(w, h, [&](const wt_frame_desc& d, bool bwd) {
      const wt::Geom g = wt::make_geom(d, bwd);
      bool ok = (uint64_t)g.tilesX * g.tilesY == g.ntiles && g.hrb > 0 && g.hrb <= wt::kMaxHistBins;
      ok &= (uint64_t)g.sX * g.SW >= g.tilesX && (uint64_t)g.sY * g.SH >= g.tilesY;
      ok &= wt::make_layout(g, 0).total > 4ull * g.NX * g.ntiles;
      expect(ok, "tables at the size limits", d, bwd);
    });
}

// Fragments of a frame in WT_SCRATCH_BYTES when it is cut into the largest power-of-two tiles (a column per thread for
// packed storage and the one-pass render), one level up to 4,096 tiles, then super-tiles doubled up to 8 x 8 tiles until
// there are at most 1,024, and one class without tables per super-tile past 8,192 of them.
static uint64_t fragments_of_largest_tiles(const wt_frame_desc& d) {
  const uint64_t C = d.channels, M = 2ull << d.rank, AL = C + 3;
  const bool temporal = d.flags & WT_TEMPORAL;
  const uint64_t per_px = 8 * (C * M + AL) + (temporal ? 4 * C * M : 0) + (d.flags & WT_TIGHT_DEPTH ? 8 : 0);
  uint32_t e = 0;
  while ((2ull << e) <= std::min<uint64_t>(163840 / per_px, 2048)) ++e;
  if (temporal || d.coeff_dtype == WT_E5B9G9R9) e = std::min(e, C == 1 ? 10u : 8u);
  auto up = [](uint64_t n, uint64_t by) { return (n + by - 1) / by; };
  const uint64_t tx = up(d.width, 1ull << (e + 1) / 2), ty = up(d.height, 1ull << e / 2), nt = tx * ty;
  uint64_t sw = 1, sh = 1, NX = 8, copies = 1, supers = 0;
  if (nt > 4096) {
    while (up(tx, sw) * up(ty, sh) > 1024 && sw * sh < 64) (sw <= sh ? sw : sh) *= 2;
    supers = up(tx, sw) * up(ty, sh);
    if (supers <= 8192) copies = 2;
    else supers = 0, NX = 1;
  }
  auto a = [&](uint64_t bytes) { return up(bytes, 256) * 256; };
  auto tables = [&](uint64_t n) { return 2 * a(4 * NX * n) + a(4 * (NX * n + 1)) + a(4 * n); };
  auto bytes = [&](uint64_t F) {
    return 256 + tables(nt) + a(4 * 257 * up(NX * nt, 16384)) + copies * (a(4 * (2 + C) * F) + a(16 * F)) +
           (copies == 2 ? tables(supers) : 0);
  };
  if (bytes(0) > WT_SCRATCH_BYTES) return 0;
  uint64_t F = (WT_SCRATCH_BYTES - bytes(0)) / (copies * 4 * (6 + C));
  while (F && bytes(F) > WT_SCRATCH_BYTES) --F;
  return F;
}

// wt_render_noalloc takes as many fragments of any frame as fit its limit with the largest tiles.
static void scratch() {
  uint32_t seed = 12345;
  auto rnd = [&](uint32_t n) {
    seed = seed * 1664525u + 1013904223u;
    return (uint32_t)((uint64_t)(seed >> 8) * n >> 24);
  };
  std::vector<wt_frame_desc> ds = {{961, 1255, 7, 1, WT_F32, 0},   {15, 2879, 10, 3, WT_F32, 0},
                                   {398, 38445, 6, 3, WT_F32, 0},  {3358, 48264, 3, 3, WT_F32, 0},
                                   {16384, 16385, 3, 1, WT_F32, 0}, {62633, 9101, 0, 1, WT_F32, 0},
                                   {20199, 7480, 4, 1, WT_F32, WT_TEMPORAL}, {19906, 19238, 1, 3, WT_E5B9G9R9, WT_TEMPORAL}};
  while (ds.size() < 40000) {
    const uint32_t w = 1 + rnd(1u << (1 + rnd(17))), h = 1 + rnd(1u << (1 + rnd(17)));
    wt_frame_desc d{w, h, rnd(11), rnd(2) ? 3u : 1u, WT_F32, rnd(3)};
    if ((uint64_t)w * h >> 32 || (d.flags == WT_TEMPORAL && d.rank > 4)) continue;
    if (d.channels == 3 && d.rank <= 4 && rnd(2)) d.coeff_dtype = WT_E5B9G9R9;
    ds.push_back(d);
  }
  for (const wt_frame_desc& d : ds) {
    wt::Geom g;
    size_t need, limit;
    const uint64_t F = fragments_of_largest_tiles(d);
    const bool ok = wt::scratch_geom(d, F, g, need, limit);
    expect(!F || (ok && need <= limit && limit <= wt::kScratchBytes), "fragments of the scratch array", d, false);
    // and no more than twice that, where the frame's own tiles are binned in one level instead of two
    expect(!wt::scratch_geom(d, WT_SCRATCH_BYTES / (4 * (6 + d.channels)) + (1u << 20), g, need, limit),
           "limit of the scratch array", d, false);
  }
}

// The least cost of all tile shapes of a frame at M <= 32, without the search's bounds: the larger of equals, the narrower
// of those.
static void all_shapes(const wt::Geom& g, uint32_t per_px, uint32_t& lTW, uint32_t& TH) {
  uint32_t most = std::min(wt::kLdsBytes / per_px, wt::kMaxTilePx);
  if (g.M >= 16) most = std::min(most, wt::kTileThreads / g.C);
  uint64_t best = ~0ull;
  for (uint32_t l = 3; l <= 6; ++l)
    for (uint32_t tw = 1u << l, th = std::min(2 * tw - 1, most / tw); th >= tw / 2 && tw * th >= wt::kMinTilePx; --th) {
      const uint32_t px = tw * th, tx = (g.W - 1) / tw + 1, ty = (g.H - 1) / th + 1;
      const uint64_t nt = (uint64_t)tx * ty;
      uint64_t cost = (nt + 255) / 256 * (px + wt::kTileFixedPx);
      uint32_t lsw, sh;
      if (nt > wt::kTwoLevelTiles) cost += wt::pick_supers(tx, ty, lsw, sh) * px;
      if (nt > wt::kMaxLdsBins * wt::kMaxSub) cost = nt << 24;
      if (cost < best || (cost == best && px > TH << lTW)) best = cost, lTW = l, TH = th;
    }
}

// The bounded search of the tile shape finds what the search of all shapes finds, in less than half of its time on frames
// that have thousands of tiles.
static void shapes() {
  uint32_t seed = 99;
  auto rnd = [&](uint32_t n) {
    seed = seed * 1664525u + 1013904223u;
    return (uint32_t)((uint64_t)(seed >> 8) * n >> 24);
  };
  for (int i = 0; i < 60000; ++i) {
    const uint32_t w = 1 + rnd(1u << (1 + rnd(17))), h = 1 + rnd(1u << (1 + rnd(17)));
    const bool bwd = rnd(2);
    const wt_frame_desc d{w, h, rnd(5), rnd(2) ? 3u : 1u, WT_F32, rnd(3)};
    if ((uint64_t)w * h >> 32) continue;
    const wt::Geom g = wt::make_geom(d, bwd);
    uint32_t l = 0, th = 0;
    all_shapes(g, wt::tile_px_bytes(g, bwd), l, th);
    expect(l == g.lTW && th == g.TH, "tile shape", d, bwd);
  }
  double all = 0, bounded = 0;
  volatile uint32_t sink = 0;
  auto now = [] { return std::chrono::duration<double>(std::chrono::steady_clock::now().time_since_epoch()).count(); };
  const std::pair<uint32_t, uint32_t> sizes[] = {{1920, 1080}, {3840, 2160}, {7680, 4320}, {16001, 16003}, {65535, 65537}};
  for (auto [w, h] : sizes) {
    const wt_frame_desc d{w, h, 3, 1, WT_F32, 0};
    const wt::Geom g = wt::make_geom(d);
    uint32_t l = 0, th = 0;
    double t = now();
    for (int i = 0; i < 500; ++i) sink = sink + wt::make_geom(d).TH;
    bounded += now() - t;
    t = now();
    for (int i = 0; i < 500; ++i) all_shapes(g, wt::tile_px_bytes(g, false), l, th), sink = sink + th;
    all += now() - t;
  }
  printf("all shapes %.2f us a frame, bounded %.2f\n", all / 2500 * 1e6, bounded / 2500 * 1e6);
  expect(bounded < 0.5 * all, "time of the search", {0, 0, 3, 1, WT_F32, 0}, false);
}

// Row numbers by one 24-bit multiply, for tiles and super-tiles of every height that frames of up to 2^14 rows get.
static void rows() {
  for (uint32_t h : {1u, 2u, 100u, 4095u, 4096u, 4097u, 8192u, 8193u, 12288u, 16383u, 16384u, 16385u})
    for (uint32_t w : {1u, 3u, 16u, 160u, 500u, 4000u})
      each_form(w, h, [&](const wt_frame_desc& d, bool bwd) {
        wt::Geom gs[2] = {wt::make_geom(d, bwd)};
        gs[1] = wt::super_geom(gs[0]);
        for (const wt::Geom& g : gs)
          if (g.mulTH)
            for (uint32_t y = 0; y < h; ++y) {
              const uint32_t p = (y & 0xffffff) * (g.mulTH & 0xffffff);
              if (p >> 20 != y / g.TH) {
                expect(false, "row of a tile", d, bwd);
                break;
              }
            }
        expect(h > 16384 || gs[0].mulTH || gs[0].TH < 4, "one multiply for the usual frames", d, bwd);
      });
}

// describe <width> <height> <rank> <channels> <flags> <gradient>: the frame's tiles and its binning levels.
static int describe(char** a) {
  auto n = [&](int i) { return (uint32_t)strtoul(a[i], nullptr, 10); };
  const wt::Geom g = wt::make_geom(wt_frame_desc{n(0), n(1), n(2), n(3), WT_F32, n(4)}, n(5) != 0);
  printf("tiles %u levels %u\nbad 0\n", g.ntiles, g.two ? 2u : g.lds_bins ? 1u : 0u);
  return 0;
}

int main(int argc, char** argv) {
  const char* what = argc > 1 ? argv[1] : "";
  if (!strcmp(what, "describe") && argc == 8) return describe(argv + 2);
  if (!strcmp(what, "last_tile")) last_tile();
  else if (!strcmp(what, "limits")) limits();
  else if (!strcmp(what, "scratch")) scratch();
  else if (!strcmp(what, "shapes")) shapes();
  else if (!strcmp(what, "rows")) rows();
  else return 2;
  printf("bad %d\n", bad);
  return bad != 0;
}
