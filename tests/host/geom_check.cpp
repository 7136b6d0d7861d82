// Host checks of the frame geometry (wt_bin.hip: make_geom, make_layout; wt_tile.h: tile addressing). One check per
// argument; prints "bad 0" when it holds.
#include <cstdio>
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

int main(int argc, char** argv) {
  const char* what = argc > 1 ? argv[1] : "";
  if (!strcmp(what, "last_tile")) last_tile();
  else if (!strcmp(what, "limits")) limits();
  else return 2;
  printf("bad %d\n", bad);
  return bad != 0;
}
