// Host check of the tile sequence of a launch (tile_regions, region_tile in
// ws_gemm_plan.hpp), built with g++ and the undefined-behaviour sanitizer by
// tests/test_tile_regions.py: for every small grid of tiles and every block
// left out of it, each tile outside the block is visited exactly once, none
// inside it is, and the indexes past the end, which the kernels ask for and
// drop, divide by nothing that is zero.  Exit status 0 when so.
#include <cstdio>
#include <vector>

#include "ws_gemm_plan.hpp"

static int check(int tm, int tn, int gm, int cm, int cn) {
  const wsg::TileRegions r = wsg::tile_regions(tm, tn, gm, cm, cn);
  const int tiles = r.num_tiles;
  std::vector<int> seen((size_t)tm * tn, 0);
  int ti, tj;
  for (int v = 0; v < tiles; ++v) {
    wsg::region_tile(r, v, &ti, &tj);
    if (ti < 0 || ti >= tm || tj < 0 || tj >= tn) return 1;
    ++seen[(size_t)ti * tn + tj];
  }
  for (int i = 0; i < tm; ++i)
    for (int j = 0; j < tn; ++j)
      if (seen[(size_t)i * tn + j] != (i < cm && j < cn ? 0 : 1)) return 1;
  for (int past = 0; past < 600; past += 7) {
    wsg::region_tile(r, tiles + past, &ti, &tj);
    if (ti < 0 || ti >= tm || tj < 0 || tj >= tn) return 1;
  }
  return 0;
}

int main() {
  for (int tm = 1; tm <= 9; ++tm)
    for (int tn = 1; tn <= 9; ++tn) {
      for (int gm = 1; gm <= tm; gm *= 2)
        if (check(tm, tn, gm, -1, -1)) return std::printf("%d x %d, groups of %d\n", tm, tn, gm), 1;
      for (int cm = 1; cm <= tm; ++cm)
        for (int cn = 1; cn <= tn; ++cn)
          if (cm * cn < tm * tn && check(tm, tn, 1, cm, cn))
            return std::printf("%d x %d without %d x %d\n", tm, tn, cm, cn), 1;
    }
  return 0;
}
