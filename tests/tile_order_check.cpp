// Checks the order in which workgroups take tiles, on the host: every tile exactly once, and what the choice between the two
// orders is for.  Prints the number of grids checked, or what failed.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../paper_2603_12440_amd/csrc/tile_order.hpp"

using namespace mi355gemm;

// tiles per XCD (workgroups are dealt round-robin), in the order in which they are taken
static std::vector<std::vector<std::pair<int, int>>> walk(int tiles_m, int tiles_n, bool strips, int spread) {
  const TileOrder o = make_tile_order(tiles_m, tiles_n, strips);
  const int n = tiles_m * tiles_n;
  std::vector<char> seen(n, 0);
  std::vector<std::vector<std::pair<int, int>>> xcd(8);
  for (int wg = 0; wg < n; ++wg) {
    int tm = -1, tn = -1;
    tile_of<true>(o, tiles_m, tiles_n, spread, strips, wg, n, tm, tn);
    if (!strips) {                                     // what the kernels with regions only compute
      int m = -1, k = -1;
      tile_of<false>(o, tiles_m, tiles_n, spread, false, wg, n, m, k);
      if (m != tm || k != tn) tm = -1;
    }
    if (tm < 0 || tm >= tiles_m || tn < 0 || tn >= tiles_n || seen[tm * tiles_n + tn]++) {
      std::printf("%dx%d strips %d spread %d: workgroup %d takes (%d, %d)\n", tiles_m, tiles_n, strips, spread, wg, tm, tn);
      std::exit(1);
    }
    xcd[wg % 8].push_back({tm, tn});
  }
  return xcd;
}

// panels that one tile of an XCD reads and no other: nobody else brings them to that L2
static int unshared(const std::vector<std::vector<std::pair<int, int>>>& xcd, int tiles_m, int tiles_n) {
  int count = 0;
  for (const auto& tiles : xcd) {
    std::vector<int> rows(tiles_m, 0), cols(tiles_n, 0);
    for (const auto& t : tiles) { ++rows[t.first]; ++cols[t.second]; }
    for (const auto& t : tiles) count += (rows[t.first] == 1) + (cols[t.second] == 1);
  }
  return count;
}

int main() {
  long grids = 0;
  for (int m = 1; m <= 50; ++m)
    for (int n = 1; n <= 50; ++n)
      for (int strips = 0; strips < 2; ++strips)
        for (int spread = 0; spread < 2; ++spread) { walk(m, n, strips, spread); ++grids; }
  const int large[][2] = {{1, 70000}, {70000, 1}, {257, 300}, {300, 257}, {17, 4099}, {4099, 17}, {512, 512}, {2, 33333}, {9, 9001}};
  for (const auto& g : large)
    for (int strips = 0; strips < 2; ++strips)
      for (int spread = 0; spread < 2; ++spread) { walk(g[0], g[1], strips, spread); ++grids; }
  // two workgroups per CU and between one and two tiles per CU: all run at once, few panels are read by one tile of an XCD alone
  long strips = 0, regions = 0;
  for (int m = 1; m < 512; ++m)
    for (int n = 1; n < 512; ++n)
      if (m >= 5 && n >= 5 && takes_strips(m, n, 128 * 128, true, 4096, true)) {
        ++grids;
        strips += unshared(walk(m, n, true, 1), m, n);
        regions += unshared(walk(m, n, false, 1), m, n);
      }
  if (strips * 2 > regions) { std::printf("panels read by one tile alone: strips %ld, regions %ld\n", strips, regions); return 1; }
  // where the line lies
  struct { int m, n, area; bool two; int k_bytes; bool whole, want; } rule[] = {
      {24, 11, 128 * 128, true, 4096, true, true},    {24, 11, 128 * 128, false, 4096, true, false}, {24, 11, 256 * 256, false, 4096, true, false},
      {16, 16, 128 * 128, true, 4096, true, false},   {32, 16, 128 * 128, true, 4096, true, false},  {5, 59, 128 * 128, true, 4096, true, false},
      {8, 40, 128 * 128, true, 4096, true, true},     {59, 5, 128 * 128, true, 4096, true, true},    {41, 61, 128 * 128, true, 512, true, true},
      {41, 61, 128 * 128, true, 514, true, false},    {40, 61, 128 * 128, true, 512, true, false},   {40, 61, 128 * 128, true, 512, false, true},
      {17, 19, 256 * 256, false, 64, true, true},     {24, 11, 64 * 64, true, 64, false, false}};
  for (const auto& r : rule)
    if (takes_strips(r.m, r.n, r.area, r.two, r.k_bytes, r.whole) != r.want) {
      std::printf("%dx%d tiles of area %d, K of %d bytes: expected %s\n", r.m, r.n, r.area, r.k_bytes, r.want ? "strips" : "regions");
      return 1;
    }
  struct { int m, n, area, k_bytes; bool any_rows, want; } deal[] = {
      {45, 5, 128 * 128, 1570, false, true},  {2, 79, 64 * 64, 8192, false, false},  {2, 79, 64 * 64, 8192, true, false}, {10, 11, 64 * 64, 8220, true, true},
      {10, 11, 64 * 64, 8220, false, false},  {10, 11, 64 * 64, 512, true, false},   {8, 9, 64 * 64, 8220, true, false},  {9, 27, 64 * 64, 8220, true, true},
      {7, 9, 64 * 64, 8220, true, false},     {1, 14, 64 * 64, 8220, true, true},    {1, 14, 64 * 64, 8220, false, false}, {1, 17, 64 * 64, 8220, true, false},
      {11, 10, 256 * 256, 8192, false, false}, {29, 9, 64 * 64, 8220, true, false}, {6, 7, 64 * 64, 8220, true, true}, {6, 7, 64 * 64, 8220, false, false}};
  for (const auto& r : deal)
    if (dealt_one_by_one(r.m, r.n, r.area, r.k_bytes, r.any_rows) != r.want) {
      std::printf("%dx%d tiles of area %d, K of %d bytes, any rows %d: expected %d\n", r.m, r.n, r.area, r.k_bytes, r.any_rows, r.want);
      return 1;
    }
  // the lines of a panel that neighbouring tiles touch: all of them, whatever the number of tiles, and none by more than a
  // workgroup has to
  for (int tiles = 1; tiles <= 20; ++tiles)
    for (int at_most = 4; at_most <= 8; at_most *= 2)
      for (int lines : {48, 56, 64}) {
        std::vector<int> by(lines, 0);
        for (int tile = 0; tile < tiles && tile < at_most; ++tile)
          for (int lane = 0; lane < 64; ++lane) {
            const int l = touched_line(lane, tile, touch_shift(tiles, at_most), lines);
            if (l < 0 || l >= lines) { std::printf("%d tiles: line %d of %d\n", tiles, l, lines); return 1; }
            by[l] |= 1 << tile;
          }
        for (int l = 0; l < lines; ++l)
          if (!by[l] || (l + 1 < lines && (tiles & (tiles - 1)) == 0 && (by[l] & (by[l] - 1)))) {
            std::printf("%d tiles, at most %d: line %d of %d touched by the set %x\n", tiles, at_most, l, lines, by[l]);
            return 1;
          }
      }
  std::printf("%ld grids ok, panels read by one tile alone: strips %ld, regions %ld\n", grids, strips, regions);
  return 0;
}
