// In which order the workgroups of one launch take the tiles of C.  Plain integer code, compiled for host and device.
//
// Workgroups are handed to the 8 XCDs round-robin; each XCD has its own L2, all of them share the last-level cache.
// Two orders:
//   * regions: 256 consecutive tile ids, what the chip works on at a time with one workgroup per CU, are a compact region
//     of up to 16 x 16 tiles (groups of 16 tile rows, every other group walked backwards), and the 32 tiles of a region
//     that one XCD gets are an 8 x 4 block, which share 12 panels in its L2.  So a region touches 32 panels instead of all
//     of A, and the next region finds half of them in the last-level cache: with operands that are not in that cache when
//     the launch begins, 8192^3 takes 756 us (820 us with every XCD walking its own eighth of the tiles).  A round whose tiles
//     do not divide by 8 is cut into runs all the same, the first XCDs' one tile longer (100x5000x4096, 158 tiles of 64x64:
//     24.6 us dealt one by one, 17.0 in runs).
//   * strips: groups of 8 tile rows, each walked column by column over the full width, one renumbering over the whole grid
//     (an eighth per XCD; none where the tiles do not divide by 8: then tile row r of a group is XCD r's).
// Strips serve two kinds of launches (us with strips / with regions, operands in the last-level cache):
//   * 128x128 tiles, two workgroups per CU, between one and two tiles per CU.  All of them run at once; the regions' second
//     round would give an XCD a few tiles far from its first 32, whose panels nothing else in that L2 reads, and a launch takes
//     as long as those: bf16, K = 2056, 24x11 tiles 33.8 / 40.3, 59x5 37.5 / 43.2; fp8, 679 drawn grids with K > 512 0.98.  Not for
//     grids at least twice as wide as high whose tiles do not divide by 8 (bf16, 5x59: 45.8 / 40.6).
//   * K of at most 512 bytes, where writing C is most of the work: full-width rows of C are written closer together in time.
//     41x61 tiles of 128x128 but 8 columns, K = 64: bf16 32.5 / 39.1; 9x28 tiles of 256x256, K = 64: bf16
//     18.0 / 18.8; fp8, 20000 drawn grids: even (0.92 to 1.06; 1.03 with 256 to 512 tiles of 128x128, twice as wide as high).  Unless the tiles divide by 8 and C's rows are whole 16-byte pieces (regions up to 5 % ahead there;
//     rows at any element, 4700 drawn products: strips 1.3 % ahead with fp32 results, even with 16-bit ones).
#pragma once

#include <stdint.h>

namespace mi355gemm {

struct TileOrder {
  uint32_t div_group, div_rows, div_h;   // reciprocals of what tile_of divides by: tiles of a group, of a strip of the last one, its rows
};

inline TileOrder make_tile_order(int tiles_m, int tiles_n, bool strips) {
  auto m = [](int64_t d) { return d < 2 ? ~0u : (uint32_t)((((uint64_t)1 << 32) + d - 1) / d); };
  const int G = strips ? 8 : 16, rows = (tiles_m - 1) % G + 1;
  return TileOrder{m((int64_t)G * tiles_n), m((int64_t)(strips ? tiles_n : 4) * rows), m(rows <= 8 ? rows : rows - 8)};
}

// Kernels whose launches may take strips: large tiles with two slabs in LDS.  (The persistent 256x256 kernels never gained more
// than 3 % by them and pay for the choice.)
template <int BM, int BN, int SLABS, bool PERSIST>
constexpr bool kEitherOrder = BM * BN >= 128 * 128 && SLABS == 2 && !(PERSIST && BM * BN > 128 * 128);

// Which of the two a launch takes.  two_per_cu: two workgroups of this kernel fit a CU; whole_rows: rows of C are whole
// 16-byte pieces.
inline bool takes_strips(int64_t tiles_m, int64_t tiles_n, int tile_area, bool two_per_cu, int64_t k_bytes, bool whole_rows) {
  const int64_t n = tiles_m * tiles_n;
  if (tile_area == 128 * 128 && two_per_cu && n > 256 && n < 512 && (n % 8 == 0 || tiles_n < 2 * tiles_m)) return true;
  return tile_area >= 128 * 128 && k_bytes <= 512 && (n % 8 != 0 || !whole_rows);
}

// Less than a round of small tiles (up to 128x128), not a multiple of 8: which launches deal the tiles to the XCDs one by one instead of
// in a run per XCD.  Over 6000 drawn grids (us in runs / dealt): wider than high 0.95 on average (100x5000x4096, 2x79 tiles of
// 64x64: 17.0 / 24.6), others 1.01 (5712x584x785, 45x5 tiles of 128x128: 14.5 / 13.9).  any_rows: operands of any alignment with B
// row-major, whose pieces of a row touch two lines each, the neighbouring columns' tiles the same ones: dealt, an XCD has all
// columns of a tile row, and from 8 rows on that is 1.19 and up to 1.4 ahead (582x661x4110, 10x11 tiles of 64x64: 81 / 57; with 128x128
// tiles 1.05), as it is 1.1 with up to 8 tile columns or 16 tiles (346x385x4845, 6x7 tiles: 98.6 / 77.6); others are 0.91 in runs.
inline bool dealt_one_by_one(int64_t tiles_m, int64_t tiles_n, int tile_area, int64_t k_bytes, bool any_rows) {
  const int64_t n = tiles_m * tiles_n;
  if (n >= 256 || n % 8 == 0 || tile_area > 128 * 128 || k_bytes <= 512) return false;
  return tiles_n <= tiles_m || (any_rows && (tiles_m >= 8 || tiles_n <= 8 || n <= 16));
}

// x / d on the scalar unit (m = ceil(2^32 / d); 2^32 - 1 for d = 1): the estimate is off by one at most.  (A division by a
// run-time value goes through vector registers, which the K loop of a persistent workgroup has none to spare of.)
__host__ __device__ __forceinline__ int div_by(int x, int d, uint32_t m) {
  const uint32_t q = (uint32_t)(((uint64_t)(uint32_t)x * m) >> 32);
  const int r = x - (int)(q * (uint32_t)d);            // -d .. d
  return (int)q + (r >= d ? 1 : 0) - (r < 0 ? 1 : 0);
}

// The tile (tm, tn) of workgroup wg of tiles_m * tiles_n; spread: renumber over the XCDs; EITHER: the launch may have strips.
// This runs before a workgroup's first loads, so every scalar counts: without EITHER the regions' sizes are constants (as
// arguments they cost a launch of one 256x256 tile per workgroup 0.1 us of 11.7), and with it they follow from one flag.  A
// branch between the two orders doubled the time of the persistent kernels.
template <bool EITHER>
__host__ __device__ __forceinline__ void tile_of(const TileOrder& o, int tiles_m, int tiles_n, bool spread, bool strips, int wg,
                                                 int n_wg, int& tm, int& tn) {
  auto least = [](int a, int b) { return a < b ? a : b; };
  const bool whole = EITHER && strips;
  const int G = whole ? 8 : 16, W = whole ? tiles_n : 4;       // tile rows of a group; tile columns of a strip of it
  int id = wg;
  if (spread) {                                        // one contiguous eighth per XCD: of the grid, or of a round of 256 ids
    const int base = whole ? 0 : wg & ~255, size = whole ? n_wg : least(256, n_wg - base);
    if (!whole) id = base + (wg & 7) * (size >> 3) + least(wg & 7, size & 7) + ((wg - base) >> 3);   // (the first size % 8 XCDs take one more)
    else if ((size & 7) == 0) id = (wg & 7) * (size >> 3) + (wg >> 3);
  }
  const int group = div_by(id, G * tiles_n, o.div_group);
  id -= group * (G * tiles_n);
  const int rows = least(G, tiles_m - group * G);
  const int strip = div_by(id, W * rows, rows == G ? (whole ? o.div_group : 1u << 26) : o.div_rows);
  id -= strip * (W * rows);
  const int cols = least(W, tiles_n - strip * W);
  const int half = id >= 8 * cols ? 1 : 0;             // 8 tile rows of the strip
  id -= half * (8 * cols);
  const int h = least(8, rows - half * 8);
  const int col = div_by(id, h, h == 8 ? 1u << 29 : o.div_h);
  tm = group * G + half * 8 + id - col * h;
  tn = strip * W + col;
  if (group & (G >> 4)) tn = tiles_n - 1 - tn;         // (regions: odd groups backwards)
}

// Prefetching a panel that several tiles read (mfma16_kernel.hpp): as many of the `tiles` along it as divide by a power of two up
// to `at_most` (4 or 8), which one XCD works on at a time, share its lines.  The power's exponent; and which of a wave's `lines`
// lines (at most 64) lane `lane` touches for the workgroup on tile `tile`.
inline int touch_shift(int tiles, int at_most) {
  const int n = tiles < at_most ? tiles : at_most;
  return (n >= 2) + (n >= 4) + (n >= 8);
}
__host__ __device__ __forceinline__ int touched_line(int lane, int tile, int shift, int lines) {
  const int line = ((lane >> shift) << shift) + (tile & ((1 << shift) - 1));
  return line < lines ? line : lines - 1;
}

}  // namespace mi355gemm
