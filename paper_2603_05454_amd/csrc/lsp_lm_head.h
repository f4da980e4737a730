// Internal: how the output head cuts the active rows into tiles.
#pragma once
#include "lsp_common.h"

namespace lsp {

constexpr int kComputeUnits = 256;

// How high row tiles are.  Up to 128 rows: one tile of 128 (64 rows of it where there are no more), which reads the weights once, or, where a
// launch then has fewer tiles than compute units, tiles of 64 (128 rows x 126 464 entries x K = 4096: 182 us, 250 in one tile of
// 256; 100 rows x 152 064 x 2048 133, 160 in two of 64).  More rows: what takes the least time in whole rounds of an XCD's 32
// workgroups, a tile of 64, 128 and 256 rows counted as 7, 10 and 17 (measured, one round each of 26 145 entries x 4096: 32, 50 and 86 us; the same
// ratios to 10 % from K = 1024 to 4096).  Tiles of 256 share a weight slice best and win where they are full and so is the last round;
// lower ones where the last of a few rounds would be nearly empty or the tiles are mostly padding.  us at 64, 128 and 256 rows, K = 4096:
// 208 rows x 126 464 entries 357, 262 and 244 (8, 4 and 2 rounds), x 66 593 227, 185 and 223 (5, 3 and 2), 140 x 40 000 101, 110 and 110,
// 450 x 40 000 202, 167 and 197, 300 x 26 145 100, 98 and 91, 580 x 26 145 162, 150 and 172, 300 x 9036 38, 49 and 81.  122 such shapes
// (140 to 700 rows, K 1024 to 4096) were 1.046x over a rule that took 256 wherever more than 384 rows gave enough tiles, and 1.047x with the best of
// each; 84 others 1.025x, and up to 1.5 % (0.2 us) slower in the smallest, whose height is the same.
// R: active rows; VT: vocabulary tiles.  (Their product over 512 fits 32 bits by far: it is what the workspace holds partials for.)
__host__ __device__ __forceinline__ int tile_rows(int R, int VT) {
  if (R <= 128) return int64_t(VT) * ((R + 63) / 64) <= kComputeUnits ? 64 : 128;
  const int per_xcd = (VT + 7) / 8;
  auto rounds = [&](int height) { return (per_xcd * ((R + height - 1) / height) + 31) >> 5; };
  const int c64 = 7 * rounds(64), c128 = 10 * rounds(128), c256 = 17 * rounds(256);
  return c256 <= (c64 < c128 ? c64 : c128) ? 256 : c128 <= c64 ? 128 : 64;
}

}  // namespace lsp
