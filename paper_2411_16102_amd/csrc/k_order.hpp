// Where a tile begins along K (plain C++).
#pragma once

namespace bs {

constexpr int K_TILE = 64;  // elements of K in a k-tile: rows of 128 bytes

// Products of few rows on whole tiles, weight rows a multiple of 4 KB apart: every tile begins 16 k-tiles further along
// K than the one before and comes round.  All of them at the same column would ask for lines on few of the memory
// channels at any moment (the activation panel, read by all, stays in the caches anyway).  64 rows, 64x128 tiles:
// 2 x 14336 columns, K = 4096 53.5 -> 44.1 us, K = 8192 164 -> 162; rows of other lengths lose up to 4 % by it.
constexpr int first_k_tile(int tile, int k, int ldb) {
  return k > 0 && ldb % 2048 == 0 && k % K_TILE == 0 ? tile * 16 % (k / K_TILE) : 0;
}

}  // namespace bs
