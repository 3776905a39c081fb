// Which of its two routes a tile-list build takes (plain C++: also built for
// the CPU by the tests).
#pragma once
#include <cstdint>

namespace gs {

// Whether a build of n Gaussians in nv views with ntiles tiles compares
// everything with everything instead of sorting.  Comparing costs, measured,
// 13 us, 0.17 us per million compares of the ranking (n^2 a view), 1.3 us per
// million (Gaussian, tile) pairs and 0.6 us per million squared tiles (each
// tile adds up the counts of all tiles before it); sorting costs 50 us for a
// hundred Gaussians and 80 to 95 for some thousands, whatever the tiles.  So
// the line lies where the first sum reaches about 85 us (us per build,
// compared / sorted, 16x16 tiles but where stated).  On this side of it:
// 1000 Gaussians in one view of 64 tiles 14 / 56, 16,000 63 / 82; 8192 in one
// of 3600 83 / 87; 12,000 in one of 2500 89 / 92; 6000 in one of 4800 8x8
// tiles 85 / 87; 2000 in one of 8160 79 / 87; 8192 in 4 of 2500 84 / 93.
// Past it: 16 in 4 of 10,000 69 / 63; 3000 in one of 8160 92 / 89; 12,000 in
// one of 3600 111 / 93; 8192 in one of 4800 8x8 tiles 105 / 89; 1000 in two of
// 16,320 175 / 86, in one of 32,400 573 / 86; 1000 in 8 of 65,280 2148 / 99.
constexpr int64_t kSmallN = 16384;      // Gaussians
constexpr int64_t kSmallTiles = 9797;   // (their square alone reaches the cost)
constexpr int64_t kSmallCost = 480ll * 1000 * 1000;
inline bool compares_all(int64_t n, int64_t nv, int64_t ntiles) {
  return n <= kSmallN && ntiles <= kSmallTiles && n * n * nv + 8 * n * ntiles + 5 * ntiles * ntiles <= kSmallCost;
}

}  // namespace gs
