// Which form a matrix's products take, from its row groups.  Host code
// without HIP types.
#pragma once

#include <cstdint>

namespace fs {

// Column-count class of a product with k columns: the kernels' compile-time
// column count (1, 2, 4, 8 or 16) and its index 0..4.
constexpr int kKmClasses = 5;
inline int32_t km_for(int32_t k)
{
    return k <= 1 ? 1 : k <= 2 ? 2 : k <= 4 ? 4 : k <= 8 ? 8 : 16;
}
inline int32_t km_index(int32_t k)
{
    return k <= 1 ? 0 : k <= 2 ? 1 : k <= 4 ? 2 : k <= 8 ? 3 : 4;
}

// Classes (bits by km_index) whose multi-column products run on the matrix
// cores.  A pattern is a tile of up to four rows with equal columns, so the
// tiles pay where rows share their columns; a row of several lanes spreads
// its entries over that many times as many steps, each with its own pass over
// the tiles.  us per product, column pairs / tiles:
//
// rows per pattern (one lane per row)   k = 4        k = 8        k = 16
//   1.5, 22 slots per row (synthetic)   24.8 / 21.1  31.5 / 34.5  57.4 / 41.6
//   2,   14 (2-D P1 elasticity 700^2)   75.3 / 76.0   112 / 121    205 / 232
//           (its solves, 96 iterations   11.6 / 12.6 ms, k = 8  19.4 / 21.8 ms)
//   2,   30 (two fields on P1 30^3)     20.3 / 15.4  24.1 / 23.6  49.0 / 29.4
//   2.33, 16 (synthetic)                18.2 / 15.2  25.0 / 24.4  45.5 / 34.4
//   2.9, 43 (P1 elasticity 24^3)        30.0 / 15.5  32.8 / 20.5  65.5 / 23.2
// lanes per row, that elasticity matrix
//   2                                   21.0 / 15.4  25.5 / 16.8  45.5 / 21.3
//   4                                   15.1 / 14.8  20.1 / 15.9  33.6 / 22.2
//     (120,000 rows of 45, synthetic)   30.6 / 32.6  47.2 / 37.4  78.6 / 51.8
//   8                                   12.7 / 25.1  21.9 / 26.6  27.0 / 31.5
// P2 elasticity 14^3 (1 to 8 lanes)     38.9 / 41.6  53.9 / 44.2  92.3 / 58.5
// two fields on P1 30^3, 4 lanes        12.9 / 13.3  19.1 / 14.9  33.3 / 27.4
//   (its solves                          2.62 / 3.03 ms, k = 8  3.57 / 3.77 ms)
constexpr double kTileRows = 2.25;      // rows per pattern, or
constexpr double kTileRowsLong = 1.9;   //   with at least so many slots per
constexpr double kTileSlotsLong = 24;   //   row and few lanes
constexpr double kTileLanesFew = 2.5;   // mean lanes per row: the class of
constexpr double kTileLanes = 4.0;      //   four columns; the wider ones
inline int32_t tile_classes(double rows, double patterns, double slots,
                            double mean_lanes)
{
    const bool shared = rows >= kTileRows * patterns;
    const bool pairs = rows >= kTileRowsLong * patterns &&
                       slots >= kTileSlotsLong * rows &&
                       mean_lanes <= kTileLanesFew;
    if (patterns <= 0 || !(shared || pairs)) return 0;
    const int32_t four = 1 << km_index(4), wide = 1 << km_index(8) | 1 << km_index(16);
    return (mean_lanes <= kTileLanesFew ? four : 0) |
           (mean_lanes <= kTileLanes ? wide : 0);
}

}  // namespace fs
