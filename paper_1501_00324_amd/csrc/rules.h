// Which form a matrix's products take, from its row groups.  Host code
// without HIP types.
#pragma once

#include <array>
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

// Value type classes of a launch.
enum { VT_F64 = 0, VT_F32 = 1, VT_BF16 = 2 };

// Which single-column products are staged (internal.h: StageGroup), bits by
// value type.  A staged group gathers each of its columns once instead of once
// per slot, and reads its list on top.  us per product, gathers per slot / staged (rows of one
// length along a band unless a mesh is named; 6 M to 18 M slots):
//
//                                    FP64          FP32          BF16
// slots per lane
//   2                                20.0 / 28.4   15.3 / 22.5   12.7 / 27.1
//   3                                21.9 / 22.1   17.8 / 15.1   15.7 / 16.1
//     (P1 line, 1 M rows)            11.3 / 11.3    7.8 /  8.7    7.4 /  8.8
//   4                                15.5 / 18.9   11.7 / 12.0    9.3 / 13.7
//   5                                21.9 / 17.7   17.3 / 12.1   14.4 / 11.8
// distinct columns per slot, of 7 slots per row
//   0.22                             42.9 / 29.4   35.5 / 21.7   32.4 / 19.7
//   0.52                             43.1 / 30.2   35.6 / 22.4   32.7 / 21.1
// of 27 (all within 60 columns of the diagonal at 0.23, 230 at 0.48)
//   0.23                             25.7 / 26.1   20.6 / 16.2   15.7 / 13.8
//   0.42                             26.0 / 27.7   20.7 / 18.6   16.0 / 16.4
//   0.55                             26.5 / 28.6   20.9 / 20.0   16.3 / 17.2
//     (Q1 Laplacian 100^3, 0.34)     52.3 / 48.8   33.5 / 30.9   24.8 / 25.0
// widest group, rows that share no columns: 32 KB of LDS are five workgroups
// on a compute unit, 40 KB three or four
//   680 (45 slots)                   26.8 / 26.2   22.3 / 17.7   17.1 / 13.4
//   900 (75)                         36.5 / 34.7   27.8 / 22.4   21.6 / 18.7
//   1080 (45)                        26.4 / 30.5   22.3 / 18.8   17.1 / 14.4
//   1280 (106)                       49.1 / 52.0   38.4 / 35.6   28.5 / 27.6
//   1500 (120)                       52.8 / 61.0   42.9 / 39.1   30.6 / 30.5
// rows that share them in threes: one copy of the positions for three
//   1280 (153)                       47.5 / 45.6   40.4 / 30.7   30.2 / 21.5
//   1900 (228, past the LDS limit)   73.5 / 66.2   56.1 / 46.4   41.4 / 32.0
// lines of 128 bytes that the 64 lanes of a slot touch, Q1 Laplacian, in
// natural numbering (5.5: whole runs of neighbours) and reverse Cuthill-McKee
// (8 to 12); short rows read by single slots gain either way
//   60^3 natural                     13.1 / 11.8    9.2 /  8.7
//   70^3 natural (FP32: 57 MB)       18.9 / 19.0   13.3 / 12.1
//   76^3 natural (73 MB)             22.5 / 23.2   14.9 / 15.1
//   80^3 natural                     25.7 / 27.7   16.9 / 17.5   12.8 / 13.5
//   84^3 natural                     30.3 / 30.1   19.5 / 21.2
//   96^3 natural                     45.1 / 43.7   26.7 / 28.0   20.1 / 22.3
//   105^3 natural (FP32: 192 MB)     60.0 / 60.7   33.3 / 35.0
//   110^3 natural                    69.9 / 69.8   38.8 / 39.0   29.2 / 30.5
//   118^3 natural                    87.3 / 84.5   48.2 / 47.3
//   126^3 natural                   106.3 / 101.6  58.6 / 55.9   43.5 / 42.3
//   70^3                             19.5 / 19.6   15.0 / 12.5   11.6 /  9.5
//   90^3                             37.7 / 37.2   25.9 / 24.0   19.5 / 18.9
// refined solves with FP32 products (ms; 192 iterations), natural numbering
//   70^3  2.58 / 2.70   80^3  3.10 / 3.21   88^3  3.75 / 3.84
//   96^3  4.50 / 4.49  105^3  5.57 / 5.53  118^3  7.80 / 7.28
constexpr int32_t kStageMax = 1280;     // columns of the widest group,
constexpr int32_t kStageMaxOwn = 1023;  //   FP64 with rows of their own
constexpr double kStageShared = 1.5;    // rows per pattern from which rows
                                        //   count as sharing
constexpr double kStageMost = 0.45;     // columns per slot
constexpr double kStageSlots = 4.5;     // mean slots per lane
constexpr double kStageLines = 7.5;     // lines per slot of rows of their own
                                        //   read by pairs; below, BF16
                                        //   gathers per slot, and FP32
constexpr double kStageRunsFrom = 64e6; //   where slots of 6 bytes take so
constexpr double kStageRunsTo = 180e6;  //   much
inline bool stage_pays(double slots, double lanes)
{
    return slots >= kStageSlots * lanes;
}
inline int32_t stage_forms(int32_t widest, double columns, double slots,
                           double rows, double patterns, int32_t vec,
                           double lines)
{
    if (widest > kStageMax || columns > kStageMost * slots) return 0;
    const bool shared = rows >= kStageShared * patterns;
    const bool f64 = shared || widest <= kStageMaxOwn;
    const bool runs = !shared && vec > 1 && 64 * lines < kStageLines * slots;
    const bool f32 = !runs || 6 * slots < kStageRunsFrom ||
                     6 * slots > kStageRunsTo;
    return (f32 ? 1 << VT_F32 : 0) | (f64 ? 1 << VT_F64 : 0) |
           (runs ? 0 : 1 << VT_BF16);
}

// Batch shape that a timed workgroup choice of cg_solve_batch_wg is kept for.
// `held`: every member's slots fit in registers, where 1024 threads stand for
// the kernel that holds them -- a choice timed with one of the two kernels
// says nothing about the other.
typedef std::array<int64_t, 7> WgKey;
inline WgKey wg_key(int64_t dev, int64_t m, int64_t rows, int64_t nnz,
                    int64_t parts, uint64_t kinds, bool held)
{
    return {dev, m, rows, nnz, parts, int64_t(kinds), held ? 1 : 0};
}

}  // namespace fs
