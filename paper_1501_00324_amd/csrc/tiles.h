// Multi-column products on the matrix cores: the device function shared by
// the plain product (tiles.hip) and the CG engine's.
#pragma once

#include "device.h"

namespace fs {
namespace {

// Multi-column product of one row group on the matrix cores, for matrices
// whose rows share their columns in runs (row patterns, internal.h): the up
// to four rows of a pattern times KM columns of Y are v_mfma_f64_4x4x4
// tiles, A(row, entry) X(column of entry, :).  What bounds the multi-column
// products is the address unit, which takes four lanes a cycle whatever they
// load (counters: 85% busy in coop_group with 16 columns): so X is read once
// per (pattern, entry) instead of once per (row, entry), and 16 bytes a lane
// -- two columns, one for each of two instructions that share their A operand
// (69% busy with 16 columns, 77% with 8 and 75% with 4, whose lanes take 8
// bytes: P1 elasticity 64^3).
//
// Lane l of the instruction is block b = l / 4 % 4; row (A) and column (B, D)
// l % 4 of the block; entry (A, B) and row (D) l / 16.  KM = 16: two blocks
// hold an entry's 16 columns as pairs, and the two entries of a lane group
// (lower and upper two blocks) accumulate apart and are added at the end.
// KM = 4 and 8: 8 bytes a lane, a block holds four columns of one of 16 / KM
// patterns; with pairs the 8-column form measured the same (49 us).
// us per product before (coop_group) and now: P1 elasticity 64^3, k = 16,
// 386 -> 235 (with the 48 us permutation of X); 41^3, k = 8, 76 -> 48;
// k = 4, 48 -> 35; Q1 elasticity 33^3, k = 5, 66 -> 39.
//
// Values and columns of S slots per lane are staged in LDS (the loads of the
// next S in flight meanwhile), the column as the byte offset of its X row
// (-1: padding), which the launcher checks to fit 31 bits.  kTiles tiles'
// accumulators stay in registers over the whole row; the patterns past them
// are other work items (`part`).  Only rows and columns that exist are
// emitted, so what the clamped lanes compute is dropped.
constexpr int kTiles = 12;
constexpr int kTileStride = 68;        // doubles per staged slot (bank shift)
struct TileBuf {
    double v[8 * kTileStride];
    int c[8 * kWave];
    int first[kWave + 1];              // first row of each pattern
};
template <int KM> constexpr int tile_parts() { return KM == 16 ? 2 : 1; }
// Occupancy floor (wavefronts per SIMD): the pairs' accumulators and gathers
// spill at 4 (326 against 235 us).
constexpr int tile_waves(int km) { return km == 16 ? 3 : 4; }

template <int V, int KM, bool N, bool ONE, class Emit>
__device__ __forceinline__ void tile_rows(const Group &g, int gi, int lane,
                                          gptr<double> val, gptr<void> col,
                                          int gb, gptr<uint8_t> lpat,
                                          gptr<double> X, int k, int ldx,
                                          TileBuf &buf, int part, Emit emit)
{
    typedef typename Pack<double, V>::T PV;
    typedef ColStream<V, N> CS;
    constexpr bool PAIR = KM == 16;
    constexpr int W = PAIR ? 2 : 1;    // columns per lane
    constexpr int E = PAIR ? 8 : 4;    // entries per step
    constexpr int PB = 16 / KM;        // patterns per tile
    constexpr int S = ONE && PAIR ? 8 : 4;   // slots per staged chunk
    constexpr int C = S / V;           // loads per chunk
    const int lt = ONE ? 0 : g.width_lt >> 24, T = 1 << lt;
    const int width = g.width_lt & 0xffffff, nch = width / V;
    const long base = long(g.base64) * kWave;
    const gptr<PV> pv = reinterpret_cast<gptr<PV>>(val + base) + lane;
    const CS cs(col, base, lane, gb);
    // the group's patterns
    const int row = lane >> lt, sub = lane & (T - 1);
    const int pat = lpat[long(gi) * kWave + lane] >> lt;
    const int up = __shfl(pat, lane >= T ? lane - T : lane, kWave);
    const bool first = sub == 0 && row < g.nrows && (row == 0 || up != pat);
    const int np = __popcll(__ballot(first));
    wave_lds_sync();
    if (first) buf.first[pat] = row;
    if (lane == 0) buf.first[np] = g.nrows;
    wave_lds_sync();
    // this lane's entry within a step, pattern within a tile, column(s)
    const int blk = (lane >> 2) & 3, kk = lane >> 4;
    const int half = blk >> 1;         // pairs: entry of the lane group
    const int psub = (lane & 15) / KM;
    const int q0 = PAIR ? 8 * (blk & 1) + 2 * (lane & 3) : lane % KM;
    const int entry = PAIR ? 2 * kk + half : kk;
    // pairs end inside the row: an odd last column is the pair's second
    const int qs = max(0, min(q0, k - W));
    const bool odd = PAIR && (k & 1);
    const bool second = q0 > qs;
    const int q8 = 8 * qs, row8 = 8 * ldx;
    const int last = (kWave >> lt) - 1;
    const auto xb = reinterpret_cast<gptr<char>>(X);
    typedef typename std::conditional<PAIR, dv2u, double>::type XV;
    for (int t0 = part * kTiles; t0 * PB < np;
         t0 += tile_parts<KM>() * kTiles) {
        const int nt = min(kTiles, (np - t0 * PB + PB - 1) / PB);
        int crow[kTiles];
        double acc[kTiles][W];
#pragma unroll
        for (int t = 0; t < kTiles; ++t) {
            crow[t] = buf.first[min((t0 + t) * PB + psub, np - 1)] << lt;
#pragma unroll
            for (int w = 0; w < W; ++w) acc[t][w] = 0.0;
        }
        typename CS::P cn[C];
        PV an[C];
        auto load = [&](int j) {
#pragma unroll
            for (int u = 0; u < C; ++u)
                if (j + u < nch) {
                    cn[u] = cs.load(j + u);
                    an[u] = __builtin_nontemporal_load(pv + (j + u) * kWave);
                }
        };
        load(0);
        for (int j = 0; j < nch; j += C) {
            wave_lds_sync();
            bool pad = false;
#pragma unroll
            for (int u = 0; u < C; ++u) {
                double a[V];
                unpack<double, double, V>(an[u], a);
#pragma unroll
                for (int t = 0; t < V; ++t) {
                    // slots past the width: padding
                    const bool in = j + u < nch;
                    const int c = in ? cs.get(cn[u], t) : -1;
                    pad |= c < 0;
                    buf.v[(u * V + t) * kTileStride + lane] = in ? a[t] : 0.0;
                    buf.c[(u * V + t) * kWave + lane] = c < 0 ? -1 : c * row8;
                }
            }
            const bool any_pad = __any(pad);
            wave_lds_sync();
            if (j + C < nch) load(j + C);
            // steps of E entries: entry e of a row is lane e % T, slot e / T
            // of the staged ones
            for (int e0 = 0; e0 < S * T; e0 += E) {
                const int e = e0 + entry, ln = e & (T - 1), sl = e >> lt;
                const double *const av = buf.v + sl * kTileStride + ln;
                const int *const cv = buf.c + sl * kWave + ln;
                constexpr int TB = 6;  // tiles per batch of gathers
#pragma unroll
                for (int h = 0; h < kTiles; h += TB) {
                    if (h >= nt) break;
                    int c[TB];
                    XV x[TB];
                    double a[TB];
#pragma unroll
                    for (int t = 0; t < TB; ++t) c[t] = cv[crow[h + t]];
#pragma unroll
                    for (int t = 0; t < TB; ++t)
                        x[t] = *reinterpret_cast<gptr<XV>>(
                            xb + unsigned(max(c[t], 0) + q8));
#pragma unroll
                    for (int t = 0; t < TB; ++t)
                        a[t] = av[min(crow[h + t] + ((lane & 3) << lt),
                                      last << lt)];
                    if constexpr (PAIR) {
                        if (odd) {
#pragma unroll
                            for (int t = 0; t < TB; ++t)
                                x[t].x = second ? x[t].y : x[t].x;
                        }
                        if (any_pad) {
#pragma unroll
                            for (int t = 0; t < TB; ++t) {
                                x[t].x = c[t] < 0 ? 0.0 : x[t].x;
                                x[t].y = c[t] < 0 ? 0.0 : x[t].y;
                            }
                        }
#pragma unroll
                        for (int t = 0; t < TB; ++t) {
                            acc[h + t][0] = __builtin_amdgcn_mfma_f64_4x4x4f64(
                                a[t], x[t].x, acc[h + t][0], 0, 0, 0);
                            acc[h + t][1] = __builtin_amdgcn_mfma_f64_4x4x4f64(
                                a[t], x[t].y, acc[h + t][1], 0, 0, 0);
                        }
                    } else {
                        if (any_pad) {
#pragma unroll
                            for (int t = 0; t < TB; ++t)
                                x[t] = c[t] < 0 ? 0.0 : x[t];
                        }
#pragma unroll
                        for (int t = 0; t < TB; ++t)
                            acc[h + t][0] = __builtin_amdgcn_mfma_f64_4x4x4f64(
                                a[t], x[t], acc[h + t][0], 0, 0, 0);
                    }
                }
            }
        }
        // lane l emits column l % KM of row l / 16 of pattern l % 16 / KM
        const int q = lane % KM;
#pragma unroll
        for (int t = 0; t < kTiles; ++t) {
            double v = acc[t][0];
            if constexpr (PAIR) {
                // the other entry of the lane group
                const double s0 = acc[t][0] + __shfl_xor(acc[t][0], 8, kWave);
                const double s1 = acc[t][1] + __shfl_xor(acc[t][1], 8, kWave);
                const int src = 16 * kk + (q >> 1);
                const double v0 = __shfl(s0, src, kWave);
                const double v1 = __shfl(s1, src, kWave);
                v = (q & 1) ? v1 : v0;
            }
            const int p = (t0 + t) * PB + psub;
            if (p < np) {
                const int rg = buf.first[p] + kk;
                if (rg < buf.first[p + 1] && q < k) emit(rg, q, v);
            }
        }
    }
}

template <int V, int KM, bool N, class Emit>
__device__ __forceinline__ void tile_group(const Group &g, int gi, int lane,
                                           gptr<double> val, gptr<void> col,
                                           int gb, gptr<uint8_t> lpat,
                                           gptr<double> X, int k, int ldx,
                                           TileBuf &buf, int part, Emit emit)
{
    if ((g.width_lt >> 24) == 0)
        tile_rows<V, KM, N, true>(g, gi, lane, val, col, gb, lpat, X, k, ldx,
                                  buf, part, emit);
    else
        tile_rows<V, KM, N, false>(g, gi, lane, val, col, gb, lpat, X, k, ldx,
                                   buf, part, emit);
}

// Whether X (rows of ldx values) is small enough for 31-bit offsets.
inline bool tile_fits(int64_t n_cols, int64_t ldx)
{
    return 8 * n_cols * ldx <= INT32_MAX - 128;
}

}  // namespace
}  // namespace fs
