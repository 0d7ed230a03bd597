// Device side of the layout build: the phases that touch every non-zero
// (column range check, bandwidth sums, slot assignment with the
// CSR-position -> slot map, 16-bit column offsets).  The row order and the
// row groups come from the host (they need only the row lengths, or the
// graph for reverse Cuthill-McKee); the results are the same arrays the
// host builder writes, bit for bit.
//
// Paper: section "Cost of Reordering Matrix Values" -- the layout's value
// map comes from one scan of the pattern, after which every value refresh is
// a device scatter; here that scan runs on the device as well.
#include <type_traits>

#include "device.h"

namespace fs {
namespace {

// Smallest CSR position whose column lies outside [0, n_cols).
__global__ __launch_bounds__(kBlock) void k_check_cols(
    const int *__restrict__ col, long nnz, int n_cols,
    unsigned long long *__restrict__ first)
{
    const long stride = long(gridDim.x) * kBlock;
    for (long k = long(blockIdx.x) * kBlock + threadIdx.x; k < nnz;
         k += stride) {
        const int c = col[k];
        if (c < 0 || c >= n_cols) atomicMin(first, (unsigned long long)k);
    }
}

__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}

// Sums of |i - c| and |iperm[i] - iperm[c]| over the entries (i, c): 16
// lanes per row (four rows per wave in flight), the lanes striding over the
// row's entries; the block's sums meet in LDS and go out as one pair of
// atomics (atomics on one address serialise, so a grid of at most
// kBandBlocks keeps them few).  Integer sums, so the order of the additions
// does not matter.
constexpr int kBandLanes = 16;
constexpr int kBandBlocks = 2048;

__global__ __launch_bounds__(kBlock) void k_band(
    int n, const int *__restrict__ rowptr, const int *__restrict__ col,
    const int *__restrict__ iperm, unsigned long long *__restrict__ sums)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int sub = lane & (kBandLanes - 1);
    const long first = (long(blockIdx.x) * kBlock + threadIdx.x) / kBandLanes;
    const long stride = long(gridDim.x) * kBlock / kBandLanes;
    unsigned long long s0 = 0, s1 = 0;
    for (long i = first; i < n; i += stride) {
        const int k0 = rowptr[i], k1 = rowptr[i + 1];
        const long ri = iperm[i];
        for (int k = k0 + sub; k < k1; k += kBandLanes) {
            const int c = col[k];
            const long d0 = i - c, d1 = ri - iperm[c];
            s0 += (unsigned long long)(d0 < 0 ? -d0 : d0);
            s1 += (unsigned long long)(d1 < 0 ? -d1 : d1);
        }
    }
    __shared__ unsigned long long part[2][kWavesPerBlock];
    s0 = wave_sum_u64(s0);
    s1 = wave_sum_u64(s1);
    const int w = threadIdx.x >> 6;
    if (lane == 0) {
        part[0][w] = s0;
        part[1][w] = s1;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        unsigned long long t = 0;
        for (int i = 0; i < kWavesPerBlock; ++i) t += part[threadIdx.x][i];
        atomicAdd(sums + threadIdx.x, t);
    }
}

__device__ __forceinline__ int layout_col(const int *__restrict__ col,
                                          const int *__restrict__ iperm,
                                          int k)
{
    const int c = col[k];
    return iperm ? iperm[c] : c;
}

// Slot assignment, one wave per row group.  A row's entries are ranked by
// their (relabelled) column: entry e of rank m goes to lane
// row_in_group * T + m % T, slot m / T of that lane, i.e. element
// base + (s / V) * 64 * V + lane * V + s % V (the column-interleaved order
// of sections "ELL-WARP" and "ELL-WARP v2 (K2)", with the columns sorted
// as in "K1rs").  Lanes hold up to 64 entries of the row; each counts the
// smaller columns over the whole row through cross-lane reads, so a row of
// length L costs L * ceil(L / 64) steps.  An entry whose column repeats an
// earlier entry of its row is a duplicate: the smallest such CSR position
// is reported through *dup.  The group's smallest and largest column go to
// lohi (0, -1 for a group without entries).  What the value refresh and the
// Jacobi scaling read is known here too: every slot's position in its CSR row
// (jpos, rows of at most 255 entries; prefilled with 255 = padding), the row
// starts, and the diagonal's slot of every row (-1: none).
__global__ __launch_bounds__(kBlock) void k_assign_slots(
    const Group *__restrict__ groups, int ngroups, int V,
    const int *__restrict__ perm, const int *__restrict__ iperm,
    const int *__restrict__ rowptr, const int *__restrict__ col,
    int *__restrict__ slot_col, int *__restrict__ map,
    uint8_t *__restrict__ jpos, int *__restrict__ rstart,
    int *__restrict__ diag, int2 *__restrict__ lohi,
    unsigned long long *__restrict__ dup)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int w0 = __builtin_amdgcn_readfirstlane(
        int(blockIdx.x) * kWavesPerBlock + int(threadIdx.x >> 6));
    const int nw = gridDim.x * kWavesPerBlock;
    for (int g = w0; g < ngroups; g += nw) {
        const Group G = load_group(gbl(groups), g);
        const int lt = G.width_lt >> 24, T = 1 << lt;
        const long base = long(G.base64) * kWave;
        int mn = INT_MAX, mx = -1;
        for (int rr = 0; rr < G.nrows; ++rr) {
            const int orow = perm[G.row0 + rr];
            const int k0 = __builtin_amdgcn_readfirstlane(rowptr[orow]);
            const int len =
                __builtin_amdgcn_readfirstlane(rowptr[orow + 1]) - k0;
            unsigned long long own = 0;      // lanes that held the diagonal
            for (int e0 = 0; e0 < len; e0 += kWave) {
                const int e = e0 + lane;
                const int c = e < len ? layout_col(col, iperm, k0 + e) : INT_MAX;
                int rank = 0;
                bool rep = false;
                for (int f0 = 0; f0 < len; f0 += kWave) {
                    int cf_lane = c;
                    if (f0 != e0) {
                        const int f = f0 + lane;
                        cf_lane = f < len ? layout_col(col, iperm, k0 + f)
                                          : INT_MAX;
                    }
                    const int nf = min(kWave, len - f0);
                    for (int t = 0; t < nf; ++t) {
                        const int cf = __builtin_amdgcn_readlane(cf_lane, t);
                        rank += cf < c ? 1 : 0;
                        rep = rep || (cf == c && f0 + t < e);
                    }
                }
                if (e < len) {
                    const int ln = rr * T + (rank & (T - 1));
                    const int s = rank >> lt;
                    const long idx = base + long(s / V) * kWave * V +
                                     long(ln) * V + s % V;
                    slot_col[idx] = c;
                    map[k0 + e] = int(idx);
                    if (jpos) jpos[idx] = uint8_t(e);
                    if (diag && c == G.row0 + rr) diag[c] = int(idx);
                    mn = min(mn, c);
                    mx = max(mx, c);
                    if (rep) atomicMin(dup, (unsigned long long)(k0 + e));
                }
                own |= __ballot(c == G.row0 + rr);
            }
            if (lane == 0) {
                if (rstart) rstart[G.row0 + rr] = k0;
                if (diag && !own) diag[G.row0 + rr] = -1;
            }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            mn = min(mn, __shfl_xor(mn, o, kWave));
            mx = max(mx, __shfl_xor(mx, o, kWave));
        }
        if (lane == 0) lohi[g] = make_int2(mx < 0 ? 0 : mn, mx);
    }
}

// 16-bit column offsets from each group's smallest column (0xffff marks
// padding), one wave per group over its whole slot region.
__global__ __launch_bounds__(kBlock) void k_offsets16(
    const Group *__restrict__ groups, int ngroups,
    const int *__restrict__ slot_col, const int2 *__restrict__ lohi,
    uint16_t *__restrict__ col16, int *__restrict__ gbase)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int w0 = __builtin_amdgcn_readfirstlane(
        int(blockIdx.x) * kWavesPerBlock + int(threadIdx.x >> 6));
    const int nw = gridDim.x * kWavesPerBlock;
    for (int g = w0; g < ngroups; g += nw) {
        const Group G = load_group(gbl(groups), g);
        const long base = long(G.base64) * kWave;
        const long region = long(G.width_lt & 0xffffff) * kWave;
        const int lo = lohi[g].x;
        for (long t = lane; t < region; t += kWave) {
            const int c = slot_col[base + t];
            col16[base + t] = c < 0 ? uint16_t(0xffff) : uint16_t(c - lo);
        }
        if (lane == 0) gbase[g] = lo;
    }
}

// Slot of every row's diagonal entry, -1 where it has none (one wavefront
// per row group): the Jacobi scaling of a solve then reads one value per row
// instead of searching the columns.
__global__ __launch_bounds__(kBlock) void k_diag_slots(
    const Group *__restrict__ groups, int ngroups, int V,
    const int *__restrict__ slot_col, int *__restrict__ diag)
{
    const int g = int(blockIdx.x) * kWavesPerBlock + int(threadIdx.x >> 6);
    if (g >= ngroups) return;
    const int lane = threadIdx.x & (kWave - 1);
    const Group G = load_group(gbl(groups), g);
    const long base = long(G.base64) * kWave;
    const int width = G.width_lt & 0xffffff, lt = G.width_lt >> 24;
    const int r = lane >> lt;
    int at = -1;
    for (int s = 0; s < width; ++s) {
        const long i = base + long(s / V) * kWave * V + lane * V + s % V;
        if (slot_col[i] == G.row0 + r) at = int(i);
    }
    for (int o = 1; o < (1 << lt); o <<= 1)
        at = max(at, __shfl_xor(at, o, kWave));
    if ((lane & ((1 << lt) - 1)) == 0 && r < G.nrows) diag[G.row0 + r] = at;
}

// ------------------------------------------------------ staged products
// Both kernels run one wavefront per workgroup and row group and find the
// group's distinct columns with a bitmap over its column span in LDS.
constexpr int kSpanNarrow = 65536;      // 16-bit offsets
constexpr int kSpanWide = 320 * 1024;   // 40 KB of bitmap, 20 KB of counts

// Smallest and largest column of the group (every lane), and their bitmap.
// False when they span more than `span` columns.
__device__ __forceinline__ bool column_bitmap(const int *__restrict__ cols,
                                              int region, int lane, int span,
                                              unsigned *bits, int &lo, int &hi)
{
    lo = INT_MAX;
    hi = -1;
    for (int t = lane; t < region; t += kWave) {
        const int c = cols[t];
        if (c >= 0) {
            lo = min(lo, c);
            hi = max(hi, c);
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        lo = min(lo, __shfl_xor(lo, o, kWave));
        hi = max(hi, __shfl_xor(hi, o, kWave));
    }
    if (hi < 0) {
        lo = 0;
        return true;
    }
    if (hi - lo >= span) return false;
    for (int w = lane; w <= (hi - lo) >> 5; w += kWave) bits[w] = 0u;
    __syncthreads();
    for (int t = lane; t < region; t += kWave) {
        const int c = cols[t];
        if (c >= 0) atomicOr(bits + ((c - lo) >> 5), 1u << ((c - lo) & 31));
    }
    __syncthreads();
    return true;
}

// Row patterns and distinct columns of a group.  Rows whose columns equal
// the previous row's share its pattern, up to four rows per pattern (the
// row tile of the multi-column products); lane j of a row of pattern p
// reads position entry p * T + j.  counts[g] = {patterns + 256 * lines,
// distinct columns or -1}; lines: what the group's gathers by slot would
// touch, as runs of lanes whose columns share 128 bytes (rows of one lane;
// else every lane counts).
__global__ __launch_bounds__(kWave) void k_stage_count(
    const Group *__restrict__ groups, int V, const int *__restrict__ slot_col,
    int span, uint8_t *__restrict__ lpat, int2 *__restrict__ counts)
{
    extern __shared__ unsigned bits[];
    const int g = int(blockIdx.x), lane = int(threadIdx.x);
    const Group G = load_group(gbl(groups), g);
    const int *cols = slot_col + long(G.base64) * kWave;
    const int width = G.width_lt & 0xffffff, lt = G.width_lt >> 24;
    const int T = 1 << lt, row = lane >> lt;
    int differs = row == 0, lines = 0;
    for (int s = 0; s < width; ++s) {
        const int c = cols[(s / V) * kWave * V + lane * V + s % V];
        const int up = __shfl(c, lane >= T ? lane - T : lane, kWave);
        differs |= c != up;
        lines += __popcll(__ballot(
            c >= 0 && (T > 1 || lane == 0 || c >> 4 != up >> 4)));
    }
    for (int o = 1; o < T; o <<= 1) differs |= __shfl_xor(differs, o, kWave);
    const unsigned long long starts = __ballot(differs != 0);
    // this row's pattern; lanes past the last row stay with its pattern
    int p = -1, run = 0;
    for (int r = 0; r <= min(row, G.nrows - 1); ++r) {
        if (((starts >> (r << lt)) & 1) || run == 4) {
            ++p;
            run = 0;
        }
        ++run;
    }
    lpat[long(g) * kWave + lane] = uint8_t(p * T + (lane & (T - 1)));
    int lo, hi, nd = 0;
    if (!column_bitmap(cols, width * kWave, lane, span, bits, lo, hi)) {
        nd = -1;
    } else if (hi >= 0) {
        for (int w = lane; w <= (hi - lo) >> 5; w += kWave) nd += __popc(bits[w]);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) nd += __shfl_xor(nd, o, kWave);
    }
    if (lane == kWave - 1)
        counts[g] = make_int2(p + 1 + (min(lines, 0x7fffff) << 8), nd);
}

// The group's column list (ascending) and every pattern's positions in it,
// four slots per entry; padding slots, and slots past the width, hold the
// list's length.
template <typename E>
__global__ __launch_bounds__(kWave) void k_stage_lists(
    const Group *__restrict__ groups, int V, const int *__restrict__ slot_col,
    int span, const int *__restrict__ gbase,
    const StageGroup *__restrict__ grp, const uint8_t *__restrict__ lpat,
    uint16_t *__restrict__ loc, E *__restrict__ list)
{
    extern __shared__ unsigned bits[];
    uint16_t *before = reinterpret_cast<uint16_t *>(bits + span / 32);
    const int g = int(blockIdx.x), lane = int(threadIdx.x);
    const Group G = load_group(gbl(groups), g);
    const StageGroup sg = grp[g];
    const int *cols = slot_col + long(G.base64) * kWave;
    const int width = G.width_lt & 0xffffff, T = 1 << (G.width_lt >> 24);
    int lo, hi;
    // every span fits (k_stage_count)
    column_bitmap(cols, width * kWave, lane, span, bits, lo, hi);
    const int words = hi < 0 ? 0 : ((hi - lo) >> 5) + 1;
    const int b0 = gbase ? gbase[g] : 0;
    int done = 0;
    for (int w0 = 0; w0 < words; w0 += kWave) {
        const int w = w0 + lane;
        unsigned m = w < words ? bits[w] : 0u;
        int n = __popc(m), at = n;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int u = __shfl_up(at, o, kWave);
            if (lane >= o) at += u;
        }
        at += done - n;                       // set bits before this word
        done = __shfl(at + n, kWave - 1, kWave);
        if (w < words) before[w] = uint16_t(at);
        for (; m; m &= m - 1)
            list[sg.list + at++] = E(lo + 32 * w + __ffs(m) - 1 - b0);
    }
    __syncthreads();
    const int me = lpat[long(g) * kWave + lane];
    const bool first =
        lane < T || lpat[long(g) * kWave + (lane >= T ? lane - T : 0)] != me;
    if (!first) return;
    for (int j = 0; j < (width + 3) / 4; ++j) {
        ushort4 o;
        uint16_t *const po = &o.x;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int s = 4 * j + t;
            const int c =
                s < width ? cols[(s / V) * kWave * V + lane * V + s % V] : -1;
            int at = sg.nd;
            if (c >= 0) {
                const int w = (c - lo) >> 5;
                at = before[w] + __popc(bits[w] & ((1u << ((c - lo) & 31)) - 1u));
            }
            po[t] = uint16_t(at);
        }
        reinterpret_cast<ushort4 *>(loc)[sg.loc + long(j) * sg.per + me] = o;
    }
}

// Inverse of the CSR-position -> slot map: imap[map[k]] = k (padding slots
// keep the -1 they were filled with).
__global__ __launch_bounds__(kBlock) void k_inverse_map(
    const int *__restrict__ map, long nnz, int *__restrict__ imap)
{
    const long stride = long(gridDim.x) * kBlock;
    for (long k = long(blockIdx.x) * kBlock + threadIdx.x; k < nnz;
         k += stride)
        imap[map[k]] = int(k);
}

// Value refresh in slot order (paper: section "Cost of Reordering Matrix
// Values", the per-Newton-step reorder of the values into the layout): one
// workgroup per row group walks the group's slot region, slot s taking
// vals[imap[s]] (0 for padding).  The slot arrays are written in full
// coalesced lines; the CSR values are gathered, but a group's region only
// touches the CSR ranges of its own rows, which stay in the CU's cache
// while the workgroup walks it.  The FP32 / BF16 copies round as the
// scatter at creation does.
__global__ __launch_bounds__(kBlock) void k_value_refresh(
    const Group *__restrict__ groups, const int *__restrict__ imap,
    const double *__restrict__ vals, double *__restrict__ val,
    float *__restrict__ f32, uint16_t *__restrict__ bf16)
{
    const int g = xcd_remap(blockIdx.x, gridDim.x);
    const Group G = load_group(gbl(groups), g);
    const long base = long(G.base64) * kWave;
    const long end = base + long(G.width_lt & 0xffffff) * kWave;
    // U slots per thread at a time: all their positions are loaded, then
    // all their values gathered, then all stored, so each thread keeps U
    // independent gathers in flight instead of one dependent pair (config
    // 1: U = 4 / 8 / 16 take 195 / 178 / 160 us; with 16 a whole row group
    // of up to 4096 slots is one batch)
    constexpr int U = 16;
    for (long t0 = base + threadIdx.x; t0 < end; t0 += U * kBlock) {
        int k[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const long t = t0 + long(u) * kBlock;
            k[u] = t < end ? __builtin_nontemporal_load(imap + t) : -1;
        }
        double a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = k[u] < 0 ? 0.0 : vals[k[u]];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const long t = t0 + long(u) * kBlock;
            if (t >= end) continue;
            const double v = a[u];
            // streamed out, so the slot arrays do not evict the rows' values
            __builtin_nontemporal_store(v, val + t);
            if (f32 || bf16) {
                const float f = float(v);
                if (f32) __builtin_nontemporal_store(f, f32 + t);
                if (bf16)
                    __builtin_nontemporal_store(f32_to_bf16_rne(f), bf16 + t);
            }
        }
    }
}

// Row starts and byte-wide positions for the refresh (one wavefront per row
// group): a row's entries fill exactly its lanes' non-padding slots, so
// the smallest CSR position among them is the row's start, and every slot
// stores its entry's offset from that start.  Rows hold at most 255
// entries (checked by the caller); 255 marks padding.
__global__ __launch_bounds__(kBlock) void k_refresh_rows(
    const Group *__restrict__ groups, int ngroups, int vec,
    const int *__restrict__ imap, uint8_t *__restrict__ jpos,
    int *__restrict__ rstart)
{
    const int g = int(blockIdx.x) * kWavesPerBlock + int(threadIdx.x >> 6);
    if (g >= ngroups) return;
    const int lane = threadIdx.x & (kWave - 1);
    const Group G = load_group(gbl(groups), g);
    const long base = long(G.base64) * kWave;
    const int nch = (G.width_lt & 0xffffff) / vec, lt = G.width_lt >> 24;
    int mn = 0x7fffffff;
    for (int j = 0; j < nch; ++j)
        for (int t = 0; t < vec; ++t) {
            const int k = imap[base + (long(j) * kWave + lane) * vec + t];
            if (k >= 0 && k < mn) mn = k;
        }
    for (int o = 1; o < (1 << lt); o <<= 1)
        mn = min(mn, __shfl_xor(mn, o, kWave));
    const int r = lane >> lt;
    if ((lane & ((1 << lt) - 1)) == 0 && r < G.nrows)
        rstart[G.row0 + r] = mn == 0x7fffffff ? 0 : mn;
    for (int j = 0; j < nch; ++j)
        for (int t = 0; t < vec; ++t) {
            const long i = base + (long(j) * kWave + lane) * vec + t;
            const int k = imap[i];
            jpos[i] = k < 0 ? uint8_t(255) : uint8_t(k - mn);
        }
}

// The refresh through row starts: the map read is one byte per slot
// instead of four.  Thread x of a group's workgroup takes the group's slots
// x, x + 256, ... -- always the same lane (256 is a multiple of 64 vec
// slots), so one row and one row start per thread.
__global__ __launch_bounds__(kBlock) void k_value_refresh_rows(
    const Group *__restrict__ groups, int vec,
    const uint8_t *__restrict__ jpos, const int *__restrict__ rstart,
    const double *__restrict__ vals, double *__restrict__ val,
    float *__restrict__ f32, uint16_t *__restrict__ bf16)
{
    const int g = xcd_remap(blockIdx.x, gridDim.x);
    const Group G = load_group(gbl(groups), g);
    const long base = long(G.base64) * kWave;
    const long end = base + long(G.width_lt & 0xffffff) * kWave;
    const int lt = G.width_lt >> 24;
    const int r = ((int(threadIdx.x) / vec) & (kWave - 1)) >> lt;
    const long rs = r < G.nrows ? long(rstart[G.row0 + r]) : 0;
    constexpr int U = 16;
    for (long t0 = base + threadIdx.x; t0 < end; t0 += U * kBlock) {
        int jp[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const long t = t0 + long(u) * kBlock;
            jp[u] = t < end ? int(__builtin_nontemporal_load(jpos + t)) : 255;
        }
        double a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = jp[u] == 255 ? 0.0 : vals[rs + jp[u]];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const long t = t0 + long(u) * kBlock;
            if (t >= end) continue;
            const double v = a[u];
            __builtin_nontemporal_store(v, val + t);
            if (f32 || bf16) {
                const float f = float(v);
                if (f32) __builtin_nontemporal_store(f, f32 + t);
                if (bf16)
                    __builtin_nontemporal_store(f32_to_bf16_rne(f), bf16 + t);
            }
        }
    }
}

// The same with the CSR rows read along their length: a wavefront takes 16
// lanes of a group (16 / T rows), copies the T * width values from each row
// start into LDS with consecutive lanes on consecutive values, and its
// slots pick theirs from there.  The direct form gathers 64 rows' values with
// every load, each from a line of its own, which leave the L1 before their
// 16 values are used: P1 elasticity 64^3 in random numbering with an FP32
// copy 210 us, this form 148 us = 4.9 TB/s (the copy rate); rows in CSR order
// (Q1 elasticity 60^3 with a BF16 copy) 186 against 188 us.  Loading the
// positions ahead of the rows: 6 us slower.  A row shorter than T * width
// reads on into the next rows' values (clamped to the array), which no slot
// picks.  Needs T <= 16 and 16 * width doubles of LDS per wavefront.
template <int V>
__global__ __launch_bounds__(kBlock) void k_value_refresh_tiles(
    const Group *__restrict__ groups, const uint8_t *__restrict__ jpos,
    const int *__restrict__ rstart, const double *__restrict__ vals, long nnz,
    int lds_wave, double *__restrict__ val, float *__restrict__ f32,
    uint16_t *__restrict__ bf16)
{
    // positions of V slots (in byte order)
    typedef typename std::conditional<V == 1, uint8_t, uint16_t>::type J;
    typedef typename Slots<V>::D D;
    extern __shared__ double rows_[];
    const int g = xcd_remap(blockIdx.x, gridDim.x);
    const Group G = load_group(gbl(groups), g);
    const int w = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const int lane = threadIdx.x & (kWave - 1);
    const int lt = G.width_lt >> 24, width = G.width_lt & 0xffffff;
    const int len = width << lt, nr = 16 >> lt;      // row length, rows
    const int row0 = w * nr;                         // in the group
    const int have = min(nr, G.nrows - row0);        // rows that exist
    double *const t = rows_ + w * lds_wave;
    // lane r (< nr) knows row r's start
    const int mine = lane < have ? rstart[G.row0 + row0 + lane] : 0;
    const int total = max(have, 0) * len;
    const float inv = 1.0f / float(len);
    const long base = long(G.base64) * kWave;
    const int nch = width / V, l = lane & 15;
    const auto pj = gbl(reinterpret_cast<const J *>(jpos + base)) + w * 16 + l;
    constexpr int U = 12;
    for (int i0 = 0; i0 < total; i0 += U * kWave) {
        double a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * kWave + lane;
            // i / len exactly: both at most 16 * 64
            const int ic = min(i, total - 1);
            const int r = int((float(ic) + 0.5f) * inv), j = ic - r * len;
            const long at = long(__shfl(mine, r, kWave)) + j;
            if (i0 + u * kWave < total) a[u] = gbl(vals)[at < nnz ? at : nnz - 1];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * kWave + lane;
            if (i < total) t[i] = a[u];
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // slots: V of 16 lanes in four chunks per step
    const int r = l >> lt;
    const bool real = r < have;
    const int tr = (real ? r : 0) * len;
    auto pick = [&](int jp) { return real && jp != 255 ? t[tr + jp] : 0.0; };
    auto step = [&](int s, J jp) {
        const int c = 4 * s + (lane >> 4);
        if (c >= nch) return;
        const long at = base / V + long(c) * kWave + w * 16 + l;
        D v;
        if constexpr (V == 1) {
            v = pick(jp);
        } else {
            v.x = pick(jp & 0xff);
            v.y = pick(jp >> 8);
        }
        __builtin_nontemporal_store(v, reinterpret_cast<D *>(val) + at);
        if (!f32 && !bf16) return;
        if constexpr (V == 1) {
            const float f = float(v);
            if (f32) __builtin_nontemporal_store(f, f32 + at);
            if (bf16) __builtin_nontemporal_store(f32_to_bf16_rne(f), bf16 + at);
        } else {
            fv2 f;
            f.x = float(v.x);
            f.y = float(v.y);
            us2 h;
            h.x = f32_to_bf16_rne(f.x);
            h.y = f32_to_bf16_rne(f.y);
            if (f32) __builtin_nontemporal_store(f, reinterpret_cast<fv2 *>(f32) + at);
            if (bf16) __builtin_nontemporal_store(h, reinterpret_cast<us2 *>(bf16) + at);
        }
    };
    for (int s = 0; 4 * s < nch; ++s)
        step(s, pj[long(min(4 * s + (lane >> 4), nch - 1)) * kWave]);
}

int wave_grid(long waves)
{
    const long b = (waves + kWavesPerBlock - 1) / kWavesPerBlock;
    return int(b < 1 ? 1 : (b > 8192 ? 8192 : b));
}

}  // namespace

hipError_t launch_inverse_map(const int32_t *map, int64_t nnz, int32_t *imap,
                              hipStream_t s)
{
    if (nnz == 0) return hipSuccess;
    const long b = (nnz + kBlock - 1) / kBlock;
    hipLaunchKernelGGL(k_inverse_map, dim3(unsigned(b > 8192 ? 8192 : b)),
                       dim3(kBlock), 0, s, map, long(nnz), imap);
    return hipGetLastError();
}

hipError_t launch_value_refresh(const Group *groups, int32_t ngroups,
                                const int32_t *imap, const double *vals,
                                double *val, float *f32, uint16_t *bf16,
                                hipStream_t s)
{
    if (ngroups == 0) return hipSuccess;
    hipLaunchKernelGGL(k_value_refresh, dim3(ngroups), dim3(kBlock), 0, s,
                       groups, imap, vals, val, f32, bf16);
    return hipGetLastError();
}

hipError_t launch_refresh_rows(const Group *groups, int32_t ngroups,
                               int32_t vec, const int32_t *imap,
                               uint8_t *jpos, int32_t *rstart, hipStream_t s)
{
    if (ngroups == 0) return hipSuccess;
    const int b = (ngroups + kWavesPerBlock - 1) / kWavesPerBlock;
    hipLaunchKernelGGL(k_refresh_rows, dim3(b), dim3(kBlock), 0, s, groups,
                       ngroups, vec, imap, jpos, rstart);
    return hipGetLastError();
}

hipError_t launch_value_refresh_rows(const Group *groups, int32_t ngroups,
                                     int32_t vec, int32_t tile_width,
                                     int64_t nnz, const uint8_t *jpos,
                                     const int32_t *rstart,
                                     const double *vals, double *val,
                                     float *f32, uint16_t *bf16,
                                     hipStream_t s)
{
    if (ngroups == 0) return hipSuccess;
    if (tile_width > 0) {
        // an odd stride between the wavefronts' tiles (banks)
        const int per = 16 * tile_width + 1;
        const size_t lds = sizeof(double) * size_t(per) * kWavesPerBlock;
        if (vec == 1)
            hipLaunchKernelGGL(k_value_refresh_tiles<1>, dim3(ngroups),
                               dim3(kBlock), lds, s, groups, jpos, rstart,
                               vals, long(nnz), per, val, f32, bf16);
        else
            hipLaunchKernelGGL(k_value_refresh_tiles<2>, dim3(ngroups),
                               dim3(kBlock), lds, s, groups, jpos, rstart,
                               vals, long(nnz), per, val, f32, bf16);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_value_refresh_rows, dim3(ngroups), dim3(kBlock), 0,
                       s, groups, vec, jpos, rstart, vals, val, f32, bf16);
    return hipGetLastError();
}

hipError_t launch_check_cols(const int32_t *col, int64_t nnz, int32_t n_cols,
                             unsigned long long *first, hipStream_t s)
{
    if (nnz == 0) return hipSuccess;
    const long b = (nnz + kBlock - 1) / kBlock;
    hipLaunchKernelGGL(k_check_cols, dim3(unsigned(b > 8192 ? 8192 : b)),
                       dim3(kBlock), 0, s, col, long(nnz), n_cols, first);
    return hipGetLastError();
}

hipError_t launch_band(int32_t n, const int32_t *rowptr, const int32_t *col,
                       const int32_t *iperm, unsigned long long *sums,
                       hipStream_t s)
{
    if (n == 0) return hipSuccess;
    const long b = (long(n) * kBandLanes + kBlock - 1) / kBlock;
    hipLaunchKernelGGL(k_band, dim3(unsigned(b > kBandBlocks ? kBandBlocks : b)),
                       dim3(kBlock), 0, s, n, rowptr, col, iperm, sums);
    return hipGetLastError();
}

hipError_t launch_assign_slots(const Group *groups, int32_t ngroups,
                               int32_t vec, const int32_t *perm,
                               const int32_t *iperm, const int32_t *rowptr,
                               const int32_t *col, int32_t *slot_col,
                               int32_t *map, uint8_t *jpos, int32_t *rstart,
                               int32_t *diag, int2 *lohi,
                               unsigned long long *dup, hipStream_t s)
{
    if (ngroups == 0) return hipSuccess;
    hipLaunchKernelGGL(k_assign_slots, dim3(wave_grid(ngroups)), dim3(kBlock),
                       0, s, groups, ngroups, vec, perm, iperm, rowptr, col,
                       slot_col, map, jpos, rstart, diag, lohi, dup);
    return hipGetLastError();
}

hipError_t launch_diag_slots(const Group *groups, int32_t ngroups, int32_t vec,
                             const int32_t *slot_col, int32_t *diag,
                             hipStream_t s)
{
    if (ngroups == 0) return hipSuccess;
    hipLaunchKernelGGL(k_diag_slots, dim3(spmv_blocks(ngroups)), dim3(kBlock),
                       0, s, groups, ngroups, vec, slot_col, diag);
    return hipGetLastError();
}

hipError_t launch_stage_count(const Group *groups, int32_t ngroups,
                              int32_t vec, const int32_t *slot_col,
                              bool narrow, uint8_t *lpat, int2 *counts,
                              hipStream_t s)
{
    if (ngroups == 0) return hipSuccess;
    const int span = narrow ? kSpanNarrow : kSpanWide;
    hipLaunchKernelGGL(k_stage_count, dim3(ngroups), dim3(kWave), span / 8, s,
                       groups, vec, slot_col, span, lpat, counts);
    return hipGetLastError();
}

hipError_t launch_stage_lists(const Group *groups, int32_t ngroups,
                              int32_t vec, const int32_t *slot_col,
                              const int32_t *gbase, const StageGroup *grp,
                              const uint8_t *lpat, uint16_t *loc, void *cols,
                              hipStream_t s)
{
    if (ngroups == 0) return hipSuccess;
    const int span = gbase ? kSpanNarrow : kSpanWide;
    const size_t lds = size_t(span / 32) * (sizeof(unsigned) + sizeof(uint16_t));
    if (gbase)
        hipLaunchKernelGGL(k_stage_lists<uint16_t>, dim3(ngroups),
                           dim3(kWave), lds, s, groups, vec, slot_col, span,
                           gbase, grp, lpat, loc,
                           static_cast<uint16_t *>(cols));
    else
        hipLaunchKernelGGL(k_stage_lists<int32_t>, dim3(ngroups), dim3(kWave),
                           lds, s, groups, vec, slot_col, span, gbase, grp,
                           lpat, loc, static_cast<int32_t *>(cols));
    return hipGetLastError();
}

hipError_t launch_offsets16(const Group *groups, int32_t ngroups,
                            const int32_t *slot_col, const int2 *lohi,
                            uint16_t *col16, int32_t *gbase, hipStream_t s)
{
    if (ngroups == 0) return hipSuccess;
    hipLaunchKernelGGL(k_offsets16, dim3(wave_grid(ngroups)), dim3(kBlock), 0,
                       s, groups, ngroups, slot_col, lohi, col16, gbase);
    return hipGetLastError();
}

}  // namespace fs
