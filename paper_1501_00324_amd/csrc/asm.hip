// Finite-element assembly as a sum-only product (paper: section
// "Description of Current GPU Methods", assembly of the global tangent
// matrix and residual as an SpMV with a vector of ones whose
// multiplications are dropped).  One lane owns one output entry and adds its
// element contributions in ascending order, so the result is bitwise the
// sequential element-by-element sum.  The index lists of a wavefront's 64
// entries are stored column-interleaved (one coalesced 256-byte load per
// step), tasks inside a window of output positions are ordered by
// contribution count so the lists of one wavefront have nearly equal length,
// and the element values are gathered through the cache hierarchy (a line
// of an element matrix serves neighbouring rows of the same node).
#include <type_traits>

#include "device.h"

namespace fs {
namespace {

__global__ __launch_bounds__(kBlock) void k_assemble(
    const int2 *__restrict__ waves, int nwaves, long ntasks,
    const int *__restrict__ tpos, const int *__restrict__ aidx,
    const double *__restrict__ in, double *__restrict__ out,
    float *__restrict__ f32, uint16_t *__restrict__ bf16)
{
    const int b = xcd_remap(blockIdx.x, gridDim.x);
    const int w = __builtin_amdgcn_readfirstlane(
        b * kWavesPerBlock + int(threadIdx.x >> 6));
    if (w >= nwaves) return;
    const int lane = threadIdx.x & (kWave - 1);
    const int2 wd = waves[w];
    const int base64 = __builtin_amdgcn_readfirstlane(wd.x);
    const int width = __builtin_amdgcn_readfirstlane(wd.y);
    const int *p = aidx + long(base64) * kWave + lane;
    // padding entries (-1) come after a lane's real ones; they read in[0]
    // (present whenever width > 0) and add +0.0, which leaves a sum that
    // started from +0.0 unchanged
    constexpr int U = 8;
    double acc = 0.0;
    int j = 0;
    for (; j + U <= width; j += U) {
        int c[U];
        double v[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            c[u] = __builtin_nontemporal_load(p + long(j + u) * kWave);
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = in[c[u] < 0 ? 0 : c[u]];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = c[u] >= 0 ? v[u] : 0.0;
#pragma unroll
        for (int u = 0; u < U; ++u) acc += v[u];
    }
    for (; j < width; ++j) {
        const int c = __builtin_nontemporal_load(p + long(j) * kWave);
        const double v = in[c < 0 ? 0 : c];
        acc += c >= 0 ? v : 0.0;
    }
    const long t = long(w) * kWave + lane;
    const int q = t < ntasks ? tpos[t] : -1;    // -1: filler task
    if (q >= 0) {
        out[q] = acc;
        if (f32 || bf16) {
            const float f = float(acc);
            if (f32) f32[q] = f;
            if (bf16) bf16[q] = f32_to_bf16_rne(f);
        }
    }
}

// Place in LDS of a group's slot: one double of padding per 64, so that the
// entries of a row, which lie 64 or 128 doubles apart, fall into different
// banks (unpadded, conflicts took 62% of the LDS cycles; now 47% of
// asm_matrix's and 34% of asm_system's).
__device__ __forceinline__ int lds_place(int slot) { return slot + (slot >> 6); }
__device__ __forceinline__ uint16_t lds_place(uint16_t off)
{
    return off == 0xffff ? off : uint16_t(lds_place(int(off)));
}

// LDS offsets of four steps of a lane side by side: out[(ob + c) * 64 + lane]
// holds steps 4c .. 4c + 3 of the batch (0xffff past its last step), one
// wavefront per batch.
__global__ __launch_bounds__(kBlock) void k_interleave_offsets(
    const int4 *__restrict__ bdesc, long nbatch,
    const uint16_t *__restrict__ off, us4 *__restrict__ out)
{
    const long b = long(blockIdx.x) * kWavesPerBlock + (threadIdx.x >> 6);
    if (b >= nbatch) return;
    const int lane = threadIdx.x & (kWave - 1);
    const int4 d = bdesc[b];
    for (int c = 0; 4 * c < d.y; ++c) {
        us4 o;
#pragma unroll
        for (int t = 0; t < 4; ++t)
            o[t] = 4 * c + t < d.y
                       ? lds_place(off[(long(d.x) + 4 * c + t) * kWave + lane])
                       : uint16_t(0xffff);
        out[(long(d.z) + c) * kWave + lane] = o;
    }
}

// Row-group assembly: the block's row group accumulates in LDS.  A wave
// takes `rows` rows at a time; at step k lane q*nde + b adds element value
// (ea_q * nde + b) of row q's k-th element row ea_q, so the nde lanes of a
// row read nde consecutive doubles and every element row is read once.
// The adds into one slot come from steps of one row in ascending order
// (a slot belongs to one row and an element touches it once), and one
// wave's LDS accesses complete in program order, so each slot receives its
// contributions in ascending element order.  With WR the element vectors
// are assembled in the same pass: row q of a batch adds re[ea_q] at every
// step (again element order) and writes r at its caller row perm[row].
//
// What bounds it is the address unit (four lanes a cycle, whatever they
// load) and one chain of loads -- index, then value -- per eight steps.  So
// a lane's LDS offsets come four steps to a load, the element rows of eight
// steps (8 rows <= 64 of them, EL = 1) as one load of which every lane takes
// its steps by shuffles, their vector entries likewise; and the indices of
// the next eight steps are in flight while the values of these are waited
// for.  12 (11 without the vector) load instructions per eight steps instead
// of 32 (24).  Elements of four to seven unknowns, whose batches hold up to
// 16 rows, take two loads (EL) of element rows per eight steps; smaller ones
// load every step's lane by lane (EL = 0), four steps at a time.  Lanes without
// work add 0.0 into a private dummy slot past the group region.
//
// With ORD the element rows come from a buffer stored in the plan's own order
// (row rec * rows + q), so they are read contiguously and ea is not needed: a
// step's values and offsets are requested together, and looking offsets up
// ahead only puts their wait before the values' (elasticity on 20^3 nodes
// 23.0 us with, 17.5 without).
//
// LAT: few row groups, whose time is the chain of one wavefront.  The next
// indices are then requested without a branch, which would make them wait for
// the values before them (asm_system of elasticity on 12^3 nodes, 81 groups,
// 18.8 -> 16.0 us; on 20^3, 375 groups, 26.4 -> 23.1); with more groups the
// branch costs less than the extra requests (64^3 493 / 501 us, triangles
// 400^2, 2,500 groups, 12.9 / 13.9).
//
// BIG: element matrices larger together than the last-level cache.  An
// element is read by the groups of all its nodes, about a level of the
// locality order apart, which an L2 does not hold: the L2s read
// 3.6 GB for 2.3 GB of elements and plan (P1 elasticity 64^3, asm_system).
// With one contiguous range per XCD the eight windows are eight places of
// the element data; in chunks of 32 groups side by side the XCDs read one
// place of it at a time, and the values stream out past the caches.  The
// L2s read as much either way (3.64 and 3.61 GB), but it comes sooner:
// 646 us in contiguous ranges, 578 in chunks.  Smaller data keeps the
// contiguous ranges (P1 Laplacian 70^3, 252 MB: 203 us, 218 in chunks).
template <int U, bool WR, bool ORD, int EL, bool BIG, bool LAT>
__global__ __launch_bounds__(kBlock) void k_assemble_lds(
    const int4 *__restrict__ gdesc, const int4 *__restrict__ bdesc,
    const int *__restrict__ ea, const us4 *__restrict__ off, int nde,
    int rows, const double *__restrict__ ke, double *__restrict__ val,
    float *__restrict__ f32, uint16_t *__restrict__ bf16,
    const Group *__restrict__ groups, const int *__restrict__ perm,
    const double *__restrict__ re, double *__restrict__ r)
{
    static_assert(U == 4 || U == 8, "offsets come four steps to a load");
    extern __shared__ double acc[];   // group region + 64 dummy slots
    int g;
    if constexpr (BIG) {
        constexpr int C = 32, R = 8 * C;   // chunk, groups per round of XCDs
        const int i = int(blockIdx.x), whole = int(gridDim.x) / R * R;
        g = i < whole ? i / R * R + i % 8 * C + i % R / 8 : i;
    } else {
        g = xcd_remap(blockIdx.x, gridDim.x);
    }
    const int4 gd = gdesc[g];
    const int region = gd.y * kWave, held = lds_place(region);
    for (int t = threadIdx.x; t < held; t += kBlock) acc[t] = 0.0;
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const int lane = threadIdx.x & (kWave - 1);
    const int q = lane / nde, b = lane - q * nde;
    const bool act = q < rows;
    const int qc = act ? q : rows - 1;
    const int dummy = held + lane;
    const auto pe = gbl(ea);
    const auto po = gbl(off);
    const auto pk = gbl(ke);
    // indices of the U steps from k of batch d
    constexpr bool EA1 = EL > 0;
    constexpr int UL = EA1 ? U / EL : U;   // steps per load of element rows
    struct Index {
        us4 o[U / 4];
        int e[EA1 ? EL : U];
    };
    auto batch = [&](int j) {
        const int4 d = bdesc[gd.z + min(j, gd.w - 1)];
        return make_int4(__builtin_amdgcn_readfirstlane(d.x),
                         __builtin_amdgcn_readfirstlane(d.y),
                         __builtin_amdgcn_readfirstlane(d.z), 0);
    };
    auto load = [&](Index &x, const int4 &d, int k) {
        const auto p = po + (long(d.z) + (k >> 2)) * kWave + lane;
        x.o[0] = __builtin_nontemporal_load(p);
        if constexpr (U == 8) {
            if constexpr (LAT)
                x.o[1] = __builtin_nontemporal_load(p + (k + 4 < d.y ? kWave : 0));
            else if (k + 4 < d.y)
                x.o[1] = __builtin_nontemporal_load(p + kWave);
        }
        if constexpr (EA1) {
            // lane u * rows + q: step u of row q (past the batch: its last)
#pragma unroll
            for (int l = 0; l < EL; ++l) {
                const int i = min((k + l * UL) * rows + lane, d.y * rows - 1);
                x.e[l] = __builtin_nontemporal_load(pe + long(d.x) * rows + i);
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (k + u < d.y)
                    x.e[u] = __builtin_nontemporal_load(
                        pe + (long(d.x) + k + u) * rows + qc);
        }
    };
    int j = wave;
    if constexpr (ORD) {
        // a step's values are `rows` rows of nde, wherever its offsets lie:
        // both are requested together, nothing is left to look up ahead
        const int len = rows * nde, at = qc * nde + b;
        for (; j < gd.w; j += kWavesPerBlock) {
            const int4 d = batch(j);
            const auto p = pk + long(d.x) * len + at;
            const auto po4 = po + long(d.z) * kWave + lane;
            for (int k = 0; k < d.y; k += U) {
                us4 o[2];
                double v[U];
                with_count<1, U>(min(U, d.y - k), [&](auto count) {
                    constexpr int R = decltype(count)::value;
#pragma unroll
                    for (int c = 0; 4 * c < R; ++c)
                        o[c] = __builtin_nontemporal_load(po4 + (k / 4 + c) * kWave);
#pragma unroll
                    for (int u = 0; u < R; ++u)
                        v[u] = __builtin_nontemporal_load(p + long(k + u) * len);
#pragma unroll
                    for (int u = 0; u < R; ++u) {
                        // (rows of dropped element rows carry 0xffff only)
                        const int to = o[u / 4][u % 4];
                        const bool use = act && to != 0xffff;
                        acc[use ? to : dummy] += use ? v[u] : 0.0;
                    }
                });
            }
        }
    } else {
        int4 d = batch(j), dn = batch(j + kWavesPerBlock);
        Index nx;
        if (j < gd.w && d.y > 0) load(nx, d, 0);
        for (; j < gd.w; j += kWavesPerBlock) {
            double racc = 0.0;
            for (int k = 0; k < d.y; k += U) {
                const Index x = nx;
                int o[U], e[U];
                double v[U], w[EA1 ? EL : 1];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    o[u] = x.o[u >> 2][u & 3];
                    if (u >= 4 && k + 4 >= d.y) o[u] = 0xffff;
                    if constexpr (EA1) e[u] = __shfl(x.e[u / UL], (u % UL) * rows + qc, kWave);
                    else e[u] = k + u < d.y ? x.e[u] : -1;
                }
                if constexpr (WR && EA1) {
#pragma unroll
                    for (int l = 0; l < EL; ++l) {
                        const bool ok = lane < UL * rows && x.e[l] >= 0;
                        w[l] = gbl(re)[ok ? x.e[l] : 0];
                        w[l] = ok ? w[l] : 0.0;
                    }
                }
                bool use[U];
                auto value = [&](int u) {
                    use[u] = act && o[u] != 0xffff && e[u] >= 0;
                    v[u] = pk[long(use[u] ? e[u] : 0) * nde + b];
                };
                // all loads before the first use, in halves: a guard per load would
                // make each wait for the one before.  Steps past the batch's last
                // have no lanes in use and read the first value.
#pragma unroll
                for (int u = 0; u < U / 2; ++u) value(u);
                if (k + U / 2 < d.y) {
#pragma unroll
                    for (int u = U / 2; u < U; ++u) value(u);
                } else {
#pragma unroll
                    for (int u = U / 2; u < U; ++u) {
                        use[u] = false;
                        v[u] = 0.0;
                    }
                }
                double wu[U];
                if constexpr (WR && !EA1) {
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const bool ok = act && b == 0 && e[u] >= 0;
                        wu[u] = ok ? gbl(re)[ok ? e[u] : 0] : 0.0;
                    }
                }
                // the next indices, behind the values in flight
                if constexpr (LAT) {
                    // of this batch, or the next one's first (a batch without any:
                    // this one's once more)
                    const bool more = k + U < d.y, go = !more && dn.y > 0;
                    load(nx, go ? dn : d, more ? k + U : 0);
                } else if (k + U < d.y) {
                    load(nx, d, k + U);
                } else if (j + kWavesPerBlock < gd.w && dn.y > 0) {
                    load(nx, dn, 0);
                }
                if constexpr (WR && EA1) {
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        wu[u] = __shfl(w[u / UL], (u % UL) * rows + qc, kWave);
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
                    acc[use[u] ? o[u] : dummy] += use[u] ? v[u] : 0.0;
                if constexpr (WR) {
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (k + u < d.y) racc += wu[u];
                }
            }
            if constexpr (WR) {
                const int rr = j * rows + q;
                const Group lg = load_group(gbl(groups), g);
                if (act && b == 0 && rr < lg.nrows) r[perm[lg.row0 + rr]] = racc;
            }
            if (d.y == 0 && j + kWavesPerBlock < gd.w && dn.y > 0) load(nx, dn, 0);
            d = dn;
            dn = batch(j + 2 * kWavesPerBlock);
        }
    }
    __syncthreads();
    const long base = long(gd.x) * kWave;
    for (int t = threadIdx.x; t < region; t += kBlock) {
        const double a = acc[lds_place(t)];
        if constexpr (BIG) __builtin_nontemporal_store(a, val + base + t);
        else val[base + t] = a;
        if (f32 || bf16) {
            const float f = float(a);
            if (f32) f32[base + t] = f;
            if (bf16) bf16[base + t] = f32_to_bf16_rne(f);
        }
    }
}

}  // namespace

// Row groups up to which the launch is one wavefront's chain (two workgroups
// on a compute unit; both sides' times at the kernel).
constexpr int32_t kAsmFew = 512;

hipError_t launch_assemble_lds(const AsmLdsPlan &P, const double *ke,
                               double *val, float *f32, uint16_t *bf16,
                               const Group *groups, const int32_t *perm,
                               const double *re, double *r, bool ordered,
                               hipStream_t s)
{
    if (P.ngroups == 0) return hipSuccess;
    const size_t lds = sizeof(double) * (size_t(P.region_max) +
                                         size_t(P.region_max / kWave) + kWave);
    auto go = [&](auto u, auto wr, auto ord, auto el, auto big, auto lat) {
        hipLaunchKernelGGL((k_assemble_lds<decltype(u)::value,
                                           decltype(wr)::value,
                                           decltype(ord)::value,
                                           decltype(el)::value,
                                           decltype(big)::value,
                                           decltype(lat)::value>),
                           dim3(P.ngroups), dim3(kBlock), lds, s,
                           reinterpret_cast<const int4 *>(P.d_gdesc),
                           reinterpret_cast<const int4 *>(P.d_bdesc), P.d_ea,
                           reinterpret_cast<const us4 *>(P.d_off), P.nde,
                           P.rows, ke, val, f32, bf16, groups, perm, re, r);
    };
    const std::true_type yes;
    const std::false_type no;
    const std::integral_constant<int, 8> eight;
    const std::integral_constant<int, 4> four;
    const std::integral_constant<int, 0> none;
    const std::integral_constant<int, 1> one;
    const std::integral_constant<int, 2> two;
    auto sized = [&](auto u, auto wr, auto el) {
        if (P.big) go(u, wr, no, el, yes, no);
        else if (P.ngroups <= kAsmFew) go(u, wr, no, el, no, yes);
        else go(u, wr, no, el, no, no);
    };
    auto stepped = [&](auto wr) {
        if (8 * P.rows <= kWave) sized(eight, wr, one);
        else if (4 * P.rows <= kWave) sized(eight, wr, two);
        else sized(four, wr, none);
    };
    if (ordered) go(eight, no, yes, none, no, no);
    else if (re) stepped(yes);
    else stepped(no);
    return hipGetLastError();
}

hipError_t launch_interleave_offsets(const int32_t *bdesc, int64_t nbatch,
                                     const uint16_t *off, uint16_t *out,
                                     hipStream_t s)
{
    if (nbatch == 0) return hipSuccess;
    hipLaunchKernelGGL(k_interleave_offsets,
                       dim3(unsigned((nbatch + kWavesPerBlock - 1) /
                                     kWavesPerBlock)),
                       dim3(kBlock), 0, s,
                       reinterpret_cast<const int4 *>(bdesc), long(nbatch),
                       off, reinterpret_cast<us4 *>(out));
    return hipGetLastError();
}

hipError_t launch_assemble(const AsmPlan &P, const double *in, double *out,
                           float *f32, uint16_t *bf16, hipStream_t s)
{
    if (P.nwaves == 0) return hipSuccess;
    hipLaunchKernelGGL(k_assemble, dim3(spmv_blocks(P.nwaves)), dim3(kBlock),
                       0, s, reinterpret_cast<const int2 *>(P.d_waves),
                       P.nwaves, long(P.ntasks), P.d_tpos, P.d_aidx, in, out,
                       f32, bf16);
    return hipGetLastError();
}

}  // namespace fs
