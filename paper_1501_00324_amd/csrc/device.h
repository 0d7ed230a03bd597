// Device helpers shared by the kernel translation units: slot loads, row
// reductions and XCD-aware block numbering.  Everything has internal
// linkage.
#pragma once

#include <cmath>
#include <type_traits>

#include "internal.h"

namespace fs {
namespace {

typedef double dv2 __attribute__((ext_vector_type(2)));
// a pair of doubles at any 8-byte address
typedef double dv2u __attribute__((ext_vector_type(2), aligned(8)));
typedef int iv2 __attribute__((ext_vector_type(2)));
typedef float fv2 __attribute__((ext_vector_type(2)));
typedef unsigned short us2 __attribute__((ext_vector_type(2)));
typedef unsigned short us4 __attribute__((ext_vector_type(4)));

constexpr int kWavesPerBlock = kBlock / kWave;

// Pointers into global memory.  Most kernels find their pointers inside
// descriptor structs, where the compiler cannot tell that they address
// global memory and emits flat accesses (which also count against the LDS
// counter, so they serialise with cross-lane shuffles, and rule out scalar
// loads of uniform data); casting them to the global address space gives
// plain global and scalar loads.
#define FS_GLOBAL __attribute__((address_space(1)))
template <class T> using gptr = const FS_GLOBAL T *;
template <class T> using gmut = FS_GLOBAL T *;
template <class T> __device__ __forceinline__ gptr<T> gbl(const T *p)
{
    return (gptr<T>)p;
}
template <class T> __device__ __forceinline__ gmut<T> gblw(T *p)
{
    return (gmut<T>)p;
}
constexpr int kVecBlocks = 1024;   // max workgroups of the vector kernels

// Workgroups are dispatched round-robin over the 8 XCDs; renumber so XCD k
// owns one contiguous range of logical blocks.  A bijection for any grid.
__device__ __forceinline__ int xcd_remap(int bid, int nblk)
{
    constexpr int NX = 8;
    const int xcd = bid % NX, idx = bid / NX;
    const int base = nblk / NX, rem = nblk % NX;
    return xcd * base + (xcd < rem ? xcd : rem) + idx;
}

// v of another lane, by a data-parallel-primitive control (a VALU move, where
// a cross-lane shuffle is an LDS access of some 60 cycles).
template <int CTRL> __device__ __forceinline__ double dpp(double v)
{
    const int2 w = __builtin_bit_cast(int2, v);
    return __builtin_bit_cast(
        double, make_int2(__builtin_amdgcn_update_dpp(0, w.x, CTRL, 0xf, 0xf, true),
                          __builtin_amdgcn_update_dpp(0, w.y, CTRL, 0xf, 0xf, true)));
}
template <int CTRL> __device__ __forceinline__ float dpp(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(
        0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
constexpr int kDppXor1 = 0xb1, kDppXor2 = 0x4e;   // quad_perm 1,0,3,2 / 2,3,0,1
constexpr int kDppHalfMirror = 0x141, kDppMirror = 0x140;
constexpr int kDppRor4 = 0x124, kDppRor8 = 0x128;

// v plus v of lane ^ 16 or lane ^ 32 (the swaps exchange 16- or 32-lane rows
// between their two results).
template <int O> __device__ __forceinline__ unsigned swap_rows(unsigned v, unsigned &w)
{
    if constexpr (O == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        w = r[1];
        return r[0];
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        w = r[1];
        return r[0];
    }
}
template <int O> __device__ __forceinline__ double add_rows(double v)
{
    const uint2 u = __builtin_bit_cast(uint2, v);
    uint2 a, b;
    a.x = swap_rows<O>(u.x, b.x);
    a.y = swap_rows<O>(u.y, b.y);
    return __builtin_bit_cast(double, a) + __builtin_bit_cast(double, b);
}
template <int O> __device__ __forceinline__ float add_rows(float v)
{
    unsigned b;
    const unsigned a = swap_rows<O>(__float_as_uint(v), b);
    return __uint_as_float(a) + __uint_as_float(b);
}

// Butterfly over the lane distances 32, 16, ..., 1 (all lanes active): the
// sums of the shuffle form, bit for bit -- once the distance-8 sums are
// equal, a rotation by 4 in a row of 16 is the distance-4 partner.  A
// six-step shuffle butterfly of a double takes about 0.35 us in a kernel
// that waits for it, this one about 0.06.
__device__ __forceinline__ double wave_sum(double v)
{
    v = add_rows<32>(v);
    v = add_rows<16>(v);
    v += dpp<kDppRor8>(v);
    v += dpp<kDppRor4>(v);
    v += dpp<kDppXor2>(v);
    v += dpp<kDppXor1>(v);
    return v;
}

// Slot element types for V slots per load: values, 32-bit columns, 16-bit
// column offsets.
template <int V> struct Slots;
template <> struct Slots<1> { typedef double D; typedef int I; typedef uint16_t H; };
template <> struct Slots<2> { typedef dv2 D; typedef iv2 I; typedef us2 H; };

// Column index stream of a group: 32-bit layout columns (NARROW = false)
// or 16-bit offsets from the group's base column gb, 0xffff marking
// padding (NARROW = true).  Both decode to a layout column, -1 = padding.
template <int V, bool NARROW> struct ColStream {
    typedef typename std::conditional<NARROW, typename Slots<V>::H,
                                      typename Slots<V>::I>::type P;
    typedef typename std::conditional<NARROW, uint16_t, int32_t>::type E;
    gptr<P> p;
    int gb;
    __device__ __forceinline__ ColStream(gptr<void> col, long base, int lane,
                                         int gbase)
        : p(reinterpret_cast<gptr<P>>(static_cast<gptr<E>>(col) + base) +
            lane),
          gb(gbase)
    {
    }
    __device__ __forceinline__ P load(int j) const
    {
        return __builtin_nontemporal_load(p + long(j) * kWave);
    }
    __device__ __forceinline__ int get(const P &c, int t) const
    {
        int v;
        if constexpr (V == 1) v = int(c);
        else v = t ? int(c.y) : int(c.x);
        if constexpr (NARROW) return v == 0xffff ? -1 : gb + v;
        else return v;
    }
};

// Padded slots (column -1) read x[0] (always in bounds: a matrix with
// slots has at least one column) and the select drops the product, so an
// Inf/NaN there never reaches the sum.
__device__ __forceinline__ void slot_fma(int c, double a, gptr<double> x,
                                         double &acc)
{
    const double xv = x[c < 0 ? 0 : c];
    acc = fma(a, c >= 0 ? xv : 0.0, acc);
}

// This lane's share of its row: sum over its slots of a * x[col].  The
// matrix stream is read in batches of 8 slots (a batch's column and value
// loads are issued together) and software-pipelined over two register sets:
// the gathers of batch b are issued first, then the stream loads of batch
// b + 1, then batch b's products consume the gathers.  Loads complete in
// issue order, so waiting for batch b's gathers leaves batch b + 1's values
// in flight, and a wavefront always has matrix stream outstanding (the
// plain order -- stream, gathers, products -- leaves the stream idle during
// every gather round).  The scheduling barriers keep the compiler from
// hoisting the next batch's loads above the gathers, which would make the
// gather wait cover them too.  The batches are taken in pairs (the two
// register sets alternate without copies, which would wait for the loads);
// an odd last batch and the slots past the last full batch follow.  The
// sums are formed in the same order as the unpipelined loop.  Costs
// registers: 4 wavefronts per SIMD instead of 8, measured 2.3-2.5% faster
// on the 0.42 GB and 1.9 GB elasticity matrices than the unpipelined loop at
// 8 wavefronts, and faster than this loop held to 6 wavefronts.
template <int V, bool NARROW>
__device__ __forceinline__ double group_lane_sum(const Group &g, int lane,
                                                 gptr<double> val,
                                                 gptr<void> col, int gb,
                                                 gptr<double> x)
{
    typedef typename Slots<V>::D D;
    typedef ColStream<V, NARROW> CS;
    typedef typename CS::P PI;
    constexpr int U = 8 / V;
    const int width = g.width_lt & 0xffffff;
    const long base = long(g.base64) * kWave;
    gptr<D> pv = reinterpret_cast<gptr<D>>(val + base) + lane;
    const CS cs(col, base, lane, gb);
    const int nch = width / V;
    const int nb = nch / U;              // full batches
    double acc0 = 0.0, acc1 = 0.0;
    auto load = [&](PI (&c)[U], D (&a)[U], int b) {
#pragma unroll
        for (int u = 0; u < U; ++u) c[u] = cs.load(b * U + u);
#pragma unroll
        for (int u = 0; u < U; ++u)
            a[u] = __builtin_nontemporal_load(pv + (b * U + u) * kWave);
    };
    // padded slots (column -1) gather x[0] and the select drops them
    auto gather = [&](const PI (&c)[U], int (&cc)[U * V],
                      double (&xv)[U * V]) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int t = 0; t < V; ++t) cc[u * V + t] = cs.get(c[u], t);
#pragma unroll
        for (int i = 0; i < U * V; ++i) xv[i] = x[cc[i] < 0 ? 0 : cc[i]];
    };
    auto products = [&](const D (&a)[U], const int (&cc)[U * V],
                        const double (&xv)[U * V]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if constexpr (V == 1) {
                double &acc = (u & 1) ? acc1 : acc0;
                acc = fma(a[u], cc[u] >= 0 ? xv[u] : 0.0, acc);
            } else {
                acc0 = fma(a[u].x, cc[2 * u] >= 0 ? xv[2 * u] : 0.0, acc0);
                acc1 = fma(a[u].y, cc[2 * u + 1] >= 0 ? xv[2 * u + 1] : 0.0,
                           acc1);
            }
        }
    };
    if (nb > 0) {
        PI c0[U], c1[U];
        D a0[U], a1[U];
        load(c0, a0, 0);
        int b = 0;
        for (; b + 2 <= nb; b += 2) {
            int cc[U * V];
            double xv[U * V];
            gather(c0, cc, xv);
            __builtin_amdgcn_sched_barrier(0);
            load(c1, a1, b + 1);
            __builtin_amdgcn_sched_barrier(0);
            products(a0, cc, xv);
            gather(c1, cc, xv);
            __builtin_amdgcn_sched_barrier(0);
            // the last pair reloads batch b + 1 (no branch in the loop)
            load(c0, a0, b + 2 < nb ? b + 2 : b + 1);
            __builtin_amdgcn_sched_barrier(0);
            products(a1, cc, xv);
        }
        if (b < nb) {                    // odd last batch, already loaded
            int cc[U * V];
            double xv[U * V];
            gather(c0, cc, xv);
            products(a0, cc, xv);
        }
    }
    for (int j = nb * U; j < nch; ++j) {
        const PI c = cs.load(j);
        const D a = __builtin_nontemporal_load(pv + j * kWave);
        if constexpr (V == 1) {
            slot_fma(cs.get(c, 0), a, x, (j & 1) ? acc1 : acc0);
        } else {
            slot_fma(cs.get(c, 0), a.x, x, acc0);
            slot_fma(cs.get(c, 1), a.y, x, acc1);
        }
    }
    return acc0 + acc1;
}

// The same sum without pipelining, in batches of B slots (one register
// set): for kernels whose register budget is already spent, such as the
// 1024-thread blocks of the persistent solve (128 registers per lane, where
// 16-slot batches fit and keep more loads in flight).  The order of the
// sums does not depend on B.
template <int V, bool NARROW, int B = 8>
__device__ __forceinline__ double group_lane_sum_plain(const Group &g,
                                                       int lane,
                                                       gptr<double> val,
                                                       gptr<void> col, int gb,
                                                       gptr<double> x)
{
    typedef typename Slots<V>::D D;
    typedef ColStream<V, NARROW> CS;
    constexpr int U = B / V;
    const int width = g.width_lt & 0xffffff;
    const long base = long(g.base64) * kWave;
    gptr<D> pv = reinterpret_cast<gptr<D>>(val + base) + lane;
    const CS cs(col, base, lane, gb);
    const int nch = width / V;
    double acc0 = 0.0, acc1 = 0.0;
    int j = 0;
    for (; j + U <= nch; j += U) {
        typename CS::P c[U];
        D a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) c[u] = cs.load(j + u);
#pragma unroll
        for (int u = 0; u < U; ++u)
            a[u] = __builtin_nontemporal_load(pv + (j + u) * kWave);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if constexpr (V == 1) {
                slot_fma(cs.get(c[u], 0), a[u], x, (u & 1) ? acc1 : acc0);
            } else {
                slot_fma(cs.get(c[u], 0), a[u].x, x, acc0);
                slot_fma(cs.get(c[u], 1), a[u].y, x, acc1);
            }
        }
    }
    for (; j < nch; ++j) {
        const typename CS::P c = cs.load(j);
        const D a = __builtin_nontemporal_load(pv + j * kWave);
        if constexpr (V == 1) {
            slot_fma(cs.get(c, 0), a, x, (j & 1) ? acc1 : acc0);
        } else {
            slot_fma(cs.get(c, 0), a.x, x, acc0);
            slot_fma(cs.get(c, 1), a.y, x, acc1);
        }
    }
    return acc0 + acc1;
}

// Sum over the T = 2^lt lanes of each row (lanes of a row are adjacent), lane
// distances 1, 2, ..., T / 2; mirrors stand for the distances 4 and 8, whose
// partners hold equal sums by then.
template <typename T>
__device__ __forceinline__ T row_reduce(T acc, int lt)
{
    if (lt > 0) acc += dpp<kDppXor1>(acc);
    if (lt > 1) acc += dpp<kDppXor2>(acc);
    if (lt > 2) acc += dpp<kDppHalfMirror>(acc);
    if (lt > 3) acc += dpp<kDppMirror>(acc);
    if (lt > 4) acc = add_rows<16>(acc);
    if (lt > 5) acc = add_rows<32>(acc);
    return acc;
}

__device__ __forceinline__ Group load_group(gptr<Group> groups, int g)
{
    Group d;
    d.base64 = __builtin_amdgcn_readfirstlane(groups[g].base64);
    d.row0 = __builtin_amdgcn_readfirstlane(groups[g].row0);
    d.nrows = __builtin_amdgcn_readfirstlane(groups[g].nrows);
    d.width_lt = __builtin_amdgcn_readfirstlane(groups[g].width_lt);
    return d;
}

// Column base of group g for 16-bit column offsets (0 when there are none).
__device__ __forceinline__ int load_gbase(gptr<int32_t> gbase, int g)
{
    return gbase ? __builtin_amdgcn_readfirstlane(gbase[g]) : 0;
}

template <typename VT, int V> struct Pack;
template <> struct Pack<double, 1> { typedef double T; };
template <> struct Pack<double, 2> { typedef dv2 T; };
template <> struct Pack<float, 1> { typedef float T; };
template <> struct Pack<float, 2> { typedef fv2 T; };
template <> struct Pack<uint16_t, 1> { typedef uint16_t T; };
template <> struct Pack<uint16_t, 2> { typedef us2 T; };

template <typename ST> __device__ __forceinline__ ST widen(double v) { return ST(v); }
template <typename ST> __device__ __forceinline__ ST widen(float v) { return ST(v); }
template <typename ST> __device__ __forceinline__ ST widen(uint16_t h)
{
    return ST(__uint_as_float(uint32_t(h) << 16));
}

template <typename VT, typename ST, int V>
__device__ __forceinline__ void unpack(typename Pack<VT, V>::T a, ST (&o)[V])
{
    if constexpr (V == 1) {
        o[0] = widen<ST>(a);
    } else {
        o[0] = widen<ST>(a.x);
        o[1] = widen<ST>(a.y);
    }
}

// Order this wavefront's LDS writes before its later LDS reads (and its
// reads before later writes): LDS operations of one wavefront execute in
// order, so only the compiler has to be kept from moving them.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// f(integral_constant<int, n>) for a uniform n in LO .. HI, each n with a
// block of its own.  The empty asm tells the blocks apart: the compiler would
// otherwise merge their equal stores into ones through a chosen pointer, which
// keeps the arrays f fills in scratch memory.
template <int LO, int HI, class F>
__device__ __forceinline__ void with_count(int n, F &&f)
{
    if (LO == HI || n == HI) {
        f(std::integral_constant<int, HI>());
        asm volatile("" ::"n"(HI));
    } else if constexpr (LO < HI) {
        constexpr int M = (LO + HI) / 2;
        if constexpr (M > LO) {
            if (n < M) return with_count<LO, M - 1>(n, f);
        }
        with_count<M, HI - 1>(n, f);
    }
}

// This wavefront's staging buffer in the block's dynamic LDS: `stage` + 1
// entries per wavefront.
template <typename ST> __device__ __forceinline__ ST *stage_buffer(int stage)
{
    extern __shared__ double stage_lds_[];
    return reinterpret_cast<ST *>(stage_lds_) +
           __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)) * (stage + 1);
}

// This lane's share of its row, as group_lane_sum forms it (even slots and
// odd slots apart, each in slot order: the same bits), with the entries of
// x staged in LDS.  The slot loop then only streams -- values and 2-byte
// positions, two batches in flight -- and reads LDS: a gather from global
// memory waits behind the stream loads issued before it (the vector cache
// returns in order), which cost the unstaged loop 13-16% of its time on
// the elasticity matrices, and their rows' three-fold repeated gathers go
// with it.  The first batch is requested before the staging.
template <typename VT, typename ST, int V, bool NARROW, bool STREAM = false>
__device__ __forceinline__ ST staged_lane_sum(const Group &g, int gi, int lane,
                                              gptr<VT> val,
                                              const StageArgs &a, gptr<ST> x,
                                              ST *xs)
{
    typedef typename Pack<VT, V>::T PV;
    // slots per batch; 16 need registers that cost wavefronts (us, 8 / 16:
    // P1 elasticity 64^3 f32 32.7 / 37.1, bf16 20.7 / 21.5; bf16 Q1 Laplacian
    // 126^3 45.3 / 47.3, 2-D P1 elasticity 700^2 12.3 / 13.0)
    constexpr int B = 8;
    constexpr int U = B / V, L = B / 4;
    const auto gp = gbl(a.grp) + gi;
    const int per = __builtin_amdgcn_readfirstlane(gp->per);
    const int nd = __builtin_amdgcn_readfirstlane(gp->nd);
    const long l0 = __builtin_amdgcn_readfirstlane(gp->list);
    const gptr<us4> pl = reinterpret_cast<gptr<us4>>(gbl(a.loc)) +
                         __builtin_amdgcn_readfirstlane(gp->loc);
    const unsigned me =
        per == kWave ? unsigned(lane) : gbl(a.lpat)[long(gi) * kWave + lane];
    const int width = g.width_lt & 0xffffff;
    const gptr<PV> pv =
        reinterpret_cast<gptr<PV>>(val + long(g.base64) * kWave);
    const int nb = (width + B - 1) / B, full = width / B, nch = width / V;
    auto position = [&](int j) {
        const auto p = pl + long(j) * per + me;
        if constexpr (STREAM) return __builtin_nontemporal_load(p);
        else return *p;
    };
    // R loads of V slots from batch b.  A partial batch has a block of its own
    // for every length: with a guard per load, each address calculation waits
    // for the loads before it (P1 Laplacian 126^3, 15 slots per row, f64 / bf16
    // us: 71.0 / 62.6 so, 61.9 / 27.4 now; 60^3 10.3 / 11.1 and 8.1 / 8.1; gathers
    // per slot 69.7 / 43.2 and 11.9 / 9.5), and repeating the last load costs
    // the address unit a useful one (Q1 Laplacian 60^3 in f32 9.7, now 8.9).
    auto load_some = [&](us4 (&c)[L], PV (&v)[U], int b, auto count) {
        constexpr int R = decltype(count)::value;
#pragma unroll
        for (int l = 0; l < (R * V + 3) / 4; ++l) c[l] = position(b * L + l);
#pragma unroll
        for (int u = 0; u < R; ++u)
            v[u] = __builtin_nontemporal_load(pv + (b * U + u) * kWave + lane);
    };
    auto load = [&](us4 (&c)[L], PV (&v)[U], int b) {
        with_count<1, U>(b < full ? U : nch - b * U, [&](auto count) {
            load_some(c, v, b, count);
        });
    };
    ST acc0 = ST(0), acc1 = ST(0);
    auto use = [&](const us4 (&c)[L], const PV (&v)[U], int b) {
        with_count<1, U>(b < full ? U : nch - b * U, [&](auto count) {
            constexpr int R = decltype(count)::value;
            ST xv[R * V];
#pragma unroll
            for (int i = 0; i < R * V; ++i) xv[i] = xs[c[i / 4][i % 4]];
#pragma unroll
            for (int u = 0; u < R; ++u) {
                ST av[V];
                unpack<VT, ST, V>(v[u], av);
#pragma unroll
                for (int t = 0; t < V; ++t) {
                    ST &acc = ((u * V + t) & 1) ? acc1 : acc0;
                    acc = fma(av[t], xv[u * V + t], acc);
                }
            }
        });
    };
    us4 c0[L], c1[L];
    PV v0[U], v1[U];
    if (nb > 0) load(c0, v0, 0);
    // x of the listed columns, up to eight gathers in flight per lane; the
    // entry after the last is the zero that padding slots read
    wave_lds_sync();
    constexpr int S = 8;
    for (int i0 = 0; i0 < nd; i0 += S * kWave) {
        int c[S];
        ST v[S];
#pragma unroll
        for (int u = 0; u < S; ++u)
            if (i0 + u * kWave < nd) {
                const int i = min(i0 + u * kWave + lane, nd - 1);
                if constexpr (NARROW)
                    c[u] = static_cast<gptr<uint16_t>>(gbl(a.cols))[l0 + i];
                else
                    c[u] = static_cast<gptr<int32_t>>(gbl(a.cols))[l0 + i];
            }
        const int gb = NARROW ? load_gbase(gbl(a.gbase), gi) : 0;
#pragma unroll
        for (int u = 0; u < S; ++u)
            if (i0 + u * kWave < nd) v[u] = x[gb + c[u]];
#pragma unroll
        for (int u = 0; u < S; ++u)
            if (i0 + u * kWave + lane < nd) xs[i0 + u * kWave + lane] = v[u];
    }
    if (lane == 0) xs[nd] = ST(0);
    wave_lds_sync();
    for (int b = 0; b < nb; b += 2) {
        if (b + 1 < nb) load(c1, v1, b + 1);
        __builtin_amdgcn_sched_barrier(0);
        use(c0, v0, b);
        if (b + 1 >= nb) break;
        if (b + 2 < nb) load(c0, v0, b + 2);
        __builtin_amdgcn_sched_barrier(0);
        use(c1, v1, b + 1);
    }
    return acc0 + acc1;
}

// y[row or yperm[row]] = (A x)[row], staged: one row group per wavefront.
template <typename VT, typename ST, int V, bool SCATTER, bool NARROW,
          bool STREAM = false>
__global__ __launch_bounds__(kBlock) void k_spmv_staged(
    const Group *__restrict__ groups, int ngroups, const VT *__restrict__ val,
    const StageArgs st, int stage, const ST *__restrict__ x,
    ST *__restrict__ y, const int *__restrict__ yperm)
{
    const int b = xcd_remap(blockIdx.x, gridDim.x);
    const int g = __builtin_amdgcn_readfirstlane(
        b * kWavesPerBlock + int(threadIdx.x >> 6));
    if (g >= ngroups) return;
    const int lane = threadIdx.x & (kWave - 1);
    const Group gd = load_group(gbl(groups), g);
    const int lt = gd.width_lt >> 24;
    const ST acc = row_reduce(
        staged_lane_sum<VT, ST, V, NARROW, STREAM>(
            gd, g, lane, gbl(val), st, gbl(x), stage_buffer<ST>(stage)),
        lt);
    const int r = lane >> lt;
    if ((lane & ((1 << lt) - 1)) == 0 && r < gd.nrows) {
        const int row = gd.row0 + r;
        y[SCATTER ? yperm[row] : row] = acc;
    }
}

// float -> bfloat16, round to nearest even; NaN stays a (quiet) NaN.
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x007fffffu))
        return uint16_t((u >> 16) | 0x0040u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return uint16_t(u >> 16);
}

inline int vec_blocks(long n)
{
    long b = (n + kBlock - 1) / kBlock;
    if (b > kVecBlocks) b = kVecBlocks;
    return b < 1 ? 1 : int(b);
}

inline int spmv_blocks(int ngroups)
{
    return (ngroups + kWavesPerBlock - 1) / kWavesPerBlock;
}


}  // namespace
}  // namespace fs
