// Y = A X on the matrix cores, for matrices whose rows share their columns
// (tiles.h).
#include <type_traits>

#include "tiles.h"

namespace fs {
namespace {

// Y[row or yperm[row], :] = (A X)[row, :], 3 <= k <= KM columns.
template <int V, int KM, bool SCATTER, bool N>
__global__ __launch_bounds__(kBlock, tile_waves(KM)) void k_spmm_tiles(
    const Group *__restrict__ groups, int ngroups,
    const double *__restrict__ val, const void *__restrict__ col,
    const int *__restrict__ gbase, const uint8_t *__restrict__ lpat,
    const double *__restrict__ X, int ldx, double *__restrict__ Y, long ldy,
    int k, const int *__restrict__ yperm)
{
    __shared__ TileBuf tiles[kWavesPerBlock];
    constexpr int NP = tile_parts<KM>();
    const int b = xcd_remap(blockIdx.x, gridDim.x);
    const int i = __builtin_amdgcn_readfirstlane(
        b * kWavesPerBlock + int(threadIdx.x >> 6));
    const int g = i / NP;
    if (g >= ngroups) return;
    const Group gd = load_group(gbl(groups), g);
    tile_group<V, KM, N>(
        gd, g, int(threadIdx.x & (kWave - 1)), gbl(val), gbl(col),
        N ? load_gbase(gbl(gbase), g) : 0, gbl(lpat), gbl(X), k, ldx,
        tiles[threadIdx.x >> 6], i % NP, [&](int rg, int q, double v) {
            const int row = gd.row0 + rg;
            Y[(SCATTER ? long(yperm[row]) : long(row)) * ldy + q] = v;
        });
}

template <int V, int KM, bool SC>
void tiles_go(const fs_csr *A, int32_t k, const double *X, int64_t ldx,
              double *Y, int64_t ldy, const int32_t *yperm, hipStream_t s)
{
    const long waves = long(A->n_groups) * tile_parts<KM>();
    const dim3 g(unsigned((waves + kWavesPerBlock - 1) / kWavesPerBlock));
    if (A->d_col16)
        hipLaunchKernelGGL((k_spmm_tiles<V, KM, SC, true>), g, dim3(kBlock),
                           0, s, A->d_groups, A->n_groups, A->d_val,
                           A->d_col16, A->d_gbase, A->d_lpat, X, int(ldx), Y,
                           long(ldy), k, yperm);
    else
        hipLaunchKernelGGL((k_spmm_tiles<V, KM, SC, false>), g, dim3(kBlock),
                           0, s, A->d_groups, A->n_groups, A->d_val, A->d_col,
                           nullptr, A->d_lpat, X, int(ldx), Y, long(ldy), k,
                           yperm);
}

}  // namespace

hipError_t launch_spmm_tiles(const fs_csr *A, int32_t k, const double *X,
                             int64_t ldx, double *Y, int64_t ldy,
                             const int32_t *yperm, hipStream_t s)
{
    if (!tile_fits(A->n_cols, ldx)) return hipErrorInvalidValue;
    auto go = [&](auto vt, auto kt) {
        constexpr int V = decltype(vt)::value, KM = decltype(kt)::value;
        if (yperm) tiles_go<V, KM, true>(A, k, X, ldx, Y, ldy, yperm, s);
        else tiles_go<V, KM, false>(A, k, X, ldx, Y, ldy, yperm, s);
    };
    auto by_k = [&](auto vt) {
        if (k <= 4) go(vt, std::integral_constant<int, 4>());
        else if (k <= 8) go(vt, std::integral_constant<int, 8>());
        else go(vt, std::integral_constant<int, 16>());
    };
    if (A->host.vec == 1) by_k(std::integral_constant<int, 1>());
    else by_k(std::integral_constant<int, 2>());
    return hipGetLastError();
}

}  // namespace fs
