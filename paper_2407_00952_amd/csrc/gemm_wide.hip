// bf16 MFMA GEMM on tiles of 128, 192 or 256 rows and 128 columns with 8 waves that own a CU (gfx950): launches of one to a
// few such tiles per CU, which 256 x 256 tiles would leave unevenly filled (T = 5376, 4096 -> 1024: 224 tiles of 192 x 128 in
// 38.7 us, against 336 of 128 x 128 in 53 and 84 of 256 x 256 in 79).  Two waves to a SIMD hide what a barrier per slab
// costs; with 4 waves of twice the tile the same loop is slower by a third to a half, for all its fewer LDS reads.
#include "gemm_tile.h"

namespace {

template <int EPI, int NZ, int TM>
__global__ __launch_bounds__(512, 2) void gemm_wide_kernel(GemmArgs a)
{
    // 2 x 4 waves of 64 x 32, or 4 x 2 of 48 x 64 and 64 x 64; as many LDS stages as fit
    constexpr int WM = TM == 128 ? 2 : 4;
    gemm_tile_body<EPI, NZ, TM, 128, WM, 8 / WM, 1, TM == 128 ? 4 : 3, false>(a, 1);
}

template <int EPI, int NZ>
int launch_wz(const GemmArgs &a, const TilePlan &p, hipStream_t st)
{
    const int tiles = ((a.M + p.tm - 1) / p.tm) * ((a.seg_n + 127) / 128) * a.nseg;
    const dim3 grid((tiles + 7) / 8 * 8), block(512);
    if (p.tm == 128) hipLaunchKernelGGL((gemm_wide_kernel<EPI, NZ, 128>), grid, block, 0, st, a);
    else if (p.tm == 192) hipLaunchKernelGGL((gemm_wide_kernel<EPI, NZ, 192>), grid, block, 0, st, a);
    else if constexpr (NZ <= 16) hipLaunchKernelGGL((gemm_wide_kernel<EPI, NZ, 256>), grid, block, 0, st, a);
    else return SL_EINVAL;
    SL_CHECK_LAUNCH("gemm wide");
    return 0;
}
template <int EPI>
int launch_we(const GemmArgs &a, int nz, const TilePlan &p, hipStream_t st)
{
    switch (nz) {
    case 0: return launch_wz<EPI, 0>(a, p, st);
    case 16: return launch_wz<EPI, 16>(a, p, st);
    case 32: if (EPI == EPI_STORE) return launch_wz<EPI_STORE, 32>(a, p, st); break;
    case 48: if (EPI == EPI_STORE) return launch_wz<EPI_STORE, 48>(a, p, st); break;
    }
    return SL_EINVAL;
}

}  // namespace

int launch_gemm_wide(const GemmArgs &a, int epi, int nz, const TilePlan &p, hipStream_t st)
{
    switch (epi) {
    case EPI_STORE: return launch_we<EPI_STORE>(a, nz, p, st);
    case EPI_RESID: return launch_we<EPI_RESID>(a, nz, p, st);
    case EPI_GELU: return launch_we<EPI_GELU>(a, nz, p, st);
    case EPI_DGELU: return launch_we<EPI_DGELU>(a, nz, p, st);
    case EPI_STORE_DELTA: return nz == 0 ? launch_wz<EPI_STORE_DELTA, 0>(a, p, st) : SL_EINVAL;
    }
    return SL_EINVAL;
}
