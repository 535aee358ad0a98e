// GEMM on MXFP8 operands on tiles smaller than 256 x 256, and the rule that picks the kernel of such a product (gfx950).
//
// With 256 x 256 tiles alone 64 rows of 4096 -> 1024 kept 4 CUs busy for 43 us (8.9 on 32 x 64 tiles), 2048 rows 32 CUs for
// 59 us (19 on 64 x 128).  Bound as the bf16 forms by the LDS (gemm_tile.h).
#include "gemm_mx_tile.h"

namespace {

// Blocks of 4 waves, two to a CU, up to 64 x 128; of 8 waves that own a CU beyond.  Ring depths: as many stages as fit.
template <int EPI, int TM, int TN>
__global__ __launch_bounds__(TM <= 64 ? 256 : 512, 2) void gemm_mx_tile_kernel(MxArgs a)
{
    constexpr int WM = TM <= 128 ? 2 : 4, WN = TM <= 64 ? 2 : TM == 128 ? 4 : 2;
    gemm_mx_body<EPI, TM, TN, WM, WN, (TM > 128 || (TM == 64 && TN == 128) ? 3 : 4)>(a);
}

// Fitted to plain-store launches of 16 to 32768 rows; a slab is 128.  Without a low-rank branch: 1318 shapes of 128 to 5120 columns,
// the form it picks is 0.2 % slower on average than the fastest.  With one: eight weight shapes (mean error 6 %; 0.1 % slower than
// the fastest there).  The branch costs the 256 x 256 kernel most (see mx.hip), so priced by the second table products without one
// were taken off it too early (8192 rows of 1024 -> 3072: 42 us on 256 x 128, 37 on 256 x 256).  Other epilogues than the plain
// store cost it as well: they are priced by the second.
constexpr Form FORMS[2][7] = {
    {{32, 64, {3.712f, .177f}, {4.127f, .305f}, {0.f, .419f}},                 // plain store, no low-rank branch
     {64, 64, {4.033f, .198f}, {4.738f, .403f}, {.576f, .573f}},
     {64, 128, {4.391f, .265f}, {5.402f, .667f}, {.049f, .907f}},
     {128, 128, {5.154f, .334f}, {}, {4.425f, .652f}},
     {192, 128, {5.494f, .454f}, {}, {4.968f, .835f}},
     {256, 128, {6.320f, .550f}, {}, {5.886f, 1.036f}},
     {256, 256, {5.932f, 1.292f}, {}, {6.131f, 1.897f}}},
    {{32, 64, {3.29f, .189f}, {2.71f, .420f}, {0.08f, .458f}},
     {64, 64, {3.51f, .228f}, {2.90f, .552f}, {0.83f, .589f}},
     {64, 128, {3.74f, .326f}, {3.07f, .837f}, {0.68f, .942f}},
     {128, 128, {4.97f, .401f}, {}, {2.55f, .775f}},
     {192, 128, {5.27f, .532f}, {}, {3.38f, .980f}},
     {256, 128, {5.82f, .641f}, {}, {4.87f, 1.196f}},
     {256, 256, {5.83f, 1.388f}, {}, {6.79f, 2.063f}}}};

template <int EPI>
int launch_e(const MxArgs &a, const TilePlan &p, hipStream_t st)
{
    const int tiles = ((a.M + p.tm - 1) / p.tm) * ((a.seg_n + p.tn - 1) / p.tn) * a.nseg;
    const dim3 grid((tiles + 7) / 8 * 8), block(p.tm <= 64 ? 256 : 512);
    switch (p.tm * 1000 + p.tn) {
    case 32064: hipLaunchKernelGGL((gemm_mx_tile_kernel<EPI, 32, 64>), grid, block, 0, st, a); break;
    case 64064: hipLaunchKernelGGL((gemm_mx_tile_kernel<EPI, 64, 64>), grid, block, 0, st, a); break;
    case 64128: hipLaunchKernelGGL((gemm_mx_tile_kernel<EPI, 64, 128>), grid, block, 0, st, a); break;
    case 128128: hipLaunchKernelGGL((gemm_mx_tile_kernel<EPI, 128, 128>), grid, block, 0, st, a); break;
    case 192128: hipLaunchKernelGGL((gemm_mx_tile_kernel<EPI, 192, 128>), grid, block, 0, st, a); break;
    case 256128: hipLaunchKernelGGL((gemm_mx_tile_kernel<EPI, 256, 128>), grid, block, 0, st, a); break;
    default: return SL_EINVAL;
    }
    SL_CHECK_LAUNCH("gemm mx tile");
    return 0;
}

}  // namespace

TilePlan plan_gemm_mx(int M, int seg_n, int nseg, int K, int epi, bool low_rank)
{
    TilePlan best = {0, 0, 1, 0};
    double least = 0;
    for (const Form &f : FORMS[low_rank || epi != EPI_STORE]) {
        const double c = form_cost(f, (long)((M + f.tm - 1) / f.tm) * ((seg_n + f.tn - 1) / f.tn) * nseg, K / 128, epi == EPI_STORE ? 16 : 0);
        if (best.tm == 0 || c < least) { best = {f.tm, f.tn, 1, 0}; least = c; }
    }
    return best;
}

int launch_gemm_mx_tile(const MxArgs &a, int epi, const TilePlan &p, hipStream_t st)
{
    switch (epi) {
    case EPI_STORE: return launch_e<EPI_STORE>(a, p, st);
    case EPI_RESID: return launch_e<EPI_RESID>(a, p, st);
    case EPI_GELU: return launch_e<EPI_GELU>(a, p, st);
    case EPI_DGELU: return launch_e<EPI_DGELU>(a, p, st);
    case EPI_STORE_DELTA: return launch_e<EPI_STORE_DELTA>(a, p, st);
    }
    return SL_EINVAL;
}
