// bf16 MFMA GEMM on small tiles with blocks of 4 waves, two to a CU, and the rule that picks the kernel of a product (gfx950).
//
// The tiles are for launches that would leave most of the chip idle on larger ones: 32 x 32 (two slabs of 64 to a barrier;
// one sequence of 128 tokens, 3072 -> 768: 6.7 us against 10.4 on 64 x 64 tiles), 32 x 64, 64 x 64 and 64 x 128, so that one
// block's waits (copies, barriers, epilogue) are the other's matrix time.  Only single layers, which do not promise that a
// sequence's bits are the same in every batch, may share a short launch's contraction over blocks (64 x 64 tiles).
#include "gemm_tile.h"
#include <algorithm>

namespace {

constexpr int SPLIT_TILES = 128;                         // most 64 x 64 tiles of a launch that shares its contraction

// Ring depths: as many stages as leave room for two blocks in the 160 KB of a CU (one with 32 x 64 tiles and a rank-space
// branch, where two stages would be 2.3 times as slow as three).
template <int EPI, int NZ, int TM, int TN>
__global__ __launch_bounds__(256, TM == 32 && NZ == 16 ? 1 : 2) void gemm_tile_kernel(GemmArgs a, int splits)
{
    constexpr bool SPLIT = TM == 64 && TN == 64 && EPI == EPI_STORE && NZ <= 16;
    constexpr int NSUB = TM == 32 ? 2 : 1, NST = TN == 64 && TM == 64 ? (NZ < 32 ? 4 : 3) : NZ < 32 ? 3 : 2;
    gemm_tile_body<EPI, NZ, TM, TN, 2, 2, NSUB, NST, SPLIT>(a, splits);
}
template <int EPI, int NZ>
__global__ __launch_bounds__(256, NZ == 48 ? 1 : 2) void gemm_tile32_kernel(GemmArgs a)
{
    gemm_tile_body<EPI, NZ, 32, 32, 2, 2, 2, NZ == 0 ? 4 : 3, false>(a, 1);
}

// 128 x 128 with 4 waves, two blocks to a CU: plain stores of short contractions, whose epilogue then has another block's loop
// beside it (13197 rows of 128 -> 2520: 26.2 us, 30.3 on 64 x 128, 31.7 on 128 x 256).
template <int EPI>
__global__ __launch_bounds__(256, 2) void gemm_tile128_kernel(GemmArgs a)
{
    gemm_tile_body<EPI, 0, 128, 128, 2, 2, 1, 2, false>(a, 1);
}

int tile_grid(const GemmArgs &a, int tm, int tn, int splits)
{
    const int tiles = ((a.M + tm - 1) / tm) * ((a.seg_n + tn - 1) / tn) * a.nseg;
    return (tiles * splits + 7) / 8 * 8;
}
template <int EPI, int NZ>
int launch_tz(const GemmArgs &a, const TilePlan &p, hipStream_t st)
{
    if (p.splits > 1 && !(p.tm == 64 && p.tn == 64 && EPI == EPI_STORE && NZ <= 16)) return SL_EINVAL;
    const dim3 grid(tile_grid(a, p.tm, p.tn, p.splits)), block(256);
    if (p.pair) {
        if constexpr (EPI == EPI_STORE && NZ == 0) hipLaunchKernelGGL((gemm_tile128_kernel<EPI>), grid, block, 0, st, a);
        else return SL_EINVAL;
    } else if (p.tm == 64 && p.tn == 64) hipLaunchKernelGGL((gemm_tile_kernel<EPI, NZ, 64, 64>), grid, block, 0, st, a, p.splits);
    else if (p.tm == 64) hipLaunchKernelGGL((gemm_tile_kernel<EPI, NZ, 64, 128>), grid, block, 0, st, a, 1);
    else if (p.tn == 64) hipLaunchKernelGGL((gemm_tile_kernel<EPI, NZ, 32, 64>), grid, block, 0, st, a, 1);
    else if constexpr (EPI != EPI_STORE_DELTA) hipLaunchKernelGGL((gemm_tile32_kernel<EPI, NZ>), grid, block, 0, st, a);
    else return SL_EINVAL;
    SL_CHECK_LAUNCH("gemm tile");
    return 0;
}
template <int EPI>
int launch_te(const GemmArgs &a, int nz, const TilePlan &p, hipStream_t st)
{
    switch (nz) {
    case 0: return launch_tz<EPI, 0>(a, p, st);
    case 16: return launch_tz<EPI, 16>(a, p, st);
    case 32: if (EPI == EPI_STORE) return launch_tz<EPI_STORE, 32>(a, p, st); break;
    case 48: if (EPI == EPI_STORE) return launch_tz<EPI_STORE, 48>(a, p, st); break;
    }
    return SL_EINVAL;
}

// Fitted to plain-store launches of 64 to 32768 rows at seven weight shapes of 768 to 5120 (mean error 2 to 6 %; the form it picks
// is 0.5 % slower on average than the fastest of such a launch).  Other epilogues are priced as that one and take up to 45 % more
// (GELU of 10240 rows of 768 -> 3072: 49 us here, 72 measured).  The third group was fitted to 32 and 48 columns together; its
// 256 x 256 row is that of 48 (32768 rows of 4096 -> 1024: 262 us, with 32 columns 233).
constexpr double FILL = 12;                              // (form_cost)
constexpr Form FORMS[3][9] = {
    {{32, 32, {2.46f, .093f}, {2.60f, .175f}, {0.97f, .170f}},          // no rank-space branch
     {32, 64, {2.33f, .129f}, {2.49f, .250f}, {0.70f, .269f}},
     {64, 64, {2.70f, .171f}, {2.85f, .344f}, {0.68f, .394f}},
     {64, 128, {2.38f, .263f}, {3.96f, .522f}, {0.65f, .658f}},
     {128, 128, {3.61f, .295f}, {}, {3.28f, .463f}},
     {192, 128, {3.97f, .366f}, {}, {4.76f, .609f}},
     {256, 128, {4.78f, .510f}, {}, {5.57f, .810f}},
     {128, 256, {5.20f, .646f}, {}, {4.93f, .865f}},
     {256, 256, {7.20f, 1.058f}, {}, {7.95f, 1.423f}}},
    {{32, 32, {3.01f, .133f}, {3.14f, .239f}, {1.30f, .232f}},          // 16 rank-space columns
     {32, 64, {3.26f, .157f}, {4.68f, .339f}, {3.14f, .345f}},
     {64, 64, {3.53f, .195f}, {3.81f, .397f}, {1.71f, .451f}},
     {64, 128, {3.45f, .289f}, {4.88f, .587f}, {1.76f, .706f}},
     {128, 128, {4.62f, .338f}, {}, {4.04f, .529f}},
     {192, 128, {5.53f, .424f}, {}, {5.53f, .689f}},
     {256, 128, {6.05f, .591f}, {}, {6.46f, .896f}},
     {},
     {256, 256, {6.80f, 1.083f}, {}, {5.00f, 1.690f}}},
    {{32, 32, {3.48f, .181f}, {5.18f, .384f}, {3.46f, .371f}},          // 32 or 48
     {32, 64, {2.51f, .355f}, {4.33f, .403f}, {2.00f, .446f}},
     {64, 64, {3.55f, .270f}, {4.37f, .474f}, {2.00f, .552f}},
     {64, 128, {2.11f, .685f}, {5.70f, .753f}, {2.27f, .931f}},
     {128, 128, {5.55f, .371f}, {}, {5.71f, .571f}},
     {192, 128, {7.54f, .515f}, {}, {7.47f, .806f}},
     {},
     {},
     {256, 256, {8.10f, 1.342f}, {}, {6.20f, 1.950f}}}};

// The pair form of 128 x 128, for plain stores without a rank-space branch and contractions below 768: of 882 such shapes it takes
// 200, the form picked is then 1.1 % slower on average than the fastest, 2.9 % without it.  (From 768 on the other forms are
// within 1 % of it wherever it wins.)
constexpr Form PAIR = {128, 128, {3.87f, .465f}, {4.351f, .896f}, {-1.789f, 1.563f}};

}  // namespace

// Over how many blocks a launch of t64 tiles of 64 x 64 and nk slabs may share its contraction, if it has scratch for that:
// 32 tiles or fewer over four, 64 over three, 128 over two, so that every block has a CU.  A block keeps 9 slabs or more.
constexpr long SPLIT_ENDS[3] = {32, 64, SPLIT_TILES};
static int split_shares(long t64, int nk)
{
    const int s = t64 > SPLIT_ENDS[2] ? 1 : t64 > SPLIT_ENDS[1] ? 2 : t64 > SPLIT_ENDS[0] ? 3 : 4;
    return std::max(1, std::min(s, nk / 9));
}

// The kernel for a product: the form that costs least (FORMS).  `whole`: the kernels of 256-column tiles may be picked too.
// A shared contraction costs its blocks 3 us to combine their partial sums, so it takes 43 slabs or more to beat the forms of
// 32 rows.
TilePlan plan_gemm_tile(int M, int seg_n, int nseg, int K, int epi, int nz, bool can_split, bool whole)
{
    const int nk = K / BK;
    auto tiles = [&](int tm, int tn) { return (long)((M + tm - 1) / tm) * ((seg_n + tn - 1) / tn) * nseg; };
    TilePlan best = {0, 0, 1, 0};
    double least = 0;
    for (const Form &f : FORMS[nz == 0 ? 0 : nz == 16 ? 1 : 2]) {
        if (f.tm == 0 || (!whole && f.tn == 256)) continue;
        if (epi == EPI_STORE_DELTA && f.tn < 64) continue;               // a head's columns in one tile
        const double c = form_cost(f, tiles(f.tm, f.tn), nk, epi == EPI_STORE ? FILL : 0);
        if (best.tm == 0 || c < least) { best = {f.tm, f.tn, 1, 0}; least = c; }
    }
    if (epi == EPI_STORE && nz == 0 && nk < 12) {
        const double c = form_cost(PAIR, tiles(PAIR.tm, PAIR.tn), nk, FILL);
        if (c < least) { best = {PAIR.tm, PAIR.tn, 1, 1}; least = c; }
    }
    if (can_split && epi == EPI_STORE && nz <= 16) {
        const int s = split_shares(tiles(64, 64), nk);
        if (s > 1 && form_cost(FORMS[nz == 0 ? 0 : 1][2], tiles(64, 64) * s, (nk + s - 1) / s, FILL) + 3.0 < least) best = {64, 64, s, 0};
    }
    return best;
}

// A plain store over counted rows (at most M) on a kernel that computes all M: up to 512 tiles of 128 x 128, which the smaller forms
// take at once, and for at most 128 rows, of which the counting kernel's 256-row tiles would fill half.  Larger launches would
// spend rounds on rows that nobody wants (40 % of a loss head's are prompt tokens).  Whole loss heads of 768 columns, us, on the
// smaller forms and on the counting kernel: 2315 tokens, V = 2000 (304 tiles) 59, 69; 1024, 8000 (504) 78.5, 86; 1500, 8000
// (756) 90, 92, with 1280 columns 112, 110; 1500, 31118 (2928; 1280 columns) 273, 220.
TilePlan plan_gemm_counted(int M, int N, int K)
{
    if (M > 128 && (long)((M + 127) / 128) * ((N + 127) / 128) > 512) return {0, 0, 0, 0};
    return plan_gemm_tile(M, N, 1, K, EPI_STORE, 0, false, M <= 128);
}

// Scratch by the decision above, so that a layer has none where its launch shares nothing.  The shared form costs the same at
// every row count of a share count and the others no less at more rows, so a share count that is ever taken is taken at its
// last row of tiles, and those say what any number of rows needs.
SplitPlan plan_gemm_split(int M, int N, int K, int nz)
{
    SplitPlan p = {false, 0, 0};
    const int nk = K / BK, cols = (N + 63) / 64, rows = (M + 63) / 64;
    if (split_shares(1, nk) == 1 || cols > SPLIT_TILES) return p;
    auto shares = [&](int m) { return plan_gemm_tile(m, N, 1, K, EPI_STORE, nz, true, true).splits; };
    long blocks = 0;
    auto count = [&](int r, int s) { if (s > 1) blocks = std::max(blocks, (long)r * cols * s); };
    for (long end : SPLIT_ENDS) {
        const int last = (int)end / cols;
        if (last == 0) continue;
        const int s = shares(last * 64);
        if (s > 1) p.most_rows = last * 64;
        if (last * 64 <= M) count(last, s);
    }
    if (M <= p.most_rows) {
        const int s = shares(M);
        p.shared = s > 1;
        count(rows, s);
    }
    // a block leaves its 64 x 64 fp32 sums and its 64 rows of rank-space ones
    p.bytes = (size_t)blocks * 64 * (64 + nz) * sizeof(float);
    return p;
}
size_t gemm_split_counter_bytes() { return SPLIT_TILES * sizeof(unsigned); }

int launch_gemm_tile(const GemmArgs &a, int epi, int nz, const TilePlan &p, hipStream_t st)
{
    if (p.tm > 64 && p.tn == 128 && !p.pair) return launch_gemm_wide(a, epi, nz, p, st);
    switch (epi) {
    case EPI_STORE: return launch_te<EPI_STORE>(a, nz, p, st);
    case EPI_RESID: return launch_te<EPI_RESID>(a, nz, p, st);
    case EPI_GELU: return launch_te<EPI_GELU>(a, nz, p, st);
    case EPI_DGELU: return launch_te<EPI_DGELU>(a, nz, p, st);
    case EPI_STORE_DELTA: return nz == 0 ? launch_tz<EPI_STORE_DELTA, 0>(a, p, st) : SL_EINVAL;
    }
    return SL_EINVAL;
}
