// bf16 MFMA GEMM on small tiles, for launches that would leave most of the chip idle on 256-row tiles (gfx950).
//
// Same product, low-rank branch and epilogues as gemm.hip:
//   out[M,N] = epilogue( X[M,K] . W[N,K]^T  +  zscale * (X . Z^T)[M,K2] . T[N,K2]^T )
//
// One block computes a TILE x TILE tile: 64 x 64 or 128 x 128 with 4 waves (2 x 2), two blocks to a CU, so that one's
// waits (copies, barriers, epilogue) are the other's matrix time; or 128 x 128 with 8 waves (2 x 4) and twice the LDS stages
// for launches that have one such tile per CU.  What bounds these launches is latency and how many CUs have work, not the
// matrix rate; plan_gemm_tile picks from the tile counts.
// Every output element is one accumulation over k in increasing order, as in gemm.hip, bit for bit: a sequence's results do
// not depend on which of the kernels its batch ran on.  Only single layers, which make no such promise, may share a short
// launch's contraction over blocks (splits): the partial accumulators of a tile's blocks go to scratch memory and the block
// that arrives last adds them in share order -- whichever block that is, so results are still reproducible.
#include "common.h"
#include "gemm_copy.h"
#include "gemm_epilogue.h"
#include <algorithm>

namespace {

constexpr int BK = 64, ROWB = BK * 2;
constexpr int SPLIT_TILES = 128;                         // most 64 x 64 tiles of a launch that shares its contraction

// Partial sums cross XCDs (each has its own L2), so they are written and read at device scope: relaxed 8-byte atomics
// go through to the memory side and need no cache flush; the order is kept by the vmcnt wait before the counter.
__device__ __forceinline__ void put_partial(float4 *p, f32x4 v)
{
    union { f32x4 f; unsigned long long u[2]; } x;
    x.f = v;
    __hip_atomic_store((unsigned long long *)p, x.u[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store((unsigned long long *)p + 1, x.u[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ f32x4 get_partial(const float4 *p)
{
    union { f32x4 f; unsigned long long u[2]; } x;
    x.u[0] = __hip_atomic_load((const unsigned long long *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    x.u[1] = __hip_atomic_load((const unsigned long long *)p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return x.f;
}

// Epilogue of 64 rows that the waves `wm` = own of the block hold: staged through LDS so that memory sees 16-byte accesses.
// INTERIOR: the rows and columns lie wholly inside the matrix, no branch (see epilogue4 in gemm.hip).
template <int EPI, int TILE, int NTHR, bool INTERIOR>
__device__ __forceinline__ void epilogue_rows(const GemmArgs &a, const float *stg, int m0, int n0, int n_end,
                                              const float (&bias8)[8])
{
    constexpr int P = TILE + 4, TPR = TILE / 8, RPP = NTHR / TPR, NP = 64 / RPP;
    const int er = (int)threadIdx.x / TPR, ec = ((int)threadIdx.x % TPR) * 8, col = n0 + ec;
    AuxRow aux[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int row = m0 + p * RPP + er;
        load_aux<EPI>(a, row, col, INTERIOR || (row < a.M && col < n_end), aux[p]);
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int rl = p * RPP + er, row = m0 + rl;
        const float4 p0 = *(const float4 *)(stg + rl * P + ec);
        const float4 p1 = *(const float4 *)(stg + rl * P + ec + 4);
        float v[8] = {p0.x + bias8[0], p0.y + bias8[1], p0.z + bias8[2], p0.w + bias8[3],
                      p1.x + bias8[4], p1.y + bias8[5], p1.z + bias8[6], p1.w + bias8[7]};
        if (INTERIOR || (row < a.M && col < n_end)) store_row8<EPI>(a, row, col, v, aux[p]);
    }
}

// NW waves, two rows of them; NST LDS stages
template <int EPI, int NZ, int TILE, int NW, int NST>
__global__ __launch_bounds__(64 * NW, 2) void gemm_tile_kernel(GemmArgs a, int splits)
{
    constexpr int NTHR = 64 * NW, WN = NW / 2;
    constexpr int XB = TILE * ROWB, ZB = NZ * ROWB, STAGE = 2 * XB + ZB;
    constexpr int MI = TILE / 32, NI = TILE / 16 / WN;   // 16 x 16 tiles of a wave along M and N
    constexpr int CP = TILE / 8 / NW;                    // copies (1 KB each) of a wave per operand and slab
    constexpr int ZI = NZ > 0 ? (NZ / 8 + NW - 1) / NW : 0;      // and of the down-projection rows (some are copied twice)
    constexpr int PER = 2 * CP + ZI;
    constexpr int NZT = NZ > 0 ? NZ / 16 : 1, MZ = MI / WN;
    constexpr int K2P = NZ > 0 ? (NZ + 31) / 32 * 32 : 32;
    constexpr int P = TILE + 4;
    constexpr int EPB = 64 * P * 4, LDSB = NST * STAGE > EPB ? NST * STAGE : EPB;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[LDSB];
    __shared__ int last_block;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int r16 = lane & 15, kg = lane >> 4;

    // tile and share of the contraction of this block; consecutive logical ids land on one XCD and walk panels of
    // PANEL row tiles column by column (operands of the tiles in flight on an XCD stay in its L2)
    const int tiles_n_seg = (a.seg_n + TILE - 1) / TILE;
    const int tiles_n = tiles_n_seg * a.nseg;
    const int tiles_m = (a.M + TILE - 1) / TILE;
    const int nb = tiles_m * tiles_n * splits;
    const int per_xcd = (nb + 7) >> 3;
    const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (logical >= nb || (int)(blockIdx.x >> 3) >= per_xcd) return;
    const int tile = logical / splits, split = logical - tile * splits;
    constexpr int PANEL = 8;
    const int pidx = tile / (PANEL * tiles_n), prem = tile - pidx * (PANEL * tiles_n);
    const int prow = min(PANEL, tiles_m - pidx * PANEL);
    const int tn = prem / prow, tm = pidx * PANEL + prem - tn * prow;
    const int seg = tn / tiles_n_seg, tns = tn - seg * tiles_n_seg;
    const int n0 = seg * a.seg_n + tns * TILE, n_end = (seg + 1) * a.seg_n, m0 = tm * TILE;
    const int nk_all = a.K / BK;
    const int ks0 = (int)((long)split * nk_all / splits), nk = (int)((long)(split + 1) * nk_all / splits) - ks0;
    const bool has_z = (NZ > 0) && (a.zmat[seg] != nullptr);

    // copies: 8 rows (1 KB) per instruction, lane l fills 16-byte slot l: row l>>3, physical k-chunk l&7 holding logical
    // chunk (l&7) ^ (l>>3)
    const int lrow = lane >> 3, lch = (lane & 7) ^ (lane >> 3);
    unsigned xo[CP], wo[CP], zo[ZI > 0 ? ZI : 1];
#pragma unroll
    for (int p = 0; p < CP; ++p) {
        xo[p] = ((unsigned)min(m0 + (wave * CP + p) * 8 + lrow, a.M - 1) * (unsigned)a.ldx + lch * 8) * 2u;
        wo[p] = ((unsigned)min(n0 + (wave * CP + p) * 8 + lrow, n_end - 1) * (unsigned)a.ldw + lch * 8) * 2u;
    }
#pragma unroll
    for (int p = 0; p < ZI; ++p) {
        const int piece = (wave * ZI + p) % (NZ > 0 ? NZ / 8 : 1);      // 8-row piece; past the last one: the first again
        zo[p] = has_z ? ((unsigned)(piece * 8 + lrow) * (unsigned)a.ldz + lch * 8) * 2u : xo[0];
    }
    const char *Xb = (const char *)a.X, *Wb = (const char *)a.W;
    const char *Zb = has_z ? (const char *)a.zmat[seg] : (const char *)a.X;
    const unsigned base = lds_addr(lds);
    // copies past the last slab repeat it (in bounds, never read), so that one constant serves every wait
#define GT_ISSUE(slot, t)                                                                              \
    {                                                                                                  \
        const size_t kb_ = (size_t)(ks0 + min((t), nk - 1)) * ROWB;                         \
        const unsigned sb_ = base + (slot) * STAGE;                                                    \
        _Pragma("unroll") for (int p = 0; p < CP; ++p) glds_soff(Xb + kb_, xo[p], sb_ + (wave * CP + p) * 1024); \
        _Pragma("unroll") for (int p = 0; p < CP; ++p) glds_soff(Wb + kb_, wo[p], sb_ + XB + (wave * CP + p) * 1024); \
        _Pragma("unroll") for (int p = 0; p < ZI; ++p)                                                 \
            glds_soff(Zb + kb_, zo[p], sb_ + 2 * XB + ((wave * ZI + p) % (NZ > 0 ? NZ / 8 : 1)) * 1024); \
    }

    f32x4 acc[MI][NI], zacc[MZ][NZT];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int h = 0; h < MZ; ++h)
#pragma unroll
        for (int q = 0; q < NZT; ++q) zacc[h][q] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int a_row = (wm * (TILE / 2) + r16) * ROWB, b_row = XB + (wn * (TILE / WN) + r16) * ROWB;
    const int z_row = a_row + wn * MZ * 16 * ROWB;
    const int sw = r16 & 7;
    // operand fragments of k-step k2 of a slab
#define GT_READ(F, slot, k2)                                                                           \
    {                                                                                                  \
        const unsigned char *S_ = lds + (slot) * STAGE;                                               \
        const int co = (((k2) * 4 + kg) ^ sw) << 4;                                                    \
        _Pragma("unroll") for (int i = 0; i < MI; ++i) F.a[i] = *(const bf16x8 *)(S_ + a_row + i * 16 * ROWB + co); \
        _Pragma("unroll") for (int j = 0; j < NI; ++j) F.b[j] = *(const bf16x8 *)(S_ + b_row + j * 16 * ROWB + co); \
        if (NZ > 0) {                     /* the waves that share rows share out the rank-space rows */ \
            _Pragma("unroll") for (int h = 0; h < MZ; ++h) F.za[h] = *(const bf16x8 *)(S_ + z_row + h * 16 * ROWB + co); \
            _Pragma("unroll") for (int q = 0; q < NZT; ++q) F.zb[q] = *(const bf16x8 *)(S_ + 2 * XB + (q * 16 + r16) * ROWB + co); \
        }                                                                                              \
    }
#define GT_MFMA(F)                                                                                     \
    {                                                                                                  \
        _Pragma("unroll") for (int i = 0; i < MI; ++i)                                                 \
            _Pragma("unroll") for (int j = 0; j < NI; ++j)                                             \
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(F.a[i], F.b[j], acc[i][j], 0, 0, 0); \
        if (NZ > 0) {                                                                                  \
            _Pragma("unroll") for (int q = 0; q < NZT; ++q)                                            \
                _Pragma("unroll") for (int h = 0; h < MZ; ++h)                                         \
                    zacc[h][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(F.za[h], F.zb[q], zacc[h][q], 0, 0, 0); \
        }                                                                                              \
    }
    struct Frags { bf16x8 a[MI], b[NI], za[MZ], zb[NZT]; } f0, f1;

    // up-projection operands, needed after the loop: requested first, so that the waits below count copies only
    bf16x8 tb[K2P / 32][NI];
    if (NZ > 0 && has_z) {
#pragma unroll
        for (int ks = 0; ks < K2P / 32; ++ks)
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                const int n = min(n0 + wn * (TILE / WN) + j * 16 + r16, n_end - 1) - seg * a.seg_n;
                tb[ks][j] = *(const bf16x8 *)(a.tmat[seg] + (size_t)n * a.ldt + ks * 32 + kg * 8);
            }
    }
#pragma unroll
    for (int s = 0; s < NST; ++s) GT_ISSUE(s, s)
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 1) * PER) : "memory");
    __syncthreads();
    GT_READ(f0, 0, 0)
    // Fragments are read one k-step ahead of their MFMAs, and the one barrier of a slab sits between its k-steps: in
    // front of it the wave's reads of the slab are done and its copies of the next slab have landed (the newer ones may
    // still be in flight); behind it the slab's slot is refilled, NST - 1 slabs before it is needed.
    int slot = 0;
    for (int t = 0; t < nk; ++t) {
        const int next = slot + 1 == NST ? 0 : slot + 1;
        GT_READ(f1, slot, 1)
        __builtin_amdgcn_sched_barrier(0);
        GT_MFMA(f0)
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NST - 2) * PER) : "memory");
        __syncthreads();
        GT_READ(f0, next, 0)
        GT_ISSUE(slot, t + NST)
        __builtin_amdgcn_sched_barrier(0);
        GT_MFMA(f1)
        __builtin_amdgcn_sched_barrier(0);
        slot = next;
    }
    // the repeated copies have landed and every wave is done with the ring before it is reused
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
#undef GT_ISSUE
#undef GT_READ
#undef GT_MFMA

    if (splits > 1) {
        constexpr int NV = MI * NI + (NZ > 0 ? MZ * NZT : 0);            // float4 per thread
        float4 *part = (float4 *)a.split_part + ((size_t)tile * splits) * NV * NTHR + tid;
        float4 *mine = part + (size_t)split * NV * NTHR;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) put_partial(mine + (i * NI + j) * NTHR, acc[i][j]);
        if (NZ > 0) {
#pragma unroll
            for (int h = 0; h < MZ; ++h)
#pragma unroll
                for (int q = 0; q < NZT; ++q) put_partial(mine + (MI * NI + h * NZT + q) * NTHR, zacc[h][q]);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                 // this wave's partial sums are in memory
        __syncthreads();
        if (tid == 0) {
            const unsigned n = __hip_atomic_fetch_add(a.split_cnt + tile, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            last_block = n + 1 == (unsigned)splits;
            // the last block leaves the counter as the next launch expects it
            if (last_block) __hip_atomic_store(a.split_cnt + tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        if (!last_block) return;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) acc[i][j] = get_partial(part + (i * NI + j) * NTHR);
        if (NZ > 0) {
#pragma unroll
            for (int h = 0; h < MZ; ++h)
#pragma unroll
                for (int q = 0; q < NZT; ++q) zacc[h][q] = get_partial(part + (MI * NI + h * NZT + q) * NTHR);
        }
        for (int s = 1; s < splits; ++s) {
            const float4 *src = part + (size_t)s * NV * NTHR;
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j) acc[i][j] += get_partial(src + (i * NI + j) * NTHR);
            if (NZ > 0) {
#pragma unroll
                for (int h = 0; h < MZ; ++h)
#pragma unroll
                    for (int q = 0; q < NZT; ++q) zacc[h][q] += get_partial(src + (MI * NI + h * NZT + q) * NTHR);
            }
        }
    }

    // ---- low-rank tail: acc += (zscale * z)[TILE,K2P] . T[n,K2P]^T ------------------------------------
    if (NZ > 0 && has_z) {
        constexpr int ZP = K2P + 8;
        bf16 *zs = (bf16 *)lds;
#pragma unroll
        for (int h = 0; h < MZ; ++h)
#pragma unroll
            for (int q = 0; q < K2P / 16; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int row = wm * (TILE / 2) + (wn * MZ + h) * 16 + 4 * kg + e;
                    zs[row * ZP + q * 16 + r16] = f2bf(q < NZT ? zacc[h][q < NZT ? q : 0][e] * a.zscale : 0.f);
                }
        __syncthreads();
        if (a.zspill[seg] != nullptr && tns == 0) {
            const int cpr = a.K2 >> 3;                   // 16-byte chunks per row
            for (int c = tid; c < TILE * cpr; c += NTHR) {
                const int row = c / cpr, cc = c - row * cpr;
                if (m0 + row < a.M)
                    *(uint4 *)(a.zspill[seg] + (size_t)(m0 + row) * a.K2 + cc * 8) = *(const uint4 *)(zs + row * ZP + cc * 8);
            }
        }
#pragma unroll
        for (int ks = 0; ks < K2P / 32; ++ks) {
            bf16x8 af[MI];
#pragma unroll
            for (int i = 0; i < MI; ++i)
                af[i] = *(const bf16x8 *)(zs + (wm * (TILE / 2) + i * 16 + r16) * ZP + ks * 32 + kg * 8);
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], tb[ks][j], acc[i][j], 0, 0, 0);
        }
        __syncthreads();                                 // the z tile has been consumed
    }

    // ---- epilogue, 64 rows at a time ---------------------------------------------------------------------
    constexpr int TPR = TILE / 8;
    const int gcol = n0 + (tid % TPR) * 8;
    float bias8[8];
    {
        bf16x8 b8;
#pragma unroll
        for (int i = 0; i < 8; ++i) b8[i] = f2bf(0.f);
        if (a.bias && gcol < n_end) b8 = *(const bf16x8 *)(a.bias + gcol);
#pragma unroll
        for (int i = 0; i < 8; ++i) bias8[i] = bf2f(b8[i]);
    }
    float *stg = (float *)lds;
    const bool interior = m0 + TILE <= a.M && n0 + TILE <= n_end;
#pragma unroll
    for (int c = 0; c < TILE / 64; ++c) {
        if (c > 0) __syncthreads();
        // 64-row chunk c: both wave rows at TILE = 64, wave row c at TILE = 128
        if (TILE == 64 || wm == c) {
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        stg[((TILE == 64 ? wm * 32 : 0) + i * 16 + 4 * kg + e) * P + wn * (TILE / WN) + j * 16 + r16] = acc[i][j][e];
        }
        if (interior) epilogue_rows<EPI, TILE, NTHR, true>(a, stg, m0 + 64 * c, n0, n_end, bias8);
        else epilogue_rows<EPI, TILE, NTHR, false>(a, stg, m0 + 64 * c, n0, n_end, bias8);
    }
}

template <int EPI, int NZ, int TILE, int NW, int NST>
int launch_tt(const GemmArgs &a, int splits, hipStream_t st)
{
    const int tiles = ((a.M + TILE - 1) / TILE) * ((a.seg_n + TILE - 1) / TILE) * a.nseg;
    hipLaunchKernelGGL((gemm_tile_kernel<EPI, NZ, TILE, NW, NST>), dim3((tiles * splits + 7) / 8 * 8), dim3(64 * NW), 0, st, a,
                       splits);
    SL_CHECK_LAUNCH("gemm tile");
    return 0;
}
template <int EPI, int NZ>
int launch_tz(const GemmArgs &a, const TilePlan &p, hipStream_t st)
{
    // LDS stages: as many as leave room for two blocks on a CU; a block of 8 waves owns its CU
    if (p.tile == 64) return launch_tt<EPI, NZ, 64, 4, NZ < 32 ? 4 : 3>(a, p.splits, st);
    return p.waves == 4 ? launch_tt<EPI, NZ, 128, 4, 2>(a, 1, st) : launch_tt<EPI, NZ, 128, 8, 4>(a, 1, st);
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

}  // namespace

// Over how many blocks a launch of t64 tiles of 64 x 64 and nk slabs shares its contraction, if it has scratch for that.
// Combining the partial sums costs about 3 us, so a block keeps 9 slabs or more.
static int split_shares(long t64, int nk)
{
    const int s = t64 > SPLIT_TILES ? 1 : t64 > 64 ? 2 : t64 > 32 ? 3 : 4;
    return std::max(1, std::min(s, nk / 9));
}

// What this launch should run on: tile 64 or 128 (with the number of wave groups and of blocks per tile), or 0 for the
// 256-row kernels of gemm.hip.  Costs are in units of a round of 256 x 256 tiles over the 256 CUs.
TilePlan plan_gemm_tile(int M, int seg_n, int nseg, int K, int nz, bool can_split)
{
    auto tiles = [&](int tm, int tn) { return (long)((M + tm - 1) / tm) * ((seg_n + tn - 1) / tn) * nseg; };
    const long t64 = tiles(64, 64), t128 = tiles(128, 128), t256 = tiles(256, 256), t128x256 = tiles(128, 256);
    // Up to two 64 x 64 tiles per CU: all of them run at once, and the smallest tile gives the most CUs work (M = 128,
    // 768 x 768: 5.4 us against 10 on 128-row tiles and 24 on 256-row ones).  With 128 tiles or fewer a long
    // contraction is shared out too.
    if (t64 <= 512) return {64, 4, can_split ? split_shares(t64, K / BK) : 1};
    // One 128 x 128 tile per CU at most: 8 waves, so that each SIMD has two, and four stages (T = 4096, 4096 -> 1024: 34.5 us
    // against 44 with 4 waves and two stages, 54 on 128-row tiles of the 4-wave kernel).
    if (t128 <= 256) return {128, 8, 1};
    // Otherwise two such tiles share a CU; a round of 512 of them costs 0.58 of a round of 256-row tiles (85 against 128
    // flop per operand byte), 0.75 with a rank-space branch (its rows are copied and multiplied for every tile: 32768
    // tokens of 1280, five rounds of 128 against three of 256: 141, 176 and 380 us against 124, 171 and 332); a partial one
    // less.  256-row tiles lose whole rounds instead.
    const long full = t128 / 512, rem = t128 - 512 * full;
    const double c128 = (nz == 0 ? 0.58 : 0.75) * (full + (rem == 0 ? 0.0 : rem <= 256 ? 0.75 : 0.9));
    double c256 = (double)((t256 + 255) / 256);
    if (nz == 0 && M >= 1024) c256 = std::min(c256, 0.58 * ((t128x256 + 255) / 256));
    return c128 < c256 ? TilePlan{128, 4, 1} : TilePlan{0, 4, 1};
}

int gemm_split_rows(int N, int K)
{
    return split_shares(1, K / BK) > 1 ? SPLIT_TILES / ((N + 63) / 64) * 64 : 0;
}
// a block leaves its 64 x 64 fp32 sums and its 64 rows of rank-space ones
size_t gemm_split_bytes(int M, int N, int K, int nz)
{
    const int cols = (N + 63) / 64, rows = std::min((M + 63) / 64, SPLIT_TILES / cols);
    long blocks = 0;
    for (int r = 1; r <= rows; ++r) {
        const int s = split_shares((long)r * cols, K / BK);
        if (s > 1) blocks = std::max(blocks, (long)r * cols * s);
    }
    return (size_t)blocks * 64 * (64 + nz) * sizeof(float);
}
size_t gemm_split_counter_bytes() { return SPLIT_TILES * sizeof(unsigned); }

int launch_gemm_tile(const GemmArgs &a, int epi, int nz, const TilePlan &p, hipStream_t st)
{
    switch (epi) {
    case EPI_STORE: return launch_te<EPI_STORE>(a, nz, p, st);
    case EPI_RESID: return launch_te<EPI_RESID>(a, nz, p, st);
    case EPI_GELU: return launch_te<EPI_GELU>(a, nz, p, st);
    case EPI_DGELU: return launch_te<EPI_DGELU>(a, nz, p, st);
    case EPI_STORE_DELTA: return nz == 0 ? launch_tz<EPI_STORE_DELTA, 0>(a, p, st) : SL_EINVAL;
    }
    return SL_EINVAL;
}
