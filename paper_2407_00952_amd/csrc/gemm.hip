// bf16 MFMA GEMM for frozen linears with the rank-r LoRA branch fused on chip (gfx950).
//
//   out[M,N] = epilogue( X[M,K] . W[N,K]^T  +  zscale * (X . Z^T)[M,K2] . T[N,K2]^T )
//
// Forward (SplitLoRA Sec. II-C: W + low-rank product):  Z = A (down-projection, rows
// padded with zeros), T = B (up-projection).  Input-gradient pass: the same kernel on the
// transposed frozen weight with Z = B^T and T = A^T, so no weight gradient is ever formed.
// The rank-space product X.Z^T is accumulated inside the K loop from the X tile that is
// already in LDS, scaled, rounded to bf16, staged through LDS and applied as K2/16 extra
// MFMA steps; the first column tile of a segment also spills it ([M,K2] bf16) because the
// adapter-gradient kernels need it.  Input gradients of large batches find it spilled already (gemm_tail4).
//
// Tiling: 256x256x64 block tile, 8 waves (2 x 4), wave tile 128x64 = 8x4 MFMA 16x16x32
// tiles (measured ~8 % faster than 32x32x16 on this power-limited part); two LDS stages filled
// by asynchronous global->LDS copies (no staging registers), 16-byte XOR-swizzled LDS rows
// so that both the copies and the MFMA operand reads are bank-conflict free.
#include "common.h"
#include "gemm_copy.h"
#include "gemm_epilogue.h"
#include "prof.h"
#include <algorithm>

namespace {

constexpr int BM = 256, BN = 256, BK = 64, NTHR = 512;
constexpr int ROWB = BK * 2;                 // bytes per LDS row (one k-slab of a tile row)
constexpr int XB = BM * ROWB, WB = BN * ROWB;

// NZ = number of rank-space columns handled in the K loop: 16 per adapter whose down-projection
// spans this K range (16, 32 or 48).  K2P = NZ rounded up to the MFMA k-step of 32.
//
// Bound by the matrix pipe's rate under the power limit once nothing waits in front of it; the loop is there to get to that.
// Fragments are read AHEAD row tiles before their MFMAs, one after each row tile's products, and the copies of the slab
// after the next go out one or two behind each row tile, so neither the LDS queue nor the copy queue ever holds a wave up;
// one barrier per slab, where the last fragments of its buffer have been read.  Every LDS read is at one of two lane
// offsets plus a scalar: with an address register for each, 28 to 96 bytes of the loop's values were spilled, which cost
// all of the gain.  us at 32768 rows, rank-space columns 16 / 32 / 48, against a loop that read all fragments of a k-step and
// then multiplied: 4096 -> 1024 254 -> 225, 257 -> 233, 270 -> 262; 1024 -> 4096 285 -> 270, 292 -> 280, 319 -> 312;
// 10240 x 768 -> 2304 48.0 -> 45.4, 49.9 -> 47.2, 55.8 -> 54.2.
template <int EPI, int NZ>
__global__ __launch_bounds__(NTHR) void gemm_kernel(GemmArgs a)
{
    constexpr int ZB = NZ * ROWB, STAGE = XB + WB + ZB;
    constexpr int K2P = (NZ + 31) / 32 * 32;
    constexpr int NZT = NZ / 16;                         // 16-column tiles of z
    // 8 where the registers hold them (4: 16 columns 225 -> 239 us at 32768 x 4096 -> 1024; 8: 48 columns spill, 262 -> 392)
    constexpr int AHEAD = NZ <= 32 ? 8 : 4;
    __shared__ __attribute__((aligned(1024))) unsigned char st0[STAGE];
    __shared__ __attribute__((aligned(1024))) unsigned char st1[STAGE];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const int r16 = lane & 15, kg = lane >> 4;           // MFMA 16x16x32: row/column r16, k-group kg

    // ---- tile of this block; consecutive logical tiles go to the same XCD (blocks are
    //      handed to the 8 XCDs round-robin) so an XCD's L2 sees each X row tile once.
    const int tiles_n_seg = (a.seg_n + BN - 1) / BN;
    const int tiles_n = tiles_n_seg * a.nseg;
    const int tiles_m = (a.M + BM - 1) / BM;
    const int nb = tiles_m * tiles_n;
    const int per_xcd = (nb + 7) >> 3;
    const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (logical >= nb) return;
    // inside an XCD's range the tiles are walked in panels of 4 row tiles, column by column, so the
    // 32 tiles in flight on an XCD form a 4 x 8 patch: each X row tile and each W column tile is
    // fetched into that L2 once per patch instead of W being re-streamed for every pair of row tiles
    constexpr int PANEL = 4;
    const int pidx = logical / (PANEL * tiles_n), prem = logical - pidx * (PANEL * tiles_n);
    const int prow = min(PANEL, tiles_m - pidx * PANEL);
    const int tn = prem / prow, tm = pidx * PANEL + prem - tn * prow;
    const int seg = tn / tiles_n_seg;
    const int tns = tn % tiles_n_seg;
    const int n0 = seg * a.seg_n + tns * BN;
    const int n_end = (seg + 1) * a.seg_n;
    const int m0 = tm * BM;

    const bool has_z = a.zmat[seg] != nullptr;

    // ---- global -> LDS: every wave copies 32 rows of the X tile and 32 rows of the W tile per
    //      stage, 8 rows (1 KB) per instruction.  Lane l fills 16-byte slot l of the 1 KB chunk:
    //      row l>>3, physical k-chunk l&7, which holds logical k-chunk (l&7) ^ (l>>3) (XOR swizzle).
    const int lrow = lane >> 3, lch = (lane & 7) ^ (lane >> 3);
    // 32-bit byte offsets from the (scalar) matrix bases keep the address registers few
    unsigned xo[4], wo[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const int row = min(m0 + wave * 32 + p * 8 + lrow, a.M - 1);
        const int n = min(n0 + wave * 32 + p * 8 + lrow, n_end - 1);
        xo[p] = ((unsigned)row * (unsigned)a.ldx + lch * 8) * 2u;
        wo[p] = ((unsigned)n * (unsigned)a.ldw + lch * 8) * 2u;
    }
    // waves 0 .. NZ/8 - 1 copy 8 rows of Z each (all ones there, otherwise no lane is active)
    const int zlanes = (wave - (has_z ? NZ / 8 : 0)) >> 31;
    const unsigned zo = ((unsigned)(wave * 8 + lrow) * (unsigned)a.ldz + lch * 8) * 2u;
    const char *Xb = (const char *)a.X, *Wb = (const char *)a.W;
    const char *Zb = has_z ? (const char *)a.zmat[seg] : (const char *)a.X;
    const int wofs = wave * 32 * ROWB;

    // wave tile 128 x 64 = 8 x 4 MFMA 16x16x32 tiles; lane holds column r16, rows 4 kg + e of each
    f32x4 acc[8][4];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.0f;
    // rank-space activations of this wave's 32-row slice (rows wm*128 + wn*32 ..): 2 x NZT tiles
    f32x4 zacc[2][NZT];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int q = 0; q < NZT; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) zacc[h][q][e] = 0.0f;

    // Row tile i of the wave is tile (i + 2 wn) mod 8 of its 128 rows: the two whose rank-space activations it forms come
    // first, so that their products use the fragments that are there.
    const int rot = 2 * wn;
    // lane offsets of k-steps 0 and 1; the tile's place is a scalar
    const unsigned v0 = r16 * ROWB + ((kg ^ (r16 & 7)) << 4), v1 = v0 ^ 64;
    const unsigned sa = wm * 128 * ROWB, sb = XB + wn * 64 * ROWB;
    const unsigned l0 = lds_addr(st0), l1 = lds_addr(st1);
    const int nk = a.K / BK;
    constexpr int NCP = 9, TURN = 8 - AHEAD;             // copies of a wave per slab; the row tile that reads the next step's first
    bf16x8 fa[AHEAD], fb[2][4], fz[NZT];
    auto rd = [&](unsigned v, unsigned s) { return *(const __attribute__((address_space(3))) bf16x8 *)(v + s); };
    auto copy1 = [&](unsigned st, int kt, int q) {
        const size_t kb = (size_t)min(kt, nk - 1) * (BK * 2);    // (behind the last slab: it once more, unread)
        if (q < 4) glds_soff(Xb + kb, xo[q & 3], st + wofs + (q & 3) * 1024);
        else if (q < 8) glds_soff(Wb + kb, wo[q & 3], st + XB + wofs + (q & 3) * 1024);
        else glds_soff_if(Zb + kb, zo, st + XB + WB + wave * 1024, zlanes);
    };
    // row tile i on the column fragments cb, then the reads that have become free: of row tile i + AHEAD, whose step has its
    // slab at S and lane offset v, and from TURN on of the next step's columns and rank-space columns
#define GEMM_ROW(i, cb, S, v)                                                                          \
    {                                                                                                  \
        _Pragma("unroll") for (int j = 0; j < 4; ++j)                                                  \
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[(i) % AHEAD], fb[cb][j], acc[i][j], 0, 0, 0); \
        if ((i) < 2 && has_z) {                                                                        \
            _Pragma("unroll") for (int q = 0; q < NZT; ++q)                                            \
                zacc[(i) & 1][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[(i) % AHEAD], fz[q], zacc[(i) & 1][q], 0, 0, 0); \
        }                                                                                              \
        fa[(i) % AHEAD] = rd(v, (S) + sa + (((i) + AHEAD + rot) & 7) * (16 * ROWB));                   \
        if ((i) >= TURN && (i) < TURN + 4) fb[1 - (cb)][((i) - TURN) & 3] = rd(v, (S) + sb + (((i) - TURN) & 3) * (16 * ROWB)); \
        if ((i) >= 4 && (i) - 4 < NZT) fz[((i) & 3) % NZT] = rd(v, (S) + XB + WB + ((i) & 3) * (16 * ROWB)); \
    }
    // one slab; behind the barrier its buffer takes the slab after the next, which has until the next slab's barrier to land.
    // (The scalars are made opaque: else the compiler keeps the sum of each with each lane offset.)
#define GEMM_SLAB(lc, ln)                                                                              \
    {                                                                                                  \
        unsigned sc = lc, sn = ln;                                                                     \
        asm volatile("" : "+s"(sc));                                                                   \
        _Pragma("unroll") for (int i = 0; i < 8; ++i) {                                                \
            if (i < TURN) GEMM_ROW(i, 0, sc, v0) else GEMM_ROW(i, 0, sc, v1)                           \
            __builtin_amdgcn_sched_barrier(0);                                                         \
        }                                                                                              \
        _Pragma("unroll") for (int i = 0; i < TURN; ++i) {                                             \
            GEMM_ROW(i, 1, sc, v1)                                                                     \
            __builtin_amdgcn_sched_barrier(0);                                                         \
        }                                                                                              \
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");                                    \
        __syncthreads();                                                                               \
        asm volatile("" : "+s"(sn));                                                                   \
        _Pragma("unroll") for (int i = TURN; i < 8; ++i) {                                             \
            GEMM_ROW(i, 1, sn, v0)                                                                     \
            _Pragma("unroll") for (int q = 0; q < NCP; ++q)                                            \
                if (q >= (i - TURN) * NCP / AHEAD && q < (i - TURN + 1) * NCP / AHEAD) copy1(lc, kt + 2, q); \
            __builtin_amdgcn_sched_barrier(0);                                                         \
        }                                                                                              \
    }
#pragma unroll
    for (int q = 0; q < NCP; ++q) copy1(l0, 0, q);
#pragma unroll
    for (int q = 0; q < NCP; ++q) copy1(l1, 1, q);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NCP) : "memory");
    __syncthreads();
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) fa[i] = rd(v0, l0 + sa + ((i + rot) & 7) * (16 * ROWB));
#pragma unroll
    for (int j = 0; j < 4; ++j) fb[0][j] = rd(v0, l0 + sb + j * (16 * ROWB));
#pragma unroll
    for (int q = 0; q < NZT; ++q) fz[q] = rd(v0, l0 + XB + WB + q * (16 * ROWB));
    for (int kt = 0;;) {
        GEMM_SLAB(l0, l1)
        if (++kt >= nk) break;
        GEMM_SLAB(l1, l0)
        if (++kt >= nk) break;
    }
#undef GEMM_ROW
#undef GEMM_SLAB
    // the copies and reads behind the last slab are done before its buffers are used for anything else
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();

    // ---- low-rank tail: acc += (zscale * z)[256,K2P] . T[n,K2P]^T -----------------------------
    if (has_z) {
        constexpr int ZP = K2P + 8;                      // LDS pitch of the z tile, in elements
        bf16 *zs = (bf16 *)st0;                          // the K loop is over: reuse stage 0
        const bf16 *tm_ = a.tmat[seg];
        // up-projection operands (L2 hits): column n0 + wn*64 + j*16 + r16, k = ks*32 + kg*8 ..
        bf16x8 tb[K2P / 32][4];
#pragma unroll
        for (int ks = 0; ks < K2P / 32; ++ks)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int n = min(n0 + wn * 64 + j * 16 + r16, n_end - 1) - seg * a.seg_n;
                tb[ks][j] = *(const bf16x8 *)(tm_ + (size_t)n * a.ldt + ks * 32 + kg * 8);
            }
        // scaled, rounded z of this wave's 32 rows; columns NZ..K2P of the tile are zero
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int q = 0; q < K2P / 16; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int row = wm * 128 + wn * 32 + h * 16 + 4 * kg + e;
                    zs[row * ZP + q * 16 + r16] = f2bf(q < NZT ? zacc[h][q < NZT ? q : 0][e] * a.zscale : 0.f);
                }
        __syncthreads();
        if (a.zspill[seg] != nullptr && tns == 0) {
            const int cpr = a.K2 >> 3;                   // 16-byte chunks per row
            for (int c = tid; c < BM * cpr; c += NTHR) {
                int row = c / cpr, cc = c - row * cpr;
                if (m0 + row < a.M)
                    *(uint4 *)(a.zspill[seg] + (size_t)(m0 + row) * a.K2 + cc * 8) =
                        *(const uint4 *)(zs + row * ZP + cc * 8);
            }
        }
#pragma unroll
        for (int ks = 0; ks < K2P / 32; ++ks) {
#pragma unroll
            for (int ih = 0; ih < 2; ++ih) {
                bf16x8 af[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    af[i] = *(const bf16x8 *)(zs + (wm * 128 + ((ih * 4 + i + rot) & 7) * 16 + r16) * ZP + ks * 32 + kg * 8);
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        acc[ih * 4 + i][j] =
                            __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], tb[ks][j], acc[ih * 4 + i][j], 0, 0, 0);
            }
        }
    }

    // ---- epilogue.  A lane holds column r16 of each 16x16 tile, rows 4 kg + e: each wave transposes
    //      its tiles through a private LDS strip (32 rows x 64 columns fp32) so that global memory
    //      sees 16-byte accesses, 8 rows x 128..256 contiguous bytes per instruction.  Only the
    //      owning wave touches its strip, so no block barrier is needed.
    constexpr int EP = 68;                               // strip pitch in floats (bank-conflict free)
    if (has_z) __syncthreads();                          // the z tile in st0 has been consumed
    float *stg = (float *)((wave < 4 ? st0 : st1) + (wave & 3) * (32 * EP * 4));
    const int er = lane >> 3, ec = (lane & 7) * 8;
    const int gcol = n0 + wn * 64 + ec;
    float bias8[8];
    {
        bf16x8 b8;
#pragma unroll
        for (int i = 0; i < 8; ++i) b8[i] = f2bf(0.f);
        if (a.bias && gcol < n_end) b8 = *(const bf16x8 *)(a.bias + gcol);
#pragma unroll
        for (int i = 0; i < 8; ++i) bias8[i] = bf2f(b8[i]);
    }
    AuxRow aux[2][4];
    const int row_base = m0 + wm * 128 + er;
    auto strip = [&](int i) { return ((2 * i + rot) & 7) * 16; };      // first row of strip i: its row tiles 2 i and 2 i + 1
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const int row = row_base + strip(0) + it * 8;
        load_aux<EPI>(a, row, gcol, row < a.M && gcol < n_end, aux[0][it]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (i + 1 < 4) {
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int row = row_base + strip(i + 1) + it * 8;
                load_aux<EPI>(a, row, gcol, row < a.M && gcol < n_end, aux[(i + 1) & 1][it]);
            }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    stg[(h * 16 + 4 * kg + e) * EP + j * 16 + r16] = acc[2 * i + h][j][e];
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int rl = it * 8 + er;
            const float4 p0 = *(const float4 *)(stg + rl * EP + ec);
            const float4 p1 = *(const float4 *)(stg + rl * EP + ec + 4);
            float v[8] = {p0.x + bias8[0], p0.y + bias8[1], p0.z + bias8[2], p0.w + bias8[3],
                          p1.x + bias8[4], p1.y + bias8[5], p1.z + bias8[6], p1.w + bias8[7]};
            const int row = m0 + wm * 128 + strip(i) + rl;
            if (row < a.M && gcol < n_end) store_row8<EPI>(a, row, gcol, v, aux[i & 1][it]);
        }
    }
}

// ---------------------------------------------------------------------------------------------------
// Products without a rank-space branch (NZ = 0): 4 waves (2 x 2), wave tile 128 x 128 = 8 x 8 MFMA tiles.
//
// One wave per SIMD owns all 512 registers of a lane: the 256 accumulators are pinned to the accumulation
// half of the file by writing the MFMA as inline assembly with "a" operands (left to itself the compiler
// shuffles them through the other half around every MFMA), and the other half holds the operand
// fragments one k-step ahead.  Per 32-deep k-step a wave reads 8 + 8 fragments for 64 MFMAs, a third less
// LDS traffic per MFMA than the 8 + 4 for 32 of the 8-wave kernel.  LDS is a ring of five 32 KB half
// stages: three for the X tile and two for the W tile, so the X copies run two slabs ahead and the W
// copies one.  With a single wave per SIMD whatever the wave issues in a clump is time the matrix pipe idles: the 32 fragment
// reads and 16 copies of a slab go one by one behind MFMAs of their own, and the fragments of a k-step have a register set of
// their own, so that the last read is 32 MFMAs old at the barrier.  Against three reads and two copies behind each row of 8
// MFMAs: 3300 -> 2920 shader cycles a slab of 2048 MFMA cycles, of which the chip, at its power limit, takes back a part
// as clock: 2.10 -> 1.94 GHz in launches with copies between them, 2.15 -> 2.06 in rounds of 18 blocks of width 1024.  us at 32768 x 4096 -> 1024 200.3 -> 195.0, 32768 x 1024 -> 4096 235.4 -> 231.2;
// a round of 18 blocks of width 1024 at 32768 tokens 39.47 -> 38.27 ms, the loss head at 32768 x 1024 -> 50257 4.27 -> 3.99 ms.
// The grid is one block per CU and a block walks its tiles itself, so that the first copies of the next
// tile are in flight under the epilogue of the current one.
// The MFMA hazards the compiler can no longer see (inline assembly) are covered by construction: every MFMA
// accumulates in place (destination = addend, the back-to-back form the hardware interlocks) and the same
// accumulator comes round again only 64 MFMAs later; fragments come from LDS reads the compiler still
// tracks; and the only way out of the loop leads through 24 wait states (see the end of the loop body).
// tests/test_kernel_isa.py verifies all three in the compiled code of every instantiation.
// ---------------------------------------------------------------------------------------------------
constexpr int NTHR4 = 256, HB = 32768;       // HB: one operand's k-slab (256 rows x 128 B)

// NI = 16-row MFMA tiles per wave along M: 8 (tile 256 x 256, wave tile 128 x 128) or 4 (tile 128 x 256, wave
// tile 64 x 128) for launches that have fewer 256-row tiles than the chip has CUs.
// COUNTED: the number of rows, and (EPI_PARTIAL) over how many blocks a tile's contraction is shared, are read from
// device memory (a.rows); share s of a tile leaves its fp32 sums in the s-th [rows, ldo] block of out0.
// TAIL: a rank-space branch whose activations are there (a.zspill): its one or two k-steps of 32 follow the main loop, on operands
// read straight into fragments while the last two slabs are multiplied.
template <int EPI, int NI, bool COUNTED, bool TAIL = false>
__device__ __forceinline__ void gemm4_body(GemmArgs a)
{
    static_assert(!TAIL || NI == 8, "the tail is for 256 x 256 tiles");
    constexpr int BM4 = 32 * NI;                         // rows of a block tile
    constexpr bool SHARED = EPI == EPI_PARTIAL;
    // Spacing, in MFMAs of a k-step, of the fragment reads and of the copies, and how many of the X copies of a slab go out
    // beside the W copies before it (the others one k-step later).  (CP, NX1) = (5, 4), (6, 2), (7, 1) are within 0.5 % of each
    // other on whole rounds; all X copies behind the W copies, (4, 8), are 1 to 4 % slower.
    constexpr int RD = 2, CP = NI == 8 ? 6 : 3, NX1 = 2;
    if constexpr (COUNTED) a.M = a.rows->rows;
    const int shares = SHARED ? a.rows->shares : 1;
    __shared__ __attribute__((aligned(1024))) unsigned char ring[5 * HB];   // X: 0, HB, 2HB;  W: 3HB, 4HB

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int r16 = lane & 15, kg = lane >> 4;

    // Tiles of this block.  The grid is at most one block per CU and a block walks its share of the tiles
    // itself: blocks are handed to the 8 XCDs round-robin, XCD x owns the logical tiles
    // [x per_xcd, (x + 1) per_xcd) and its blocks take them in turn, so that the tiles in flight on an XCD are
    // consecutive ones of the same panel walk as in the 8-wave kernel (a 4 x 8 patch per XCD's L2).  Owning
    // the CU for the whole launch is what lets the first copies of the next tile run under the epilogue of
    // the current one (2.5 us per tile otherwise, a tenth of a K = 1024 tile).
    const int tiles_n_seg = (a.seg_n + BN - 1) / BN;
    const int tiles_n = tiles_n_seg * a.nseg;
    const int tiles_m = (a.M + BM4 - 1) / BM4;
    const int nt = tiles_m * tiles_n, nb = SHARED ? nt * shares : nt;    // shares of one tile are nt apart
    const int per_xcd = (nb + 7) >> 3;
    const int slots = gridDim.x >> 3;
    const int t_end = min(((int)(blockIdx.x & 7) + 1) * per_xcd, nb);
    int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (logical >= t_end) return;
    // measurement hook: block 0 owns its CU from the first tile to the last, so the shader-clock and the
    // 100 MHz reference counter at its start and end give the clock the chip held under this launch
    if (a.clk != nullptr && blockIdx.x == 0 && tid == 0) {
        a.clk[0] = __builtin_amdgcn_s_memtime();
        a.clk[1] = __builtin_amdgcn_s_memrealtime();
    }
    const int lrow = lane >> 3, lch = (lane & 7) ^ (lane >> 3);
    const char *Xb = (const char *)a.X, *Wb = (const char *)a.W;
    const unsigned ringa_x = lds_addr(ring) + wave * (8 * NI) * ROWB, ringa_w = lds_addr(ring) + wave * 64 * ROWB;
    const int a_row = (wm * (16 * NI) + r16) * ROWB, b_row = (wn * 128 + r16) * ROWB;
    const int sw = r16 & 7;
    int nk = a.K / BK, klast = (nk - 1) * BK;
    int k1 = min(BK, klast), k2 = min(2 * BK, klast);
    const int nk_all = nk;
    // the epilogue's staging strips live in the third X buffer, the one the next tile's early copies leave alone
    float *stg = (float *)(ring + 2 * HB + wave * (16 * EP4 * 4));

    int m0, n0, n_end, share = 0, zseg = 0;
    float *const part0 = (float *)a.out0;
    unsigned xo[8], wo[8];
    // tile `t` of the panel walk: its origin, and this wave's copy offsets (every wave copies a quarter of the
    // rows of each operand tile per slab -- 8 NI of X, 64 of W --, 8 rows = 1 KB per instruction; lane l fills
    // 16-byte slot l: row l>>3, physical k-chunk l&7 holding logical chunk (l&7) ^ (l>>3))
#define G4_TILE(id)                                                                                    \
    {                                                                                                  \
        constexpr int PANEL = 4;                                                                       \
        int t = (id);                                                                                  \
        unsigned kb = 0;                                 /* byte offset of the share's first slab */   \
        if constexpr (SHARED) {                                                                        \
            share = t / nt;                                                                            \
            t -= share * nt;                                                                           \
            const int ks = (int)((long)share * nk_all / shares);                                       \
            nk = (int)((long)(share + 1) * nk_all / shares) - ks;                                      \
            klast = (nk - 1) * BK;                                                                     \
            k1 = min(BK, klast);                                                                       \
            k2 = min(2 * BK, klast);                                                                   \
            kb = (unsigned)ks * ROWB;                                                                  \
        }                                                                                              \
        const int pidx = t / (PANEL * tiles_n), prem = t - pidx * (PANEL * tiles_n);                   \
        const int prow = min(PANEL, tiles_m - pidx * PANEL);                                           \
        const int tn = prem / prow, tm = pidx * PANEL + prem - tn * prow;                              \
        const int seg = tn / tiles_n_seg, tns = tn % tiles_n_seg;                                      \
        zseg = seg;                                                                                    \
        n0 = seg * a.seg_n + tns * BN;                                                                 \
        n_end = (seg + 1) * a.seg_n;                                                                   \
        m0 = tm * BM4;                                                                                 \
        _Pragma("unroll") for (int p = 0; p < 8; ++p) {                                                \
            const int row = min(m0 + wave * (8 * NI) + (p % NI) * 8 + lrow, a.M - 1);                  \
            const int n = min(n0 + wave * 64 + p * 8 + lrow, n_end - 1);                               \
            xo[p] = ((unsigned)row * (unsigned)a.ldx + lch * 8) * 2u + kb;                             \
            wo[p] = ((unsigned)n * (unsigned)a.ldw + lch * 8) * 2u + kb;                               \
        }                                                                                              \
    }
#define G4_COPYX(k0, ldsb, p) glds_soff(Xb + (size_t)(k0) * 2, xo[p], ringa_x + (ldsb) + (p) * 1024);
#define G4_COPYW(k0, ldsb, p) glds_soff(Wb + (size_t)(k0) * 2, wo[p], ringa_w + (ldsb) + (p) * 1024);
    // the first copies of a tile.  Copies past the last slab repeat it (in bounds, never read), so the in-order
    // copy counter can be waited on with the same constants from the first slab to the last.
#define G4_HEAD4                                                                                       \
    {                                                                                                  \
        _Pragma("unroll") for (int p = 0; p < 8; ++p) G4_COPYW(0, 3 * HB, p)                           \
        _Pragma("unroll") for (int p = 0; p < NI; ++p) G4_COPYX(0, 0, p)                               \
        _Pragma("unroll") for (int p = 0; p < 8; ++p) G4_COPYW(k1, 4 * HB, p)                          \
        _Pragma("unroll") for (int p = 0; p < NI; ++p) G4_COPYX(k1, HB, p)                             \
    }
#define G4_HEAD5 { _Pragma("unroll") for (int p = 0; p < NX1; ++p) G4_COPYX(k2, 2 * HB, p) }
#define G4_LDA(nb_, i, xs, k2_) fa[nb_][i] = *(const bf16x8 *)(ring + (xs) + a_row + (i) * 16 * ROWB + ((((k2_) * 4 + kg) ^ sw) << 4));
#define G4_LDB(nb_, j, ws, k2_) fb[nb_][j] = *(const bf16x8 *)(ring + (ws) + b_row + (j) * 16 * ROWB + ((((k2_) * 4 + kg) ^ sw) << 4));
    // One k-step: 8 NI MFMAs on fragment set cb.  Behind an MFMA goes at most one fragment read of the next k-step (set nb_)
    // or one copy, so that the wave has its next MFMA ready before the matrix pipe has finished this one.
#define G4_STEP(cb, nb_, xs, ws, k2_, COPIES)                                                          \
    {                                                                                                  \
        _Pragma("unroll") for (int i = 0; i < NI; ++i) _Pragma("unroll") for (int j = 0; j < 8; ++j) { \
            asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[i][j]) : "v"(fa[cb][i]), "v"(fb[cb][j])); \
            const int s_ = 8 * i + j;                                                                  \
            if (s_ % RD == 0 && s_ / RD < 8) G4_LDB(nb_, (s_ / RD) & 7, ws, k2_)                       \
            if (s_ % RD == 0 && s_ / RD >= 8 && s_ / RD < 8 + NI) G4_LDA(nb_, (s_ / RD - 8) & (NI - 1), xs, k2_) \
            COPIES(s_)                                                                                 \
            __builtin_amdgcn_sched_barrier(0);                                                         \
        }                                                                                              \
    }
    // k-step 0 of slab kt: the rest of X of slab kt + 2; k-step 1, behind the barrier that frees the slab's buffers: W of slab
    // kt + 2, then the first NX1 copies of X of slab kt + 3
#define G4_COPIES0(s_) { if ((s_) % CP == 1 && (s_) / CP < NI - NX1) glds_soff(x2, xo[((s_) / CP + NX1) & (NI - 1)], lx2 + (((s_) / CP + NX1) & (NI - 1)) * 1024); }
#define G4_COPIES1(s_) { if ((s_) % CP == 1 && (s_) / CP < 8) glds_soff(w2, wo[((s_) / CP) & 7], lw + (((s_) / CP) & 7) * 1024); \
                         if ((s_) % CP == 1 && (s_) / CP >= 8 && (s_) / CP < 8 + NX1) glds_soff(x3, xo[((s_) / CP - 8) & (NI - 1)], lx + (((s_) / CP - 8) & (NI - 1)) * 1024); }

    G4_TILE(logical)
    G4_HEAD4                                             // copy queue: W0 X0 W1 X1 ...
    for (;;) {
        G4_HEAD5                                         // ... X2
        // Everything but X2 (NX1 copies) has landed: W0, X0 (and W1, X1, requested just before them or, from the second
        // tile on, before the previous tile's epilogue).  The counter is in order, so this also waits for
        // the previous tile's stores to be acknowledged, which they are within 0.2 us of being issued.
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NX1) : "memory");
        __syncthreads();
        f32x4 acc[NI][8];
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.0f;
        bf16x8 fa[2][NI], fb[2][8];
        int xcur = 0, wcur = 3 * HB;                     // buffers of the slab being computed
#pragma unroll
        for (int i = 0; i < 8; ++i) { G4_LDB(0, i, 3 * HB, 0) if (i < NI) { G4_LDA(0, i & (NI - 1), 0, 0) } }
        // rows of z and of the up-projection: k-step ks of the tail
        bf16x8 za[TAIL ? 8 : 1], tb[TAIL ? 8 : 1];
        auto tail_operands = [&](int ks) {
            const char *zp = (const char *)a.zspill[zseg], *tp = (const char *)a.tmat[zseg];
            int lane_ = lane;
            asm volatile("" : "+v"(lane_));              // (else 16 addresses are held in registers through the loop)
            const int r_ = lane_ & 15, k_ = ks * 32 + (lane_ >> 4) * 8;
            const bool zok = k_ < a.K2;                  // columns past K2 count as zero
#pragma unroll
            for (int i = 0; i < (TAIL ? 8 : 0); ++i) {
                const int row = min(m0 + wm * 128 + i * 16 + r_, a.M - 1), n = min(n0 + wn * 128 + i * 16 + r_, n_end - 1) - zseg * a.seg_n;
                za[i] = *(const bf16x8 *)(zp + ((unsigned)row * (unsigned)a.K2 + (zok ? k_ : 0)) * 2u);
                tb[i] = *(const bf16x8 *)(tp + ((unsigned)n * (unsigned)a.ldt + k_) * 2u);
            }
        };
        const bool has_z = TAIL && a.zmat[zseg] != nullptr;
        const int kt_tail = max(nk - 2, 0);
        for (int kt = 0;; ++kt) {                        // nk >= 1 (checked by the launcher)
            if (TAIL) {
                if (has_z && kt == kt_tail) tail_operands(0);
            }
            const int xnxt = xcur == 2 * HB ? 0 : xcur + HB, wnxt = wcur ^ (3 * HB ^ 4 * HB);
            const int c2 = min((kt + 2) * BK, klast), c3 = min((kt + 3) * BK, klast);
            const char *x2 = Xb + (size_t)c2 * 2, *w2 = Wb + (size_t)c2 * 2, *x3 = Xb + (size_t)c3 * 2;
            const unsigned lx2 = ringa_x + (xcur == 0 ? 2 * HB : xcur - HB), lx = ringa_x + xcur, lw = ringa_w + wcur;
            G4_STEP(0, 1, xcur, wcur, 1, G4_COPIES0)     // MFMAs (slab kt, step 0); fetch (kt, step 1)
            // slab kt+1 has landed (X of kt+2 may still be in flight); nobody reads slab kt's buffers any more
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(NI) : "memory");
            __syncthreads();
            G4_STEP(1, 0, xnxt, wnxt, 0, G4_COPIES1)
            xcur = xnxt; wcur = wnxt;
            // The compiler takes an accumulator for finished where its MFMA is issued, and it moves
            // accumulators between registers right where the loop ends.  The only way out of the loop is
            // through these wait states, which let the last MFMAs retire first (a 16-pass result needs 19;
            // tests/test_kernel_isa.py follows every path from the last MFMA in the compiled code).
            if (kt + 1 >= nk) {
                asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");
                break;
            }
        }
        // all copies have landed and every wave is out of the loop before the ring is reused
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __syncthreads();
        if (TAIL) {
            if (has_z) {
                for (int ks = 0;;) {
                    if (ks * 32 + kg * 8 >= a.K2) {
#pragma unroll
                        for (int i = 0; i < (TAIL ? 8 : 0); ++i)
#pragma unroll
                            for (int e = 0; e < 8; ++e) za[i][e] = f2bf(0.f);
                    }
                    // a vector write, then an MFMA the compiler does not see: 2 wait states (tests/test_kernel_isa.py); the barriers,
                    // because nothing else ties the zeros above to this side of them
                    __builtin_amdgcn_sched_barrier(0);
                    asm volatile("s_nop 1" ::: "memory");
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int i = 0; i < NI; ++i)
#pragma unroll
                        for (int j = 0; j < 8; ++j)
                            asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[i][j]) : "v"(za[TAIL ? i : 0]), "v"(tb[TAIL ? j : 0]));
                    if (++ks * 32 >= a.K2) break;
                    tail_operands(ks);
                }
                asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");          // (as behind the main loop)
            }
        }
        // the next tile's first four half stages are requested now and arrive under this tile's epilogue
        const int em0 = m0, en0 = n0, en_end = n_end;
        if constexpr (SHARED) a.out0 = part0 + (size_t)share * a.M * a.ldo;
        const int next = logical + slots;
        if (next < t_end) {
            G4_TILE(next)
            G4_HEAD4
        }
        if (em0 + BM4 <= a.M && en0 + BN <= en_end) epilogue4<EPI, true, NI>(a, acc, stg, em0, en0, en_end, wm, wn, lane);
        else epilogue4<EPI, false, NI>(a, acc, stg, em0, en0, en_end, wm, wn, lane);
        if (next >= t_end) break;
        logical = next;
        // the staging reads are done before the copy into the buffer they used is requested
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __syncthreads();
    }
    if (a.clk != nullptr && blockIdx.x == 0 && tid == 0) {
        a.clk[2] = __builtin_amdgcn_s_memtime();
        a.clk[3] = __builtin_amdgcn_s_memrealtime();
    }
#undef G4_TILE
#undef G4_HEAD4
#undef G4_HEAD5
#undef G4_COPYX
#undef G4_COPYW
#undef G4_LDA
#undef G4_LDB
#undef G4_STEP
#undef G4_COPIES0
#undef G4_COPIES1
}

template <int EPI, int NI>
__global__ __launch_bounds__(NTHR4) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_kernel4(GemmArgs a)
{
    gemm4_body<EPI, NI, false>(a);
}
template <int EPI, int NI>
__global__ __launch_bounds__(NTHR4) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_counted4(GemmArgs a)
{
    gemm4_body<EPI, NI, true>(a);
}

// The 4-wave kernel for a product whose rank-space activations are there (rank_grad.hip forms them in the pass that forms dB):
// bound as gemm_kernel4; there is no room in LDS to form them in its loop, and the loop that forms them (gemm_kernel) reads
// half as much again from LDS.  The tail adds 32 or 64 to the contraction, its operands come under way two slabs before the end.
// us at 32768 rows, gemm_kernel and this: 3072 -> 1024 with 32 columns 178, 150; 4096 -> 1024 229, 193; 1024 -> 4096 with the
// saved GELU' 331, 273 (no branch at all: 194 and 273).  It has all 512 registers and spills three of the epilogue's, read back once a tile.
template <int EPI>
__global__ __launch_bounds__(NTHR4) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_tail4(GemmArgs a)
{
    gemm4_body<EPI, 8, false, true>(a);
}

template <int EPI>
int launch_tail4(const GemmArgs &a, hipStream_t st)
{
    const int nb = ((a.M + 255) / 256) * ((a.seg_n + BN - 1) / BN) * a.nseg;
    hipLaunchKernelGGL(gemm_tail4<EPI>, dim3(std::min(((nb + 7) / 8) * 8, 256)), dim3(NTHR4), 0, st, a);
    SL_CHECK_LAUNCH("gemm");
    return 0;
}

template <int EPI>
int launch_t4(const GemmArgs &a, int rows, hipStream_t st)
{
    const int nb = ((a.M + rows - 1) / rows) * ((a.seg_n + BN - 1) / BN) * a.nseg;
    const int grid = std::min(((nb + 7) / 8) * 8, 256);    // one block per CU, each walks its tiles
    if (rows == 128) hipLaunchKernelGGL((gemm_kernel4<EPI, 4>), dim3(grid), dim3(NTHR4), 0, st, a);
    else hipLaunchKernelGGL((gemm_kernel4<EPI, 8>), dim3(grid), dim3(NTHR4), 0, st, a);
    SL_CHECK_LAUNCH("gemm");
    return 0;
}

template <int EPI, int NZ>
int launch_t(const GemmArgs &a, hipStream_t st)
{
    const int tiles_n = ((a.seg_n + BN - 1) / BN) * a.nseg;
    const int tiles_m = (a.M + BM - 1) / BM;
    const int nb = tiles_m * tiles_n;
    const int grid = ((nb + 7) / 8) * 8;
    hipLaunchKernelGGL((gemm_kernel<EPI, NZ>), dim3(grid), dim3(NTHR), 0, st, a);
    SL_CHECK_LAUNCH("gemm");
    return 0;
}

template <int EPI>
int launch_e(const GemmArgs &a, int nz, int rows, hipStream_t st)
{
    if constexpr (EPI == EPI_STORE || EPI == EPI_DGELU) {
        if (nz > 0 && a.z_ready && rows == 256) return launch_tail4<EPI>(a, st);
    }
    switch (nz) {
    case 0: return launch_t4<EPI>(a, rows, st);          // no rank-space branch: the 4-wave kernel
    case 16: return launch_t<EPI, 16>(a, st);
    case 32: return launch_t<EPI, 32>(a, st);
    case 48: return launch_t<EPI, 48>(a, st);
    }
    return SL_EINVAL;
}

}  // namespace

static int launch_gemm_inner(const GemmArgs &a, int epi, int nz, hipStream_t st);
static int launch_gemm_counted(const GemmArgs &a, int epi, hipStream_t st);

int launch_gemm(const GemmArgs &a, int epi, int nz, hipStream_t st)
{
    const bool rec = prof_begin(PK_GEMM, st, a.rows ? &a.rows->rows : nullptr);
    GemmArgs b = a;
    b.clk = prof_clock_words(rec);
    const int rc = epi == EPI_PARTIAL || (a.rows && plan_gemm_counted(a.M, a.N, a.K).tm == 0)
                       ? launch_gemm_counted(b, epi, st)
                       : launch_gemm_inner(b, epi, nz, st);
    // algorithmic work of this launch: the frozen product only (the rank-r branch adds < 1 % and is left
    // out, which understates the achieved rate slightly)
    const double row = 2.0 * (double)a.N * a.K;
    prof_end(rec, PK_GEMM, a.rows ? 0.0 : row * a.M, st, a.rows ? row : 0.0);
    return rc;
}

static int launch_gemm_inner(const GemmArgs &a, int epi, int nz, hipStream_t st)
{
    if (a.M <= 0 || a.N <= 0 || a.K <= 0 || (a.K % BK) != 0 || a.nseg < 1 || a.nseg > 3 ||
        a.nseg * a.seg_n != a.N || (a.ldx % 8) || (a.ldw % 8) || (a.seg_n % 8) || (a.ldo % 8))
        return SL_EINVAL;
    if (a.mx) return launch_gemm_mx_stack(a, epi, nz, st);
    // the copies address both operands with 32-bit byte offsets from their bases
    if ((unsigned long long)a.M * a.ldx * 2ull >= (1ull << 32) || (unsigned long long)a.N * a.ldw * 2ull >= (1ull << 32))
        return SL_EINVAL;
    if (nz > 0 && (a.K2 != nz || (a.ldt % 8) || a.ldt < (nz + 31) / 32 * 32 || (a.ldz % 8))) return SL_EINVAL;
    if (epi == EPI_STORE_DELTA && (nz != 0 || !a.dl_o || !a.dl_lo || !a.dl_out || !a.out0 || (a.N % 64) || a.nseg != 1))
        return SL_EINVAL;                                // no rank-space branch, whole heads of 64 columns
    const TilePlan plan = a.rows ? plan_gemm_counted(a.M, a.N, a.K)
                                 : plan_gemm_tile(a.M, a.seg_n, a.nseg, a.K, epi, nz, a.split_part != nullptr && a.split_cnt != nullptr, true);
    if (plan.tn < 256) return launch_gemm_tile(a, epi, nz, plan, st);
    switch (epi) {
    case EPI_STORE: return launch_e<EPI_STORE>(a, nz, plan.tm, st);
    case EPI_RESID: return launch_e<EPI_RESID>(a, nz, plan.tm, st);
    case EPI_GELU: return launch_e<EPI_GELU>(a, nz, plan.tm, st);
    case EPI_DGELU: return launch_e<EPI_DGELU>(a, nz, plan.tm, st);
    case EPI_STORE_DELTA: return launch_t4<EPI_STORE_DELTA>(a, plan.tm, st);
    }
    return SL_EINVAL;
}

// A product over the rows that a kernel before it counted (a.rows; a.M is their upper bound), without rank-space branch.
// EPI_STORE or EPI_PARTIAL.
static int launch_gemm_counted(const GemmArgs &a, int epi, hipStream_t st)
{
    if (a.M <= 0 || a.N <= 0 || a.K <= 0 || (a.K % BK) != 0 || a.nseg != 1 || a.seg_n != a.N || (a.ldx % 8) ||
        (a.ldw % 8) || (a.N % 8) || (a.ldo % 8) || !a.rows || !a.out0)
        return SL_EINVAL;
    if ((unsigned long long)a.M * a.ldx * 2ull >= (1ull << 32) || (unsigned long long)a.N * a.ldw * 2ull >= (1ull << 32))
        return SL_EINVAL;
    const int bm = gemm_counted_rows(a.M);
    const int tiles = ((a.M + bm - 1) / bm) * ((a.N + BN - 1) / BN);
    // shares are chosen where the rows are counted, so that launch always has a block for every CU
    const dim3 grid(epi == EPI_PARTIAL ? 256 : std::min((tiles + 7) / 8 * 8, 256)), block(NTHR4);
    // (up to 128 rows the plain store runs on kernels that compute all of them: plan_gemm_counted)
    if (epi == EPI_STORE && bm == 256) hipLaunchKernelGGL((gemm_counted4<EPI_STORE, 8>), grid, block, 0, st, a);
    else if (epi == EPI_PARTIAL && bm == 256) hipLaunchKernelGGL((gemm_counted4<EPI_PARTIAL, 8>), grid, block, 0, st, a);
    else if (epi == EPI_PARTIAL) hipLaunchKernelGGL((gemm_counted4<EPI_PARTIAL, 4>), grid, block, 0, st, a);
    else return SL_EINVAL;
    SL_CHECK_LAUNCH("gemm counted");
    return 0;
}
