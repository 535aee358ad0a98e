// Body of the bf16 GEMM kernels on tiles smaller than 256 x 256 (gfx950): gemm_tile.hip instantiates it with 4 waves a block,
// gemm_wide.hip with 8.
//
//   out[M,N] = epilogue( X[M,K] . W[N,K]^T  +  zscale * (X . Z^T)[M,K2] . T[N,K2]^T )       (see gemm.hip)
//
// Every output element is one accumulation over k in increasing order, as in gemm.hip, bit for bit: a sequence's results do
// not depend on which of the kernels its batch ran on.
//
// What bounds these launches is the LDS: with the operand fragments read as 16-byte pieces and the tiles written by the
// asynchronous copies, a slab of 64 takes 16 waves (MI + NI) + (TM + TN) cycles of its 128 bytes per cycle (128 x 128 with 8
// waves: 1024 cycles for 512 of matrix time; measured 0.45 us a slab).  So the loop is arranged around that pipe: fragments
// are read one k-step ahead, each between two MFMAs, copies likewise, and nothing in the loop branches (a branch per copy of Z
// cost 0.1 us a slab).  T = 4096, 4096 -> 1024 on 128 x 128 tiles: 36.3 us with the reads and copies of a k-step issued in
// front of its MFMAs, 31.1 with them spread; with a rank-space branch 46.5 -> 37.
#pragma once
#include "common.h"
#include "gemm_copy.h"
#include "gemm_epilogue.h"

namespace {

constexpr int BK = 64, ROWB = BK * 2;

// What a tile form costs, in us as a + b (slabs of the contraction).  Blocks of 4 waves: `one` for at most 256 tiles, `both` for
// 257 to 512, `full` for each 512 before those (two of them share a CU, but for 32 x 64 with 16 rank-space columns and 32 x 32
// with 48, whose 86 KB of LDS leave room for one; those are fitted the same way).  Blocks that own a CU (both.b 0): between `one`
// for a few tiles and `full` for 256, as full as the last round is, and `full` for each 256 before it.
// A full round of two blocks to a CU is priced at sqrt(nk^2 + fill) slabs: the line through the long contractions the table was
// fitted to leaves out what a tile costs at any length (its ring is filled whatever there is to fill it with: 0.65 us for
// 64 x 128 by the line, 3.0 measured at one slab and 3.8 at three), and small tiles were picked where a few large ones cost half
// (fp8, 10803 rows of 128 -> 4224: 42 us on 64 x 128, 24 on 256 x 256; bf16, 20820 of 64 -> 3072: 46, 34).  `fill`: the largest of
// 0 to 25 (bf16, 12) and of 8 to 16 (fp8, 16) that takes no shape of 1894 off a form by more than 3 and 5 %.  The form picked is
// then 0.9 % (bf16) and 0.2 % (fp8) slower on average than the fastest, 2.1 and 4.7 % without.  Plain stores only (else `fill` is 0):
// the others' epilogues take longer, most of all on large tiles, where nothing runs beside them, and narrow stacks lost by it
// (two blocks of 256 -> 4032 columns, 9472 tokens: 605 -> 631 us; fp8, 256 -> 1024, 17856 tokens: 677 -> 720).
struct Cost { float a, b; };
struct Form { int tm, tn; Cost one, both, full; };
inline double form_cost(const Form &f, long tiles, int nk, double fill)
{
    auto us = [&](const Cost &c) { return c.a + (double)c.b * nk; };
    const bool two = f.both.b > 0;
    const long round = two ? 512 : 256, before = (tiles - 1) / round, last = tiles - before * round;
    if (two) return before * (f.full.a + f.full.b * sqrt((double)nk * nk + fill)) + us(last > 256 ? f.both : f.one);
    const double part = last / 256.0;
    return (before + part) * us(f.full) + (1 - part) * us(f.one);
}

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

// Epilogue of CR rows staged in LDS, so that memory sees 16-byte accesses.
// INTERIOR: the rows and columns lie wholly inside the matrix, no branch (see epilogue4 in gemm_epilogue.h).
template <int EPI, int TN, int CR, int NTHR, bool INTERIOR, class Args>
__device__ __forceinline__ void epilogue_rows(const Args &a, const float *stg, int m0, int n0, int n_end,
                                              const float (&bias8)[8])
{
    constexpr int P = TN + 4, TPR = TN / 8, RPP = NTHR / TPR, NP = CR > RPP ? CR / RPP : 1;
    const int er = (int)threadIdx.x / TPR, ec = ((int)threadIdx.x % TPR) * 8, col = n0 + ec;
    const bool mine = RPP <= CR || er < CR;              // more threads than rows: the others only keep the barriers
    AuxRow aux[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int row = m0 + p * RPP + er;
        load_aux<EPI>(a, row, col, mine && (INTERIOR || (row < a.M && col < n_end)), aux[p]);
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int rl = p * RPP + er, row = m0 + rl;
        if (!mine) continue;
        const float4 p0 = *(const float4 *)(stg + rl * P + ec);
        const float4 p1 = *(const float4 *)(stg + rl * P + ec + 4);
        float v[8] = {p0.x + bias8[0], p0.y + bias8[1], p0.z + bias8[2], p0.w + bias8[3],
                      p1.x + bias8[4], p1.y + bias8[5], p1.z + bias8[6], p1.w + bias8[7]};
        if (INTERIOR || (row < a.M && col < n_end)) store_row8<EPI>(a, row, col, v, aux[p]);
    }
}

// LDS of a block: the ring of stages, which the z tile and the epilogue's staging reuse
template <int NZ, int TM, int TN, int NSUB, int NST>
constexpr int gemm_tile_lds()
{
    constexpr int ring = NST * NSUB * (TM + TN + NZ) * ROWB, z = NZ > 0 ? TM * ((NZ + 31) / 32 * 32 + 8) * 2 : 0;
    constexpr int epi = (TM % 64 == 0 ? 64 : 32) * (TN + 4) * 4;
    return ring > z ? (ring > epi ? ring : epi) : (z > epi ? z : epi);
}

// Tile and share of the contraction of this block; consecutive logical ids land on one XCD and walk panels of PANEL row
// tiles column by column (operands of the tiles in flight on an XCD stay in its L2).
struct TileOf { int m0, n0, n_end, seg, tns, tile, split; bool any; };
template <int TM, int TN, class Args>
__device__ __forceinline__ TileOf gemm_tile_of(const Args &a, int splits)
{
    TileOf t;
    const int tiles_n_seg = (a.seg_n + TN - 1) / TN;
    const int tiles_n = tiles_n_seg * a.nseg;
    const int tiles_m = (a.M + TM - 1) / TM;
    const int nb = tiles_m * tiles_n * splits;
    const int per_xcd = (nb + 7) >> 3;
    const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    t.any = logical < nb && (int)(blockIdx.x >> 3) < per_xcd;
    t.tile = logical / splits;
    t.split = logical - t.tile * splits;
    constexpr int PANEL = 8;
    const int pidx = t.tile / (PANEL * tiles_n), prem = t.tile - pidx * (PANEL * tiles_n);
    const int prow = max(1, min(PANEL, tiles_m - pidx * PANEL));
    const int tn = prem / prow, tm = pidx * PANEL + prem - tn * prow;
    t.seg = tn / tiles_n_seg;
    t.tns = tn - t.seg * tiles_n_seg;
    t.n0 = t.seg * a.seg_n + t.tns * TN;
    t.n_end = (t.seg + 1) * a.seg_n;
    t.m0 = tm * TM;
    return t;
}

// Epilogue of a block's tile, CR rows at a time; row tile i of a wave is tile (i + rot) mod MI of its rows.
template <int EPI, int TM, int TN, int WM, int WN, class Args>
__device__ __forceinline__ void gemm_tile_epilogue(const Args &a, const f32x4 (&acc)[TM / 16 / WM][TN / 16 / WN], unsigned char *lds,
                                                   int m0, int n0, int n_end, int rot)
{
    constexpr int NTHR = 64 * WM * WN, MI = TM / 16 / WM, NI = TN / 16 / WN;
    constexpr int P = TN + 4, CR = TM % 64 == 0 ? 64 : 32, CT = CR / 16;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN, r16 = lane & 15, kg = lane >> 4;
    constexpr int TPR = TN / 8;
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
    const bool interior = m0 + TM <= a.M && n0 + TN <= n_end;
#pragma unroll
    for (int c = 0; c < TM / CR; ++c) {
        if (c > 0) __syncthreads();
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int rt = wm * MI + (i + rot) % MI - c * CT;         // 16-row tile within the chunk
            if (rt >= 0 && rt < CT) {
#pragma unroll
                for (int j = 0; j < NI; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) stg[(rt * 16 + 4 * kg + e) * P + (wn * NI + j) * 16 + r16] = acc[i][j][e];
            }
        }
        if (interior) epilogue_rows<EPI, TN, CR, NTHR, true>(a, stg, m0 + CR * c, n0, n_end, bias8);
        else epilogue_rows<EPI, TN, CR, NTHR, false>(a, stg, m0 + CR * c, n0, n_end, bias8);
    }
}

// TM x TN tile, WM x WN waves; a stage of the LDS ring holds NSUB slabs of 64 (one barrier per stage), NST stages.
// SPLIT: `splits` blocks share a tile's contraction; their partial accumulators go to scratch memory and the block that
// arrives last adds them in share order -- whichever block that is, so results are still reproducible.
template <int EPI, int NZ, int TM, int TN, int WM, int WN, int NSUB, int NST, bool SPLIT>
__device__ __forceinline__ void gemm_tile_block(const GemmArgs &a, const TileOf &at, int splits, unsigned char *lds)
{
    constexpr int NW = WM * WN, NTHR = 64 * NW;
    constexpr int XB = TM * ROWB, WB = TN * ROWB, SUBB = XB + WB + NZ * ROWB, STAGE = NSUB * SUBB;
    constexpr int MI = TM / 16 / WM, NI = TN / 16 / WN;  // 16 x 16 tiles of a wave along M and N
    // copies (8 rows, 1 KB each) of a wave per slab; those of Z are left to the first waves
    constexpr int PX = TM / 8, PW = TN / 8, PZ = NZ / 8;
    constexpr int CX = PX / NW, CW = PW / NW, CZ = (PZ + NW - 1) / NW;
    constexpr int NC = CX + CW + CZ;
    constexpr int NZT = NZ > 0 ? NZ / 16 : 1;
    constexpr int MZ = (MI + WN - 1) / WN;               // 16-row tiles of z that a wave forms
    constexpr int K2P = NZ > 0 ? (NZ + 31) / 32 * 32 : 32;
    static_assert(EPI != EPI_STORE_DELTA || TN % 64 == 0, "a head's columns in one tile");
    static_assert(PX % NW == 0 && PW % NW == 0, "every wave copies as much");
    static_assert(NSUB * NC * NST < 64, "copies in flight fit the counter");

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int r16 = lane & 15, kg = lane >> 4;

    const int m0 = at.m0, n0 = at.n0, n_end = at.n_end, seg = at.seg, tns = at.tns, tile = at.tile, split = at.split;
    const int nk_all = a.K / BK;
    const int ks0 = (int)((long)split * nk_all / splits), nk = (int)((long)(split + 1) * nk_all / splits) - ks0;
    const bool has_z = (NZ > 0) && (a.zmat[seg] != nullptr);

    // copies: 8 rows (1 KB) per instruction, lane l fills 16-byte slot l: row l>>3, physical k-chunk l&7 holding logical
    // chunk (l&7) ^ (l>>3)
    const int lrow = lane >> 3, lch = (lane & 7) ^ (lane >> 3);
    unsigned xo[CX], wo[CW], zo = 0;
#pragma unroll
    for (int p = 0; p < CX; ++p)
        xo[p] = ((unsigned)min(m0 + (wave * CX + p) * 8 + lrow, a.M - 1) * (unsigned)a.ldx + lch * 8) * 2u;
#pragma unroll
    for (int p = 0; p < CW; ++p)
        wo[p] = ((unsigned)min(n0 + (wave * CW + p) * 8 + lrow, n_end - 1) * (unsigned)a.ldw + lch * 8) * 2u;
    if (NZ > 0) zo = ((unsigned)(wave * 8 + lrow) * (unsigned)a.ldz + lch * 8) * 2u;
    const char *Xb = (const char *)a.X, *Wb = (const char *)a.W;
    const char *Zb = has_z ? (const char *)a.zmat[seg] : nullptr;
    const unsigned zstep = (unsigned)(NW * 8) * (unsigned)a.ldz * 2u;
    int zlanes[CZ > 0 ? CZ : 1];
#pragma unroll
    for (int p = 0; p < CZ; ++p) zlanes[p] = (wave + p * NW - (has_z ? PZ : 0)) >> 31;      // -1 or 0
    const unsigned base = lds_addr(lds);
    // Copy q (of NC) of slab `sub` of stage t into ring slot `slot`.  Copies past the last slab repeat it (in bounds, never
    // read), and a wave without a piece of Z issues its copy with no lane enabled, so that one constant serves every wait.
    auto copy1 = [&](int slot, int t, int sub, int q) {
        const size_t kb = (size_t)(ks0 + min(t * NSUB + sub, nk - 1)) * ROWB;
        const unsigned sb = base + slot * STAGE + sub * SUBB;
        if (q < CX) glds_soff(Xb + kb, xo[q < CX ? q : 0], sb + (wave * CX + q) * 1024);
        else if (q < CX + CW) glds_soff(Wb + kb, wo[q >= CX && q < CX + CW ? q - CX : 0], sb + XB + (wave * CW + q - CX) * 1024);
        else if (NZ > 0) {
            const int piece = wave + (q - CX - CW) * NW;
            glds_soff_if(Zb + kb, zo + (q - CX - CW) * zstep, sb + XB + WB + piece * 1024, zlanes[q >= CX + CW ? q - CX - CW : 0]);
        }
    };
    // everything but the newest NST - 2 stages' copies of this wave has landed, and its fragments are in registers
#define GT_WAIT() asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NST - 2) * NSUB * NC) : "memory")

    f32x4 acc[MI][NI], zacc[MZ][NZT];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int h = 0; h < MZ; ++h)
#pragma unroll
        for (int q = 0; q < NZT; ++q) zacc[h][q] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Row tile i of the wave is tile (i + wn MZ) mod MI of its rows, so that each of the WN waves that share rows has the
    // rank-space rows it forms as its first MZ tiles (where they do not divide, two waves form the same ones).
    const int rot = NZ > 0 ? wn * MZ : 0;
    int a_off[MI];
#pragma unroll
    for (int i = 0; i < MI; ++i) a_off[i] = (wm * MI * 16 + ((i + rot) % MI) * 16 + r16) * ROWB;
    const int b_off = XB + (wn * NI * 16 + r16) * ROWB, sw = r16 & 7;
    struct Frags { bf16x8 a[MI], b[NI], zb[NZT]; } f[2];
    constexpr int NR = MI + NI + (NZ > 0 ? NZT : 0), NM = MI * NI;
    // operand fragment q of k-step `step` (two to a slab) of the stage in `slot`
    auto read1 = [&](Frags &F, int slot, int step, int q) {
        const unsigned char *S = lds + slot * STAGE + (step >> 1) * SUBB;
        const int co = (((step & 1) * 4 + kg) ^ sw) << 4;
        if (q < MI) F.a[q < MI ? q : 0] = *(const bf16x8 *)(S + a_off[q < MI ? q : 0] + co);
        else if (q < MI + NI) F.b[q >= MI && q < MI + NI ? q - MI : 0] = *(const bf16x8 *)(S + b_off + (q - MI) * 16 * ROWB + co);
        else F.zb[q >= MI + NI ? q - MI - NI : 0] = *(const bf16x8 *)(S + XB + WB + ((q - MI - NI) * 16 + r16) * ROWB + co);
    };
    auto mfma_z = [&](const Frags &F) {
        if (NZ > 0) {
#pragma unroll
            for (int q = 0; q < NZT; ++q)
#pragma unroll
                for (int h = 0; h < MZ; ++h) zacc[h][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(F.a[h], F.zb[q], zacc[h][q], 0, 0, 0);
        }
    };
    // One k-step: the MFMAs of fragment set cb, and spread between them the reads of the next k-step's fragments (in the
    // first three quarters) and copies c0 .. c1 - 1 of stage ct.
    auto step = [&](int cb, int rslot, int rstep, int cslot, int ct, int c0, int c1) {
        constexpr int SPAN = NM * 3 / 4 > 0 ? NM * 3 / 4 : 1;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            const int ra = m < SPAN ? m * NR / SPAN : NR, rb = m + 1 < SPAN ? (m + 1) * NR / SPAN : NR;
#pragma unroll
            for (int q = 0; q < NR; ++q)
                if (q >= ra && q < rb) read1(f[1 - cb], rslot, rstep, q);
#pragma unroll
            for (int c = 0; c < NSUB * NC; ++c)
                if (c >= c0 && c < c1 && (c - c0) >= m * (c1 - c0) / NM && (c - c0) < (m + 1) * (c1 - c0) / NM)
                    copy1(cslot, ct, c / NC, c % NC);
            acc[m / NI][m % NI] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[cb].a[m / NI], f[cb].b[m % NI], acc[m / NI][m % NI], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        mfma_z(f[cb]);
        __builtin_amdgcn_sched_barrier(0);
    };

    // up-projection operands, needed after the loop: requested first, so that the waits below count copies only
    bf16x8 tb[K2P / 32][NI];
    if (NZ > 0 && has_z) {
#pragma unroll
        for (int ks = 0; ks < K2P / 32; ++ks)
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                const int n = min(n0 + (wn * NI + j) * 16 + r16, n_end - 1) - seg * a.seg_n;
                tb[ks][j] = *(const bf16x8 *)(a.tmat[seg] + (size_t)n * a.ldt + ks * 32 + kg * 8);
            }
    }
    // A stage's copies go out NST - 1 stages ahead into the slot of the stage before the current one: the first C1 of them
    // in that stage's last k-step, behind its barrier, the others in the current stage's k-steps but the last.
    constexpr int STEPS = 2 * NSUB, NCS = NSUB * NC, C1 = NST > 2 ? (NCS + STEPS - 1) / STEPS : 0;
#pragma unroll
    for (int s = 0; s < NST - 1; ++s)
#pragma unroll
        for (int c = 0; c < NCS; ++c) copy1(s, s, c / NC, c % NC);
    GT_WAIT();
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NR; ++q) read1(f[0], 0, 0, q);
#pragma unroll
    for (int c = 0; c < C1; ++c) copy1(NST - 1, NST - 1, c / NC, c % NC);
    // Fragments are read one k-step ahead of their MFMAs, and the one barrier of a stage sits in front of its last k-step's
    // MFMAs: the wave's reads of the stage are done there and its copies of the next stage have landed (the newer ones may
    // still be in flight).
    const int nfull = nk / NSUB;
    int slot = 0;
    for (int t = 0; t < nfull; ++t) {
        const int next = slot + 1 == NST ? 0 : slot + 1, prev = slot == 0 ? NST - 1 : slot - 1;
#pragma unroll
        for (int st = 0; st < STEPS - 1; ++st)
            step(st & 1, slot, st + 1, prev, t + NST - 1, C1 + (NCS - C1) * st / (STEPS - 1), C1 + (NCS - C1) * (st + 1) / (STEPS - 1));
        GT_WAIT();
        __syncthreads();
        step(1, next, 0, slot, t + NST, 0, C1);
        slot = next;
    }
    if (NSUB > 1) {                                      // slabs that fill no stage
        const int rem = nk - nfull * NSUB;
#pragma unroll
        for (int s = 0; s < 2 * (NSUB - 1); ++s)
            if (s < 2 * rem) {
#pragma unroll
                for (int q = 0; q < NR; ++q) read1(f[0], slot, s, q);
#pragma unroll
                for (int m = 0; m < NM; ++m)
                    acc[m / NI][m % NI] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[0].a[m / NI], f[0].b[m % NI], acc[m / NI][m % NI], 0, 0, 0);
                mfma_z(f[0]);
            }
    }
    // the repeated copies have landed and every wave is done with the ring before it is reused
#undef GT_WAIT
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();

    if constexpr (SPLIT) if (splits > 1) {
        __shared__ int last_block;
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

    // ---- low-rank tail: acc += (zscale * z)[TM,K2P] . T[n,K2P]^T ------------------------------------
    if (NZ > 0 && has_z) {
        constexpr int ZP = K2P + 8;
        bf16 *zs = (bf16 *)lds;
#pragma unroll
        for (int h = 0; h < MZ; ++h) {
            const int rt = wm * MI + (h + rot) % MI;
#pragma unroll
            for (int q = 0; q < K2P / 16; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    zs[(rt * 16 + 4 * kg + e) * ZP + q * 16 + r16] = f2bf(q < NZT ? zacc[h][q < NZT ? q : 0][e] * a.zscale : 0.f);
        }
        __syncthreads();
        if (a.zspill[seg] != nullptr && tns == 0) {
            const int cpr = a.K2 >> 3;                   // 16-byte chunks per row
            for (int c = tid; c < TM * cpr; c += NTHR) {
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
                af[i] = *(const bf16x8 *)(zs + ((wm * MI + (i + rot) % MI) * 16 + r16) * ZP + ks * 32 + kg * 8);
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], tb[ks][j], acc[i][j], 0, 0, 0);
        }
        __syncthreads();                                 // the z tile has been consumed
    }

    gemm_tile_epilogue<EPI, TM, TN, WM, WN>(a, acc, lds, m0, n0, n_end, rot);
}

// the block's tile; a segment without adapter, which q|k|v has when not all three carry one, runs without the branch
template <int EPI, int NZ, int TM, int TN, int WM, int WN, int NSUB, int NST, bool SPLIT>
__device__ __forceinline__ void gemm_tile_body(const GemmArgs &a, int splits)
{
    __shared__ __attribute__((aligned(1024))) unsigned char lds[gemm_tile_lds<NZ, TM, TN, NSUB, NST>()];
    const int shares = SPLIT ? splits : 1;
    const TileOf at = gemm_tile_of<TM, TN>(a, shares);
    if (!at.any) return;
    if constexpr (NZ == 16 && EPI == EPI_STORE) {
        if (a.zmat[at.seg] == nullptr) {
            gemm_tile_block<EPI, 0, TM, TN, WM, WN, NSUB, NST, SPLIT>(a, at, shares, lds);
            return;
        }
    }
    gemm_tile_block<EPI, NZ, TM, TN, WM, WN, NSUB, NST, SPLIT>(a, at, shares, lds);
}

}  // namespace
