// GEMM on MXFP8 operands (gfx950): arguments and the body of its kernels.
//
//   out[M,N] = epilogue( zs[M,K2] . tmat[N,K2]^T  +  deq(X)[M,K] . deq(W)[N,K]^T )
//
// The body is that of the bf16 kernels (gemm_tile.h): a 128-byte LDS row is one k-slab of a tile row and spans 128 elements, a
// stage of the ring also carries the 4 scale bytes of every row.  A slab is one k-step of V_MFMA_SCALE_F32_16X16X128_F8F6F4, so
// a stage's fragments are in registers when its k-step begins, its slot is free behind that step's barrier, and the copies run
// NST stages ahead.
#pragma once
#include "gemm_tile.h"

struct MxArgs {
    const unsigned char *X, *XS;     // codes [M,K], scales [M,K/32]
    const unsigned char *W, *WS;     // codes [N,K], scales [N,K/32]   (N = nseg * seg_n)
    const bf16 *bias;                // [N] or null
    int M, N, K;
    int nseg, seg_n;
    // low-rank branch kept in bf16, per segment (null zs = segment not adapted): out += zs . tmat^T
    const bf16 *zs[3];               // [M,K2]: scaled rank-space activations, zero beyond the rank(s)
    const bf16 *tmat[3];             // [seg_n,ldt]: up-projection(s), ldt = K2 rounded up to 32, zero padded
    int K2, ldt;
    // epilogue (meaning as in GemmArgs)
    void *out0; void *out1; const void *aux; int ldo;
    const bf16 *dl_o, *dl_lo; float *dl_out;   // EPI_STORE_DELTA (meaning as in GemmArgs)
    unsigned char *oq, *os;          // optional MXFP8 copy of the epilogue's bf16 tensor (see GemmArgs)
    static constexpr bool kEmitCodes = true;
};

// the tile of a product with fp8 weights: 256 x 256 is that of mx.hip, the others those of gemm_mx.hip
extern "C" TilePlan plan_gemm_mx(int M, int seg_n, int nseg, int K, int epi, bool low_rank);
int launch_gemm_mx_tile(const MxArgs &a, int epi, const TilePlan &p, hipStream_t st);

namespace {

typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

template <int TM, int TN, int NST>
constexpr int gemm_mx_lds()
{
    constexpr int ring = NST * ((TM + TN) * 128 + ((TM + 63) / 64 + (TN + 63) / 64) * 256);
    constexpr int epi = (TM % 64 == 0 ? 64 : 32) * (TN + 4) * 4;
    return ring > epi ? ring : epi;
}

template <int EPI, int TM, int TN, int WM, int WN, int NST>
__device__ __forceinline__ void gemm_mx_body(const MxArgs &a)
{
    constexpr int NW = WM * WN, BKB = 128;
    constexpr int XB = TM * BKB, WB = TN * BKB;
    constexpr int MI = TM / 16 / WM, NI = TN / 16 / WN;
    // copies of a wave per slab: 8 rows (1 KB) of codes, 64 rows' scale dwords (256 bytes; left to the first waves)
    constexpr int PX = TM / 8, PW = TN / 8, SX = (TM + 63) / 64, SW = (TN + 63) / 64;
    constexpr int CX = PX / NW, CW = PW / NW, PER = CX + CW + 1;
    constexpr int STAGE = XB + WB + (SX + SW) * 256;
    static_assert(PX % NW == 0 && PW % NW == 0 && SX + SW <= NW, "every wave copies as much");
    static_assert(NST * PER < 64, "copies in flight fit the counter");
    __shared__ __attribute__((aligned(1024))) unsigned char lds[gemm_mx_lds<TM, TN, NST>()];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int r16 = lane & 15, kg = lane >> 4;
    const TileOf at = gemm_tile_of<TM, TN>(a, 1);
    if (!at.any) return;
    const int m0 = at.m0, n0 = at.n0, n_end = at.n_end, seg = at.seg;
    const int nk = a.K / BKB;

    // Low-rank operands first (SplitLoRA Sec. II-C: W + BA with the adapter kept in bf16; a few MB: cache hits).  Columns of the
    // rank-space activations beyond K2 and of the up-projection beyond the ranks are zero.  Their products stand behind the
    // first copies of every stage, which the compiler cannot count: it waits for all of these, so a tile with an adapter
    // begins when the whole ring is filled, not when its first stage is.
    f32x4 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const bool has_z = a.zs[seg] != nullptr;
    bf16x8 za[MI], tb[NI];
    auto load_z = [&](int ks) {
        const bool zok = ks * 32 + kg * 8 < a.K2;
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int n = min(n0 + (wn * NI + j) * 16 + r16, n_end - 1) - seg * a.seg_n;
            tb[j] = *(const bf16x8 *)(a.tmat[seg] + (size_t)n * a.ldt + ks * 32 + kg * 8);
        }
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int row = min(m0 + (wm * MI + i) * 16 + r16, a.M - 1);
#pragma unroll
            for (int q = 0; q < 8; ++q) za[i][q] = f2bf(0.f);
            if (zok) za[i] = *(const bf16x8 *)(a.zs[seg] + (size_t)row * a.K2 + ks * 32 + kg * 8);
        }
    };
    auto mfma_z = [&]() {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(za[i], tb[j], acc[i][j], 0, 0, 0);
    };
    if (has_z) load_z(0);

    // lane l -> row l>>3, physical 16-byte chunk l&7 holding logical chunk (l&7)^(l>>3)
    const int lrow = lane >> 3, lch = (lane & 7) ^ (lane >> 3);
    unsigned xo[CX], wo[CW];
#pragma unroll
    for (int p = 0; p < CX; ++p) xo[p] = (unsigned)min(m0 + (wave * CX + p) * 8 + lrow, a.M - 1) * (unsigned)a.K + lch * 16;
#pragma unroll
    for (int p = 0; p < CW; ++p) wo[p] = (unsigned)min(n0 + (wave * CW + p) * 8 + lrow, n_end - 1) * (unsigned)a.K + lch * 16;
    const bool sx = wave < SX;
    const int srow = sx ? min(m0 + wave * 64 + lane, a.M - 1) : min(n0 + (wave - SX) * 64 + lane, n_end - 1);
    const unsigned so = (unsigned)srow * (unsigned)(a.K >> 5);
    const unsigned char *Sb = sx ? a.XS : a.WS;
    const int slanes = (wave - (SX + SW)) >> 31;         // -1: this wave copies scales, 0: it does not
    const unsigned base = lds_addr(lds);
    // copy q (of PER) of stage t into ring slot `slot`; copies past the last slab repeat it (in bounds, never read)
    auto copy1 = [&](int slot, int t, int q) {
        const int kt = min(t, nk - 1);
        const unsigned sb = base + slot * STAGE;
        if (q < CX) glds_soff(a.X + (size_t)kt * BKB, xo[q < CX ? q : 0], sb + (wave * CX + q) * 1024);
        else if (q < CX + CW)
            glds_soff(a.W + (size_t)kt * BKB, wo[q >= CX && q < CX + CW ? q - CX : 0], sb + XB + (wave * CW + q - CX) * 1024);
        else glds4_soff_if(Sb + (size_t)kt * 4, so, sb + XB + WB + wave * 256, slanes);
    };

    const int sw = r16 & 7, c0 = (kg ^ sw) << 4, c1 = ((4 + kg) ^ sw) << 4;     // the lane's two 16-byte chunks
    const int a_off = (wm * MI * 16 + r16) * BKB, b_off = XB + (wn * NI * 16 + r16) * BKB;
    const int as_off = XB + WB + (wm * MI * 16 + r16) * 4 + kg, bs_off = XB + WB + SX * 256 + (wn * NI * 16 + r16) * 4 + kg;
    struct Frags { i32x8 a[MI], b[NI]; int as[MI], bs[NI]; } f[2];
    constexpr int NR = MI + NI, NM = MI * NI;
    auto read1 = [&](Frags &F, int slot, int q) {
        const unsigned char *S = lds + slot * STAGE;
        if (q < MI) {
            const unsigned char *r = S + a_off + q * 16 * BKB;
            F.a[q < MI ? q : 0].lo = *(const i32x4 *)(r + c0);
            F.a[q < MI ? q : 0].hi = *(const i32x4 *)(r + c1);
            F.as[q < MI ? q : 0] = S[as_off + q * 64];
        } else {
            const unsigned char *r = S + b_off + (q - MI) * 16 * BKB;
            F.b[q >= MI ? q - MI : 0].lo = *(const i32x4 *)(r + c0);
            F.b[q >= MI ? q - MI : 0].hi = *(const i32x4 *)(r + c1);
            F.bs[q >= MI ? q - MI : 0] = S[bs_off + (q - MI) * 64];
        }
    };
    // the slab of fragment set cb; between its MFMAs the reads of the next slab (first three quarters) and the copies
    auto step = [&](int cb, int rslot, int cslot, int ct) {
        constexpr int SPAN = NM * 3 / 4 > 0 ? NM * 3 / 4 : 1;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            const int ra = m < SPAN ? m * NR / SPAN : NR, rb = m + 1 < SPAN ? (m + 1) * NR / SPAN : NR;
#pragma unroll
            for (int q = 0; q < NR; ++q)
                if (q >= ra && q < rb) read1(f[1 - cb], rslot, q);
#pragma unroll
            for (int c = 0; c < PER; ++c)
                if (c >= m * PER / NM && c < (m + 1) * PER / NM) copy1(cslot, ct, c);
            acc[m / NI][m % NI] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(f[cb].a[m / NI], f[cb].b[m % NI], acc[m / NI][m % NI],
                                                                                   0, 0, 0, f[cb].as[m / NI], 0, f[cb].bs[m % NI]);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

#pragma unroll
    for (int s = 0; s < NST; ++s)
#pragma unroll
        for (int c = 0; c < PER; ++c) copy1(s, s, c);
    if (has_z) {
        mfma_z();
        for (int ks = 1; ks < (a.ldt >> 5); ++ks) {
            load_z(ks);
            mfma_z();
        }
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 1) * PER) : "memory");
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NR; ++q) read1(f[0], 0, q);
    int slot = 0;
    auto slab = [&](int cb, int t) {
        const int next = slot + 1 == NST ? 0 : slot + 1;
        // stage t + 1 has landed (the newer ones may be in flight); every wave's fragments of stage t are in registers
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NST - 2) * PER) : "memory");
        __syncthreads();
        step(cb, next, slot, t + NST);
        slot = next;
    };
    for (int t = 0; t < nk; t += 2) {
        slab(0, t);
        if (t + 1 == nk) break;
        slab(1, t + 1);
    }
    // the repeated copies have landed and every wave is done with the ring before it is reused
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
    gemm_tile_epilogue<EPI, TM, TN, WM, WN>(a, acc, lds, m0, n0, n_end, 0);
}

}  // namespace
