// Causal multi-head attention, forward and backward, head size 64, bf16 MFMA with fp32
// softmax arithmetic (gfx950).  Part of the server-side forward/backward of SplitLoRA
// Sec. III-B step a3; the attention block itself is the public GPT-2 one
// (softmax(Q K^T / sqrt(64)) V with future keys excluded).
//
// Layout: qkv [T, 3d] bf16 (q | k | v column blocks, head a at columns 64a..64a+63 of each),
// o / dO [T, d], lse [n_seq, H, S] fp32 in log2 units of the scaled scores, delta likewise.
//
// Forward, and the backward for sequences longer than 512 (a dQ kernel, then a dK/dV kernel): 4 wavefronts
// per block, each owning 32 rows (queries or keys), online-softmax tiles of 64 staged in LDS by asynchronous
// global->LDS copies, double buffered.  Scores are produced with the lane owning one query (forward, dQ) or
// one key (dK/dV), which makes the softmax statistics per-lane scalars and lets the probabilities feed the
// next MFMA straight from registers.  Operands that must be read along the token axis (V, K for dQ, Q and
// dO for dK/dV) come from the same row-major tiles through the LDS transpose read, so nothing is
// transposed in memory.
// Backward for sequences up to 512 (the default at the paper's sequence length): one block of 8 wavefronts
// per (sequence, head) forms dQ, dK and dV in one pass; K of the whole sequence stays in LDS, scores,
// probabilities and dP are formed once (see attn_bwd_fused_kernel).
// No kernel uses floating-point atomics, so results are bit-reproducible.
#include "common.h"
#include "gemm_copy.h"
#include "prof.h"

namespace {

constexpr float kScaleLog2 = 0.125f * 1.4426950408889634f;   // log2(e) / sqrt(64)
constexpr int TILE_B = 64 * 128;                             // one 64-row x 64-column bf16 tile

typedef short v4s __attribute__((ext_vector_type(4)));

// One 1 KB asynchronous copy: scalar base, the lane's byte offset, LDS place.  (The compiler's own form of it is known to
// the compiler as a write of LDS: it then waits for the copies in flight, those of the NEXT tile, in front of the first
// LDS read of every inner iteration of the two backward kernels.)
#define AT_GLDS(gp, off, lp) glds_soff(gp, off, lds_addr(lp))
#define AT_WAIT_VM0() __builtin_amdgcn_s_waitcnt(0x0F70)

// XOR mask of a tile row for the 16-byte chunks of its 128-byte LDS row.  Eight consecutive rows get
// eight different masks (row-major fragment reads: 8 lanes = 8 rows, one logical chunk), and four
// consecutive rows get masks that differ in bits 1-2 (transpose reads: 16 lanes = 4 rows x 2 adjacent
// chunks), so both kinds of operand read are bank-conflict free.
__device__ __forceinline__ int swm(int row) { return ((row & 3) << 1) | ((row >> 2) & 1); }
__device__ __forceinline__ int swz128(int row, int chunk) { return row * 128 + ((chunk ^ swm(row)) << 4); }

__device__ __forceinline__ f32x16 zero16()
{
    f32x16 z;
#pragma unroll
    for (int e = 0; e < 16; ++e) z[e] = 0.f;
    return z;
}

// Asynchronous copy of a 64 x 64 bf16 tile (global pitch ld) into a swizzled row-major LDS tile.
// Four waves, two 1 KB pieces (8 rows) each: lane l fills slot l = (row l>>3, physical chunk l&7).
__device__ __forceinline__ void tile_copy_async(unsigned char *dst, const bf16 *src, int ld, int wave, int lane)
{
    const int lrow = lane >> 3, lch = (lane & 7) ^ swm(lane >> 3);
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int r0 = (wave * 2 + p) * 8;
        AT_GLDS(src + (size_t)r0 * ld, (unsigned)(lrow * ld + lch * 8) * 2u, dst + r0 * 128);
    }
}

// MFMA operand fragment from a row-major tile: row (base + lane%32), k-step ks (16 columns)
__device__ __forceinline__ bf16x8 frag_rm(const unsigned char *t, int row, int ks, int g)
{
    return *(const bf16x8 *)(t + swz128(row, ks * 2 + g));
}

// MFMA operand fragment along the ROW axis of a row-major tile (the transposed operand): lane
// (m = lane%32, g = lane/32) receives column col0 + m at the 8 rows tok0 + 8h + 4g + e
// (h = 0,1; e = 0..3), element index 4h + e.  Uses the LDS transpose read: inside each group of
// 16 lanes, lane i receives element i%4 of the 8-byte pieces addressed by lanes i/4 + 4e.
__device__ __forceinline__ bf16x8 frag_tr(const unsigned char *t, int col0, int tok0, int lane)
{
    const int q = lane & 3, e = (lane >> 2) & 3, half = (lane >> 4) & 1, g = lane >> 5;
    const int col = col0 + 16 * half + 4 * q;
    const int row0 = tok0 + 4 * g + e, row1 = row0 + 8;
    const unsigned char *a0 = t + row0 * 128 + (((col >> 3) ^ swm(row0)) << 4) + (col & 7) * 2;
    const unsigned char *a1 = t + row1 * 128 + (((col >> 3) ^ swm(row1)) << 4) + (col & 7) * 2;
    union { v4s s[2]; bf16x8 v; } u;
    u.s[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s *)a0);
    u.s[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s *)a1);
    return u.v;
}

// The lane's byte offsets of both kinds of fragment inside a 32-row piece of a tile (neither swizzle looks above bit 2
// of the row): row-major fragment of k-step ks at rm[ks]; transposed fragment of columns 32 dt .. and rows 16 hh .. at
// tr[dt] + 2048 hh.
__device__ __forceinline__ void frag_offsets(int lane, int (&rm)[4], int (&tr)[2])
{
    const int r32 = lane & 31, g = lane >> 5, q = lane & 3, e = (lane >> 2) & 3, half = (lane >> 4) & 1;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) rm[ks] = swz128(r32, ks * 2 + g);
#pragma unroll
    for (int dt = 0; dt < 2; ++dt) {
        const int col = 32 * dt + 16 * half + 4 * q;
        tr[dt] = swz128(4 * g + e, col >> 3) + (col & 7) * 2;
    }
}
__device__ __forceinline__ bf16x8 read_tr(const unsigned char *p)
{
    union { v4s s[2]; bf16x8 v; } u;
    u.s[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s *)p);
    u.s[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s *)(p + 1024));
    return u.v;
}

__device__ __forceinline__ bf16x8 lds_b128(unsigned a) { return *(const __attribute__((address_space(3))) bf16x8 *)a; }
__device__ __forceinline__ bf16x8 lds_tr(unsigned a)
{
    union { v4s s[2]; bf16x8 v; } u;
    u.s[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s *)a);
    u.s[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s *)(a + 1024));
    return u.v;
}

constexpr int OST_PITCH = 144;                                // bytes per staged output row (128 + pad: see fwd_store)
constexpr int OST_B = 32 * OST_PITCH;

// One wave's asynchronous copy of 32 rows of 128 bytes (global pitch ld) into a swizzled row-major piece of its own: whole
// lines, where reading the MFMA fragments straight from memory touches 32 lines with 32 bytes each per instruction.
__device__ __forceinline__ void rows32_copy_async(unsigned char *dst, const bf16 *src, int ld, int lane)
{
    const int lrow = lane >> 3, lch = (lane & 7) ^ swm(lane >> 3);
#pragma unroll
    for (int p = 0; p < 4; ++p) AT_GLDS(src + (size_t)(p * 8) * ld, (unsigned)(lrow * ld + lch * 8) * 2u, dst + p * 1024);
}

// 32 rows x 64 columns held as two MFMA accumulators (a lane has 4 consecutive columns of row r32 per register group)
// leave through the wave's staging area as whole lines (see fwd_store)
__device__ __forceinline__ void store_rows32(unsigned char *stg, const f32x16 (&acc)[2], float scale, bf16 *dst, int ld, int lane)
{
    const int r32 = lane & 31, g = lane >> 5, orow = lane >> 3, och = lane & 7;
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
            bf16x4 w;
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = f2bf(acc[dt][4 * e4 + i] * scale);
            *(bf16x4 *)(stg + r32 * OST_PITCH + (32 * dt + 8 * e4 + 4 * g) * 2) = w;
        }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    bf16x8 rows[4];
#pragma unroll
    for (int it = 0; it < 4; ++it) rows[it] = *(const bf16x8 *)(stg + (8 * it + orow) * OST_PITCH + och * 16);
#pragma unroll
    for (int it = 0; it < 4; ++it) *(bf16x8 *)(dst + (size_t)(8 * it + orow) * ld + och * 8) = rows[it];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// ------------------------------------------------------------------------------------------

__global__ __launch_bounds__(256, 3) void attn_fwd_kernel(const bf16 *__restrict__ qkv, bf16 *__restrict__ o,
                                                       bf16 *__restrict__ o_lo, float *__restrict__ lse, int S,
                                                       int H, int n_seq)
{
    __shared__ __attribute__((aligned(1024))) unsigned char K0[TILE_B], V0[TILE_B], K1[TILE_B], V1[TILE_B];
    __shared__ __attribute__((aligned(16))) unsigned char Ost[4 * OST_B];
    // Block -> (two query tiles, head, sequence).  Workgroups go to the 8 XCDs round-robin and, inside an XCD,
    // to its compute units in a fixed rotation as well: with one 128-query tile per block and tiles ordered
    // inside a (sequence, head) pair, every compute unit kept receiving tiles of the SAME length (the rotation's
    // period is a multiple of the tiles per pair), a 4:1 load imbalance at S = 512 that left two thirds of the
    // block slots empty for most of the launch.  So a block takes query tiles j and nqt-1-j of its pair, the
    // long one first: all blocks then do the same number of key tiles (nqt + 1 halves of a tile), whatever the
    // rotation.  The blocks of one pair still get ids that land on ONE XCD, next to each other in dispatch
    // order, so its L2 serves their re-reads of K and V.
    const int nqt = (S + 127) >> 7, npb = (nqt + 1) >> 1;
    const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
    const int pair = (idx / npb) * 8 + xcd;             // (sequence, head) pair
    if (pair >= H * n_seq) return;
    const int qtA = nqt - 1 - idx % npb, qtB = idx % npb;                 // qtA >= qtB
    const int ntA = min(S, qtA * 128 + 128) >> 6;                       // key tiles of 64 per query tile
    const int ntB = qtA != qtB ? (qtB * 128 + 128) >> 6 : 0;
    const int nt = ntA + ntB;
    const int a = pair % H, n = pair / H;
    const int d = H * 64, ld = 3 * d;
    const int tid = threadIdx.x, lane = tid & 63, r32 = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bf16 *base = qkv + (size_t)n * S * ld + a * 64;
    int qb = qtA * 128 + wave * 32;
    bool active = qb < S;
    int q = qb + r32;

    bf16x8 qf[4];
    if (active) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) qf[ks] = *(const bf16x8 *)(base + (size_t)q * ld + ks * 16 + g * 8);
    }
    f32x16 oacc[2] = {zero16(), zero16()};
    // The softmax is VALU-bound at head size 64, so the per-element work is kept to one FMA, one
    // exp2 and a share of a max and of a bf16 pack:
    //  * the row sum is taken over the bf16-ROUNDED probabilities, two per instruction (bf16 dot product
    //    against (1, 1) with an fp32 addend); a lane sums the keys it holds, the two lanes of a query are
    //    added at the end.  Summing the rounded values makes O an exact convex combination of V rows, which
    //    the backward's rowsum(dO*O) relies on.  (An all-ones MFMA did the same for 16 registers and 128
    //    cycles of the matrix pipe per tile.)
    //  * the running maximum m (log2 units, scaled) is only raised when a tile exceeds it by more
    //    than 8, so most tiles skip the rescaling of the accumulators; p <= 2^8 meanwhile.
    float lsum = 0.f;
    const bf16x2 ones2 = {(__bf16)1.0f, (__bf16)1.0f};
    float m = -INFINITY;

    // Output of one query tile: O = oacc / l, its low-order bf16 term, and the log-sum-exp.  A lane holds 4
    // consecutive columns of ONE row per register group, so direct stores would touch 32 different 128-byte
    // lines per instruction with 8 bytes each; the wave's 32 x 64 outputs go through a private LDS area
    // instead (row pitch 144 bytes: rows 16 apart share banks, a 2-way conflict on the 8-byte writes) and
    // leave as whole lines, 16 bytes per lane.  LDS operations of one wave complete in issue order, so the
    // area needs no barrier, only that the compiler keeps the order.
    auto fwd_store = [&]() {
        if (!active) return;
        unsigned char *stg = Ost + wave * OST_B;
        const float lh = lsum + __shfl_xor(lsum, 32, 64);
        const float inv = 1.0f / lh;
        const int orow = lane >> 3, och = lane & 7;
        const size_t ooff = ((size_t)n * S + qb + orow) * d + a * 64 + och * 8;
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {          // 0: O, 1: its low-order term
            bf16 *dst = pass ? o_lo : o;
            if (!dst) break;
#pragma unroll
            for (int dt = 0; dt < 2; ++dt)
#pragma unroll
                for (int e4 = 0; e4 < 4; ++e4) {
                    bf16x4 w;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float v = oacc[dt][4 * e4 + i] * inv;
                        const bf16 hi = f2bf(v);
                        w[i] = pass ? f2bf(v - bf2f(hi)) : hi;       // o + o_lo carries ~16 bits
                    }
                    *(bf16x4 *)(stg + r32 * OST_PITCH + (32 * dt + 8 * e4 + 4 * g) * 2) = w;
                }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            bf16x8 rows[4];
#pragma unroll
            for (int it = 0; it < 4; ++it) rows[it] = *(const bf16x8 *)(stg + (8 * it + orow) * OST_PITCH + och * 16);
#pragma unroll
            for (int it = 0; it < 4; ++it) *(bf16x8 *)(dst + ooff + (size_t)(8 * it) * d) = rows[it];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        if (g == 0) lse[((size_t)n * H + a) * S + q] = m + log2f(lh);
    };

    // All 8 K fragments and all 16 V fragment reads of a tile are issued before the first MFMA, so the LDS
    // latency is paid once per tile instead of once per fragment (left inline in the MFMA calls the compiler
    // emitted read, wait, MFMA for every one of them), and the two score accumulators advance alternately.
#define FWD_TILE(Ks, Vs, k0)                                                                           \
    if (active && (k0) <= qb + 31) {                                                                   \
        bf16x8 kf[2][4];                                                                               \
        _Pragma("unroll") for (int ks = 0; ks < 4; ++ks)                                               \
            _Pragma("unroll") for (int mt = 0; mt < 2; ++mt) kf[mt][ks] = frag_rm(Ks, mt * 32 + r32, ks, g); \
        __builtin_amdgcn_sched_barrier(0);                                                             \
        f32x16 sacc[2] = {zero16(), zero16()};                                                         \
        _Pragma("unroll") for (int ks = 0; ks < 4; ++ks)                                               \
            _Pragma("unroll") for (int mt = 0; mt < 2; ++mt)                                           \
                sacc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[mt][ks], qf[ks], sacc[mt], 0, 0, 0); \
        if ((k0) + 63 > qb) {                                                                          \
            _Pragma("unroll") for (int mt = 0; mt < 2; ++mt)                                           \
                _Pragma("unroll") for (int e = 0; e < 16; ++e) {                                       \
                    const int key = (k0) + 32 * mt + 8 * (e >> 2) + 4 * g + (e & 3);                   \
                    if (key > q) sacc[mt][e] = -INFINITY;                                              \
                }                                                                                      \
        }                                                                                              \
        float tmax = sacc[0][0];                                                                       \
        _Pragma("unroll") for (int mt = 0; mt < 2; ++mt)                                               \
            _Pragma("unroll") for (int e = 0; e < 16; ++e) tmax = fmaxf(tmax, sacc[mt][e]);            \
        tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64)) * kScaleLog2;                                     \
        if (__builtin_amdgcn_ballot_w64(tmax > m + 8.0f) != 0) {                                       \
            const float m_new = fmaxf(m, tmax);                                                        \
            const float alpha = __builtin_amdgcn_exp2f(m - m_new);                                     \
            m = m_new;                                                                                 \
            lsum *= alpha;                                                                             \
            _Pragma("unroll") for (int dt = 0; dt < 2; ++dt)                                           \
                _Pragma("unroll") for (int e = 0; e < 16; ++e) oacc[dt][e] *= alpha;                   \
        }                                                                                              \
        _Pragma("unroll") for (int mt = 0; mt < 2; ++mt) {                                             \
            bf16x8 vf[2][2];                             /* this half's V fragments, under way during its exponentials */ \
            _Pragma("unroll") for (int hh = 0; hh < 2; ++hh)                                           \
                _Pragma("unroll") for (int dt = 0; dt < 2; ++dt)                                       \
                    vf[hh][dt] = frag_tr(Vs, 32 * dt, 32 * mt + 16 * hh, lane);                        \
            __builtin_amdgcn_sched_barrier(0);                                                         \
            _Pragma("unroll") for (int hh = 0; hh < 2; ++hh) {                                         \
                bf16x8 pb;                                                                             \
                float pe[8];                                                                           \
                _Pragma("unroll") for (int i = 0; i < 8; ++i) pe[i] = fmaf(sacc[mt][8 * hh + i], kScaleLog2, -m); \
                _Pragma("unroll") for (int i = 0; i < 8; ++i) pe[i] = __builtin_amdgcn_exp2f(pe[i]);   \
                _Pragma("unroll") for (int i = 0; i < 8; ++i) pb[i] = f2bf(pe[i]);                     \
                _Pragma("unroll") for (int i = 0; i < 4; ++i) {                                        \
                    const bf16x2 pr = {pb[2 * i], pb[2 * i + 1]};                                    \
                    lsum = __builtin_amdgcn_fdot2_f32_bf16(pr, ones2, lsum, false);                    \
                }                                                                                      \
                _Pragma("unroll") for (int dt = 0; dt < 2; ++dt)                                       \
                    oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[hh][dt], pb, oacc[dt], 0, 0, 0); \
            }                                                                                          \
        }                                                                                              \
    }
    // Step t of the block's flat tile sequence (ntA tiles of the long query tile, then ntB of the short one);
    // at the switch the finished tile goes out and the wave's state is set up for the other query rows.
#define FWD_STEP(Ks, Vs, t)                                                                            \
    {                                                                                                  \
        if ((t) == ntA) {                                                                              \
            /* the short tile's Q rows have been waiting in this wave's output staging area since the   \
               first copies: fetched from memory here they would cost the block one exposed latency */  \
            bf16x8 qn[4];                                                                              \
            _Pragma("unroll") for (int ks = 0; ks < 4; ++ks) qn[ks] = frag_rm(Ost + wave * OST_B, r32, ks, g); \
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   /* read before fwd_store overwrites */ \
            fwd_store();                                                                               \
            qb = qtB * 128 + wave * 32; q = qb + r32; active = true;                                   \
            _Pragma("unroll") for (int ks = 0; ks < 4; ++ks) qf[ks] = qn[ks];                          \
            oacc[0] = zero16(); oacc[1] = zero16(); lsum = 0.f; m = -INFINITY;                    \
        }                                                                                              \
        const int k0_ = ((t) < ntA ? (t) : (t) - ntA) * 64;                                            \
        FWD_TILE(Ks, Vs, k0_)                                                                          \
    }
#define FWD_COPY(Kd, Vd, t)                                                                            \
    {                                                                                                  \
        const size_t off_ = (size_t)((t) < ntA ? (t) : (t) - ntA) * 64 * ld;                           \
        tile_copy_async(Kd, kg + off_, ld, wave, lane);                                                \
        tile_copy_async(Vd, vg + off_, ld, wave, lane);                                                \
    }

    const bf16 *kg = base + d, *vg = base + 2 * d;
    FWD_COPY(K0, V0, 0)
    if (ntB > 0) {                                       // this wave's 32 Q rows of the short tile -> its staging area
        rows32_copy_async(Ost + wave * OST_B, base + (size_t)(qtB * 128 + wave * 32) * ld, ld, lane);
    }
    AT_WAIT_VM0();
    __syncthreads();
    for (int t = 0; t < nt; t += 2) {
        if (t + 1 < nt) FWD_COPY(K1, V1, t + 1)
        FWD_STEP(K0, V0, t)
        AT_WAIT_VM0();
        __syncthreads();
        if (t + 1 >= nt) break;
        if (t + 2 < nt) FWD_COPY(K0, V0, t + 2)
        FWD_STEP(K1, V1, t + 1)
        AT_WAIT_VM0();
        __syncthreads();
    }
#undef FWD_COPY
#undef FWD_STEP
#undef FWD_TILE
    fwd_store();
}

// ------------------------------------------------------------------------------------------
// dQ (and delta = rowsum(dO * O), which the dK/dV kernel reads afterwards)
// Bound by the vector work between the products and by the operand rows of each query tile, which nothing hides but
// the CU's other blocks.  So: one copy of the 32 x 32 body (all operand reads of a product issued before its first MFMA;
// a copy per case spilled), LDS offsets formed once per lane, -delta carried into dP as the accumulator's start, the
// mask only on the diagonal half, and Q, dO, O and dQ moved as whole 128-byte lines.  S = 1024, 32 x 16 heads, with the
// dK/dV kernel: 412 -> 372 us.  With copies that the compiler does not wait for in front of the operand reads (see
// AT_GLDS), at 32 x 20 heads: 219 -> 187 us, dK/dV 235 -> 210.  A half's 12 MFMAs (384 cycles) and 16 exponentials with
// what belongs to them (about 520) overlap only between waves, so three blocks share a CU, for which -delta is written to
// the 16 registers of dP's start anew for each half (held over the loop, they make 44 bytes spill): 187 -> 173 us.  The
// dK/dV kernel, with four accumulators, would spill 180 bytes.
__global__ __launch_bounds__(256, 3) void attn_bwd_dq_kernel(const bf16 *__restrict__ qkv, const bf16 *__restrict__ o,
                                                          const bf16 *__restrict__ o_lo,
                                                          const bf16 *__restrict__ dout,
                                                          const float *__restrict__ lse, float *__restrict__ delta,
                                                          bf16 *__restrict__ dqkv, int S, int H, int n_seq)
{
    __shared__ __attribute__((aligned(1024))) unsigned char KV[2][2 * TILE_B];
    __shared__ __attribute__((aligned(1024))) unsigned char Ost[4 * OST_B];
    // block ids decoded as in the forward: the query tiles of a (sequence, head) share an XCD, and a block
    // takes the tiles j and nqt-1-j one after the other so that every block has the same work
    const int nqt = (S + 127) >> 7, npb = (nqt + 1) >> 1;
    const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
    const int pair = (idx / npb) * 8 + xcd;
    if (pair >= H * n_seq) return;
    const int a = pair % H, n = pair / H;
    const int d = H * 64, ld = 3 * d;
    const int tid = threadIdx.x, lane = tid & 63, r32 = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bf16 *base = qkv + (size_t)n * S * ld + a * 64;
    int rm[4], tr[2];
    frag_offsets(lane, rm, tr);
#pragma clang loop unroll(disable)
    for (int ph = 0; ph < 2; ++ph) {
    const int qt = ph == 0 ? nqt - 1 - idx % npb : idx % npb;
    if (ph == 1) {
        if (qt == nqt - 1 - idx % npb) break;            // odd tile count: the middle tile stands alone
        __syncthreads();                                 // the first pass's tiles are no longer read
    }
    const int qb = qt * 128 + wave * 32;
    const bool active = qb < S;
    const int q = qb + r32;

    // first tile, and this wave's rows of Q (its staging area) and dO (the second buffer, still free) as whole lines
    const bf16 *kg = base + d, *vg = base + 2 * d;
    unsigned char *stg = Ost + wave * OST_B, *dO_s = KV[1] + wave * 4096;
    tile_copy_async(KV[0], kg, ld, wave, lane);
    tile_copy_async(KV[0] + TILE_B, vg, ld, wave, lane);
    bf16x8 qf[4], dof[4];
    float lse_q = 0.f, dl = 0.f;
    if (active) {
        rows32_copy_async(stg, base + (size_t)qb * ld, ld, lane);
        rows32_copy_async(dO_s, dout + ((size_t)n * S + qb) * d + a * 64, d, lane);
        // delta = rowsum(dO * O) with O to ~16 bits (o + o_lo): when the value rows of a head share a
        // large common component, dP - delta cancels it, and a delta built from bf16 O alone would not.
        // 8 lanes per row, 8 rows per pass
        const size_t off = ((size_t)n * S + qb + (lane >> 3)) * d + a * 64 + (lane & 7) * 8;
        bf16x8 ov[4], lv[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            ov[p] = *(const bf16x8 *)(o + off + (size_t)(8 * p) * d);
            lv[p] = *(const bf16x8 *)(o_lo + off + (size_t)(8 * p) * d);
        }
        lse_q = lse[((size_t)n * H + a) * S + q];
        AT_WAIT_VM0();
        asm volatile("" ::: "memory");
        float t[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const bf16x8 dv = *(const bf16x8 *)(dO_s + swz128(8 * p + (lane >> 3), lane & 7));
            t[p] = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) t[p] += bf2f(dv[i]) * (bf2f(ov[p][i]) + bf2f(lv[p][i]));
            t[p] += __shfl_xor(t[p], 1, 64);
            t[p] += __shfl_xor(t[p], 2, 64);
            t[p] += __shfl_xor(t[p], 4, 64);
        }
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const float v = __shfl(t[p], (r32 & 7) * 8, 64);
            if ((r32 >> 3) == p) dl = v;
        }
        if (g == 0) delta[((size_t)n * H + a) * S + q] = dl;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            qf[ks] = *(const bf16x8 *)(stg + rm[ks]);
            dof[ks] = *(const bf16x8 *)(dO_s + rm[ks]);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // read before the second buffer is filled
    }
    f32x16 dqacc[2] = {zero16(), zero16()};
    const int kv_end = min(S, qt * 128 + 128);
    const int ntile = kv_end >> 6;

    for (int j = 0; j < ntile; ++j) {
        AT_WAIT_VM0();
        __syncthreads();                                 // tile j has landed and nobody reads the other buffer any more
        if (j + 1 < ntile) {
            tile_copy_async(KV[(j + 1) & 1], kg + (size_t)(j + 1) * 64 * ld, ld, wave, lane);
            tile_copy_async(KV[(j + 1) & 1] + TILE_B, vg + (size_t)(j + 1) * 64 * ld, ld, wave, lane);
        }
        // the tile's 32-key halves at or below the diagonal, one copy of the body for all of them; all operand reads of
        // a product go out before its first MFMA
        const int nhalf = active ? min(max((qb + 32 - j * 64) >> 5, 0), 2) : 0;
#pragma clang loop unroll(disable)
        for (int mt = 0; mt < nhalf; ++mt) {
            const unsigned char *kt_ = KV[j & 1] + mt * 4096, *vt_ = kt_ + TILE_B;
            bf16x8 fk[4], fv[4];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                fk[ks] = *(const bf16x8 *)(kt_ + rm[ks]);
                fv[ks] = *(const bf16x8 *)(vt_ + rm[ks]);
            }
            __builtin_amdgcn_sched_barrier(0);
            // -delta as the addend of the dP product: dP - delta leaves the matrix cores ready (opaque: else it is written
            // out ahead of the loop and held)
            float nd = -dl;
            asm volatile("" : "+v"(nd));
            f32x16 sacc = zero16(), dpacc;
#pragma unroll
            for (int e = 0; e < 16; ++e) dpacc[e] = nd;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fk[ks], qf[ks], sacc, 0, 0, 0);
                dpacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fv[ks], dof[ks], dpacc, 0, 0, 0);
            }
            bf16x8 ft[2][2];
#pragma unroll
            for (int hh = 0; hh < 2; ++hh)
#pragma unroll
                for (int dt = 0; dt < 2; ++dt) ft[hh][dt] = read_tr(kt_ + hh * 2048 + tr[dt]);
            __builtin_amdgcn_sched_barrier(0);
            if (j * 64 + mt * 32 == qb) {                // the half on the diagonal: keys behind the query leave nothing
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    if (8 * (e >> 2) + 4 * g + (e & 3) > r32) sacc[e] = -INFINITY;
            }
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                bf16x8 dsb;
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    dsb[i] = f2bf(__builtin_amdgcn_exp2f(fmaf(sacc[8 * hh + i], kScaleLog2, -lse_q)) * dpacc[8 * hh + i]);
#pragma unroll
                for (int dt = 0; dt < 2; ++dt)
                    dqacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ft[hh][dt], dsb, dqacc[dt], 0, 0, 0);
            }
        }
    }

    if (active) store_rows32(stg, dqacc, 0.125f, dqkv + ((size_t)n * S + qb) * ld + a * 64, ld, lane);
    }   // pass
}

// ------------------------------------------------------------------------------------------
// dK, dV: each wavefront owns 32 keys and walks the query tiles that can see them (bound and layout as in the dQ kernel)
__global__ __launch_bounds__(256, 2) void attn_bwd_dkv_kernel(const bf16 *__restrict__ qkv,
                                                           const bf16 *__restrict__ dout,
                                                           const float *__restrict__ lse,
                                                           const float *__restrict__ delta,
                                                           bf16 *__restrict__ dqkv, int S, int H, int n_seq)
{
    __shared__ __attribute__((aligned(1024))) unsigned char QD[2][2 * TILE_B];
    __shared__ __attribute__((aligned(1024))) unsigned char Ost[4 * OST_B];
    __shared__ __align__(16) float st[2][128];           // lse | -delta of the 64 queries of a tile
    // block ids decoded as in the forward: the key tiles of a (sequence, head) share an XCD, and a block takes
    // the tiles j (most query tiles to walk) and nkt-1-j one after the other: equal work per block
    const int nkt = (S + 127) >> 7, npb = (nkt + 1) >> 1;
    const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
    const int pair = (idx / npb) * 8 + xcd;
    if (pair >= H * n_seq) return;
    const int a = pair % H, n = pair / H;
    const int d = H * 64, ld = 3 * d;
    const int tid = threadIdx.x, lane = tid & 63, r32 = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bf16 *base = qkv + (size_t)n * S * ld + a * 64;
    const bf16 *dbase = dout + (size_t)n * S * d + a * 64;
    const float *lse_b = lse + ((size_t)n * H + a) * S, *dl_b = delta + ((size_t)n * H + a) * S;
    int rm[4], tr[2];
    frag_offsets(lane, rm, tr);
#pragma clang loop unroll(disable)
    for (int ph = 0; ph < 2; ++ph) {
    const int kvt = ph == 0 ? idx % npb : nkt - 1 - idx % npb;
    if (ph == 1) {
        if (kvt == idx % npb) break;                     // odd tile count: the middle tile stands alone
        __syncthreads();                                 // the first pass's tiles and statistics are no longer read
    }
    const int kb = kvt * 128 + wave * 32;
    const bool active = kb < S;
    const int key = kb + r32;

    f32x16 dkacc[2] = {zero16(), zero16()}, dvacc[2] = {zero16(), zero16()};
    const int q_first = kvt * 128;
    const int ntile = (S - q_first) >> 6;

    // per-query statistics travel through a register so that their LDS store (which has to wait for the load) sits
    // after the MFMA work of the current tile
    float stat = 0.f;
    auto issue = [&](int j) {
        const int q0 = q_first + j * 64;
        tile_copy_async(QD[j & 1], base + (size_t)q0 * ld, ld, wave, lane);
        tile_copy_async(QD[j & 1] + TILE_B, dbase + (size_t)q0 * d, d, wave, lane);
        if (tid < 128) stat = (tid < 64 ? lse_b : dl_b - 64)[q0 + tid];      // (the sign of delta: at the store, behind the wait)
    };
    issue(0);
    // this wave's rows of K (its staging area) and V (the second buffer, still free) as whole lines
    unsigned char *stg = Ost + wave * OST_B, *v_s = QD[1] + wave * 4096;
    bf16x8 kf[4], vf[4];
    if (active) {
        rows32_copy_async(stg, base + d + (size_t)kb * ld, ld, lane);
        rows32_copy_async(v_s, base + 2 * d + (size_t)kb * ld, ld, lane);
    }
    if (tid < 128) st[0][tid] = tid < 64 ? stat : -stat;
    AT_WAIT_VM0();
    asm volatile("" ::: "memory");
    if (active) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            kf[ks] = *(const bf16x8 *)(stg + rm[ks]);
            vf[ks] = *(const bf16x8 *)(v_s + rm[ks]);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // read before the second buffer is filled
    }
    for (int j = 0; j < ntile; ++j) {
        AT_WAIT_VM0();
        __syncthreads();                                 // tile j has landed and nobody reads the other buffer any more
        if (j + 1 < ntile) issue(j + 1);
        // the tile's 32-query halves at or above this wave's keys, one copy of the body for all of them
        const int h0 = active ? min(max((kb - q_first - j * 64) >> 5, 0), 2) : 2;
#pragma clang loop unroll(disable)
        for (int hf = h0; hf < 2; ++hf) {
            const unsigned char *qt_ = QD[j & 1] + hf * 4096, *dt_ = qt_ + TILE_B;
            const float *sl = st[j & 1] + 32 * hf + 4 * g;
            bf16x8 fq[4], fd[4];
            f32x4 ls[4];
            f32x16 sacc = zero16(), dpacc;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                fq[ks] = *(const bf16x8 *)(qt_ + rm[ks]);
                fd[ks] = *(const bf16x8 *)(dt_ + rm[ks]);
            }
            // -delta as the addend of the dP product: dP - delta leaves the matrix cores ready
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4) {
                ls[e4] = *(const f32x4 *)(sl + 8 * e4);
                const f32x4 dd = *(const f32x4 *)(sl + 64 + 8 * e4);
#pragma unroll
                for (int i = 0; i < 4; ++i) dpacc[4 * e4 + i] = dd[i];
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fq[ks], kf[ks], sacc, 0, 0, 0);
                dpacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fd[ks], vf[ks], dpacc, 0, 0, 0);
            }
            bf16x8 tq[2][2], td[2][2];
#pragma unroll
            for (int hh = 0; hh < 2; ++hh)
#pragma unroll
                for (int dt = 0; dt < 2; ++dt) {
                    td[hh][dt] = read_tr(dt_ + hh * 2048 + tr[dt]);
                    tq[hh][dt] = read_tr(qt_ + hh * 2048 + tr[dt]);
                }
            __builtin_amdgcn_sched_barrier(0);
            if (q_first + j * 64 + hf * 32 == kb) {      // the half on the diagonal
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    if (r32 > 8 * (e >> 2) + 4 * g + (e & 3)) sacc[e] = -INFINITY;
            }
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                bf16x8 pb, dsb;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int e = 8 * hh + i;
                    const float p = __builtin_amdgcn_exp2f(fmaf(sacc[e], kScaleLog2, -ls[e >> 2][e & 3]));
                    pb[i] = f2bf(p);
                    dsb[i] = f2bf(p * dpacc[e]);
                }
#pragma unroll
                for (int dt = 0; dt < 2; ++dt) {
                    dvacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(td[hh][dt], pb, dvacc[dt], 0, 0, 0);
                    dkacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tq[hh][dt], dsb, dkacc[dt], 0, 0, 0);
                }
            }
        }
        if (j + 1 < ntile && tid < 128) st[(j + 1) & 1][tid] = tid < 64 ? stat : -stat;
    }

    if (active) {
        bf16 *out = dqkv + ((size_t)n * S + kb) * ld + d + a * 64;
        store_rows32(stg, dkacc, 0.125f, out, ld, lane);
        store_rows32(stg, dvacc, 1.0f, out + d, ld, lane);
    }
    }   // pass
}

// ------------------------------------------------------------------------------------------
// Fused backward for sequences of at most 512 tokens: one block of 8 wavefronts per (sequence, head)
// produces dQ, dK and dV in one pass, so the scores, the probabilities and dP are formed once instead
// of once per kernel, and K, V, Q, dO are read from memory once.
//   * K of the whole sequence sits in LDS; every wave owns two 32-key blocks (w and nb-1-w, which
//     balances the causal triangle; one where there are no more blocks than waves: S = 128 with two blocks on two
//     of the waves took 13.6 us), keeps their V fragments and their dK, dV accumulators in
//     registers, and walks the 32-query tiles that can see them (phase 1, as in the dK/dV kernel).
//   * dS of a query tile is written to LDS as dS^T [key][32 queries] bf16; after one barrier the 8
//     waves each form one 16 x 16 piece of dQ = dS K over all visible keys (phase 2), in a fixed
//     order -- no floating-point atomics, results stay bit-reproducible.
//   * Q / dO tiles (4 KB each) are double buffered asynchronous copies that also bring the tile's 32 K rows,
//     dS^T is double buffered too, so there is one barrier per query tile: phase 2 of tile i runs next to
//     phase 1 of tile i + 1.
//   * Before the arithmetic starts the block waits for two rounds of memory traffic: the first tile with lse (whose LDS store
//     stands in front of the other loads), then the wave's V fragments and delta, or the operands of delta =
//     rowsum(dO * O) of all rows, every load of which is issued before the first is used.  (All blocks of a launch run in
//     step, so these rounds are read by every
//     compute unit at once, at the memory's speed, with the matrix cores idle; forming delta tile by tile
//     behind the arithmetic, from rows streamed into LDS, was measured and only moved the same time into the
//     steps, whose length is set by the latency of the tile copies.)
//   * The two blocks' accumulators and V fragments leave 96 registers.  With an address register for every buffer and
//     offset, 84 bytes of V were spilled, and each reload waited for the copies in flight; offsets formed once per lane
//     and buffers as scalars: 216 -> 189 us (S = 512, 64 x 16 heads), 12.3 -> 9.0 (S = 128, 12 heads).
//   * The limit of 512 tokens is what K, dS^T and the tiles take of LDS.  From 257 on the split pair could run too (and the product
//     that forms dO would not have to form delta): whole rounds, 64 x 16 heads of 512 tokens 38.16 ms with this kernel, 38.62
//     with the pair; 20 x 12 of 512 4.860, 4.867; 12 x 16 of 448 9.88, 10.01; 8 x 16 of 512, a block on every other CU, 2.276,
//     2.237.  The line may not depend on the number of heads, else a sequence's bits would on its batch.
constexpr int FB_MAXS = 512;

// XOR mask of the 8-byte slots of a dS^T row (64 bytes = 32 queries): conflict-free both for the
// phase-1 stores (16 lanes = 16 consecutive keys, one slot) and for the phase-2 transpose reads
// (16 lanes = 4 consecutive keys x 4 slots)
__device__ __forceinline__ int dsm(int key) { return (((key >> 1) & 1) << 2) | ((key >> 2) & 3); }

constexpr int FB_TILE = 32 * 128;
__global__ __launch_bounds__(512) void attn_bwd_fused_kernel(const bf16 *__restrict__ qkv, const bf16 *__restrict__ o,
                                                             const bf16 *__restrict__ o_lo,
                                                             const bf16 *__restrict__ dout,
                                                             const float *__restrict__ lse, bf16 *__restrict__ dqkv,
                                                             int S, int H, const float *__restrict__ delta_in)
{
    __shared__ __attribute__((aligned(1024))) unsigned char Ks[FB_MAXS * 128];
    __shared__ __attribute__((aligned(1024))) unsigned char dS0[FB_MAXS * 64], dS1[FB_MAXS * 64];
    __shared__ __attribute__((aligned(1024))) unsigned char QD0[2 * FB_TILE], QD1[2 * FB_TILE];      // a tile of Q, then of dO
    __shared__ __align__(16) float lse_s[2 * FB_MAXS];                                               // lse, then delta
    float *const dl_s = lse_s + FB_MAXS;
    const int a = blockIdx.x, n = blockIdx.y;
    const int d = H * 64, ld = 3 * d;
    const int tid = threadIdx.x, lane = tid & 63, r32 = lane & 31, g = lane >> 5;
    const int i16 = lane & 15, kg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bf16 *base = qkv + (size_t)n * S * ld + a * 64;
    const bf16 *dbase = dout + (size_t)n * S * d + a * 64;
    const int nb = S >> 5;                               // 32-row blocks (even: S is a multiple of 64)

    // one 1 KB piece per wave and tile of Q (waves 0-3) and dO (waves 4-7), and the tile's 32 K rows (waves 0-3)
#define FB_COPY(QD, it)                                                                                \
    {                                                                                                  \
        const int lrow_c = lane >> 3, lch_c = (lane & 7) ^ swm(lane >> 3);                             \
        const int row_c = 32 * (it) + (wave & 3) * 8;                                                  \
        if (wave < 4) {                                                                                \
            const unsigned off_c = (unsigned)(lrow_c * ld + lch_c * 8) * 2u;                           \
            AT_GLDS(base + (size_t)row_c * ld, off_c, (QD) + (wave & 3) * 1024);                       \
            AT_GLDS(base + d + (size_t)row_c * ld, off_c, Ks + (it) * 4096 + (wave & 3) * 1024);       \
        } else AT_GLDS(dbase + (size_t)row_c * d, (unsigned)(lrow_c * d + lch_c * 8) * 2u, (QD) + FB_TILE + (wave & 3) * 1024); \
    }
    // ---- prologue: first tile (Q, dO, K rows), log-sum-exp and delta of all rows, this wave's V fragments
    FB_COPY(QD0, 0)
    if (tid < S) lse_s[tid] = lse[((size_t)n * H + a) * S + tid];
    // up to 8 key blocks (256 tokens) every wave owns one at most; waves without a block only do phase 2
    const bool single = nb <= 8;
    const bool owner = wave < (single ? nb : nb >> 1);
    const int jb[2] = {wave, single ? FB_MAXS : nb - 1 - wave};          // (no tile reaches block FB_MAXS)
    bf16x8 vf[2][4];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int key = min(32 * jb[b] + r32, S - 1);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
            vf[b][ks] = *(const bf16x8 *)(base + 2 * d + (size_t)(owner ? key : 0) * ld + ks * 16 + g * 8);
    }
    // delta = rowsum(dO * (O + O_lo)): [T, H] from the product that formed dO (its epilogue has dO in registers
    // and reads O there, which saves this kernel a second pass over dO and half of its prologue's traffic), or
    if (delta_in != nullptr) {
        if (tid < S) dl_s[tid] = delta_in[((size_t)n * S + tid) * H + a];
    } else {
        // formed here: 8 lanes per row (16 bytes each, one full 128-byte line per row and
        // operand), 64 rows per pass, reduced with three shuffles; the loads of all passes go out first
        bf16x8 dv[FB_MAXS / 64], ov[FB_MAXS / 64], lv[FB_MAXS / 64];
        const size_t off_d = ((size_t)n * S + (tid >> 3)) * d + a * 64 + (tid & 7) * 8;
#pragma unroll
        for (int ps = 0; ps < FB_MAXS / 64; ++ps)
            if (64 * ps < S) {
                dv[ps] = *(const bf16x8 *)(dout + off_d + (size_t)64 * ps * d);
                ov[ps] = *(const bf16x8 *)(o + off_d + (size_t)64 * ps * d);
                lv[ps] = *(const bf16x8 *)(o_lo + off_d + (size_t)64 * ps * d);
            }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ps = 0; ps < FB_MAXS / 64; ++ps)
            if (64 * ps < S) {
                float dl = 0.f;
#pragma unroll
                for (int i = 0; i < 8; ++i) dl += bf2f(dv[ps][i]) * (bf2f(ov[ps][i]) + bf2f(lv[ps][i]));
                dl += __shfl_xor(dl, 1, 64);
                dl += __shfl_xor(dl, 2, 64);
                dl += __shfl_xor(dl, 4, 64);
                if ((tid & 7) == 0) dl_s[64 * ps + (tid >> 3)] = dl;
            }
    }
    f32x16 dkacc[2][2], dvacc[2][2];
    // lane offsets of the operand reads and of the dS^T stores (row r32: its swizzle does not look above bit 3); the
    // buffers come in as scalars that the compiler cannot see through, else it keeps the sum of each with each offset
    int rm[4], tr[2];
    frag_offsets(lane, rm, tr);
    const unsigned ds_st = r32 * 64 + ((g ^ dsm(r32)) << 3);
    // phase 1 for query tile `it` (rows 32 it ..) against this wave's blocks that it can see.  Only the
    // block on the diagonal (j == it) needs the causal mask; the blocks below it run a copy without it.
#define FB_BLOCK(QD, dSw, it, b, j, DIAG)                                                              \
    {                                                                                                  \
        f32x16 sacc = zero16(), dpacc = zero16();                                                      \
        unsigned s_q = lds_addr(QD), s_k = lds_addr(Ks) + (j) * 4096, s_l = lds_addr(lse_s) + (it) * 128, \
                 s_d = lds_addr(dSw) + (j) * 2048;                                                     \
        asm volatile("" : "+s"(s_q), "+s"(s_k), "+s"(s_l), "+s"(s_d));                                 \
        _Pragma("unroll") for (int ks = 0; ks < 4; ++ks) {                                             \
            const unsigned aq = s_q + rm[ks];                                                          \
            sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_b128(aq), lds_b128(s_k + rm[ks]), sacc, 0, 0, 0); \
            dpacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_b128(aq + FB_TILE), vf[b][ks], dpacc, 0, 0, 0); \
        }                                                                                              \
        const unsigned al = s_l + 16 * g, ad = s_d + ds_st;                                            \
        _Pragma("unroll") for (int e4 = 0; e4 < 4; ++e4) {                                             \
            const int ql = 8 * e4 + 4 * g;                                                             \
            const f32x4 ls = *(const __attribute__((address_space(3))) f32x4 *)(al + 32 * e4);         \
            const f32x4 dd = *(const __attribute__((address_space(3))) f32x4 *)(al + 32 * e4 + FB_MAXS * 4); \
            bf16x4 dst4;                                                                               \
            _Pragma("unroll") for (int i = 0; i < 4; ++i) {                                            \
                const int e = 4 * e4 + i;                                                              \
                float p = __builtin_amdgcn_exp2f(fmaf(sacc[e], kScaleLog2, -ls[i]));                   \
                if (DIAG && r32 > ql + i) p = 0.f;                                                     \
                sacc[e] = p;                                                                           \
                dpacc[e] = p * (dpacc[e] - dd[i]);                                                     \
                dst4[i] = f2bf(dpacc[e]);                                                              \
            }                                                                                          \
            *(__attribute__((address_space(3))) bf16x4 *)(ad ^ (e4 << 4)) = dst4;                      \
        }                                                                                              \
        _Pragma("unroll") for (int hh = 0; hh < 2; ++hh) {                                             \
            bf16x8 pb, dsb;                                                                            \
            _Pragma("unroll") for (int i = 0; i < 8; ++i) {                                            \
                pb[i] = f2bf(sacc[8 * hh + i]);                                                        \
                dsb[i] = f2bf(dpacc[8 * hh + i]);                                                      \
            }                                                                                          \
            _Pragma("unroll") for (int dt = 0; dt < 2; ++dt) {                                         \
                const unsigned at = s_q + tr[dt] + 2048 * hh;                                          \
                dvacc[b][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_tr(at + FB_TILE), pb, dvacc[b][dt], 0, 0, 0); \
                dkacc[b][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_tr(at), dsb, dkacc[b][dt], 0, 0, 0); \
            }                                                                                          \
        }                                                                                              \
    }
#define FB_PHASE1(QD, dSw, it)                                                                         \
    if (owner) {                                                                                       \
        _Pragma("unroll") for (int b = 0; b < 2; ++b) {                                                \
            const int j = jb[b];                                                                       \
            if (j <= (it)) { const bool diag = j == (it); FB_BLOCK(QD, dSw, it, b, j, diag) }          \
            __builtin_amdgcn_sched_barrier(0);           /* keep the two blocks' live ranges apart */   \
        }                                                                                              \
    }
    // phase 2 for query tile `it`: wave w forms dQ[16 qt .. +15][16 dt .. +15], qt = w / 4, dt = w % 4,
    // as (K^T dS^T)^T over all visible keys; the lane ends up with 4 consecutive columns of one query
    // The rows a lane reads are 32 kk + (a lane constant below 32) and neither swizzle looks above bit 3 of
    // the row, so everything but the 32 kk step is formed once here (left in the loop the compiler rebuilt the
    // swizzles for every key block: 17 VALU instructions per MFMA).
    const int p2_qt = wave >> 2, p2_dt = wave & 3;
    int p2_k[2], p2_d[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int row = 8 * kg + 4 * h + (i16 >> 2);
        const int colk = 16 * p2_dt + 4 * (i16 & 3);
        p2_k[h] = row * 128 + (((colk >> 3) ^ swm(row)) << 4) + (colk & 7) * 2;
        p2_d[h] = row * 64 + (((4 * p2_qt + (i16 & 3)) ^ dsm(row)) << 3);
    }
#define FB_PHASE2(dSr, it)                                                                             \
    {                                                                                                  \
        f32x4 qacc = {0.f, 0.f, 0.f, 0.f};                                                             \
        _Pragma("unroll 2") for (int kk = 0; kk <= (it); ++kk) {                                       \
            union { v4s s[2]; bf16x8 v; } ua, ub;                                                      \
            _Pragma("unroll") for (int h = 0; h < 2; ++h) {                                            \
                const unsigned char *pk = Ks + kk * 4096 + p2_k[h];                                    \
                const unsigned char *pd = (dSr) + kk * 2048 + p2_d[h];                                 \
                ua.s[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s *)pk); \
                ub.s[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s *)pd); \
            }                                                                                          \
            qacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ua.v, ub.v, qacc, 0, 0, 0);                 \
        }                                                                                              \
        const int q = 32 * (it) + 16 * p2_qt + i16;                                                    \
        bf16x4 w4;                                                                                     \
        _Pragma("unroll") for (int e = 0; e < 4; ++e) w4[e] = f2bf(qacc[e] * 0.125f);                  \
        *(bf16x4 *)(dqkv + ((size_t)n * S + q) * ld + a * 64 + 16 * p2_dt + 4 * kg) = w4;              \
    }

    AT_WAIT_VM0();
    __syncthreads();                                     // tile 0, its K rows and the statistics it needs are in LDS
    if (nb > 1) FB_COPY(QD1, 1)
#pragma unroll
    for (int b = 0; b < 2; ++b) { dkacc[b][0] = zero16(); dkacc[b][1] = zero16(); dvacc[b][0] = zero16(); dvacc[b][1] = zero16(); }
    FB_PHASE1(QD0, dS0, 0)
    for (int it = 0; it < nb; it += 2) {
        AT_WAIT_VM0();
        __syncthreads();                                 // dS^T of tile it complete; tile it + 1 and its K rows landed
        if (it + 2 < nb) FB_COPY(QD0, it + 2)
        FB_PHASE2(dS0, it)
        if (it + 1 < nb) FB_PHASE1(QD1, dS1, it + 1)
        if (it + 1 < nb) {
            AT_WAIT_VM0();
            __syncthreads();
            if (it + 3 < nb) FB_COPY(QD1, it + 3)
            FB_PHASE2(dS1, it + 1)
            if (it + 2 < nb) FB_PHASE1(QD0, dS0, it + 2)
        }
    }
#undef FB_COPY
#undef FB_PHASE1
#undef FB_BLOCK
#undef FB_PHASE2

    // dK, dV of the two key blocks leave through LDS (the dS^T buffers, free after one more barrier) as whole
    // 128-byte lines: a lane holds 4 consecutive columns of one key per register group, direct stores would
    // touch 32 lines per instruction with 8 bytes each
    __syncthreads();
    if (owner) {
        unsigned char *stg = wave < 4 ? dS0 + wave * OST_B : dS1 + (wave - 4) * OST_B;      // 4.5 KB per wave
        const int orow = lane >> 3, och = lane & 7;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            if (b == 1 && single) break;
            bf16 *out = dqkv + ((size_t)n * S + 32 * jb[b] + orow) * ld + d + a * 64 + och * 8;
#pragma unroll
            for (int which = 0; which < 2; ++which) {     // 0: dK (scaled), 1: dV
#pragma unroll
                for (int dt = 0; dt < 2; ++dt)
#pragma unroll
                    for (int e4 = 0; e4 < 4; ++e4) {
                        bf16x4 w;
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            w[i] = which ? f2bf(dvacc[b][dt][4 * e4 + i]) : f2bf(dkacc[b][dt][4 * e4 + i] * 0.125f);
                        *(bf16x4 *)(stg + r32 * OST_PITCH + (32 * dt + 8 * e4 + 4 * g) * 2) = w;
                    }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                bf16x8 rows[4];
#pragma unroll
                for (int it = 0; it < 4; ++it)
                    rows[it] = *(const bf16x8 *)(stg + (8 * it + orow) * OST_PITCH + och * 16);
#pragma unroll
                for (int it = 0; it < 4; ++it) *(bf16x8 *)(out + (size_t)(8 * it) * ld + which * d) = rows[it];
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
        }
    }
}

}  // namespace

int launch_attn_fwd(const bf16 *qkv, bf16 *o, bf16 *o_lo, float *lse, int n_seq, int S, int H, hipStream_t st)
{
    if (n_seq <= 0 || S <= 0 || (S % 64) || H <= 0) return SL_EINVAL;
    const long long pairs8 = ((long long)H * n_seq + 7) / 8 * 8;
    const long long nblk = pairs8 * (((S + 127) / 128 + 1) / 2);     // two query tiles of 128 per block
    if (nblk > 0x7fffffffLL) return SL_EINVAL;
    // algorithmic work: two products over the lower triangle, 2 S d flop per token (d = 64 H)
    const bool rec = prof_begin(PK_ATTN_FWD, st);
    hipLaunchKernelGGL(attn_fwd_kernel, dim3((unsigned)nblk), dim3(256), 0, st, qkv, o, o_lo, lse, S, H, n_seq);
    prof_end(rec, PK_ATTN_FWD, 2.0 * S * 64.0 * H * ((double)n_seq * S), st);
    SL_CHECK_LAUNCH("attn_fwd");
    return 0;
}

bool attn_bwd_takes_delta(int S) { return S > 0 && S <= FB_MAXS && (S % 64) == 0; }

int launch_attn_bwd(const bf16 *qkv, const bf16 *o, const bf16 *o_lo, const bf16 *dout, const float *lse,
                    float *delta, bf16 *dqkv, int n_seq, int S, int H, hipStream_t st, bool delta_ready)
{
    if (delta_ready && !attn_bwd_takes_delta(S)) return SL_EINVAL;
    if (n_seq <= 0 || S <= 0 || (S % 64) || H <= 0) return SL_EINVAL;
    // algorithmic work: four products over the lower triangle (the recomputed scores are not counted)
    const double work = 4.0 * S * 64.0 * H * ((double)n_seq * S);
    const bool rec = prof_begin(PK_ATTN_BWD, st);
    if (S <= FB_MAXS) {
        hipLaunchKernelGGL(attn_bwd_fused_kernel, dim3(H, n_seq), dim3(512), 0, st, qkv, o, o_lo, dout, lse, dqkv, S, H,
                           delta_ready ? (const float *)delta : nullptr);
        prof_end(rec, PK_ATTN_BWD, work, st);
        SL_CHECK_LAUNCH("attn_bwd_fused");
        return 0;
    }
    const long long pairs8 = ((long long)H * n_seq + 7) / 8 * 8;
    const long long nblk = pairs8 * (((S + 127) / 128 + 1) / 2);     // two tiles of 128 rows per block
    if (nblk > 0x7fffffffLL) return SL_EINVAL;
    const dim3 grid((unsigned)nblk);
    hipLaunchKernelGGL(attn_bwd_dq_kernel, grid, dim3(256), 0, st, qkv, o, o_lo, dout, lse, delta, dqkv, S, H, n_seq);
    SL_CHECK_LAUNCH("attn_bwd_dq");
    hipLaunchKernelGGL(attn_bwd_dkv_kernel, grid, dim3(256), 0, st, qkv, dout, lse, delta, dqkv, S, H, n_seq);
    prof_end(rec, PK_ATTN_BWD, work, st);
    SL_CHECK_LAUNCH("attn_bwd_dkv");
    return 0;
}
