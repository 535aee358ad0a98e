// Single-precision LoRA-adapted linear layer (SplitLoRA Sec. II-C), forward and backward.
//
// Every operand and every sum is fp32: the frozen product and the rank-space projections run on the fp32 matrix
// instruction (V_MFMA_F32_16X16X4_F32: fp32 operands, fp32 accumulation, the same rate as packed vector FMAs but
// one instruction per 1024 of them), the adapter gradients on vector FMAs.  Each sum has one fixed order, so
// results are reproducible.
//
//   forward   z = x A^T                                 f32_project_kernel
//             y = x W^T + bias + s z B^T                f32_tile_kernel / f32_gemm_kernel / f32_gemm_direct_kernel
//   backward  z = x A^T, p = dy B                       f32_project_kernel (both in one launch)
//             dx = dy W + s p A                         the same product kernels, W read as [k, n]
//             dA = s p^T x, dB = s dy^T z               f32_grad_kernel (both in one launch)
//
// At T = 1024, 768 -> 768, r = 4 (2.5 GFLOP, 15 MB: 16 us at the fp32 matrix rate) forward + backward took 1113 us
// as nine launches of one vector-FMA kernel: single floats moved one by one, the rank-4 products as mostly empty 64 x 64
// tiles, the adapter gradients as 12 blocks that walk all tokens.  Five launches of the kernels below: 47 us (59 before the
// products that fill the chip took the ring kernel).
#include "common.h"
#include "gemm_copy.h"
#include <type_traits>

// the tile of a product's kernel and the stages of its ring of copies (0: a kernel without one); vec: operands of 16-byte rows
struct F32Plan { int tm, tn, stages; };
extern "C" F32Plan plan_f32(int M, int N, int K, bool vec);

namespace {

constexpr int BK = 32;                       // contraction elements per LDS slab
constexpr int KP = BK + 4;                   // pitch of an LDS row with the contraction contiguous: 16 rows x 16 bytes hit 64 banks

// four floats of a row at offset o, zeros from offset `lim` on (VEC: both multiples of 4; no branch around the load, which
// would make the compiler drain every load in flight)
template <bool VEC>
__device__ __forceinline__ float4 load4_lim(const float *__restrict__ row, int o, int lim)
{
    if (VEC) {
        float4 v = *(const float4 *)(row + max(min(o, lim - 4), 0));
        const bool in = o < lim;
        return make_float4(in ? v.x : 0.f, in ? v.y : 0.f, in ? v.z : 0.f, in ? v.w : 0.f);
    }
    float4 v;
    v.x = o < lim ? row[o] : 0.f;
    v.y = o + 1 < lim ? row[o + 1] : 0.f;
    v.z = o + 2 < lim ? row[o + 2] : 0.f;
    v.w = o + 3 < lim ? row[o + 3] : 0.f;
    return v;
}

// The same in two parts, so that nothing waits for the load where it is issued: the load from a clamped offset, and the
// zeros for what lies beyond the limit when the values are used.
template <bool VEC>
__device__ __forceinline__ float4 load4_clamped(const float *__restrict__ row, int o, int lim)
{
    if (VEC) return *(const float4 *)(row + max(min(o, lim - 4), 0));
    return load4_lim<false>(row, o, lim);
}
__device__ __forceinline__ float4 zero_beyond(float4 v, bool in)
{
    return make_float4(in ? v.x : 0.f, in ? v.y : 0.f, in ? v.z : 0.f, in ? v.w : 0.f);
}

// k-index convention of every operand fragment: a lane (m = lane%16, g = lane/16) holds k = 16 i + 4 g .. + 3 in one
// float4 and feeds component c to the c-th of four MFMAs.  Both operands use it, so each product meets its partner.
__device__ __forceinline__ void mfma4(f32x4 &acc, const float4 &a, const float4 &b)
{
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b.x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, b.y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, b.z, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, b.w, acc, 0, 0, 0);
}

// ---- rank-space projections -------------------------------------------------------------------------------------
// out[t][j] = sum_k X[t][k] Z(j,k), j < zp (rows r .. zp-1 of Z are zero).  One block per 16 tokens, the contraction
// split over 8 waves whose partial tiles are added in wave order.  Bound by reading X (latency at small T).
struct ProjJob { const float *X; const float *Z; long zj, zk; int K; float *out; };
struct ProjJobs { ProjJob j[2]; };

template <bool VEC>
__global__ __launch_bounds__(512) void f32_project_kernel(ProjJobs jobs, int T, int r, int zp)
{
    __shared__ float red[8][16][17];
    const ProjJob &jb = jobs.j[blockIdx.y];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r16 = lane & 15, g = lane >> 4;
    const int t0 = blockIdx.x * 16, K = jb.K;
    const float *xr = jb.X + (size_t)min(t0 + r16, T - 1) * K;
    const bool zok = r16 < r;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    const int steps = (K + 15) >> 4, per = (steps + 7) >> 3;
    const int s0 = wave * per, s1 = min(s0 + per, steps);
    for (int s = s0; s < s1; ++s) {
        const int k = s * 16 + 4 * g;
        const float4 a = load4_lim<VEC>(xr, k, K);
        float4 b = make_float4(0.f, 0.f, 0.f, 0.f);
        if (zok) {
            if (VEC && jb.zk == 1) b = load4_lim<true>(jb.Z + (size_t)r16 * jb.zj, k, K);
            else {
                const float *q = jb.Z + (size_t)r16 * jb.zj + (size_t)k * jb.zk;
                b.x = k < K ? q[0] : 0.f;
                b.y = k + 1 < K ? q[jb.zk] : 0.f;
                b.z = k + 2 < K ? q[2 * jb.zk] : 0.f;
                b.w = k + 3 < K ? q[3 * jb.zk] : 0.f;
            }
        }
        mfma4(acc, a, b);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) red[wave][4 * g + e][r16] = acc[e];
    __syncthreads();
    if (threadIdx.x < 256) {
        const int m = threadIdx.x >> 4, j = threadIdx.x & 15;
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < 8; ++w) v += red[w][m][j];
        // zero beyond the rank also where an infinity met a zero of Z
        if (t0 + m < T && j < zp) jb.out[(size_t)(t0 + m) * zp + j] = j < r ? v : 0.f;
    }
}

// ---- frozen product + low-rank term -------------------------------------------------------------------------------
// C[m,n] = sum_k A[m,k] B(k,n) + bias[n] + s sum_j z[m,j] U(j,n)
// A [M,K] dense; B is [N,K] dense (BT) or [K,N] dense; z [M,zp]; U(j,n) = U[j uj + n un].
struct GemmF32 {
    const float *A, *B, *bias, *z, *U;
    float *C;
    int M, N, K, zp, r;
    long uj, un;
    float s;
};

// The low-rank term is one more step of 16 contraction elements: operand fragments z[m, 4g ..] and U(4g .., n), zero
// beyond the rank.  They are requested before the main loop, whose last step they follow.  Its sum is formed on its own and
// added, scaled, in one rounding, after the bias: in the accumulators it would cost one more rounding at the size of the result for every element of the rank
// (r = 16: 1.37 times the error at n_in = 16, 1.016 times at 768).
__device__ __forceinline__ float4 up_frag_z(const GemmF32 &a, int m, int g)
{
    if (4 * g >= a.zp) return make_float4(0.f, 0.f, 0.f, 0.f);
    return *(const float4 *)(a.z + (size_t)m * a.zp + 4 * g);
}
__device__ __forceinline__ float4 up_frag_u(const GemmF32 &a, int n, int g)
{
    const float *q = a.U + (size_t)n * a.un + (size_t)(4 * g) * a.uj;
    float4 v;
    v.x = 4 * g < a.r ? q[0] : 0.f;
    v.y = 4 * g + 1 < a.r ? q[a.uj] : 0.f;
    v.z = 4 * g + 2 < a.r ? q[2 * a.uj] : 0.f;
    v.w = 4 * g + 3 < a.r ? q[3 * a.uj] : 0.f;
    return v;
}

// TM x TN tile per block, KS groups of 4 waves (2 x 2) that take the slabs of the contraction in turn, each with two LDS
// stages of its own; a group's next slab is on its way from memory in registers while the matrix cores work on the
// current one, and the groups' accumulators are added in group order at the end.  With one tile per CU a slab costs a
// memory round trip, not its arithmetic, which a second group hides; 128 x 128 tiles halve the operand traffic where there are
// enough of them.  For contractions that are no multiple of 64 and rows that are no whole float4s; the figures it was chosen by
// are from when it ran all products: T = 1024, 768 -> 768 in 64.6 us forward + backward with one group, 59.2 with two (22 us per
// product, 55 TFLOP/s), 58.9 with four, which were slower at T = 4096; 96 TFLOP/s at T = 8192, 1280 -> 5120.
template <int TM, int TN, int KS, bool BT, bool VEC>
__global__ __launch_bounds__(256 * KS) void f32_gemm_kernel(GemmF32 a)
{
    constexpr int NP = TN + 4;                           // pitch of a [k][n] slab: the four k-groups of a read are 16 banks apart
    constexpr int ASZ = TM * KP, BSZ = BT ? TN * KP : BK * NP;
    constexpr int MI = TM / 32, NI = TN / 32;
    constexpr int LA = TM * BK / 1024, LB = TN * BK / 1024;          // float4 per thread and slab
    __shared__ __attribute__((aligned(16))) float lds[KS][2][ASZ + BSZ];
    static_assert(KS == 1 || 2 * (ASZ + BSZ) >= MI * NI * 4 * 256, "a group's stages hold its accumulators");
    const int tid = threadIdx.x & 255, lane = tid & 63, wave = tid >> 6, r16 = lane & 15, g = lane >> 4;
    const int grp = threadIdx.x >> 8;
    const int wm = wave >> 1, wn = wave & 1;
    // blocks go to the 8 XCDs in turn: each XCD gets a contiguous range of the tiles, walked in panels of 4 row tiles
    // column by column, so that its L2 holds the operands of the tiles in flight on it
    const int tiles_n = (a.N + TN - 1) / TN, tiles_m = (a.M + TM - 1) / TM, nb = tiles_m * tiles_n, per_xcd = (nb + 7) >> 3;
    const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (tile >= nb) return;
    const int panel = tile / (4 * tiles_n), rem = tile - panel * 4 * tiles_n, rows = min(4, tiles_m - 4 * panel);
    const int m0 = (4 * panel + rem % rows) * TM, n0 = (rem / rows) * TN;

    float4 ra[LA], rb[LB];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            const int row = (tid >> 3) + 32 * i, k = k0 + (tid & 7) * 4;
            ra[i] = load4_clamped<VEC>(a.A + (size_t)min(m0 + row, a.M - 1) * a.K, k, a.K);
        }
#pragma unroll
        for (int i = 0; i < LB; ++i) {
            if (BT) {
                const int row = (tid >> 3) + 32 * i, k = k0 + (tid & 7) * 4;
                rb[i] = load4_clamped<VEC>(a.B + (size_t)min(n0 + row, a.N - 1) * a.K, k, a.K);
            } else {
                constexpr int TPR = TN / 4;              // threads per row of n
                const int k = k0 + tid / TPR + (256 / TPR) * i, n = n0 + (tid % TPR) * 4;
                rb[i] = load4_clamped<VEC>(a.B + (size_t)min(k, a.K - 1) * a.N, n, a.N);
            }
        }
    };
    auto commit = [&](float *st, int k0) {
#pragma unroll
        for (int i = 0; i < LA; ++i)
            *(float4 *)(st + ((tid >> 3) + 32 * i) * KP + (tid & 7) * 4) = zero_beyond(ra[i], !VEC || k0 + (tid & 7) * 4 < a.K);
#pragma unroll
        for (int i = 0; i < LB; ++i) {
            if (BT) *(float4 *)(st + ASZ + ((tid >> 3) + 32 * i) * KP + (tid & 7) * 4) = zero_beyond(rb[i], !VEC || k0 + (tid & 7) * 4 < a.K);
            else {
                constexpr int TPR = TN / 4;
                const int k = tid / TPR + (256 / TPR) * i;
                *(float4 *)(st + ASZ + k * NP + (tid % TPR) * 4) = zero_beyond(rb[i], k0 + k < a.K);
            }
        }
    };

    f32x4 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    float4 uz[MI], uu[NI];
    float bias[NI];
    if (grp == 0) {
#pragma unroll
        for (int i = 0; i < MI; ++i) uz[i] = up_frag_z(a, min(m0 + wm * (TM / 2) + i * 16 + r16, a.M - 1), g);
#pragma unroll
        for (int j = 0; j < NI; ++j) uu[j] = up_frag_u(a, min(n0 + wn * (TN / 2) + j * 16 + r16, a.N - 1), g);
#pragma unroll
        for (int j = 0; j < NI; ++j) bias[j] = a.bias ? a.bias[min(n0 + wn * (TN / 2) + j * 16 + r16, a.N - 1)] : 0.f;
    }
    // Fragments are read one half slab ahead of their MFMAs (the waves of a block leave the barrier together, and LDS
    // reads issued there would keep all of them waiting in front of idle matrix pipes), the slab after next is on its
    // way from memory, and the one barrier of a slab sits between its halves.
    float4 f0a[MI], f0b[NI], f1a[MI], f1b[NI];
    auto frags = [&](const float *st, int ks, float4 *fa, float4 *fb) {
#pragma unroll
        for (int i = 0; i < MI; ++i) fa[i] = *(const float4 *)(st + (wm * (TM / 2) + i * 16 + r16) * KP + ks * 16 + 4 * g);
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int n = wn * (TN / 2) + j * 16 + r16;
            if (BT) fb[j] = *(const float4 *)(st + ASZ + n * KP + ks * 16 + 4 * g);
            else {
                const float *q = st + ASZ + (ks * 16 + 4 * g) * NP + n;
                fb[j] = make_float4(q[0], q[NP], q[2 * NP], q[3 * NP]);
            }
        }
    };
    // component by component, so that an accumulator is not needed again by the very next MFMA
    auto mfmas = [&](const float4 *fa, const float4 *fb) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32((&fa[i].x)[c], (&fb[j].x)[c], acc[i][j], 0, 0, 0);
    };
    // slabs past the end read nothing and count as zeros, so every group runs the same number of steps
    const int nk = (a.K + BK - 1) / BK, steps = (nk + KS - 1) / KS;
    fetch(grp * BK);
    commit(lds[grp][0], grp * BK);
    fetch((KS + grp) * BK);
    __syncthreads();
    frags(lds[grp][0], 0, f0a, f0b);
    for (int kt = 0; kt < steps; ++kt) {
        frags(lds[grp][kt & 1], 1, f1a, f1b);
        __builtin_amdgcn_sched_barrier(0);
        mfmas(f0a, f0b);
        __builtin_amdgcn_sched_barrier(0);
        commit(lds[grp][(kt + 1) & 1], ((kt + 1) * KS + grp) * BK);
        fetch(((kt + 2) * KS + grp) * BK);
        __syncthreads();
        frags(lds[grp][(kt + 1) & 1], 0, f0a, f0b);
        __builtin_amdgcn_sched_barrier(0);
        mfmas(f1a, f1b);
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    if (KS > 1) {
        float4 *mine = (float4 *)lds[grp][0];
        if (grp > 0) {
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j) mine[(i * NI + j) * 256 + tid] = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
        }
        __syncthreads();
        if (grp > 0) return;
#pragma unroll
        for (int q = 1; q < KS; ++q)
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j) {
                    const float4 v = ((const float4 *)lds[q][0])[(i * NI + j) * 256 + tid];
                    acc[i][j][0] += v.x; acc[i][j][1] += v.y; acc[i][j][2] += v.z; acc[i][j][3] += v.w;
                }
    }
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            f32x4 low = {0.f, 0.f, 0.f, 0.f};
            mfma4(low, uz[i], uu[j]);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i][j][e] = fmaf(a.s, low[e], acc[i][j][e] + bias[j]);
        }
    // lane: column r16, rows 4 g + e of each 16 x 16 tile; a tile inside the matrix is stored without a branch
    float *cp = a.C + (size_t)(m0 + wm * (TM / 2) + 4 * g) * a.N + n0 + wn * (TN / 2) + r16;
    const bool inside = m0 + TM <= a.M && n0 + TN <= a.N;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                const float v = acc[i][j][e];
                if (inside) cp[(size_t)(i * 16 + e) * a.N + j * 16] = v;
                else if (m0 + wm * (TM / 2) + i * 16 + 4 * g + e < a.M && n0 + wn * (TN / 2) + j * 16 + r16 < a.N)
                    cp[(size_t)(i * 16 + e) * a.N + j * 16] = v;
            }
}

// The same product where the contraction is a multiple of 64: TM x TN tile, two groups of WM x WN waves that take the slabs of
// 32 in turn.  A stage of the LDS ring holds a slab for each group, filled by asynchronous copies NST - 1 stages ahead (a
// slab's arithmetic is shorter than the round trip that the kernel above has one slab in flight for); operand rows of
// 128 bytes with the 16-byte chunks XORed with the row, W read as [k, n] as rows of TN floats with the chunks rotated by the
// k-group, so that the four k-groups of a read meet different banks.  The sums and their order are those of f32_gemm_kernel with
// two groups (its 128 x 128 form has one, and one chain of sums instead of two).
template <int TM, int TN, int WM, int WN, int NST, bool BT>
__global__ __launch_bounds__(512) void f32_tile_kernel(GemmF32 a)
{
    static_assert(WM * WN == 4, "four waves in a group");
    constexpr int MI = TM / 16 / WM, NI = TN / 16 / WN;
    constexpr int ASZ = TM * 128, SUB = ASZ + TN * 128, STAGE = 2 * SUB;
    constexpr int CA = 2 * TM / 64, PER = CA + (2 * TN + 63) / 64;    // 1 KB copies of a wave per stage
    constexpr int RW = TN / 4;                           // 16-byte chunks of a row of W as [k, n]
    static_assert((2 * TM) % 64 == 0 && NST * PER < 64, "copies");
    __shared__ __attribute__((aligned(1024))) unsigned char lds[NST * STAGE];
    const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, g = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), grp = wv >> 2, wave = wv & 3;
    const int wm = wave / WN, wn = wave % WN;
    const int tiles_n = (a.N + TN - 1) / TN, tiles_m = (a.M + TM - 1) / TM, nb = tiles_m * tiles_n, per_xcd = (nb + 7) >> 3;
    const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (tile >= nb || (int)(blockIdx.x >> 3) >= per_xcd) return;
    const int panel = tile / (4 * tiles_n), rem = tile - panel * 4 * tiles_n, rows = min(4, tiles_m - 4 * panel);
    const int m0 = (4 * panel + rem % rows) * TM, n0 = (rem / rows) * TN;

    // operands of the low-rank term and the bias, needed after the loop: requested first, so that the waits below count
    // copies only
    float4 uz[MI], uu[NI];
    float bias[NI];
    if (grp == 0) {
#pragma unroll
        for (int i = 0; i < MI; ++i) uz[i] = up_frag_z(a, min(m0 + (wm * MI + i) * 16 + r16, a.M - 1), g);
#pragma unroll
        for (int j = 0; j < NI; ++j) uu[j] = up_frag_u(a, min(n0 + (wn * NI + j) * 16 + r16, a.N - 1), g);
#pragma unroll
        for (int j = 0; j < NI; ++j) bias[j] = a.bias ? a.bias[min(n0 + (wn * NI + j) * 16 + r16, a.N - 1)] : 0.f;
    }

    // copies: piece p of a stage (1 KB), the pieces of both groups' slabs dealt over the 8 waves; lane l fills 16-byte slot l
    const int nst = a.K / 64;                            // stages of the contraction
    unsigned ao[CA], bo[PER - CA];
    int al[CA], bl[PER - CA], blanes[PER - CA];
#pragma unroll
    for (int c = 0; c < CA; ++c) {
        const int p = wv * CA + c, sub = p / (TM / 8), row = (p % (TM / 8)) * 8 + (lane >> 3);
        ao[c] = (unsigned)min(m0 + row, a.M - 1) * (unsigned)a.K * 4u + sub * 128 + (((lane & 7) ^ (row & 7)) << 4);
        al[c] = sub * SUB + (p % (TM / 8)) * 1024;
    }
#pragma unroll
    for (int c = 0; c < PER - CA; ++c) {
        constexpr int NB = 2 * (TN / 8);                 // pieces of B per stage
        const int p = min(wv * (PER - CA) + c, NB - 1), sub = p / (TN / 8), q = p % (TN / 8);
        blanes[c] = (wv * (PER - CA) + c - NB) >> 31;    // -1, or 0 where there is no such piece
        bl[c] = sub * SUB + ASZ + q * 1024;
        if (BT) {
            const int row = q * 8 + (lane >> 3);
            bo[c] = (unsigned)min(n0 + row, a.N - 1) * (unsigned)a.K * 4u + sub * 128 + (((lane & 7) ^ (row & 7)) << 4);
        } else {
            const int slot = q * 64 + lane, k = slot / RW, ch = (slot % RW + RW - 4 * ((k >> 2) & 3) % RW) % RW;
            bo[c] = ((unsigned)(sub * 32 + k) * (unsigned)a.N + (unsigned)min(n0 + ch * 4, a.N - 4)) * 4u;
        }
    }
    const unsigned base = lds_addr(lds);
    const size_t bstep = BT ? 256 : 256 * (size_t)a.N;   // bytes of B per stage
    // copies past the last stage repeat it (in bounds, never read)
    auto copy1 = [&](int slot, int t, int c) {
        const size_t tt = (size_t)min(t, nst - 1);
        if (c < CA) glds_soff((const char *)a.A + tt * 256, ao[c < CA ? c : 0], base + slot * STAGE + al[c < CA ? c : 0]);
        else {
            const int b = c >= CA ? c - CA : 0;
            glds_soff_if((const char *)a.B + tt * bstep, bo[b], base + slot * STAGE + bl[b], blanes[b]);
        }
    };

    f32x4 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    struct Frags { float4 a[MI], b[NI]; } f[2];
    const int sw = r16 & 7;
    auto frags = [&](Frags &F, int slot, int ks) {
        const unsigned char *S = lds + slot * STAGE + grp * SUB;
        const int co = ((ks * 4 + g) ^ sw) << 4;
#pragma unroll
        for (int i = 0; i < MI; ++i) F.a[i] = *(const float4 *)(S + ((wm * MI + i) * 16 + r16) * 128 + co);
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int n = (wn * NI + j) * 16 + r16;
            if (BT) F.b[j] = *(const float4 *)(S + ASZ + n * 128 + co);
            else {
                const float *q = (const float *)(S + ASZ) + (ks * 16 + 4 * g) * TN + (((n >> 2) + 4 * g) % RW) * 4 + (n & 3);
                F.b[j] = make_float4(q[0], q[TN], q[2 * TN], q[3 * TN]);
            }
        }
    };
    // component by component, so that an accumulator is not needed again by the very next MFMA
    auto mfmas = [&](const Frags &F) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32((&F.a[i].x)[c], (&F.b[j].x)[c], acc[i][j], 0, 0, 0);
    };
#pragma unroll
    for (int s = 0; s < NST - 1; ++s)
#pragma unroll
        for (int c = 0; c < PER; ++c) copy1(s, s, c);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 2) * PER) : "memory");
    __syncthreads();
    frags(f[0], 0, 0);
    int slot = 0;
    for (int t = 0; t < nst; ++t) {
        const int next = slot + 1 == NST ? 0 : slot + 1, prev = slot == 0 ? NST - 1 : slot - 1;
        frags(f[1], slot, 1);
#pragma unroll
        for (int c = 0; c < PER; ++c) copy1(prev, t + NST - 1, c);
        __builtin_amdgcn_sched_barrier(0);
        mfmas(f[0]);
        __builtin_amdgcn_sched_barrier(0);
        // the wave's reads of the stage are done and its copies of the next one have landed
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NST - 2) * PER) : "memory");
        __syncthreads();
        frags(f[0], next, 0);
        __builtin_amdgcn_sched_barrier(0);
        mfmas(f[1]);
        __builtin_amdgcn_sched_barrier(0);
        slot = next;
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();                                     // the ring takes the second group's sums
    float4 *part = (float4 *)lds;
    if (grp == 1) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
                part[(i * NI + j) * 256 + (tid & 255)] = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
    }
    __syncthreads();
    if (grp == 1) return;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const float4 v = part[(i * NI + j) * 256 + (tid & 255)];
            acc[i][j][0] += v.x; acc[i][j][1] += v.y; acc[i][j][2] += v.z; acc[i][j][3] += v.w;
            f32x4 low = {0.f, 0.f, 0.f, 0.f};
            mfma4(low, uz[i], uu[j]);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i][j][e] = fmaf(a.s, low[e], acc[i][j][e] + bias[j]);
        }
    float *cp = a.C + (size_t)(m0 + wm * MI * 16 + 4 * g) * a.N + n0 + wn * NI * 16 + r16;
    const bool inside = m0 + TM <= a.M && n0 + TN <= a.N;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                const float v = acc[i][j][e];
                if (inside) cp[(size_t)(i * 16 + e) * a.N + j * 16] = v;
                else if (m0 + (wm * MI + i) * 16 + 4 * g + e < a.M && n0 + (wn * NI + j) * 16 + r16 < a.N)
                    cp[(size_t)(i * 16 + e) * a.N + j * 16] = v;
            }
}

// Few output tiles (small T): 16 x 16 outputs per block, the contraction split over 8 waves that read their fragments
// straight from memory, partial tiles added in wave order.  Latency-bound; the operands are re-read N / 16 and
// M / 16 times, which the caches carry up to a few hundred rows.
template <bool BT, bool VEC>
__global__ __launch_bounds__(512) void f32_gemm_direct_kernel(GemmF32 a)
{
    __shared__ float red[8][16][17];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r16 = lane & 15, g = lane >> 4;
    const int tiles_m = (a.M + 15) >> 4;
    const int m0 = (blockIdx.x % tiles_m) * 16, n0 = (blockIdx.x / tiles_m) * 16;
    const float *xr = a.A + (size_t)min(m0 + r16, a.M - 1) * a.K;
    const int nc = min(n0 + r16, a.N - 1);
    float4 uz, uu;
    if (wave == 7) {
        uz = up_frag_z(a, min(m0 + r16, a.M - 1), g);
        uu = up_frag_u(a, nc, g);
    }
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    const int steps = (a.K + 15) >> 4, per = (steps + 7) >> 3;
    const int s0 = wave * per, s1 = min(s0 + per, steps);
    for (int s = s0; s < s1; ++s) {
        const int k = s * 16 + 4 * g;
        const float4 x = load4_lim<VEC>(xr, k, a.K);
        float4 b;
        if (BT) b = load4_lim<VEC>(a.B + (size_t)nc * a.K, k, a.K);
        else {
            const float *q = a.B + (size_t)k * a.N + nc;
            b.x = k < a.K ? q[0] : 0.f;
            b.y = k + 1 < a.K ? q[a.N] : 0.f;
            b.z = k + 2 < a.K ? q[2 * (size_t)a.N] : 0.f;
            b.w = k + 3 < a.K ? q[3 * (size_t)a.N] : 0.f;
        }
        mfma4(acc, x, b);
    }
    if (wave == 7) {                                     // (the last wave has the shortest share)
        f32x4 low = {0.f, 0.f, 0.f, 0.f};
        mfma4(low, uz, uu);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = fmaf(a.s, low[e], acc[e]);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) red[wave][4 * g + e][r16] = acc[e];
    __syncthreads();
    if (threadIdx.x < 256) {
        const int m = m0 + (threadIdx.x >> 4), n = n0 + (threadIdx.x & 15);
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < 7; ++w) v += red[w][threadIdx.x >> 4][threadIdx.x & 15];
        if (m < a.M && n < a.N) {
            if (a.bias) v += a.bias[n];                  // before the share that holds the low-rank term
            a.C[(size_t)m * a.N + n] = v + red[7][threadIdx.x >> 4][threadIdx.x & 15];
        }
    }
}

// ---- adapter gradients --------------------------------------------------------------------------------------------
// G[c,j] = s sum_t X[t,c] Y[t,j], j < r: dA (written [r,C]) from X = x, Y = p and dB (written [C,r]) from X = dy, Y = z.
// One block per 32 columns walks all tokens with 32 half-waves (a half-wave reads 128 bytes of a row), whose sums
// are added in order.  Bound by reading X once; no second launch for a reduction.  A wave's rows are a chain of round trips, so
// for up to 4 columns of Y 16 of them are in flight, then 4, then single ones (us, backward of a 768 -> 768 layer, r = 4, T = 300,
// 500, 1000, 8192: 4 rows and single ones 19.4, 20.9, 28.6, 148; 16 and single ones 20.1, 22.3, 29.1, 140; as it is 18.9, 20.7,
// 27.7, 138); more columns leave registers for 4 rows.
struct GradJob { const float *X; const float *Y; int C; float *out; int rxC; };
struct GradJobs { GradJob j[2]; };

template <int ZP>
__global__ __launch_bounds__(1024) void f32_grad_kernel(GradJobs jobs, int T, int r, float s)
{
    __shared__ float red[32][ZP][33];
    const GradJob &jb = jobs.j[blockIdx.y];
    if ((int)blockIdx.x * 32 >= jb.C) return;
    const int hw = threadIdx.x >> 5, l = threadIdx.x & 31, c = blockIdx.x * 32 + l;
    const int cc = min(c, jb.C - 1);
    float acc[ZP];
#pragma unroll
    for (int j = 0; j < ZP; ++j) acc[j] = 0.f;
    // N rows of this half-wave from t on, all requested before the first is used
    auto rows = [&](int t, auto n) {
        constexpr int N = decltype(n)::value;
        float x[N];
        float4 y[N][ZP / 4];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            x[u] = jb.X[(size_t)(t + 32 * u) * jb.C + cc];
#pragma unroll
            for (int q = 0; q < ZP / 4; ++q) y[u][q] = ((const float4 *)(jb.Y + (size_t)(t + 32 * u) * ZP))[q];
        }
#pragma unroll
        for (int u = 0; u < N; ++u)
#pragma unroll
            for (int q = 0; q < ZP / 4; ++q) {
                const float4 v = y[u][q];
                acc[4 * q] = fmaf(x[u], v.x, acc[4 * q]);
                acc[4 * q + 1] = fmaf(x[u], v.y, acc[4 * q + 1]);
                acc[4 * q + 2] = fmaf(x[u], v.z, acc[4 * q + 2]);
                acc[4 * q + 3] = fmaf(x[u], v.w, acc[4 * q + 3]);
            }
    };
    int t = hw;
    if (ZP == 4) {
        for (; t + 15 * 32 < T; t += 16 * 32) rows(t, std::integral_constant<int, 16>());
        for (; t + 3 * 32 < T; t += 4 * 32) rows(t, std::integral_constant<int, 4>());
    }
#pragma unroll(ZP == 4 ? 1 : 4)
    for (; t < T; t += 32) rows(t, std::integral_constant<int, 1>());
#pragma unroll
    for (int j = 0; j < ZP; ++j) red[hw][j][l] = acc[j];
    __syncthreads();
    for (int i = threadIdx.x; i < 32 * r; i += 1024) {
        const int j = i >> 5, k = i & 31, col = blockIdx.x * 32 + k;
        float v = 0.f;
#pragma unroll
        for (int h = 0; h < 32; ++h) v += red[h][j][k];
        if (col < jb.C) jb.out[jb.rxC ? (size_t)j * jb.C + col : (size_t)col * r + j] = s * v;
    }
}

inline int pad_rank(int r) { return r <= 4 ? 4 : r <= 8 ? 8 : 16; }
inline bool aligned16(const void *p) { return (((uintptr_t)p) & 15) == 0; }

template <int TM, int TN, int KS, bool BT, bool VEC>
void launch_tile(const GemmF32 &a, hipStream_t st)
{
    const long tiles = (long)((a.M + TM - 1) / TM) * ((a.N + TN - 1) / TN);
    hipLaunchKernelGGL((f32_gemm_kernel<TM, TN, KS, BT, VEC>), dim3((unsigned)((tiles + 7) / 8 * 8)), dim3(256 * KS), 0, st, a);
}
template <int TM, int TN, int WM, int WN, int NST, bool BT>
void launch_ring(const GemmF32 &a, hipStream_t st)
{
    const long tiles = (long)((a.M + TM - 1) / TM) * ((a.N + TN - 1) / TN);
    hipLaunchKernelGGL((f32_tile_kernel<TM, TN, WM, WN, NST, BT>), dim3((unsigned)((tiles + 7) / 8 * 8)), dim3(512), 0, st, a);
}
// The kernel for a product.  16 x 16 outputs per block (f32_gemm_direct_kernel) while 64 x 64 tiles would leave most CUs without
// work: drawn at 96 of them against f32_gemm_kernel.  Against the ring the line would lie at about 36 (projection + product,
// 1024 -> 1024: 32 tiles 15.3 us direct, 17.2 on the ring; 48: 20.3, 17.4; 80: 27.2, 17.6; 4096 -> 1024: 51.2, 56.0; 66.0, 58.7;
// 92.3, 59.7).  The ring needs whole stages of 64 and 32-bit byte offsets and runs on the form that costs least, in us as measured
// (T = 64 to 8192 at five weight shapes): rounds of 256 tiles, or of 512 where two blocks share a CU, at a + b (K / 64) each.
// 32 x 64 and 64 x 48 fill the chip where 64 x 64 tiles leave a part of it idle (T = 1024, 768 -> 768: 256 tiles of 64 x 48 in
// 13.5 us, 192 of 64 x 64 in 16.1).  Without the ring (f32_gemm_kernel) 128 x 128 tiles once two of them per CU are there (below
// that the idle CUs cost more than the operand traffic saved).
template <bool BT, bool VEC>
int launch_product(const GemmF32 &a, const F32Plan &p, hipStream_t st)
{
    if (p.tm == 16) {
        const long tiles = (long)((a.M + 15) / 16) * ((a.N + 15) / 16);
        hipLaunchKernelGGL((f32_gemm_direct_kernel<BT, VEC>), dim3((unsigned)tiles), dim3(512), 0, st, a);
    } else if (p.stages == 0) {
        if (p.tm == 64) launch_tile<64, 64, 2, BT, VEC>(a, st);
        else launch_tile<128, 128, 1, BT, VEC>(a, st);
    } else if constexpr (VEC) {
        switch (p.tm * 1000 + p.tn + p.stages) {
        case 32064 + 4: launch_ring<32, 64, 2, 2, 4, BT>(a, st); break;
        case 64048 + 4: launch_ring<64, 48, 4, 1, 4, BT>(a, st); break;
        case 64064 + 4: launch_ring<64, 64, 2, 2, 4, BT>(a, st); break;
        case 64064 + 2: launch_ring<64, 64, 2, 2, 2, BT>(a, st); break;
        case 128128 + 2: launch_ring<128, 128, 2, 2, 2, BT>(a, st); break;
        default: return SL_EINVAL;
        }
    } else return SL_EINVAL;
    SL_CHECK_LAUNCH("f32 product");
    return 0;
}
int product(const GemmF32 &a, bool bt, hipStream_t st)
{
    // float4 loads need rows of a multiple of four floats on 16-byte bases
    const bool vec = (a.K % 4) == 0 && aligned16(a.A) && aligned16(a.B) && (bt || (a.N % 4) == 0);
    const F32Plan p = plan_f32(a.M, a.N, a.K, vec);
    if (bt) return vec ? launch_product<true, true>(a, p, st) : launch_product<true, false>(a, p, st);
    return vec ? launch_product<false, true>(a, p, st) : launch_product<false, false>(a, p, st);
}

int project(const ProjJob *j, int n, int T, int r, int zp, hipStream_t st)
{
    ProjJobs jobs;
    bool vec = true;
    for (int i = 0; i < n; ++i) {
        jobs.j[i] = j[i];
        vec = vec && (j[i].K % 4) == 0 && aligned16(j[i].X) && (j[i].zk != 1 || aligned16(j[i].Z));
    }
    const dim3 grid((T + 15) / 16, n);
    if (vec) hipLaunchKernelGGL((f32_project_kernel<true>), grid, dim3(512), 0, st, jobs, T, r, zp);
    else hipLaunchKernelGGL((f32_project_kernel<false>), grid, dim3(512), 0, st, jobs, T, r, zp);
    SL_CHECK_LAUNCH("f32 projection");
    return 0;
}

}  // namespace

F32Plan plan_f32(int M, int N, int K, bool vec)
{
    struct Form { int tm, tn, stages, per_cu; float a, b; };
    constexpr Form forms[5] = {{32, 64, 4, 1, 3.1f, .545f}, {64, 48, 4, 1, 3.6f, .765f}, {64, 64, 4, 1, 3.8f, .995f},
                               {64, 64, 2, 2, 4.6f, 1.90f}, {128, 128, 2, 1, 7.5f, 3.68f}};
    auto tiles = [&](int tm, int tn) { return (long)((M + tm - 1) / tm) * ((N + tn - 1) / tn); };
    if (tiles(64, 64) < 96) return {16, 16, 0};
    const bool ring = vec && K % 64 == 0 && (unsigned long long)M * K < (1ull << 30) && (unsigned long long)N * K < (1ull << 30);
    if (!ring) return tiles(128, 128) < 512 ? F32Plan{64, 64, 0} : F32Plan{128, 128, 0};
    F32Plan best = {0, 0, 0};
    double least = 0;
    for (const Form &f : forms) {
        const long round = 256 * f.per_cu;
        const double c = (double)((tiles(f.tm, f.tn) + round - 1) / round) * (f.a + f.b * (K / 64));
        if (best.tm == 0 || c < least) { best = {f.tm, f.tn, f.stages}; least = c; }
    }
    return best;
}

size_t f32_lora_linear_ws_floats(int T, int r) { return 2 * (size_t)T * pad_rank(r); }

// ws: z [T,zp] then p [T,zp], zp = r rounded up to 4, 8 or 16 (16-byte aligned)
int f32_lora_linear_fwd(int T, int n_in, int n_out, int r, float s, const float *x, const float *W,
                        const float *bias, const float *A, const float *B, float *y, float *ws, hipStream_t st)
{
    const int zp = pad_rank(r);
    const ProjJob j = {x, A, n_in, 1, n_in, ws};
    int rc;
    if ((rc = project(&j, 1, T, r, zp, st))) return rc;
    GemmF32 a = {x, W, bias, ws, B, y, T, n_out, n_in, zp, r, 1, r, s};
    return product(a, true, st);
}

int f32_lora_linear_bwd(int T, int n_in, int n_out, int r, float s, const float *x, const float *dy,
                        const float *W, const float *A, const float *B, float *dx, float *dA, float *dB, float *ws,
                        hipStream_t st)
{
    const int zp = pad_rank(r);
    float *z = ws, *p = ws + (size_t)T * zp;
    const ProjJob pj[2] = {{x, A, n_in, 1, n_in, z}, {dy, B, 1, r, n_out, p}};
    int rc;
    if ((rc = project(pj, 2, T, r, zp, st))) return rc;
    GemmF32 a = {dy, W, nullptr, p, A, dx, T, n_in, n_out, zp, r, n_in, 1, s};
    if ((rc = product(a, false, st))) return rc;
    const GradJobs gj = {{{x, p, n_in, dA, 1}, {dy, z, n_out, dB, 0}}};
    const dim3 grid(((n_in > n_out ? n_in : n_out) + 31) / 32, 2);
    if (zp == 4) hipLaunchKernelGGL((f32_grad_kernel<4>), grid, dim3(1024), 0, st, gj, T, r, s);
    else if (zp == 8) hipLaunchKernelGGL((f32_grad_kernel<8>), grid, dim3(1024), 0, st, gj, T, r, s);
    else hipLaunchKernelGGL((f32_grad_kernel<16>), grid, dim3(1024), 0, st, gj, T, r, s);
    SL_CHECK_LAUNCH("f32 adapter gradients");
    return 0;
}
