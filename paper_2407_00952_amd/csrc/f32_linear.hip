// Single-precision LoRA-adapted linear layer (SplitLoRA Sec. II-C), forward and backward.
//
// Every operand and every sum is fp32.  Products whose shapes allow it run on the bf16 matrix instruction with each operand, times
// 2^24, as the exact sum of three bf16 numbers (f32_tile_kernel; closer to the sum in 64 bits than the fp32 instruction; operands
// and sums too large for that on the fp32 one), the others and the rank-space projections on the fp32 one
// (V_MFMA_F32_16X16X4_F32), the adapter gradients on vector FMAs.  Each sum has one fixed order, so results are reproducible.
//
//   forward   z = x A^T                                 f32_tile_kernel on small tiles forms z itself; else f32_project_kernel
//             y = x W^T + bias + s z B^T                f32_tile_kernel / f32_gemm_kernel / f32_gemm_direct_kernel
//   backward  z = x A^T, p = dy B                       as in the forward
//             dx = dy W + s p A                         the same product kernels, W read as [k, n]
//             dA = s p^T x, dB = s dy^T z               f32_grad_kernel (both in one launch)
//
// At T = 1024, 768 -> 768, r = 4 (2.5 GFLOP, 15 MB) forward + backward take three launches and 38 us; with the products on the fp32
// instruction (64 x 48 tiles on a ring in LDS, 0.64 of 0.77 us a stage of 64 being matrix time) and projections of their own
// five launches and 46 us.  Whole layers in us, before and now: 64 rows of 1024 -> 3072, r = 16, 63.2 and 50.4; 200 of
// 1280 -> 5120, r = 8, 164 and 95; 1024 of 3072 -> 768 133 and 99; 2048 of 1280 -> 1280, r = 16, 208 and 167; 8192 of 1280 -> 5120
// 1719 and 1390.
#include "common.h"
#include "gemm_copy.h"
#include <type_traits>

// the tile of a product's kernel and the last argument of f32_tile_kernel (0: another kernel); vec: operands of 16-byte rows
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
    // f32_wave_tile forms z itself where Z is there ([r,K] beside a B of [N,K], [K,r] beside one of [K,N]), and stores it to
    // zout if that is there; and z2 [M,zp] = x2 A2^T, if asked for, with x2 [M,K2], A2 [r,K2]
    const float *Z;
    float *zout;
    const float *x2, *A2;
    float *z2;
    int K2;
};

// The low-rank term is one more step of 16 contraction elements: operand fragments z[m, 4g ..] and U(4g .., n), zero
// beyond the rank.  They are requested before the main loop, whose last step they follow.  Its sum is formed on its own and
// added, scaled, in one rounding, after the bias: in the accumulators it would cost one more rounding at the size of the result
// for every element of the rank (r = 16: 1.37 times the error at n_in = 16, 1.016 times at 768).
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

// ---- products on the bf16 matrix instruction ----------------------------------------------------------------------
// An fp32 number is the sum of three bf16 ones (8 bits each: round to nearest, subtract exactly, again; Henry, Tang and Heinecke,
// "Leveraging the bfloat16 artificial intelligence datatype for higher-precision computations", 2019), so a product of two is
// six bf16 products, exact in fp32, and three left out that are below 2^-24 of it.  V_MFMA_F32_16X16X32_BF16 does sixteen times
// the work of V_MFMA_F32_16X16X4_F32 in a pass and rounds its sum once where that rounds eight times: six of them take 0.375
// of the time, and the result is closer to the sum in 64 bits (errors in the 2-norm, chains of 768 and 5120 products of normal
// numbers: 4.1e-7 against 5.1e-7, 1.1e-6 against 1.3e-6; of absolute values 3.0e-7, 4.3e-7 and 6.0e-7, 9.7e-7).  Rounded, not
// cut: cut pieces all have the sign of their number, and what is left out adds up (5120 absolute values: 1.1e-5).
// The pieces are those of 2^24 times the number, which are normal numbers or zero whatever it was (its last bit is 2^-149 or more:
// unscaled, the last piece loses bits below 2^-110 and nothing is left at 2^-134); a sum gets its own scale back where the waves'
// shares of it have been added.
// Infinities and NaN, numbers that bf16 rounds to an infinity (from 2^104 on) and sums from 2^80 on come out as NaN or infinity:
// such a sum is formed again with the fp32 instruction, and only that one, so that a row's bits are the same whatever its neighbours hold.
constexpr float PIECES = 0x1p24f, SUM_SCALE = 0x1p-48f;
__device__ __forceinline__ void split3(const float4 &u, const float4 &v, bf16x8 (&p)[3])
{
    float x[8] = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] *= PIECES;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        union { unsigned w[4]; bf16x8 v; } c;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            // (the instruction by name: the compiler would convert each of the two once more to take them apart)
            asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(c.w[e]) : "v"(x[2 * e]), "v"(x[2 * e + 1]));
            if (q < 2) {
                x[2 * e] -= __uint_as_float(c.w[e] << 16);
                x[2 * e + 1] -= __uint_as_float(c.w[e] & 0xFFFF0000u);
            }
        }
        p[q] = c.v;
    }
}
// An MFMA wants 2 wait states behind the vector instruction that wrote its operand; the compiler does not count the
// conversions, which it does not see (tests/test_kernel_isa.py does).
__device__ __forceinline__ void split_done()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 1");
    __builtin_amdgcn_sched_barrier(0);
}
// Ask for the conversion of one fragment (52 instructions) between the products of MI row tiles with another, 44 of them spaced
// evenly: us of forward products 4096 x 768 -> 3072 and 8192 x 1280 -> 5120 with 3 behind each product, all 52 spaced evenly and
// these 44 132.3, 129.4, 127.1 and 653, 641, 638 (unscaled pieces, 44 instructions, 2 behind each: 131.5 and 611).
template <int MI, int I = 0>
__device__ __forceinline__ void spread_split()
{
    if constexpr (I < 6 * MI) {
        constexpr int before = I * 44 / (6 * MI), upto = (I + 1) * 44 / (6 * MI);
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);               // an MFMA
        __builtin_amdgcn_sched_group_barrier(0x002, upto - before, 0);
        spread_split<MI, I + 1>();
    } else split_done();
}
// the six products, the small ones first; neighbours work on different accumulators.  With sums of their own for the small
// ones (to be added at the end) the error is 0.4 of it.
template <int MI>
__device__ __forceinline__ void mfma_split(f32x4 *acc, int stride, f32x4 *small, int small_stride, const bf16x8 (&pa)[MI][3],
                                           const bf16x8 (&pb)[3])
{
    constexpr int PA[6] = {0, 2, 1, 0, 1, 0}, PB[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            f32x4 &c = q < 5 ? small[i * small_stride] : acc[i * stride];
            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pa[i][PA[q]], pb[PB[q]], c, 0, 0, 0);
        }
}
// whether the wave holds a sum that is no finite number (0 times it is NaN)
__device__ __forceinline__ bool any_not_finite(const f32x4 *acc, int n)
{
    float c = 0.f;
#pragma unroll
    for (int i = 0; i < n; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) c = fmaf(acc[i][e], 0.f, c);
    return __any(c != 0.f);
}
// those sums of a 16 x 16 tile formed again: `chains` sums of the fp32 instruction, one for each k in [at(c), at(c + 1)), added in
// order.  x: the lane's row of A; y: its column of B, elements ys apart, zeros unless yok
template <class At>
__device__ __forceinline__ void sum_again(f32x4 &v, const float *x, const float *y, size_t ys, bool yok, int chains, At at, int g)
{
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    for (int c = 0; c < chains; ++c) {
        f32x4 part = {0.f, 0.f, 0.f, 0.f};
        at(c, [&](int k) {
            float4 b = make_float4(0.f, 0.f, 0.f, 0.f);
            if (yok) {
                const float *q = y + (size_t)(k + 4 * g) * ys;
                b = make_float4(q[0], q[ys], q[2 * ys], q[3 * ys]);
            }
            mfma4(part, *(const float4 *)(x + k + 4 * g), b);
        });
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[e] += part[e];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (v[e] * 0.f != 0.f) v[e] = sum[e];
}

// TM x TN tile per block of NW waves, each of which takes its share of the contraction for the whole tile; the waves' sums are added
// in wave order through LDS.  So every operand is converted once per block and nothing in the loop waits at a barrier: a wave
// has a piece of LDS of its own for a k-step's operands, filled by asynchronous copies, reads its fragments from there, and
// requests the next step's operands into what it has read before it multiplies.  (Fragments read straight from memory go
// 16 bytes at a time, neighbouring lanes being different rows: 30 GB/s per CU where whole rows reach 100.)  The rank-space
// activations z = A Z^T are one more column tile, formed by every column tile's block for its rows (a third more matrix
// work at TN = 48, where a launch of their own took 5 us) and stored by the first.  The blocks of a launch also deal out the rows of a
// second projection (backward: x A^T, which nothing here waits for).
// One of them to a CU with 8 waves, for launches of about a tile per CU, or two with 4 (64 x 64 of short contractions).
template <int TM, int TN, int NW, bool BT>
struct F32Wave {
    static constexpr int MI = TM / 16, NI = TN / 16, NT = MI * (NI + 1);
    static constexpr int NA = TM / 8, NB = TN / 8, NZ = BT ? 2 : 0;   // copies of 1 KB per k-step: A, B, rows of Z
    static constexpr int SLAB = (NA + NB + NZ) * 1024;
    static constexpr int LDS = NW * (SLAB > NT * 1024 ? SLAB : NT * 1024);
};
template <int TM, int TN, int NW, bool BT>
__device__ __forceinline__ void f32_wave_tile(const GemmF32 &a, unsigned char *lds)
{
    typedef F32Wave<TM, TN, NW, BT> F;
    constexpr int MI = F::MI, NI = F::NI, NT = F::NT, NQ = (MI * NI + NW - 1) / NW, RW = TN / 4;
    const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, g = lane >> 4, sw = r16 & 7;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tiles_n = (a.N + TN - 1) / TN, tiles_m = (a.M + TM - 1) / TM, nb = tiles_m * tiles_n, per_xcd = (nb + 7) >> 3;
    const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (tile >= nb || (int)(blockIdx.x >> 3) >= per_xcd) return;
    const int panel = tile / (4 * tiles_n), rem = tile - panel * 4 * tiles_n, rows = min(4, tiles_m - 4 * panel);
    const int m0 = (4 * panel + rem % rows) * TM, tn = rem / rows, n0 = tn * TN;
    const bool fold = a.Z != nullptr;

    // copies: 8 rows of 128 bytes each, 16-byte chunks XORed with the row; W as [k, n]: rows of TN floats, chunks rotated by
    // the k-group, so that the four k-groups of a read meet different banks
    const int crow = lane >> 3, cch = ((lane & 7) ^ (lane >> 3)) << 4;
    unsigned ao[F::NA], bo[F::NB], zo[2];
#pragma unroll
    for (int p = 0; p < F::NA; ++p) ao[p] = (unsigned)min(m0 + p * 8 + crow, a.M - 1) * (unsigned)a.K * 4u + cch;
#pragma unroll
    for (int p = 0; p < F::NB; ++p) {
        if (BT) bo[p] = (unsigned)min(n0 + p * 8 + crow, a.N - 1) * (unsigned)a.K * 4u + cch;
        else {
            const int slot = p * 64 + lane, k = slot / RW, ch = (slot % RW + RW - 4 * ((k >> 2) & 3) % RW) % RW;
            bo[p] = ((unsigned)k * (unsigned)a.N + (unsigned)min(n0 + ch * 4, a.N - 4)) * 4u;
        }
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) zo[p] = fold ? (unsigned)min(p * 8 + crow, a.r - 1) * (unsigned)a.K * 4u + cch : ao[0];
    // (without a branch: the waits below count these copies whether they are wanted or not)
    const char *const zsrc = (const char *)(fold ? a.Z : a.A);
    const unsigned char *mine = lds + wave * F::SLAB;
    const unsigned base = lds_addr(mine);
    const size_t bstep = BT ? 128 : 128 * (size_t)a.N;   // bytes of B per k-step
    auto copy_a = [&](int s) {
#pragma unroll
        for (int p = 0; p < F::NA; ++p) glds_soff((const char *)a.A + (size_t)s * 128, ao[p], base + p * 1024);
    };
    auto copy_b = [&](int s) {
#pragma unroll
        for (int p = 0; p < F::NB; ++p) glds_soff((const char *)a.B + s * bstep, bo[p], base + (F::NA + p) * 1024);
#pragma unroll
        for (int p = 0; p < F::NZ; ++p) glds_soff(zsrc + (size_t)s * 128, zo[p], base + (F::NA + F::NB + p) * 1024);
    };
    const int steps = a.K >> 5, s0 = wave * steps / NW, s1 = (wave + 1) * steps / NW;
    if (s0 < s1) {
        copy_a(s0);
        copy_b(s0);
    }
    // rows of the second projection: a wave each
    if (a.z2) {
        typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
        const int per = (a.M + nb - 1) / nb;
        for (int i = wave; i < per; i += NW) {
            const int t = tile * per + i;
            if (t >= a.M) break;
            for (int j0 = 0; j0 < a.zp; j0 += 4) {
                float v[4] = {0.f, 0.f, 0.f, 0.f};
                for (int c = lane * 4; c < a.K2; c += 256) {
                    const f32x4u x = *(const f32x4u *)(a.x2 + (size_t)t * a.K2 + c);
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const f32x4u w = *(const f32x4u *)(a.A2 + (size_t)min(j0 + j, a.r - 1) * a.K2 + c);
                        v[j] = fmaf(x.x, w.x, v[j]); v[j] = fmaf(x.y, w.y, v[j]);
                        v[j] = fmaf(x.z, w.z, v[j]); v[j] = fmaf(x.w, w.w, v[j]);
                    }
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] = wave_sum(v[j]);
                if (lane < 4) {
                    const float w = lane == 0 ? v[0] : lane == 1 ? v[1] : lane == 2 ? v[2] : v[3];
                    a.z2[(size_t)t * a.zp + j0 + lane] = j0 + lane < a.r ? w : 0.f;
                }
            }
        }
    }

    f32x4 acc[NT];                                       // column tile NI is z
#pragma unroll
    for (int i = 0; i < NT; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    // the input gradient's z enters the adapter's gradient, where the fp32 instruction's 8 shorter chains stood
    f32x4 zsmall[BT ? 1 : MI];
#pragma unroll
    for (int i = 0; i < (BT ? 1 : MI); ++i) zsmall[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    const bool zok = fold && r16 < a.r;
    // Z as the caller's B [K, r] (backward): neighbouring lanes are neighbours in memory, a load per element
    const float *zcol = a.Z + min(r16, a.r - 1);
    auto load_z = [&](int s, float4 (&z)[2]) {
        if (BT || !fold) return;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float *q = zcol + (size_t)(s * 32 + 16 * h + 4 * g) * a.r;
            z[h] = make_float4(q[0], q[a.r], q[2 * a.r], q[3 * a.r]);
        }
    };
    for (int s = s0; s < s1; ++s) {
        const int next = min(s + 1, s1 - 1);             // (behind the last step: it once more, unread)
        bf16x8 pa[MI][3], pb[2][3], pz[3];
        float4 b[NI][2], z[2];
        {
            float4 f[MI][2];
            load_z(s, z);
            // A has landed (B of this step, requested behind it, and z may not have)
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(F::NB + F::NZ) : "memory");
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int h = 0; h < 2; ++h) f[i][h] = *(const float4 *)(mine + (i * 16 + r16) * 128 + (((h * 4 + g) ^ sw) << 4));
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            // (a load the compiler waits for: converted here, where nothing else is in flight)
            if (!BT) split3(zero_beyond(z[0], zok), zero_beyond(z[1], zok), pz);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const unsigned char *S = mine + F::NA * 1024;
#pragma unroll
                for (int j = 0; j < NI; ++j) {
                    const int n = j * 16 + r16;
                    if (BT) b[j][h] = *(const float4 *)(S + n * 128 + (((h * 4 + g) ^ sw) << 4));
                    else {
                        const float *q = (const float *)S + (h * 16 + 4 * g) * TN + (((n >> 2) + 4 * g) % RW) * 4 + (n & 3);
                        b[j][h] = make_float4(q[0], q[TN], q[2 * TN], q[3 * TN]);
                    }
                }
                if (BT) z[h] = *(const float4 *)(S + F::NB * 1024 + r16 * 128 + (((h * 4 + g) ^ sw) << 4));
            }
            copy_a(next);
#pragma unroll
            for (int i = 0; i < MI; ++i) split3(f[i][0], f[i][1], pa[i]);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            copy_b(next);
            if (BT) split3(zero_beyond(z[0], zok), zero_beyond(z[1], zok), pz);
        }
        split3(b[0][0], b[0][1], pb[0]);
        split_done();
#pragma unroll
        for (int j = 0; j <= NI; ++j) {
            if (j + 1 < NI) split3(b[j + 1][0], b[j + 1][1], pb[(j + 1) & 1]);
            if (j < NI) mfma_split<MI>(acc + j, NI + 1, acc + j, NI + 1, pa, pb[j & 1]);
            else if (BT) mfma_split<MI>(acc + NI, NI + 1, acc + NI, NI + 1, pa, pz);
            else mfma_split<MI>(acc + NI, NI + 1, zsmall, 1, pa, pz);
            spread_split<MI>();
        }
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    if (!BT) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i * (NI + 1) + NI][e] += zsmall[BT ? 0 : i][e];
    }
    // operands of the low-rank term and the bias for the tiles this wave finishes
    float4 uu[NQ];
    float bias[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int n = min(n0 + ((wave + q * NW) % NI) * 16 + r16, a.N - 1);
        uu[q] = up_frag_u(a, n, g);
        bias[q] = a.bias ? a.bias[n] : 0.f;
    }
    __syncthreads();                                     // the waves' pieces of LDS take their sums
    float4 *part = (float4 *)lds;
#pragma unroll
    for (int i = 0; i < NT; ++i) part[(wave * NT + i) * 64 + lane] = make_float4(acc[i][0], acc[i][1], acc[i][2], acc[i][3]);
    __syncthreads();
    auto sum = [&](int t) {
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float4 q = part[(w * NT + t) * 64 + lane];
            v[0] += q.x; v[1] += q.y; v[2] += q.z; v[3] += q.w;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] *= SUM_SCALE;
        if (any_not_finite(&v, 1)) {
            const int i = t / (NI + 1), j = t % (NI + 1), n = j < NI ? min(n0 + j * 16 + r16, a.N - 1) : r16;
            const float *y = j < NI ? a.B : a.Z;         // as [n, k] in the forward, [k, n] in the input gradient
            const size_t ld = BT ? a.K : j < NI ? a.N : a.r;
            sum_again(v, a.A + (size_t)min(m0 + i * 16 + r16, a.M - 1) * a.K, y + (BT ? n * ld : n), BT ? 1 : ld, j < NI || zok, NW,
                      [&](int w, auto step) { for (int k = w * steps / NW * 32; k < (w + 1) * steps / NW * 32; k += 16) step(k); }, g);
        }
        return v;
    };
    // z of the block's rows, in the place of the first wave's share of it as [16 rows][16]
    if (fold) {
        for (int i = wave; i < MI; i += NW) {
            const f32x4 v = sum(i * (NI + 1) + NI);
            float *zt = (float *)(part + (i * (NI + 1) + NI) * 64);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float w = zok ? v[e] : 0.f;        // also where an infinity met a zero of Z
                zt[(4 * g + e) * 16 + r16] = w;
                const int m = m0 + i * 16 + 4 * g + e;
                if (a.zout && tn == 0 && m < a.M && r16 < a.zp) a.zout[(size_t)m * a.zp + r16] = w;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int t = wave + q * NW, i = t / NI, j = t % NI;
        if (t >= MI * NI) break;
        const float4 uz = fold ? part[(i * (NI + 1) + NI) * 64 + r16 * 4 + g] : up_frag_z(a, min(m0 + i * 16 + r16, a.M - 1), g);
        f32x4 v = sum(i * (NI + 1) + j), low = {0.f, 0.f, 0.f, 0.f};
        mfma4(low, uz, uu[q]);
        const int n = n0 + j * 16 + r16;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int m = m0 + i * 16 + 4 * g + e;
            if (m < a.M && n < a.N) a.C[(size_t)m * a.N + n] = fmaf(a.s, low[e], v[e] + bias[q]);
        }
    }
}

// 128 x 128 tile per block, two groups of 2 x 2 waves (wave tile 64 x 64) that take the slabs of 32 in turn, for launches with
// enough such tiles.  A stage of the LDS ring holds a slab for each group, filled by asynchronous copies; a wave takes its
// fragments into registers, a barrier frees the stage for the copies of the stage after the next, and the wave converts and
// multiplies while they arrive; its SIMD's other wave fills the matrix pipe while it converts.  Operand rows of 128 bytes with the
// 16-byte chunks XORed with the row, W read as [k, n] as rows of 128 floats with the chunks rotated by the k-group, so that
// the four k-groups of a read meet different banks.
template <int NST, bool BT>
__device__ __forceinline__ void f32_ring_tile(const GemmF32 &a, unsigned char *lds)
{
    constexpr int TM = 128, TN = 128, WN = 2, MI = 4, NI = 4;
    constexpr int ASZ = TM * 128, SUB = ASZ + TN * 128, STAGE = 2 * SUB;
    constexpr int CA = 2 * TM / 64, PER = CA + 2 * TN / 64;           // 1 KB copies of a wave per stage
    constexpr int RW = TN / 4;                           // 16-byte chunks of a row of W as [k, n]
    static_assert(NST * PER < 64, "copies");
    const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, g = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), grp = wv >> 2, wave = wv & 3;
    const int wm = wave / WN, wn = wave % WN;
    const int tiles_n = (a.N + TN - 1) / TN, tiles_m = (a.M + TM - 1) / TM, nb = tiles_m * tiles_n, per_xcd = (nb + 7) >> 3;
    const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (tile >= nb || (int)(blockIdx.x >> 3) >= per_xcd) return;
    const int panel = tile / (4 * tiles_n), rem = tile - panel * 4 * tiles_n, rows = min(4, tiles_m - 4 * panel);
    const int m0 = (4 * panel + rem % rows) * TM, n0 = (rem / rows) * TN;

    // copies: piece p of a stage (1 KB), the pieces of both groups' slabs dealt over the 8 waves; lane l fills 16-byte slot l
    const int nst = a.K / 64;                            // stages of the contraction
    unsigned ao[CA], bo[PER - CA];
    int al[CA], bl[PER - CA];
#pragma unroll
    for (int c = 0; c < CA; ++c) {
        const int p = wv * CA + c, sub = p / (TM / 8), row = (p % (TM / 8)) * 8 + (lane >> 3);
        ao[c] = (unsigned)min(m0 + row, a.M - 1) * (unsigned)a.K * 4u + sub * 128 + (((lane & 7) ^ (row & 7)) << 4);
        al[c] = sub * SUB + (p % (TM / 8)) * 1024;
    }
#pragma unroll
    for (int c = 0; c < PER - CA; ++c) {
        const int p = wv * (PER - CA) + c, sub = p / (TN / 8), q = p % (TN / 8);
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
        else glds_soff((const char *)a.B + tt * bstep, bo[c >= CA ? c - CA : 0], base + slot * STAGE + bl[c >= CA ? c - CA : 0]);
    };

    f32x4 acc[MI * NI];
#pragma unroll
    for (int i = 0; i < MI * NI; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int sw = r16 & 7;
#pragma unroll
    for (int s = 0; s < NST; ++s)
#pragma unroll
        for (int c = 0; c < PER; ++c) copy1(s, s, c);
    int slot = 0;
    for (int t = 0; t < nst; ++t) {
        // this wave's copies of the stage have landed, then everybody's
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 1) * PER) : "memory");
        __syncthreads();
        float4 fa[MI][2], fb[NI][2];
        const unsigned char *S = lds + slot * STAGE + grp * SUB;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int co = ((h * 4 + g) ^ sw) << 4;
#pragma unroll
            for (int i = 0; i < MI; ++i) fa[i][h] = *(const float4 *)(S + ((wm * MI + i) * 16 + r16) * 128 + co);
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                const int n = (wn * NI + j) * 16 + r16;
                if (BT) fb[j][h] = *(const float4 *)(S + ASZ + n * 128 + co);
                else {
                    const float *q = (const float *)(S + ASZ) + (h * 16 + 4 * g) * TN + (((n >> 2) + 4 * g) % RW) * 4 + (n & 3);
                    fb[j][h] = make_float4(q[0], q[TN], q[2 * TN], q[3 * TN]);
                }
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __syncthreads();
#pragma unroll
        for (int c = 0; c < PER; ++c) copy1(slot, t + NST, c);
        bf16x8 pa[MI][3], pb[2][3];
#pragma unroll
        for (int i = 0; i < MI; ++i) split3(fa[i][0], fa[i][1], pa[i]);
        split3(fb[0][0], fb[0][1], pb[0]);
        split_done();
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            if (j + 1 < NI) split3(fb[j + 1][0], fb[j + 1][1], pb[(j + 1) & 1]);
            mfma_split<MI>(acc + j, NI, acc + j, NI, pa, pb[j & 1]);
            spread_split<MI>();
        }
        slot = slot + 1 == NST ? 0 : slot + 1;
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    // operands of the low-rank term, and of the sums that have to be formed again
    unsigned ar[MI], br[NI];
#pragma unroll
    for (int i = 0; i < MI; ++i) ar[i] = (unsigned)min(m0 + (wm * MI + i) * 16 + r16, a.M - 1);
#pragma unroll
    for (int j = 0; j < NI; ++j) br[j] = (unsigned)min(n0 + (wn * NI + j) * 16 + r16, a.N - 1);
    __syncthreads();                                     // the ring takes the second group's sums
    float4 *part = (float4 *)lds;
    if (grp == 1) {
#pragma unroll
        for (int i = 0; i < MI * NI; ++i) part[i * 256 + (tid & 255)] = make_float4(acc[i][0], acc[i][1], acc[i][2], acc[i][3]);
    }
    __syncthreads();
    if (grp == 1) return;
    float4 uz[MI], uu[NI];
    float bias[NI];
#pragma unroll
    for (int i = 0; i < MI * NI; ++i) {
        const float4 v = part[i * 256 + (tid & 255)];
        acc[i][0] += v.x; acc[i][1] += v.y; acc[i][2] += v.z; acc[i][3] += v.w;
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i][e] *= SUM_SCALE;
    }
    if (any_not_finite(acc, MI * NI)) {                  // (tile by tile: through the half of the ring that is free)
        static_assert(NST * STAGE >= 2 * 256 * MI * NI * 16, "room for both groups' sums");
        f32x4 *own = (f32x4 *)(part + 256 * MI * NI) + wave * MI * NI * 64 + lane;
#pragma unroll
        for (int i = 0; i < MI * NI; ++i) own[i * 64] = acc[i];
#pragma unroll 1
        for (int i = 0; i < MI * NI; ++i) {
            f32x4 v = own[i * 64];
            if (!any_not_finite(&v, 1)) continue;
            const size_t m = min(m0 + (wm * MI + i / NI) * 16 + r16, a.M - 1), n = min(n0 + (wn * NI + i % NI) * 16 + r16, a.N - 1);
            sum_again(v, a.A + m * a.K, a.B + (BT ? n * a.K : n), BT ? 1 : a.N, true, 2,
                      [&](int c, auto step) { for (int k = c * 32; k < a.K; k += k & 16 ? 48 : 16) step(k); }, g);
            own[i * 64] = v;
        }
#pragma unroll
        for (int i = 0; i < MI * NI; ++i) acc[i] = own[i * 64];
    }
#pragma unroll
    for (int i = 0; i < MI; ++i) uz[i] = up_frag_z(a, (int)ar[i], g);
#pragma unroll
    for (int j = 0; j < NI; ++j) { uu[j] = up_frag_u(a, (int)br[j], g); bias[j] = a.bias ? a.bias[br[j]] : 0.f; }
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            f32x4 &c = acc[i * NI + j];
            f32x4 low = {0.f, 0.f, 0.f, 0.f};
            mfma4(low, uz[i], uu[j]);
#pragma unroll
            for (int e = 0; e < 4; ++e) c[e] = fmaf(a.s, low[e], c[e] + bias[j]);
        }
    float *cp = a.C + (size_t)(m0 + wm * MI * 16 + 4 * g) * a.N + n0 + wn * NI * 16 + r16;
    const bool inside = m0 + TM <= a.M && n0 + TN <= a.N;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                const float v = acc[i * NI + j][e];
                if (inside) cp[(size_t)(i * 16 + e) * a.N + j * 16] = v;
                else if (m0 + (wm * MI + i) * 16 + 4 * g + e < a.M && n0 + (wn * NI + j) * 16 + r16 < a.N)
                    cp[(size_t)(i * 16 + e) * a.N + j * 16] = v;
            }
}

// FORM: pairs of waves of f32_wave_tile's block, or the stages of f32_ring_tile's ring
template <int TM, int TN, int FORM, bool BT>
__global__ __launch_bounds__(TM == 128 ? 512 : 128 * FORM, TM == 128 ? 1 : FORM == 2 ? 2 : 1) void f32_tile_kernel(GemmF32 a)
{
    if constexpr (TM == 128) {
        __shared__ __attribute__((aligned(1024))) unsigned char lds[FORM * 2 * 256 * 128];
        f32_ring_tile<FORM, BT>(a, lds);
    } else {
        __shared__ __attribute__((aligned(1024))) unsigned char lds[F32Wave<TM, TN, 2 * FORM, BT>::LDS];
        f32_wave_tile<TM, TN, 2 * FORM, BT>(a, lds);
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
template <int TM, int TN, int FORM, bool BT>
void launch_split(const GemmF32 &a, hipStream_t st)
{
    const long tiles = (long)((a.M + TM - 1) / TM) * ((a.N + TN - 1) / TN);
    hipLaunchKernelGGL((f32_tile_kernel<TM, TN, FORM, BT>), dim3((unsigned)((tiles + 7) / 8 * 8)), dim3(TM == 128 ? 512 : 128 * FORM), 0, st, a);
}
// The kernel for a product (plan_f32).  f32_tile_kernel needs whole stages of 64, rows of whole float4s and 32-bit byte offsets; without
// them 16 x 16 outputs per block while there are fewer than 96 tiles of 64 x 64 and 128 x 128 tiles of f32_gemm_kernel
// once two of them per CU are there (below that the idle CUs cost more than the operand traffic saved).
// With them the form that costs least in us as fitted to forward calls of 64 to 8192 rows at nine weight shapes (mean error 2 to 3 %):
// a launch, then rounds of tiles at a + b (K / 64) each, the last of up to 256 at a1 + b1 (K / 64); the 128 x 128 form with
// the projections' launch.  Forward, r = 4, us on 16 x 16, 32 x 64, 64 x 48, 64 x 64, two blocks of 64 x 64 to a CU, 128 x 128:
// 64 rows of 768 -> 768 10.6, 11.9, 14.6, 16.6, 18.2, 40; 256 of 1024 -> 1024 25.2, 14.0, 17.5, 19.6, 21.6, 51; 1024 of
// 768 -> 768 41, 21.6, 16.3, 16.6, 18.4, 41; 1024 of 1024 -> 1024 66, 25.8, 29.5, 21.8, 22.6, 51; 2048 of 1280 -> 1280 -, 73, 75, 67, 58, 67;
// 4096 of 768 -> 3072 -, 241, 211, 186, 145, 124.
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
        case 32064 + 4: launch_split<32, 64, 4, BT>(a, st); break;
        case 64048 + 4: launch_split<64, 48, 4, BT>(a, st); break;
        case 64064 + 4: launch_split<64, 64, 4, BT>(a, st); break;
        case 64064 + 2: launch_split<64, 64, 2, BT>(a, st); break;
        case 128128 + 2: launch_split<128, 128, 2, BT>(a, st); break;
        default: return SL_EINVAL;
        }
    } else return SL_EINVAL;
    SL_CHECK_LAUNCH("f32 product");
    return 0;
}
// float4 loads need rows of a multiple of four floats on 16-byte bases
bool vec_rows(const GemmF32 &a, bool bt) { return (a.K % 4) == 0 && aligned16(a.A) && aligned16(a.B) && (bt || (a.N % 4) == 0); }
// whether the product's kernel forms the rank-space activations (and the second projection) itself
bool projects(const GemmF32 &a, const float *Z, bool bt)
{
    const F32Plan p = plan_f32(a.M, a.N, a.K, vec_rows(a, bt));
    return p.stages > 0 && p.tm < 128 && (!bt || aligned16(Z));
}
int product(const GemmF32 &a, bool bt, hipStream_t st)
{
    const bool vec = vec_rows(a, bt);
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
    struct Form { int tm, tn, stages; float launch; int round; float a, b, a1, b1; };
    constexpr Form forms[5] = {{32, 64, 4, 2.8f, 256, 4.18f, .485f, 4.18f, .485f}, {64, 48, 4, 2.8f, 256, 5.90f, .610f, 5.90f, .610f},
                               {64, 64, 4, 2.8f, 256, 6.78f, .725f, 6.78f, .725f}, {64, 64, 2, 2.8f, 512, 5.94f, 1.518f, 5.74f, .864f},
                               {128, 128, 2, 5.5f, 256, 6.80f, 2.688f, 6.80f, 2.688f}};
    auto tiles = [&](int tm, int tn) { return (long)((M + tm - 1) / tm) * ((N + tn - 1) / tn); };
    const bool split = vec && K % 64 == 0 && (unsigned long long)M * K < (1ull << 30) && (unsigned long long)N * K < (1ull << 30);
    if (!split) {
        if (tiles(64, 64) < 96) return {16, 16, 0};
        return tiles(128, 128) < 512 ? F32Plan{64, 64, 0} : F32Plan{128, 128, 0};
    }
    const double nk = K / 64;
    F32Plan best = {0, 0, 0};
    double least = 0;
    if (tiles(16, 16) <= 1024) {
        best = {16, 16, 0};
        least = 5.9 + nk * (.25 + .27 * ((tiles(16, 16) + 255) / 256));
    }
    for (const Form &f : forms) {
        const long t = tiles(f.tm, f.tn), before = (t - 1) / f.round;
        const double c = f.launch + before * (f.a + f.b * nk) + (t - before * f.round > 256 ? f.a + f.b * nk : f.a1 + f.b1 * nk);
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
    GemmF32 a = {x, W, bias, ws, B, y, T, n_out, n_in, zp, r, 1, r, s, nullptr, nullptr, nullptr, nullptr, nullptr, 0};
    if (projects(a, A, true)) a.Z = A;
    else {
        const ProjJob j = {x, A, n_in, 1, n_in, ws};
        const int rc = project(&j, 1, T, r, zp, st);
        if (rc) return rc;
    }
    return product(a, true, st);
}

int f32_lora_linear_bwd(int T, int n_in, int n_out, int r, float s, const float *x, const float *dy,
                        const float *W, const float *A, const float *B, float *dx, float *dA, float *dB, float *ws,
                        hipStream_t st)
{
    const int zp = pad_rank(r);
    float *z = ws, *p = ws + (size_t)T * zp;
    GemmF32 a = {dy, W, nullptr, p, A, dx, T, n_in, n_out, zp, r, n_in, 1, s, nullptr, nullptr, nullptr, nullptr, nullptr, 0};
    int rc;
    if (projects(a, B, false)) {
        a.Z = B;
        a.zout = p;
        if (zp <= 8) {                                   // (16 rows of A for each row of x: a launch of its own is less)
            a.x2 = x;
            a.A2 = A;
            a.z2 = z;
            a.K2 = n_in;
        } else {
            const ProjJob j = {x, A, n_in, 1, n_in, z};
            if ((rc = project(&j, 1, T, r, zp, st))) return rc;
        }
    } else {
        const ProjJob pj[2] = {{x, A, n_in, 1, n_in, z}, {dy, B, 1, r, n_out, p}};
        if ((rc = project(pj, 2, T, r, zp, st))) return rc;
    }
    if ((rc = product(a, false, st))) return rc;
    const GradJobs gj = {{{x, p, n_in, dA, 1}, {dy, z, n_out, dB, 0}}};
    const dim3 grid(((n_in > n_out ? n_in : n_out) + 31) / 32, 2);
    if (zp == 4) hipLaunchKernelGGL((f32_grad_kernel<4>), grid, dim3(1024), 0, st, gj, T, r, s);
    else if (zp == 8) hipLaunchKernelGGL((f32_grad_kernel<8>), grid, dim3(1024), 0, st, gj, T, r, s);
    else hipLaunchKernelGGL((f32_grad_kernel<16>), grid, dim3(1024), 0, st, gj, T, r, s);
    SL_CHECK_LAUNCH("f32 adapter gradients");
    return 0;
}
