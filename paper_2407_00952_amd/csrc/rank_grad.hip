// One pass over the gradient of an adapted projection's output for the two products of the backward pass that read it beside
// the frozen one (gfx950), per job:
//
//   ps [T,16] = s dY B                    (row-wise, into columns of the rank-space gradients; bf16)
//   partial sums of dB = dY^T zs          (token-wise; zs [T,16] saved by the forward; fp32, added by lora_grad_reduce_kernel)
//   and, if asked for, dY's MXFP8 codes and scales
//
// A block of 8 waves owns HT times 128 tokens and walks all C columns in slabs of 256.  Asynchronous copies bring 64 tokens of a
// slab at a time into a ring in LDS, three such units ahead, and B's rows beside them: a wave's 16 tokens of every 128 meet B along
// the columns, and its 32 columns meet zs along the tokens (operand fragments by the LDS transpose read, zs held in
// registers).  The sum over the columns is one chain in increasing order, 32 a step, which is the one that a product kernel
// forms in its main loop: the rank-space gradients, and with them a sequence's results, are the same bits either way.
//
// Bound by reading dY once, in pieces of 512 bytes of a row: all blocks walk the columns in step, and a tensor whose rows
// are kilobytes apart is read at 2.7 TB/s in pieces of 256; and a block that waits for one unit with nothing behind it leaves its
// CU's memory path idle for a round trip (72 KB at a time: 2.9 TB/s).  32768 x 4096 with codes (422 MB) 112 us, where the
// conversion with the projection took 98 and dB's share of the gradients' launch 69.  The partial sums are r / (64 HT) of dY: HT = 1 up
// to rank 4, 2 beyond.
#include "common.h"
#include "gemm_copy.h"
#include "mx_codec.h"
#include "prof.h"

namespace {

constexpr int RG_MAX_JOBS = 3;
struct RankGradJobs { RankGradDesc j[RG_MAX_JOBS]; };

typedef short v4s_t __attribute__((ext_vector_type(4)));
// column `lane % 16` of four rows: lane e * 4 + q of a group of 16 addresses columns 4 q .. + 3 of row e
__device__ __forceinline__ bf16x8 rows8_tr(const unsigned char *lo, const unsigned char *hi)
{
    union { v4s_t s[2]; bf16x8 v; } u;
    u.s[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s_t *)lo);
    u.s[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s_t *)hi);
    return u.v;
}

template <int HT, bool QUANT>
__global__ __launch_bounds__(512, 1) void rank_grad_kernel(RankGradJobs jobs, int T, int r, float s)
{
    constexpr int R = HT * 128, U = HT * 2;              // tokens of the block, units of a slab
    constexpr int UNIT = 4 * 64 * 128, ZB = 4 * 2048;    // 64 rows, 16 rows of B^T, each by pieces of 64 columns
    constexpr int NST = 4, NZS = 3;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[NST * UNIT + NZS * ZB];
    const RankGradDesc &jb = jobs.j[blockIdx.y];
    const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, kg = lane >> 4, sw = r16 & 7;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t0 = blockIdx.x * R, ns = jb.C / 256;
    const int lrow = lane >> 3, lch = (lane & 7) ^ (lane >> 3);

    // zs as MFMA operands: through LDS, [R][16], rows past the last token zero
    bf16x8 zb[U][2];
    {
        if (tid < R) {
            uint4 a = {0, 0, 0, 0}, b = a;
            if (t0 + tid < T) {
                const uint4 *q = (const uint4 *)(jb.zs + (size_t)(t0 + tid) * SL_RP);
                a = q[0];
                b = q[1];
            }
            *(uint4 *)(lds + tid * 32) = a;
            *(uint4 *)(lds + tid * 32 + 16) = b;
        }
        __syncthreads();
        const unsigned char *z = lds + (kg * 8 + ((lane >> 2) & 3)) * 32 + (lane & 3) * 8;
#pragma unroll
        for (int k = 0; k < U * 2; ++k) zb[k >> 1][k & 1] = rows8_tr(z + k * 32 * 32, z + k * 32 * 32 + 4 * 32);
        __syncthreads();
    }

    // copies (1 KB, 8 rows of a piece): a wave's 8 rows of each piece of a unit; with a slab's first unit 8 rows of one piece of B^T
    unsigned xo[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
        xo[u] = ((unsigned)min(t0 + u * 64 + wave * 8 + lrow, T - 1) * (unsigned)jb.ldx + lch * 8) * 2u;
    const int zrow = (wave & 1) * 8, zsub = wave >> 1;
    const unsigned zo = ((unsigned)(zrow + lrow) * (unsigned)jb.ldz + zsub * 64 + lch * 8) * 2u;
    const unsigned base = lds_addr(lds) + wave * 1024, zl = lds_addr(lds) + NST * UNIT + zsub * 2048 + zrow * 128;
    // unit u of slab k (past the last slab: it once more, in bounds, never read) into ring slot `slot`, B^T into zslot
    auto copy = [&](int slot, int k, int u, int zslot) {
        const size_t kb = (size_t)min(k, ns - 1) * 512;
        if (u == 0) glds_soff((const char *)jb.Z + kb, zo, zl + zslot * ZB);
#pragma unroll
        for (int p = 0; p < 4; ++p) glds_soff((const char *)jb.X + kb + p * 128, xo[u], base + slot * UNIT + p * 8192);
    };
#pragma unroll
    for (int n = 0; n < 3; ++n) copy(n, n / U, n % U, n / U);

    f32x4 zacc[HT], g[2];
#pragma unroll
    for (int h = 0; h < HT; ++h) zacc[h] = f32x4{0.f, 0.f, 0.f, 0.f};
    // the wave's columns: two chunks of 8 in each of column tiles 2 wave, 2 wave + 1 (four to a piece); token rows of the transposed
    // reads: 8 kg + e, and 4 more, of a step of 32
    const int te = kg * 8 + ((lane >> 2) & 3), tc = (wave & 1) * 4 + ((lane & 3) >> 1), tb = (lane & 1) * 8;
    float *const out = jb.partials + ((size_t)blockIdx.x * r + min(r16, r - 1)) * jb.C + wave * 32 + 4 * kg;
    const bool whole = t0 + R <= T;
    // The unit to be read has landed, the two newer ones may be in flight (4 copies each, 5 for a slab's first).  The counter
    // is in order and counts stores too: where every row is a token, two units' stores of codes, 8 each
    // (tests/test_kernel_isa.py), lie behind a unit's copies from the third on; elsewhere none are allowed for.
    constexpr int STORES = QUANT ? 8 : 0;
    int slot = 0, zslot = 0;
    for (int k = 0; k < ns; ++k) {
        g[0] = g[1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < U; ++u) {
            constexpr int LAST = U - 1;
            const int ahead = u + 2 > LAST ? 9 : 8;
            if (QUANT && whole && (k > 0 || u > 1)) {
                if (ahead == 9) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(9 + 2 * STORES) : "memory");
                else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(8 + 2 * STORES) : "memory");
            } else if (ahead == 9) asm volatile("s_waitcnt vmcnt(9)" ::: "memory");
            else asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
            __syncthreads();
            const int nz = zslot + (u + 3) / U;
            copy(slot == 0 ? NST - 1 : slot - 1, k + (u + 3) / U, (u + 3) % U, nz >= NZS ? nz - NZS : nz);
            const unsigned char *S = lds + slot * UNIT;
            // rank-space gradients: a unit's tokens against B, by four of the waves
            if ((wave >> 2) == (u & 1)) {
                const unsigned char *Z = lds + NST * UNIT + zslot * ZB;
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int co = (((q & 1) * 4 + kg) ^ sw) << 4;
                    const bf16x8 b = *(const bf16x8 *)(Z + (q >> 1) * 2048 + r16 * 128 + co);
                    const bf16x8 a = *(const bf16x8 *)(S + (q >> 1) * 8192 + ((wave & 3) * 16 + r16) * 128 + co);
                    zacc[u >> 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, zacc[u >> 1], 0, 0, 0);
                }
            }
            // dB: the wave's columns against zs
            const unsigned char *P = S + (wave >> 1) * 8192 + tb;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int ra = i * 32 + te, rb = ra + 4;
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const bf16x8 a = rows8_tr(P + ra * 128 + (((tc + 2 * c) ^ (ra & 7)) << 4), P + rb * 128 + (((tc + 2 * c) ^ (rb & 7)) << 4));
                    g[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, zb[u][i], g[c], 0, 0, 0);
                }
            }
            if (QUANT) {
                // 32 lanes to a row, four to a block of 32 columns
                auto encode = [&](int i, bool all) {
                    const int rl = wave * 8 + i * 2 + (lane >> 5), ch = lane & 31;
                    const int row = t0 + u * 64 + rl, col = k * 256 + ch * 8;
                    union { bf16x8 b; unsigned w[4]; } x;
                    x.b = *(const bf16x8 *)(S + (ch >> 3) * 8192 + rl * 128 + (((ch & 7) ^ (rl & 7)) << 4));
                    unsigned mag = 0u;
#pragma unroll
                    for (int j = 0; j < 4; ++j) mag = max(mag, max(x.w[j] & 0x7FFFu, (x.w[j] >> 16) & 0x7FFFu));
                    mag = max(mag, (unsigned)__shfl_xor((int)mag, 1, 64));
                    mag = max(mag, (unsigned)__shfl_xor((int)mag, 2, 64));
                    const int scode = mx_scale_code(mag);
                    unsigned q[2];
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        q[j] = mx_encode_pair_bf16(x.w[2 * j] & 0xFFFFu, x.w[2 * j] >> 16, scode) |
                               (mx_encode_pair_bf16(x.w[2 * j + 1] & 0xFFFFu, x.w[2 * j + 1] >> 16, scode) << 16);
                    if (all || row < T) {
                        *(uint2 *)(jb.codes + (size_t)row * jb.C + col) = make_uint2(q[0], q[1]);
                        if ((lane & 3) == 0) jb.scales[(size_t)row * (jb.C >> 5) + (col >> 5)] = (unsigned char)scode;
                    }
                };
                if (whole) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) encode(i, true);
                } else {
                    for (int i = 0; i < 4; ++i) encode(i, false);
                }
            }
            slot = slot + 1 == NST ? 0 : slot + 1;
        }
        zslot = zslot + 1 == NZS ? 0 : zslot + 1;
        if (r16 < r) {
#pragma unroll
            for (int c = 0; c < 2; ++c) *(float4 *)(out + k * 256 + c * 16) = make_float4(g[c][0], g[c][1], g[c][2], g[c][3]);
        }
    }
#pragma unroll
    for (int h = 0; h < HT; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = t0 + h * 128 + wave * 16 + 4 * kg + e;
            // zero beyond the rank also where an infinity met a zero of B^T
            if (row < T) jb.ps[(size_t)row * jb.ldp + r16] = f2bf(r16 < r ? zacc[h][e] * s : 0.f);
        }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // the copies past the last slab land before the block's LDS is given back
}

}  // namespace

int rank_grad_rows(int r) { return r <= 4 ? 128 : 256; }
// Layers with MXFP8 weights, forward + backward in us, as separate passes and as this one: 8192 x 1024 -> 4096 (64 blocks) 156, 184;
// 18432 x 768 -> 2304 (144) 171, 179; 20480 x 768 -> 2304 (160) 191, 185; 20480 x 4096 -> 1024 407, 397; 20480 x 1024 -> 4096 384, 354;
// 32768 x 1024 -> 4096 (256) 584, 521; rank 8: 12000 x 1280 -> 5120 (47) 318, 408; 40960 x 1280 -> 3840 (160) 769, 717.  Stacks of two
// layers: 1280 wide, q, v, 20480 tokens, rank 8 (160 blocks) 4130, 4066; all six, rank 4 4755, 4691; 24576 tokens (192) 5341, 5250;
// 768 wide, all six, 20480 tokens, rank 4, passes in front of products of 768 among them, 2237, 2254: what a narrow product saves, a pass
// costs.  `width` is the product's contraction, for q, k and v that of the three slices though a pass reads one: three layers 768
// wide, 12800 tokens, q and v, rank 4 (200 blocks) 2101, 2090; 16384, q, k and v, rank 8 (192) 2446, 2411; 40960, q, rank 8 (160) 5341, 5310.
bool rank_grad_fills(int T, int njobs, int r, int width)
{
    return (long)((T + rank_grad_rows(r) - 1) / rank_grad_rows(r)) * njobs >= (width >= 1024 ? 160 : 224);
}

int launch_rank_grad(const RankGradDesc *d, int njobs, int r, float s, int T, hipStream_t st)
{
    if (njobs < 1 || njobs > RG_MAX_JOBS || T <= 0 || r < 1 || r > SL_RP) return SL_EINVAL;
    RankGradJobs jobs;
    double bytes = 0.0;
    const bool quant = d[0].codes != nullptr;
    for (int k = 0; k < njobs; ++k) {
        const RankGradDesc &q = d[k];
        if (!q.X || !q.Z || !q.zs || !q.ps || !q.partials || q.C <= 0 || (q.C % 256) || (q.ldx % 8) || (q.ldz % 8) ||
            (unsigned long long)T * q.ldx * 2ull >= (1ull << 32) || (q.codes != nullptr) != quant || (quant && !q.scales))
            return SL_EINVAL;
        jobs.j[k] = q;
        bytes += 2.0 * T * (double)q.C;
    }
    const int R = rank_grad_rows(r);
    const dim3 grid((T + R - 1) / R, njobs), block(512);
    const bool rec = prof_begin(PK_LORA_GRAD, st);
    if (R == 128 && quant) hipLaunchKernelGGL((rank_grad_kernel<1, true>), grid, block, 0, st, jobs, T, r, s);
    else if (R == 128) hipLaunchKernelGGL((rank_grad_kernel<1, false>), grid, block, 0, st, jobs, T, r, s);
    else if (quant) hipLaunchKernelGGL((rank_grad_kernel<2, true>), grid, block, 0, st, jobs, T, r, s);
    else hipLaunchKernelGGL((rank_grad_kernel<2, false>), grid, block, 0, st, jobs, T, r, s);
    prof_end(rec, PK_LORA_GRAD, bytes, st);
    SL_CHECK_LAUNCH("rank grad");
    return 0;
}
