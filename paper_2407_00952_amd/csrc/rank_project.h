// Rank-space activations of a tall operand, out[M,16] = scale * X[M,K] . Z^T (Z [16,K], rows beyond the rank count as
// zero), rounded to bf16, with the MXFP8 codes and scales of X written in the same pass if asked for.
//
// Bound by HBM (2 bytes per element in, 1.03 more out with codes), so rows are read as whole 1 KB pieces: a block takes 16
// rows in pieces of 512 columns, each of its 4 waves loads, converts and stages 4 of the rows, and a quarter of the
// piece's MFMA steps is each wave's share; the 4 partial tiles are added in wave order.  (Reading the MFMA operands
// straight from memory, 16 rows x 64 bytes per instruction, moved [32768, 4096] at 3.0 TB/s.)
#pragma once
#include "common.h"
#include "mx_codec.h"

constexpr int RP_COLS = 512, RP_ROWB = RP_COLS * 2;
constexpr int RP_LDS = 2 * 16 * RP_ROWB;                 // two pieces; the partial tiles reuse the first

// Z: bf16 [16,K] padded with zero rows (ZF32 false), or the fp32 adapter [r,K] itself
template <bool QUANT, bool ZF32>
__device__ __forceinline__ void rank_project_rows(const bf16 *__restrict__ x, int M, int K, const void *__restrict__ Z, int r,
                                                  float scale, bf16 *__restrict__ out, unsigned char *__restrict__ codes,
                                                  unsigned char *__restrict__ scales, int row0, unsigned char *lds)
{
    typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));       // an adapter need not be 16-byte aligned
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r16 = lane & 15, kg = lane >> 4;
    bf16x8 v[4];
    auto fetch = [&](int c0) {
        const int col = min(c0 + lane * 8, K - 8);
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = *(const bf16x8 *)(x + (size_t)min(row0 + wave * 4 + i, M - 1) * K + col);
    };
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    fetch(0);
    int buf = 0;
    for (int c0 = 0; c0 < K; c0 += RP_COLS, buf ^= 1) {
        unsigned char *st = lds + buf * (16 * RP_ROWB);
        // this wave's k-steps of the piece: wave, wave + 4, ..
        bf16x8 zb[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int k = min(c0 + (wave + 4 * s) * 32, K - 32) + kg * 8;
            if (ZF32) {
                const float *zp = (const float *)Z + (size_t)min(r16, r - 1) * K + k;
                const f32x4u a0 = *(const f32x4u *)zp, a1 = *(const f32x4u *)(zp + 4);
                zb[s] = bf16x8{f2bf(a0.x), f2bf(a0.y), f2bf(a0.z), f2bf(a0.w), f2bf(a1.x), f2bf(a1.y), f2bf(a1.z), f2bf(a1.w)};
            } else {
                zb[s] = *(const bf16x8 *)((const bf16 *)Z + (size_t)r16 * K + k);
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int rl = wave * 4 + i, row = row0 + rl, col = c0 + lane * 8;
            // 16-byte chunks XORed with the row: the 16 rows an operand read touches fall into different banks
            *(bf16x8 *)(st + rl * RP_ROWB + ((lane ^ rl) << 4)) = v[i];
            if (QUANT) {
                union { bf16x8 b; unsigned w[4]; } u;
                u.b = v[i];
                unsigned mag = 0u;
#pragma unroll
                for (int j = 0; j < 4; ++j) mag = max(mag, max(u.w[j] & 0x7FFFu, (u.w[j] >> 16) & 0x7FFFu));
                mag = max(mag, (unsigned)__shfl_xor((int)mag, 1, 64));
                mag = max(mag, (unsigned)__shfl_xor((int)mag, 2, 64));
                const int scode = mx_scale_code(mag);
                unsigned q[2];
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    q[j] = mx_encode_pair_bf16(u.w[2 * j] & 0xFFFFu, u.w[2 * j] >> 16, scode) |
                           (mx_encode_pair_bf16(u.w[2 * j + 1] & 0xFFFFu, u.w[2 * j + 1] >> 16, scode) << 16);
                if (row < M && col < K) {
                    *(uint2 *)(codes + (size_t)row * K + col) = make_uint2(q[0], q[1]);
                    if ((lane & 3) == 0) scales[(size_t)row * (K >> 5) + (col >> 5)] = (unsigned char)scode;
                }
            }
        }
        if (c0 + RP_COLS < K) fetch(c0 + RP_COLS);
        __syncthreads();                                 // (two buffers: one barrier per piece)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int ks = wave + 4 * s;
            if (c0 + ks * 32 < K) {
                const bf16x8 xa = *(const bf16x8 *)(st + r16 * RP_ROWB + (((ks * 4 + kg) ^ r16) << 4));
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa, zb[s], acc, 0, 0, 0);
            }
        }
    }
    __syncthreads();
    float(*red)[16][17] = (float(*)[16][17])lds;
#pragma unroll
    for (int e = 0; e < 4; ++e) red[wave][4 * kg + e][r16] = acc[e];
    __syncthreads();
    const int m = threadIdx.x >> 4, j = threadIdx.x & 15;
    float t = red[0][m][j];
#pragma unroll
    for (int w = 1; w < 4; ++w) t += red[w][m][j];
    if (row0 + m < M) out[(size_t)(row0 + m) * SL_RP + j] = f2bf(j < r ? t * scale : 0.f);
}
