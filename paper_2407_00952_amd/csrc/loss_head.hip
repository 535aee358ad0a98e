// Loss head of the server (SplitLoRA Sec. III-B: the clients send their labels with the activations
// in step a2; in step a3 the server turns its predicted value and the labels into the loss and starts
// the backward pass from it).  GPT-2's head: final LayerNorm, logits against the frozen token-embedding
// matrix Wv [V, d], token cross-entropy averaged over the labeled tokens; nothing here is trainable, so
// the only gradient produced is dY, the input of the server stack's backward pass.
//
// Only labeled tokens have a loss and a gradient (in prompt-completion records a quarter to a half of the tokens are
// prompt), so everything runs on them alone: the device lists the labeled rows first and the others behind them, and the
// kernels take the number of rows from memory; nothing synchronises the stream.  (Logits that fit a few small tiles are
// formed for the chunk's other rows too, from whatever u holds there; nobody reads them.)  Per chunk of at most 16384 listed rows
// (HBM is large: the chunk's logits are materialised once as bf16, 1.65 GB, instead of being recomputed):
//   u      = LN(y)                                 wave-per-row LayerNorm of the listed rows
//   logits = u . WvP^T            [rows, Vp]       bf16 MFMA GEMM (Vp = V rounded up to 64, zero rows)
//   dlogits = (softmax(logits) - onehot) / n       one block per row, the row held in registers,
//   loss_tok = logsumexp - logits[label]           written over the logits
//   du     = dlogits . Wv         [rows, d]        the same GEMM on the transposed copy WvT [d, Vp], its long
//                                                  contraction shared over blocks, the shares' sums kept in fp32
//   dY     = LN^T(du)                              LayerNorm input gradient, all rows (du = 0 on unlabeled ones)
// and one fixed-order reduction of loss_tok.
// Measured, d = 1024, V = 50257: 32768 tokens, 20 k of them labeled, 6.43 -> 4.31 ms (all rows, unshared contraction before;
// the two products run at 1.09 and 1.48 PFLOP/s); 1098 tokens 952 -> 239 us; 65 tokens of 768 902 -> 118 us.
#include "../../include/slora.h"
#include "common.h"
#include "prof.h"

#include <cstring>

namespace {

// 1024 threads, so that a thread's share of the longest row leaves room for 8 waves on each SIMD, two rows on a CU: one row's
// loads and stores run under the other's arithmetic (16384 rows of 50304: 764 us with one row on a CU, 671 with 512
// threads and two, 604 here = 5.5 TB/s)
constexpr int CE_THR = 1024;
constexpr int CE_MAXCH = 8;              // 16-byte chunks per thread: padded vocabulary <= 65536
// short rows, most of whose 1024 threads would only wait at the reductions (16384 rows of 1000: 94 us with 512 threads, 101 with
// 1024, 24 here; the whole head of 4096 tokens, width 1024, vocabulary 2000: 96, 111 and 93 us)
constexpr int CE_SHORT_THR = 256;
constexpr int CE_SHORT_MAXCH = 2;        // padded vocabulary <= 4096
constexpr int LH_CHUNK = 16384;          // labeled tokens per pass
constexpr int LH_MAXC = 8;               // 256-column chunks of a LayerNorm row: d <= 2048
constexpr int LH_SHARES = 64;            // most blocks a tile's contraction is shared over (one per lane below)
constexpr int LH_PART_ROWS = 65536;      // rows of partial sums a large batch has scratch for
constexpr int LH_SHARE_SLABS = 4;        // fewest slabs of a share

struct LabelCount { int n; float inv_n; };

inline size_t al256(size_t v) { return (v + 255) & ~(size_t)255; }
inline int vocab_padded(int V) { return (V + 63) / 64 * 64; }

// Rows of partial sums for up to `rows` labeled ones: the shares that the slabs of the vocabulary allow, and for every 1024 rows those
// of one round of 256 blocks.  list_labels_kernel picks no more than that of itself (checked for every row count, width
// and a sweep of vocabularies), so the limit changes no result.
inline int part_rows(int rows, int d, int V)
{
    const int slabs = vocab_padded(V) / 64 / LH_SHARE_SLABS;
    const int shares = slabs < 1 ? 1 : slabs < LH_SHARES ? slabs : LH_SHARES;
    const int rounds = (rows + 1023) / 1024 * (256 * 256 / ((d + 255) / 256));
    const int most = rounds < LH_PART_ROWS ? rounds : LH_PART_ROWS;
    return rows * shares < most ? rows * shares : most;
}

template <int THR>
__device__ __forceinline__ float block_reduce(float v, bool is_max, float *red)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float w = __shfl_xor(v, o, 64);
        v = is_max ? fmaxf(v, w) : v + w;
    }
    const int wave = threadIdx.x >> 6;
    __syncthreads();                     // `red` may still be read from the previous reduction
    if ((threadIdx.x & 63) == 0) red[wave] = v;
    __syncthreads();
    float r = red[0];
#pragma unroll
    for (int i = 1; i < THR / 64; ++i) r = is_max ? fmaxf(r, red[i]) : r + red[i];
    return r;
}

// labels >= 0 (and < V) carry a loss; anything else marks a token without label
__device__ __forceinline__ bool labeled(int l, int V) { return l >= 0 && l < V; }

// perm = the labeled rows in order, then the others in order; their number; and per chunk the rows of its products and
// over how many blocks a tile of the input-gradient product shares its contraction.  One block: a wave counts, then
// places, a contiguous piece of the rows (32768 rows: 128 KB read twice).
//
// Shares.  That product has few tiles (d / 256 columns of them) and a contraction of Vp, up to 50304: unshared, the 4096 rows
// that a second chunk of 20480 labeled tokens holds would keep 64 of 256 CUs busy as long as 16384 rows keep all of them.
// Cost of s shares in us: rounds of 256 blocks, each 1.41 us per slab of its share and about 8 to fill and drain, and the
// sums' way through HBM (written and read once, about 5 TB/s).
__global__ __launch_bounds__(1024) void list_labels_kernel(const int *__restrict__ labels, int T, int V, int d, int nk,
                                                           int tile_rows, int part_rows, int *__restrict__ perm,
                                                           LabelCount *__restrict__ out, CountedRows *__restrict__ chunks)
{
    __shared__ int cnt[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int per = ((T + 1023) / 1024) * 64;            // rows of a wave
    const int lo = (int)min((long long)wave * per, (long long)T), hi = min(lo + per, T);
    int n = 0;
    for (int i = lo; i < hi; i += 64 * 8) {              // eight loads in flight
        int l[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) l[k] = labels[min(i + k * 64 + lane, T - 1)];
#pragma unroll
        for (int k = 0; k < 8; ++k) n += __popcll(__ballot(i + k * 64 + lane < hi && labeled(l[k], V)));
    }
    if (lane == 0) cnt[wave] = n;
    __syncthreads();
    int before = 0, total = 0;
    for (int w = 0; w < 16; ++w) {
        before += w < wave ? cnt[w] : 0;
        total += cnt[w];
    }
    int yes = before, no = total + lo - before;          // where the wave's next labeled and unlabeled rows go
    for (int i = lo; i < hi; i += 64 * 8) {
        int l[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) l[k] = labels[min(i + k * 64 + lane, T - 1)];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int r = i + k * 64 + lane;
            const bool in = r < hi, is = in && labeled(l[k], V);
            const unsigned long long m = __ballot(is);
            const int lb = __popcll(m & ((1ull << lane) - 1));
            if (in) perm[is ? yes + lb : no + lane - lb] = r;
            yes += __popcll(m);
            no += max(0, min(64, hi - i - k * 64)) - __popcll(m);
        }
    }
    if (threadIdx.x == 0) {
        out->n = total;
        out->inv_n = total > 0 ? 1.0f / (float)total : 0.0f;
    }
    for (int c = wave; (long long)c * LH_CHUNK < T; c += 16) {
        const int rows = max(0, min(total - c * LH_CHUNK, LH_CHUNK));
        const int tiles = ((rows + tile_rows - 1) / tile_rows) * ((d + 255) / 256);
        const int s = lane + 1;
        const int rounds = (tiles * s + 255) / 256;
        const bool ok = s == 1 || (s * LH_SHARE_SLABS <= nk && (long long)s * rows <= part_rows);
        float cost = ok ? rounds * (1.41f * ((nk + s - 1) / s) + 8.0f) + (float)s * rows * d * 1.6e-6f : INFINITY;
        int best = s;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const float oc = __shfl_xor(cost, o, 64);
            const int ob = __shfl_xor(best, o, 64);
            if (oc < cost || (oc == cost && ob < best)) { cost = oc; best = ob; }
        }
        if (lane == 0) chunks[c] = CountedRows{rows, best};
    }
}

// Mean and reciprocal deviation of a row of y held by one wave (v: in the row's values, out the centred ones); the same
// operations in the same order as the stack's LayerNorm kernels.
__device__ __forceinline__ void row_stats(const bf16 *y, int d, int lane, float eps, float (&v)[LH_MAXC][4],
                                          float &mu, float &rho)
{
    float s = 0.f;
#pragma unroll
    for (int c = 0; c < LH_MAXC; ++c) {
        const int col = c * 256 + lane * 4;
        if (col < d) {
            const bf16x4 t = *(const bf16x4 *)(y + col);
#pragma unroll
            for (int i = 0; i < 4; ++i) { v[c][i] = bf2f(t[i]); s += v[c][i]; }
        }
    }
    mu = wave_sum(s) / (float)d;
    float q = 0.f;
#pragma unroll
    for (int c = 0; c < LH_MAXC; ++c) {
        if (c * 256 + lane * 4 < d) {
#pragma unroll
            for (int i = 0; i < 4; ++i) { v[c][i] -= mu; q += v[c][i] * v[c][i]; }
        }
    }
    rho = rsqrtf(wave_sum(q) / (float)d + eps);
}

// u = LN(y) of the chunk's labeled rows.  HBM-bound: 4 B per element.
__global__ __launch_bounds__(256) void head_ln_fwd_kernel(const bf16 *__restrict__ y, const int *__restrict__ perm,
                                                          const CountedRows *__restrict__ chunk,
                                                          const bf16 *__restrict__ gamma, const bf16 *__restrict__ beta,
                                                          float eps, bf16 *__restrict__ u, int d)
{
    const int lane = threadIdx.x & 63, i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= chunk->rows) return;
    float v[LH_MAXC][4], mu, rho;
    row_stats(y + (size_t)perm[i] * d, d, lane, eps, v, mu, rho);
#pragma unroll
    for (int c = 0; c < LH_MAXC; ++c) {
        const int col = c * 256 + lane * 4;
        if (col < d) {
            const bf16x4 gm = *(const bf16x4 *)(gamma + col), bt = *(const bf16x4 *)(beta + col);
            bf16x4 o;
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j] = f2bf(v[c][j] * rho * bf2f(gm[j]) + bf2f(bt[j]));
            *(bf16x4 *)(u + (size_t)i * d + col) = o;
        }
    }
}

// dY of `n` listed rows: the chunk's labeled ones from the shares' sums of du, the rest with du = 0 (which also carries
// a NaN of y into dY, as the formula has it).  The statistics are formed again from y (2 B per element) instead of
// being read with an fp32 copy of it.
__global__ __launch_bounds__(256) void head_ln_bwd_kernel(const bf16 *y, const int *__restrict__ perm, int n,
                                                          const CountedRows *__restrict__ chunk,
                                                          const float *__restrict__ part,
                                                          const bf16 *__restrict__ gamma, float eps,
                                                          bf16 *dy, int d)      // (dy may be y)
{
    const int lane = threadIdx.x & 63, i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= n) return;
    const int rows = chunk->rows, shares = i < rows ? chunk->shares : 0;
    const size_t row = (size_t)perm[i] * d;
    float xh[LH_MAXC][4], g[LH_MAXC][4], mu, rho;
    row_stats(y + row, d, lane, eps, xh, mu, rho);
#pragma unroll
    for (int c = 0; c < LH_MAXC; ++c)
#pragma unroll
        for (int j = 0; j < 4; ++j) g[c][j] = 0.f;
    const float *p = part + (size_t)i * d + lane * 4;
    for (int s = 0; s < shares; ++s, p += (size_t)rows * d) {
#pragma unroll
        for (int c = 0; c < LH_MAXC; ++c) {
            if (c * 256 + lane * 4 < d) {
                const float4 t = *(const float4 *)(p + c * 256);
                g[c][0] += t.x; g[c][1] += t.y; g[c][2] += t.z; g[c][3] += t.w;
            }
        }
    }
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int c = 0; c < LH_MAXC; ++c) {
        const int col = c * 256 + lane * 4;
        if (col < d) {
            const bf16x4 gm = *(const bf16x4 *)(gamma + col);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                g[c][j] *= bf2f(gm[j]);
                xh[c][j] *= rho;
                s1 += g[c][j];
                s2 += g[c][j] * xh[c][j];
            }
        }
    }
    const float m1 = wave_sum(s1) / (float)d, m2 = wave_sum(s2) / (float)d;
#pragma unroll
    for (int c = 0; c < LH_MAXC; ++c) {
        const int col = c * 256 + lane * 4;
        if (col < d) {
            bf16x4 o;
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j] = f2bf(0.f + rho * (g[c][j] - m1 - xh[c][j] * m2));
            *(bf16x4 *)(dy + row + col) = o;
        }
    }
}

// two bf16 values of a dword as floats
__device__ __forceinline__ float lo_f(unsigned w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_f(unsigned w) { return __uint_as_float(w & 0xFFFF0000u); }
__device__ __forceinline__ float pair_max(unsigned w) { return fmaxf(lo_f(w), hi_f(w)); }

// One block per listed row.  logits [rows, ldl] bf16 in; the same memory receives
// d loss / d logits = (softmax - onehot) * inv_n (zero in the padding columns).  Rows past the labeled ones have none.
template <int THR, int MAXCH>
__global__ __launch_bounds__(THR) __attribute__((amdgpu_waves_per_eu(8, 8))) void softmax_ce_kernel(bf16 *__restrict__ logits, int ldl, int V,
                                                            const int *__restrict__ labels,
                                                            const int *__restrict__ perm,
                                                            const CountedRows *__restrict__ chunk,
                                                            const LabelCount *__restrict__ cnt,
                                                            float *__restrict__ loss_tok)
{
    __shared__ float red[THR / 64];
    const int tid = threadIdx.x, row = perm[blockIdx.x];
    if ((int)blockIdx.x >= chunk->rows) {
        if (tid == 0) loss_tok[row] = 0.f;
        return;
    }
    const int label = labels[row];
    bf16 *p = logits + (size_t)blockIdx.x * ldl;
    const int nch = ldl >> 3;
    const float picked = bf2f(p[label]);     // read before any thread overwrites the row (barriers below)
    const float l2e = 1.4426950408889634f;
    uint4 v[MAXCH];                       // the row's bf16 values, two to a dword
    float m = -INFINITY;
#pragma unroll
    for (int c = 0; c < MAXCH; ++c) {
        const int ch = tid + c * THR;
        if (ch < nch) v[c] = *(const uint4 *)(p + ch * 8);
    }
#pragma unroll
    for (int c = 0; c < MAXCH; ++c) {
        const int ch = tid + c * THR;
        if (ch < nch) {
            if (ch * 8 + 8 > V) {            // padding columns become -inf: no probability, no gradient
                unsigned *w = (unsigned *)&v[c];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (ch * 8 + 2 * i >= V) w[i] = 0xFF80FF80u;
                    else if (ch * 8 + 2 * i + 1 >= V) w[i] = (w[i] & 0xFFFFu) | 0xFF800000u;
                }
            }
            m = fmaxf(m, fmaxf(fmaxf(pair_max(v[c].x), pair_max(v[c].y)), fmaxf(pair_max(v[c].z), pair_max(v[c].w))));
        }
    }
    m = block_reduce<THR>(m, true, red);
    // The unpacked values would not all fit in registers beside the packed ones: without this the compiler keeps
    // them from pass to pass and half the waves have no room.
#pragma unroll
    for (int c = 0; c < MAXCH; ++c) asm volatile("" : "+v"(v[c].x), "+v"(v[c].y), "+v"(v[c].z), "+v"(v[c].w));
    float s = 0.f;
#pragma unroll
    for (int c = 0; c < MAXCH; ++c) {
        const int ch = tid + c * THR;
        if (ch < nch) {
            const unsigned w[4] = {v[c].x, v[c].y, v[c].z, v[c].w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                s += __builtin_amdgcn_exp2f((lo_f(w[i]) - m) * l2e);
                s += __builtin_amdgcn_exp2f((hi_f(w[i]) - m) * l2e);
            }
        }
    }
    s = block_reduce<THR>(s, false, red);
#pragma unroll
    for (int c = 0; c < MAXCH; ++c) asm volatile("" : "+v"(v[c].x), "+v"(v[c].y), "+v"(v[c].z), "+v"(v[c].w));
    const float lse = m + __logf(s);
    if (tid == 0) loss_tok[row] = lse - picked;
    const float inv_n = cnt->inv_n;
#pragma unroll
    for (int c = 0; c < MAXCH; ++c) {
        const int ch = tid + c * THR;
        if (ch < nch) {
            const unsigned w[4] = {v[c].x, v[c].y, v[c].z, v[c].w};
            bf16x8 o;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                o[2 * i] = f2bf(__builtin_amdgcn_exp2f((lo_f(w[i]) - lse) * l2e) * inv_n);
                o[2 * i + 1] = f2bf(__builtin_amdgcn_exp2f((hi_f(w[i]) - lse) * l2e) * inv_n);
            }
            *(bf16x8 *)(p + ch * 8) = o;
            // the thread that owns the label's column stores that one again
            if (ch == label >> 3) p[label] = f2bf((__builtin_amdgcn_exp2f((picked - lse) * l2e) - 1.0f) * inv_n);
        }
    }
}

// loss = (sum_t loss_tok[t]) / n, one block, fixed order, double accumulation
__global__ __launch_bounds__(1024) void loss_mean_kernel(const float *__restrict__ loss_tok, int T,
                                                         const LabelCount *__restrict__ cnt, float *__restrict__ loss)
{
    __shared__ double red[1024];
    double a = 0.0;
    for (int i = threadIdx.x; i < T; i += 1024 * 8) {    // eight loads in flight
        float v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = loss_tok[min(i + k * 1024, T - 1)];
#pragma unroll
        for (int k = 0; k < 8; ++k) a += i + k * 1024 < T ? (double)v[k] : 0.0;
    }
    red[threadIdx.x] = a;
    __syncthreads();
    for (int o = 512; o > 0; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = (float)(red[0] / (double)cnt->n);   // n = 0: 0/0 = NaN marks "no labeled token"
}

struct HeadWs {
    size_t WvP, WvT;                     // persistent: independent of the token count
    size_t cnt, chunks, perm, u, part, logits, total;
};

HeadWs head_ws(int T, int d, int V)
{
    const size_t Vp = (size_t)vocab_padded(V);
    HeadWs w;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += al256(bytes); return o; };
    w.WvP = take(2 * Vp * d);
    w.WvT = take(2 * Vp * d);
    const int rows = T < LH_CHUNK ? T : LH_CHUNK;
    w.cnt = take(sizeof(LabelCount));
    w.chunks = take(sizeof(CountedRows) * ((size_t)(T - 1) / LH_CHUNK + 1));
    w.perm = take(4 * (size_t)T);
    w.u = take(2 * (size_t)rows * d);
    w.part = take(4 * (size_t)part_rows(rows, d, V) * d);
    w.logits = take(2 * (size_t)rows * Vp);
    w.total = off;
    return w;
}

bool head_args_ok(int T, int d, int V)
{
    if (T <= 0 || d <= 0 || V <= 0) return false;
    if ((d % 64) || d > 2048) return false;
    if (vocab_padded(V) > CE_MAXCH * CE_THR * 8) return false;
    return true;
}

GemmArgs plain_gemm(const bf16 *X, int ldx, const bf16 *W, int ldw, int M, int N, int K, void *out, int ldo)
{
    GemmArgs a;
    memset(&a, 0, sizeof(a));
    a.X = X; a.ldx = ldx; a.W = W; a.ldw = ldw; a.M = M; a.N = N; a.K = K;
    a.nseg = 1; a.seg_n = N; a.ldo = ldo; a.out0 = out; a.K2 = 16; a.ldz = K; a.ldt = 32;
    return a;
}

}  // namespace

extern "C" {

size_t slora_loss_head_ws_bytes(int32_t max_tokens, int32_t d_model, int32_t vocab)
{
    if (!head_args_ok(max_tokens, d_model, vocab)) return 0;
    return head_ws(max_tokens, d_model, vocab).total;
}

int slora_loss_head_prepare(int32_t d_model, int32_t vocab, const void *Wv, void *ws, size_t ws_bytes, void *stream)
{
    if (!head_args_ok(1, d_model, vocab) || !Wv || !ws) return SLORA_EINVAL;
    if ((((uintptr_t)ws) & 255) || (((uintptr_t)Wv) & 15)) return SLORA_EINVAL;
    const HeadWs w = head_ws(1, d_model, vocab);
    if (ws_bytes < w.total) return SLORA_ENOSPC;
    hipStream_t st = (hipStream_t)stream;
    char *base = (char *)ws;
    const int Vp = vocab_padded(vocab);
    const hipError_t e = hipMemcpyAsync(base + w.WvP, Wv, 2 * (size_t)vocab * d_model, hipMemcpyDeviceToDevice, st);
    if (e != hipSuccess) { set_hip_error(e, "loss_head_prepare copy"); return SLORA_EHIP; }
    int rc;
    if ((rc = launch_fill_zero(base + w.WvP + 2 * (size_t)vocab * d_model, 2 * (size_t)(Vp - vocab) * d_model, st)))
        return rc;
    return launch_transpose_bf16((const bf16 *)(base + w.WvP), Vp, d_model, (bf16 *)(base + w.WvT), st);
}

int slora_loss_head(int32_t T, int32_t d_model, int32_t vocab, const void *y, const void *lnf_g, const void *lnf_b,
                    float eps, const int32_t *labels, void *ws, size_t ws_bytes, float *loss_tok, float *loss,
                    void *dy, void *stream)
{
    if (!head_args_ok(T, d_model, vocab) || !y || !lnf_g || !lnf_b || !labels || !ws || !loss_tok || !loss || !dy)
        return SLORA_EINVAL;
    if ((((uintptr_t)ws) & 255) || ((((uintptr_t)y) | ((uintptr_t)dy)) & 15)) return SLORA_EINVAL;
    const HeadWs w = head_ws(T, d_model, vocab);
    if (ws_bytes < w.total) return SLORA_ENOSPC;
    hipStream_t st = (hipStream_t)stream;
    char *base = (char *)ws;
    const int d = d_model, Vp = vocab_padded(vocab);
    bf16 *u = (bf16 *)(base + w.u), *logits = (bf16 *)(base + w.logits);
    float *part = (float *)(base + w.part);
    int *perm = (int *)(base + w.perm);
    LabelCount *cnt = (LabelCount *)(base + w.cnt);
    CountedRows *chunks = (CountedRows *)(base + w.chunks);
    const bf16 *gamma = (const bf16 *)lnf_g, *beta = (const bf16 *)lnf_b;
    int rc;

    const int most = T < LH_CHUNK ? T : LH_CHUNK;
    hipLaunchKernelGGL(list_labels_kernel, dim3(1), dim3(1024), 0, st, labels, T, vocab, d, Vp / 64,
                       gemm_counted_rows(most), part_rows(most, d, vocab), perm, cnt, chunks);
    SL_CHECK_LAUNCH("list_labels");
    for (int c = 0, r0 = 0; r0 < T; ++c, r0 += LH_CHUNK) {
        const int rows = (T - r0 < LH_CHUNK) ? T - r0 : LH_CHUNK;
        const CountedRows *cr = chunks + c;
        const int *list = perm + r0;
        bool rec = prof_begin(PK_LN_FWD, st, &cr->rows);
        hipLaunchKernelGGL(head_ln_fwd_kernel, dim3((rows + 3) / 4), dim3(256), 0, st, (const bf16 *)y, list, cr, gamma,
                           beta, eps, u, d);
        prof_end(rec, PK_LN_FWD, 0.0, st, 4.0 * d);
        SL_CHECK_LAUNCH("head_ln_fwd");
        GemmArgs a = plain_gemm(u, d, (const bf16 *)(base + w.WvP), d, rows, Vp, d, logits, Vp);
        a.rows = cr;
        if ((rc = launch_gemm(a, EPI_STORE, 0, st))) return rc;
        if (Vp <= CE_SHORT_MAXCH * CE_SHORT_THR * 8)
            hipLaunchKernelGGL((softmax_ce_kernel<CE_SHORT_THR, CE_SHORT_MAXCH>), dim3(rows), dim3(CE_SHORT_THR), 0, st, logits,
                               Vp, vocab, labels, list, cr, cnt, loss_tok);
        else
            hipLaunchKernelGGL((softmax_ce_kernel<CE_THR, CE_MAXCH>), dim3(rows), dim3(CE_THR), 0, st, logits, Vp, vocab,
                               labels, list, cr, cnt, loss_tok);
        SL_CHECK_LAUNCH("softmax_ce");
        GemmArgs b = plain_gemm(logits, Vp, (const bf16 *)(base + w.WvT), Vp, most, d, Vp, part, d);
        b.rows = cr;
        if ((rc = launch_gemm(b, EPI_PARTIAL, 0, st))) return rc;
        rec = prof_begin(PK_LN_BWD, st, &cr->rows);
        hipLaunchKernelGGL(head_ln_bwd_kernel, dim3((rows + 3) / 4), dim3(256), 0, st, (const bf16 *)y, list, rows, cr,
                           part, gamma, eps, (bf16 *)dy, d);
        prof_end(rec, PK_LN_BWD, 4.0 * rows * (double)d, st, 4.0 * d);
        SL_CHECK_LAUNCH("head_ln_bwd");
    }
    hipLaunchKernelGGL(loss_mean_kernel, dim3(1), dim3(1024), 0, st, loss_tok, T, cnt, loss);
    SL_CHECK_LAUNCH("loss_mean");
    return SLORA_OK;
}

}  // extern "C"
