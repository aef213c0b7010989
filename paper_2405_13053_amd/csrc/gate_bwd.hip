// Gradients of the gate of a MeteoRA module (Sec. 3.2, Eq. 4; App. "Top-k strategy"): W, A_i, B_i are
// frozen, only W_gate and its bias are trained.
//
// With dy = dL_lm/do, v_j = scale * (x A_{a_j}) B_{a_j} the contribution of the j-th selected adapter and w the
// Eq. 3 weights, the language-model loss reaches the selected logits as
//     dL/dw_j = <dy, v_j> = scale * sum_q (x A_{a_j})_q * (B_{a_j} dy)_q,      dL/dg_{a_j} = w_j (dL/dw_j - sum_i w_i dL/dw_i)
// and the LoRA-classification loss (cross entropy of the softmax over all N logits against the token's
// label, weight beta) adds beta * (softmax(g) - onehot(label)) to every logit's gradient.  Then
//     dW_gate = x^T d_logits,   dbias = sum_t d_logits[t].
//
// Launches: the two r-vectors come from dense MFMA products, as in the mid-batch forward path:
// x * Wcat^T gives the logits and x A_i of EVERY adapter (the forward's own first launch, so the logits and with
// them the top-k are bit-identical to that path's), dy * Bflat^T with Bflat = B viewed as [N*r, d_out] gives
// B_i dy of every adapter; both as fp32 K-split partials.  gate_bwd_dlogits_kernel (this file) turns them
// into d_logits per token, gate_bwd_wgrad_kernel accumulates x^T d_logits over token slices
// (a [d_in, T] x [T, 32] product whose x operand is not K-contiguous), and gate_bwd_reduce_kernel adds the
// slices in order.
//
// Input gradient (optional): dx = dy W + scale * sum_j w_j (B_{a_j} dy) A_{a_j}^T + d_logits W_gate^T is the
// forward's fused GEMM with the roles swapped: dy times W^T's storage (the caller's transposed copy
// W_t[d_in, d_out]) with the K loop continued over an extension operand hx[T, E] against Xt[d_in, E]:
//   columns a*r + q:        hx = scale * w * (B_a dy)_q for the selected adapters, else 0;   Xt[c] = A[a][c][q]
//   next 3 blocks of 32:    hx = hi(d_logits) | hi(d_logits) | lo(d_logits);  Xt[c] = hi(W_gate[c]) | lo(W_gate[c]) | hi(W_gate[c])
// (two-term bf16 splits, the lo * lo product dropped: the gate term to about 2^-16 of its size).
// gate_bwd_dlogits_kernel writes hx and Xt (W_gate changes with every optimizer step).
#include <initializer_list>
#include "common.hpp"
#include "kernels.hpp"
#include "topk_key.hpp"
#include "dense_logits.hpp"

namespace meteora {

// Tokens per workgroup of the d_logits kernel: it waits on two rounds of loads, so many small workgroups (4096 tokens:
// 512).  With Xt written by the same launch it takes 11.5 us; 16 tokens per workgroup, the splits four at a time and Xt in
// a launch of its own took 11.9 + 6.0.
constexpr int kBwdTokens = 8;
constexpr int kBwdTokensPerWave = 2;
constexpr int kBwdThreads = kBwdTokens / kBwdTokensPerWave * 64;
constexpr int kBwdNP = 32;              // logit columns (N <= 32, as the dense products require)

struct DlogitsArgs {
    const float* part_x;     // [S1][T][CR]  x * Wcat^T
    const float* part_dy;    // [S2][T][NR]  dy * Bflat^T
    const float* bias;       // [N] or NULL
    const int32_t* idx_in;   // [T,k] routing of the forward call, or NULL: rank again here
    const float* w_in;       // [T,k]
    const int32_t* labels;   // [T] or NULL
    bf16_t* dgs;             // d_logits in three bf16 terms, see split3: [blocks of 8 tokens][term][32][8 tokens]
    float* d_logits;         // [T,N] or NULL
    bf16_t* hx;              // [T][ext] extension operand of the input-gradient GEMM, or NULL
    int ext;                 // columns of hx: N*r + 96 rounded up to 64
    int S1, S2, CR, NR, T, N, r, k;
    float scale, beta;
    // an even number of token blocks (past T they write zeros); workgroups from token_blocks on write Xt instead (a launch of
    // its own would cost more than its work)
    int token_blocks;
    const uint16_t* A;       // [N, d_in, r]
    const float* W_gate;     // [d_in, N]
    int d_in;
    uint16_t* Xt;            // [d_in][ext]
};

// The three bf16 terms of an fp32 value: its 24 significand bits, 8 to a term (cut, not rounded: the largest values stay
// finite).  hi + mid + lo == v from about 2^-102 up; of smaller values the bits below bf16's smallest normal one may be lost.
// What is not finite is its first term alone.
struct Split3 { uint16_t term[3]; };
__device__ __forceinline__ Split3 split3(float v) {
    const uint32_t hi = __float_as_uint(v) & 0xffff0000u;
    const bool finite = (hi & 0x7f800000u) != 0x7f800000u;
    const float r1 = finite ? v - __uint_as_float(hi) : 0.f;
    const uint32_t mid = __float_as_uint(r1) & 0xffff0000u;
    const float r2 = r1 - __uint_as_float(mid);
    // a NaN keeps its quiet bit (its payload may lie in the bits cut off)
    return {{(uint16_t)((hi >> 16) | (v != v ? 0x40u : 0u)), (uint16_t)(mid >> 16), (uint16_t)(__float_as_uint(r2) >> 16)}};
}

__device__ void pack_xt(const uint16_t* __restrict__ A, const float* __restrict__ W_gate, int d_in, int N, int r, int ext,
                        size_t e, uint16_t* __restrict__ Xt);

__global__ __launch_bounds__(kBwdThreads) void gate_bwd_dlogits_kernel(const DlogitsArgs a) {
    if ((int)blockIdx.x >= a.token_blocks) {   // uniform
        pack_xt(a.A, a.W_gate, a.d_in, a.N, a.r, a.ext,
                (size_t)(blockIdx.x - a.token_blocks) * kBwdThreads + threadIdx.x, a.Xt);
        return;
    }
    constexpr int NP = kBwdNP;
    constexpr int TPP = 64 / NP;
    constexpr int G = kBwdTokensPerWave / TPP;
    constexpr int kChunks = kMaxRank / 8;
    __shared__ int s_idx[kBwdTokens][kMaxTopK];
    __shared__ float s_w[kBwdTokens][kMaxTopK];
    __shared__ float s_dot[kBwdTokens][kMaxTopK][kChunks];
    __shared__ float s_dg[kBwdTokens][NP];
    extern __shared__ __attribute__((aligned(16))) float s_u[];   // [kBwdTokens][k][r]: B_a dy, only when hx is written
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & (NP - 1), sub = lane / NP;
    const int t0 = blockIdx.x * kBwdTokens;
    const int T = a.T, N = a.N, r = a.r, k = a.k;

    float g[G];
    int lt[G];
#pragma unroll
    for (int i = 0; i < G; ++i) lt[i] = wave * kBwdTokensPerWave + i * TPP + sub;
    dense_logits<NP, G>(a.part_x, a.S1, a.CR, a.bias, T, N, t0, lt, col, g);

    int sel_i[G];
    float sel_w[G];
    if (a.idx_in != nullptr) {
#pragma unroll
        for (int i = 0; i < G; ++i) {
            const int t = min(t0 + lt[i], T - 1);
            sel_i[i] = col < k ? min(max(a.idx_in[(size_t)t * k + col], 0), N - 1) : 0;   // stay inside the partials
            sel_w[i] = col < k ? a.w_in[(size_t)t * k + col] : 0.f;
        }
    } else {
        wave_topk_softmax<NP, G>(g, lane, N, k, 1.0f, sel_i, sel_w);
    }
#pragma unroll
    for (int i = 0; i < G; ++i) {
        if (col < k) { s_idx[lt[i]][col] = sel_i[i]; s_w[lt[i]][col] = sel_w[i]; }
        // classification part: beta * (softmax over the N logits - onehot(label)); labels outside [0, N) carry none
        float ce = 0.f;
        const int t = min(t0 + lt[i], T - 1);
        const int label = a.labels != nullptr ? a.labels[t] : -1;
        float gmax = col < N ? g[i] : -INFINITY;
#pragma unroll
        for (int off = NP / 2; off >= 1; off >>= 1) gmax = fmaxf(gmax, __shfl_xor(gmax, off));
        const float e = col < N ? expf(g[i] - gmax) : 0.f;
        float sum = e;
#pragma unroll
        for (int off = NP / 2; off >= 1; off >>= 1) sum += __shfl_xor(sum, off);
        if (label >= 0 && label < N && col < N) ce = a.beta * (e / sum - (col == label ? 1.f : 0.f));
        s_dg[lt[i]][col] = ce;
    }
    __syncthreads();

    // ---- dL/dw of every (token, slot): a thread takes 8 of the r products, splits added in order ----
    const int R8 = r / 8;
    for (int e = threadIdx.x; e < kBwdTokens * k * R8; e += kBwdThreads) {
        const int tl = e / (k * R8), rem = e - tl * (k * R8);
        const int s = rem / R8, c = rem - s * R8;
        const int t = min(t0 + tl, T - 1);
        const int ad = s_idx[tl][s];
        const float* ph = a.part_x + (size_t)t * a.CR + 3 * NP + ad * r + c * 8;
        const float* pu = a.part_dy + (size_t)t * a.NR + ad * r + c * 8;
        f32x4 h0 = {0.f, 0.f, 0.f, 0.f}, h1 = h0, u0 = h0, u1 = h0;
        f32x4 x0[8], x1[8], y0[8], y1[8];   // both products' splits in one round of loads: there are at most 8 of each
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float* p = ph + (size_t)min(u, a.S1 - 1) * T * a.CR;
            x0[u] = *reinterpret_cast<const f32x4*>(p);
            x1[u] = *reinterpret_cast<const f32x4*>(p + 4);
            p = pu + (size_t)min(u, a.S2 - 1) * T * a.NR;
            y0[u] = *reinterpret_cast<const f32x4*>(p);
            y1[u] = *reinterpret_cast<const f32x4*>(p + 4);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (u < a.S1) { h0 += x0[u]; h1 += x1[u]; }
            if (u < a.S2) { u0 += y0[u]; u1 += y1[u]; }
        }
        float d = 0.f;
#pragma unroll
        for (int q = 0; q < 4; ++q) d += h0[q] * u0[q];
#pragma unroll
        for (int q = 0; q < 4; ++q) d += h1[q] * u1[q];
        s_dot[tl][s][c] = d;
        if (a.hx != nullptr) {
            float* su = s_u + ((size_t)tl * k + s) * r + c * 8;
            *reinterpret_cast<f32x4*>(su) = u0;
            *reinterpret_cast<f32x4*>(su + 4) = u1;
        }
    }
    __syncthreads();

    // ---- softmax backward over the k selected, scattered onto the token's logit row ----
#pragma unroll
    for (int i = 0; i < G; ++i) {
        float dw = 0.f;
        if (col < k) {
            for (int c = 0; c < R8; ++c) dw += s_dot[lt[i]][col][c];
            dw *= a.scale;
        }
        float mean = col < k ? sel_w[i] * dw : 0.f;
#pragma unroll
        for (int off = 1; off < kMaxTopK; off <<= 1) mean += __shfl_xor(mean, off);
        // the k selected adapters of a token are distinct: no two lanes add to the same entry
        if (col < k) s_dg[lt[i]][sel_i[i]] += sel_w[i] * (dw - mean);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < G; ++i) {
        const int t = t0 + lt[i];
        if (t >= T) continue;
        if (a.d_logits != nullptr && col < N) a.d_logits[(size_t)t * N + col] = s_dg[lt[i]][col];
    }
    static_assert(kBwdTokens == 8 && kBwdThreads >= 6 * kBwdNP, "one 8-byte piece per thread: 4 tokens of a term's column");
    if (threadIdx.x < 6 * NP) {
        const int half = threadIdx.x & 1, term = threadIdx.x / (2 * NP), n = threadIdx.x / 2 % NP;
        uint16_t v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const Split3 sp = split3(t0 + half * 4 + j < T && n < N ? s_dg[half * 4 + j][n] : 0.f);
            v[j] = term == 0 ? sp.term[0] : term == 1 ? sp.term[1] : sp.term[2];
        }
        *reinterpret_cast<uint2*>(a.dgs + ((size_t)blockIdx.x * 6 * NP + threadIdx.x) * 4) =
            uint2{(uint32_t)v[0] | (uint32_t)v[1] << 16, (uint32_t)v[2] | (uint32_t)v[3] << 16};
    }
    if (a.hx == nullptr) return;

    // ---- rows of hx: a thread owns 8 columns of one token ----
    const int C8 = a.ext / 8, NR = N * r;
    for (int e = threadIdx.x; e < kBwdTokens * C8; e += kBwdThreads) {
        const int tl = e / C8, c0 = (e - tl * C8) * 8;
        const int t = t0 + tl;
        if (t >= T) continue;
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = 0.f;
        if (c0 < NR) {                                       // the adapter part: scale * w * (B_a dy)
            const int ad = c0 / r;
            for (int sl = 0; sl < k; ++sl)
                if (s_idx[tl][sl] == ad) {
                    const float sw = a.scale * s_w[tl][sl];
                    const float* su = s_u + ((size_t)tl * k + sl) * r + (c0 - ad * r);
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[i] = sw * su[i];
                }
        } else if (c0 < NR + 3 * NP) {                       // the gate part: hi | hi | lo of d_logits
            const int term = (c0 - NR) / NP, n0 = (c0 - NR) - term * NP;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float d = s_dg[tl][n0 + i];            // columns >= N are not written above and hold 0 or the
                const float dz = n0 + i < N ? d : 0.f;       // classification part of a padding lane: masked here
                const float hi = static_cast<float>(static_cast<bf16_t>(dz));
                v[i] = term == 2 ? dz - hi : hi;
            }
        }
        u32x4 pk;
        pk[0] = pack_bf16x2(v[0], v[1]); pk[1] = pack_bf16x2(v[2], v[3]);
        pk[2] = pack_bf16x2(v[4], v[5]); pk[3] = pack_bf16x2(v[6], v[7]);
        *reinterpret_cast<u32x4*>(a.hx + (size_t)t * a.ext + c0) = pk;
    }
}

// Xt[c][ext] for the input-gradient GEMM: A[a][c][:] at columns a*r.., then hi | lo | hi of W_gate[c][:] in blocks
// of 32 columns, zero elsewhere.  Piece e: 8 columns of one row c.
__device__ void pack_xt(const uint16_t* __restrict__ A, const float* __restrict__ W_gate, int d_in, int N, int r, int ext,
                        size_t e, uint16_t* __restrict__ Xt) {
    const int C8 = ext / 8, NR = N * r;
    if (e >= (size_t)d_in * C8) return;
    const int c = (int)(e / C8), c0 = (int)(e - (size_t)c * C8) * 8;
    u32x4 pk = {0u, 0u, 0u, 0u};
    if (c0 < NR) {
        const int ad = c0 / r, q0 = c0 - ad * r;
        pk = *reinterpret_cast<const u32x4*>(A + ((size_t)ad * d_in + c) * r + q0);
    } else if (c0 < NR + 3 * kBwdNP) {
        const int term = (c0 - NR) / kBwdNP, n0 = (c0 - NR) - term * kBwdNP;
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float w = n0 + i < N ? W_gate[(size_t)c * N + n0 + i] : 0.f;
            const float hi = static_cast<float>(static_cast<bf16_t>(w));
            v[i] = term == 1 ? w - hi : hi;
        }
        pk[0] = pack_bf16x2(v[0], v[1]); pk[1] = pack_bf16x2(v[2], v[3]);
        pk[2] = pack_bf16x2(v[4], v[5]); pk[3] = pack_bf16x2(v[6], v[7]);
    }
    *reinterpret_cast<u32x4*>(Xt + (size_t)c * ext + c0) = pk;
}

// ---- dW_gate partials: wpart[slice][c][32] = sum over the slice's tokens of x[t][c] * dg[t][:] ----
// The contraction runs over tokens: an operand of v_mfma_f32_32x32x16_bf16 is 8 consecutive tokens of a column per lane.
// x[T, d_in] is not token-contiguous, so a lane loads 4 columns of 8 tokens (8 bytes each, whole lines per half wavefront)
// and pairs the halves of its registers (two v_perm per 4 values).  d_logits comes as three bf16 terms that add up to its
// fp32 value, in the operand's own order: every product is exact in fp32, as in the forward gate, and a multiply of K = 16
// takes 32 cycles where the fp32 MFMA takes 512.  Bound by the latency of the loads: a wavefront owns 128 columns and one of
// PARTS shares of the workgroup's tokens, all of whose loads are in flight for up to 64 tokens.  The sums meet in LDS.
// Workgroups of column tile 0 also add up dg for dbias.
constexpr int kWgCols = 128, kWgChunk = 16;                      // chunk: tokens per MFMA
constexpr int kWgRing = 4;                                       // chunks whose loads are in flight per wavefront
constexpr int wgrad_lds(int parts) { return parts * 16 * 64 * 16; }   // the accumulators of every wavefront

template <int PARTS>
__global__ __launch_bounds__(PARTS * 64) void gate_bwd_wgrad_kernel(const uint16_t* __restrict__ x,
                                                                     const uint16_t* __restrict__ dgs, int T, int d_in,
                                                                     int slice_chunks, float* __restrict__ wpart,
                                                                     float* __restrict__ bpart) {
    extern __shared__ __attribute__((aligned(16))) f32x4 red[];  // [part][fragment * 4 + entry group][lane]
    __shared__ float s_b[PARTS][kBwdNP];
    const int lane = threadIdx.x & 63, l31 = lane & 31, kh = lane >> 5;
    const int part = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c0 = blockIdx.x * kWgCols, slice = blockIdx.y;
    const int c = min(c0 + 4 * l31, d_in - 4);                   // d_in % 8 == 0: 4 columns inside or the last ones again
    const int chunks = ceil_div(T, kWgChunk);
    const int s_begin = slice * slice_chunks, s_n = min(slice_chunks, chunks - s_begin);
    const int k0 = s_begin + part * s_n / PARTS, k1 = s_begin + (part + 1) * s_n / PARTS;

    struct Chunk { uint2 x[8]; u32x4 d[3]; };
    auto load = [&](Chunk& f, int ch) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {   // tokens past the last one: the last one again, their dg is zero
            const int t = min(ch * kWgChunk + kh * 8 + j, T - 1);
            f.x[j] = *reinterpret_cast<const uint2*>(x + (size_t)t * d_in + c);
        }
        const uint16_t* d = dgs + ((size_t)(ch * 2 + kh) * 3 * kBwdNP + l31) * 8;
#pragma unroll
        for (int term = 0; term < 3; ++term) f.d[term] = *reinterpret_cast<const u32x4*>(d + term * kBwdNP * 8);
    };
    f32x16 acc[4];
#pragma unroll
    for (int f = 0; f < 4; ++f)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[f][i] = 0.f;
    float bsum = 0.f;
    const bool bias_tile = blockIdx.x == 0;                      // uniform
    auto operand = [&](const Chunk& f, int q) {                  // column c + q
        u32x4 v;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t even = q < 2 ? f.x[2 * j].x : f.x[2 * j].y, odd = q < 2 ? f.x[2 * j + 1].x : f.x[2 * j + 1].y;
            v[j] = __builtin_amdgcn_perm(odd, even, q % 2 == 0 ? 0x05040100u : 0x07060302u);
        }
        return __builtin_bit_cast(bf16x8, v);
    };
    auto multiply = [&](f32x16& sum, const Chunk& f, int term, bf16x8 xq) {
        sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, f.d[term]), xq, sum, 0, 0, 0);
    };
    auto add_bias = [&](const Chunk& f) {
        float b[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            b[j] = ((bf16_bits_to_float(f.d[2][j] & 0xffffu) + bf16_bits_to_float(f.d[1][j] & 0xffffu)) +
                    bf16_bits_to_float(f.d[0][j] & 0xffffu)) +
                   ((bf16_bits_to_float(f.d[2][j] >> 16) + bf16_bits_to_float(f.d[1][j] >> 16)) +
                    bf16_bits_to_float(f.d[0][j] >> 16));
        bsum += (b[0] + b[1]) + (b[2] + b[3]);
    };
    Chunk f[kWgRing];
#pragma unroll
    for (int u = 0; u < kWgRing; ++u)
        if (k0 + u < k1) load(f[u], k0 + u);
    // One rounding of a full-sized sum for each chunk, not three: the small terms come first, or have sums of their own
    if constexpr (PARTS == 2) {                                  // no more chunks than the ring holds
#pragma unroll
        for (int u = 0; u < kWgRing; ++u) {
            if (k0 + u >= k1) break;                             // uniform per wavefront
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const bf16x8 xq = operand(f[u], q);
                multiply(acc[q], f[u], 2, xq);
                multiply(acc[q], f[u], 1, xq);
            }
        }
#pragma unroll
        for (int u = 0; u < kWgRing; ++u) {
            if (k0 + u >= k1) break;
#pragma unroll
            for (int q = 0; q < 4; ++q) multiply(acc[q], f[u], 0, operand(f[u], q));
            if (bias_tile) add_bias(f[u]);
        }
    } else {
        f32x16 low[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < 16; ++i) low[q][i] = 0.f;
        for (int ch = k0; ch < k1; ch += kWgRing) {
#pragma unroll
            for (int u = 0; u < kWgRing; ++u) {
                if (ch + u >= k1) break;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const bf16x8 xq = operand(f[u], q);
                    multiply(low[q], f[u], 2, xq);
                    multiply(acc[q], f[u], 0, xq);
                    multiply(low[q], f[u], 1, xq);
                }
                if (bias_tile) add_bias(f[u]);
                if (ch + u + kWgRing < k1) load(f[u], ch + u + kWgRing);
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] += low[q];
    }
    // accumulator entry i of lane l: adapter 8*(i/4) + 4*(l/32) + i%4, column c0 + 4 * (l%32) + fragment
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            red[(part * 16 + q * 4 + g) * 64 + lane] = f32x4{acc[q][4 * g], acc[q][4 * g + 1], acc[q][4 * g + 2], acc[q][4 * g + 3]};
    bsum += __shfl_xor(bsum, 32);
    if (kh == 0) s_b[part][l31] = bsum;
    __syncthreads();
    // 16-byte pieces in the order of wpart, the parts added in order
    for (int p = threadIdx.x; p < kWgCols * kBwdNP / 4; p += PARTS * 64) {
        const int col = p / (kBwdNP / 4), piece = p % (kBwdNP / 4);
        const int at = ((col & 3) * 4 + piece / 2) * 64 + (piece & 1) * 32 + col / 4;
        f32x4 v = red[at];
#pragma unroll
        for (int w = 1; w < PARTS; ++w) v += red[w * 16 * 64 + at];
        if (c0 + col < d_in) *reinterpret_cast<f32x4*>(wpart + ((size_t)slice * d_in + c0 + col) * kBwdNP + piece * 4) = v;
    }
    if (bias_tile && threadIdx.x < kBwdNP) {
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < PARTS; ++w) v += s_b[w][threadIdx.x];
        bpart[slice * kBwdNP + threadIdx.x] = v;
    }
}

// dW_gate[c][n] = sum of the slices in order (thread per (c, padded n)); the last workgroup does dbias.
__global__ __launch_bounds__(256) void gate_bwd_reduce_kernel(const float* __restrict__ wpart,
                                                               const float* __restrict__ bpart, int slices, int d_in,
                                                               int N, float* __restrict__ dW_gate,
                                                               float* __restrict__ dbias) {
    const size_t total = (size_t)d_in * kBwdNP;
    if (blockIdx.x == gridDim.x - 1) {
        if (dbias != nullptr && threadIdx.x < N) {
            float s = 0.f;
            for (int sl = 0; sl < slices; ++sl) s += bpart[sl * kBwdNP + threadIdx.x];
            dbias[threadIdx.x] = s;
        }
        return;
    }
    const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= total) return;
    const int n = (int)(e % kBwdNP);
    const size_t cidx = e / kBwdNP;
    float s = 0.f;
    for (int s0 = 0; s0 < slices; s0 += 8) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = wpart[(size_t)min(s0 + u, slices - 1) * total + e];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (s0 + u < slices) s += v[u];
    }
    if (n < N) dW_gate[cidx * N + n] = s;
}

// ---- host side ----
bool gate_backward_applies(int T, int d_in, int d_out, int N, int r, bool bf16) {
    return bf16 && N <= kBwdNP && r % 8 == 0 && prep_wcat_rows(N, r) <= kWcatMaxRows && d_in % 64 == 0 && d_out % 64 == 0 &&
           T >= 1 && T <= kGateBackwardMaxTokens && r <= kMaxRank &&
           gemm_dense_splitk_ok(T, d_in, prep_wcat_rows(N, r)) && gemm_dense_splitk_ok(T, d_out, N * r);
}

// One workgroup per CU at most, since a few more take a second round, and 8 slices or, of more than 256 chunks, one for every
// 32: a slice costs the reduction about 0.1 us.  Four wavefronts to a workgroup, two where a slice has 8 chunks or fewer: the
// way of more sums through LDS costs more than the longer chains.  Whole gate_backward calls with 64 outputs, us: 5120 inputs
// on 280 and 240 workgroups, 1000 tokens 38.0 and 31.3, 4096 57.2 and 48.3; 256 inputs in 8, 16 and 64 slices, 4096 tokens
// 26.8, 26.0, 33.5, 8192 43.1, 40.5, 47.4; 4096 inputs with 8, 4 and 2 wavefronts, 64 tokens 24.3, 22.6, 22.0, 300 25.9, 24.3,
// 23.8, 1000 31.1, 29.8, 29.3, 4096 44.0, 42.5, 43.1.
// most_slices never falls with more tokens, as the slices in use do: it is what a workspace has room for.
struct WgradPlan { int parts, slice_chunks, most_slices; };
static WgradPlan wgrad_plan(int T, int d_in) {
    const int chunks = ceil_div(T, kWgChunk), col_tiles = ceil_div(d_in, kWgCols);
    int n = chunks / 32 < 8 ? 8 : chunks / 32 < 32 ? chunks / 32 : 32;
    for (const int most : {256 / col_tiles, ceil_div(chunks, 4)})
        if (n > most) n = most;
    if (n < 1) n = 1;
    const int slice_chunks = ceil_div(chunks, n);
    return {slice_chunks > 2 * kWgRing ? 4 : 2, slice_chunks, n};
}

// One after the other in the same place: the products until the kernel of d_logits has read them, and the input gradient's K splits.
// (The weight gradient's slices have one of their own: behind the products the launch that adds them took 3.6 us, so 2.5, 600 x 2048.)
// reserve: room for any batch of up to T tokens, else what a call of T tokens writes (dx: with the input gradient).
GateBackwardLayout gate_backward_layout(int T, int d_in, int d_out, int N, int r, bool dx, bool reserve) {
    GateBackwardLayout L{};
    const int CR = prep_wcat_rows(N, r), NR = N * r;
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t o = off; off = align_up(off + bytes, 256); return o; };
    auto pairs = [&](int K, int rows) {
        return reserve ? (size_t)gemm_dense_pairs_reserved(T, K, rows) : (size_t)gemm_dense_splits(T, K, rows) * T;
    };
    size_t dx_bytes = 0;
    if (reserve) dx_bytes = gemm_few_tile_bytes(T, d_out, d_in);
    else if (const int S = dx ? gemm_few_tile_splits(T, d_out, d_in) : 0) dx_bytes = (size_t)S * T * d_in * sizeof(float);
    else if (dx) dx_bytes = gemm_splitk_bytes(T, d_out, d_in, true);
    L.dxpart = L.part_x = take(pairs(d_in, CR) * CR * sizeof(float));
    L.part_dy = take(pairs(d_out, NR) * NR * sizeof(float));
    if (off < dx_bytes) off = align_up(dx_bytes, 256);
    // whole pairs of 8-token blocks, 3072 bytes each: less than 192 T + 3072
    L.dgs = take((size_t)T * 192 + 3072);
    const int slices = wgrad_plan(T, d_in).most_slices;
    L.wpart = take((size_t)slices * d_in * kBwdNP * sizeof(float));
    L.bpart = take((size_t)slices * kBwdNP * sizeof(float));
    L.ext = (int)align_up((size_t)NR + 3 * kBwdNP, 64);
    L.hx = take(dx || reserve ? (size_t)T * L.ext * sizeof(uint16_t) : 0);
    L.xt = take(dx || reserve ? (size_t)d_in * L.ext * sizeof(uint16_t) : 0);
    L.total = off;
    return L;
}

hipError_t gate_bwd_init_kernels() {
    return ensure_lds_limit(reinterpret_cast<const void*>(&gate_bwd_wgrad_kernel<4>), wgrad_lds(4));
}

hipError_t launch_gate_backward(const void* x, const void* dy, const void* wcat, const void* B, const float* bias,
                                const int32_t* idx_in, const float* w_in, const int32_t* labels, float beta, int T,
                                int d_in, int d_out, int N, int r, int k, float scale, float* dW_gate, float* dbias,
                                float* d_logits, const float* part_x_given, int part_x_splits, const void* A,
                                const float* W_gate, const void* W_t, void* dx, char* ws, hipStream_t stream) {
    if ((dx != nullptr) && (!A || !W_gate || !W_t)) return hipErrorInvalidValue;
    if (!gate_backward_applies(T, d_in, d_out, N, r, true) || k < 1 || k > kMaxTopK || k > N)
        return hipErrorInvalidValue;
    const GateBackwardLayout L = gate_backward_layout(T, d_in, d_out, N, r, dx != nullptr, false);
    const int CR = prep_wcat_rows(N, r), NR = N * r;
    const float* part_x = part_x_given != nullptr ? part_x_given : reinterpret_cast<float*>(ws + L.part_x);
    float* part_dy = reinterpret_cast<float*>(ws + L.part_dy);
    bf16_t* dgs = reinterpret_cast<bf16_t*>(ws + L.dgs);
    float* wpart = reinterpret_cast<float*>(ws + L.wpart);
    float* bpart = reinterpret_cast<float*>(ws + L.bpart);
    hipError_t e = hipSuccess;
    if (part_x_given == nullptr) e = launch_gemm_dense_splitk(x, wcat, T, d_in, CR, reinterpret_cast<float*>(ws + L.part_x), stream);
    if (e != hipSuccess) return e;
    e = launch_gemm_dense_splitk(dy, B, T, d_out, NR, part_dy, stream);
    if (e != hipSuccess) return e;
    DlogitsArgs a{};
    a.part_x = part_x; a.part_dy = part_dy; a.bias = bias; a.idx_in = idx_in; a.w_in = w_in; a.labels = labels;
    a.dgs = dgs; a.d_logits = d_logits;
    a.hx = dx != nullptr ? reinterpret_cast<bf16_t*>(ws + L.hx) : nullptr;
    a.ext = L.ext;
    a.S1 = (part_x_given != nullptr && part_x_splits > 0) ? part_x_splits : gemm_dense_splits(T, d_in, CR);
    a.S2 = gemm_dense_splits(T, d_out, NR);
    a.CR = CR; a.NR = NR; a.T = T; a.N = N; a.r = r; a.k = k; a.scale = scale; a.beta = beta;
    const size_t u_bytes = dx != nullptr ? (size_t)kBwdTokens * k * r * sizeof(float) : 0;   // at most 16 KB
    if (a.S1 > 8 || a.S2 > 8) return hipErrorInvalidValue;
    a.token_blocks = (int)align_up(ceil_div(T, kBwdTokens), 2);
    uint16_t* xt = reinterpret_cast<uint16_t*>(ws + L.xt);
    int64_t blocks_all = a.token_blocks;
    if (dx != nullptr) {
        a.A = (const uint16_t*)A; a.W_gate = W_gate; a.d_in = d_in; a.Xt = xt;
        blocks_all += ceil_div64((int64_t)d_in * (L.ext / 8), kBwdThreads);
    }
    gate_bwd_dlogits_kernel<<<(unsigned)blocks_all, kBwdThreads, u_bytes, stream>>>(a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (dx != nullptr) {
        // dx = dy * W_t^T continued over hx * Xt^T: the forward's GEMM with d_in and d_out swapped
        float* dxpart = reinterpret_cast<float*>(ws + L.dxpart);
        e = gemm_few_tile_splits(T, d_out, d_in) > 0
                ? launch_gemm_few_tiles(dy, W_t, T, d_out, d_in, ws + L.hx, L.ext, xt, L.ext, dx, dxpart, stream)
                : launch_gemm(dy, W_t, T, d_out, d_in, true, ws + L.hx, L.ext, xt, L.ext, dx, 0, T <= 64 ? dxpart : nullptr, stream);
        if (e != hipSuccess) return e;
    }
    const WgradPlan plan = wgrad_plan(T, d_in);
    const int slices = ceil_div(ceil_div(T, kWgChunk), plan.slice_chunks);
    auto wgrad = [&](auto kern) {
        kern<<<dim3(ceil_div(d_in, kWgCols), slices), plan.parts * 64, wgrad_lds(plan.parts), stream>>>(
            (const uint16_t*)x, (const uint16_t*)dgs, T, d_in, plan.slice_chunks, wpart, bpart);
        return hipGetLastError();
    };
    if (plan.parts == 4 && (e = gate_bwd_init_kernels()) != hipSuccess) return e;
    e = plan.parts == 4 ? wgrad(gate_bwd_wgrad_kernel<4>) : wgrad(gate_bwd_wgrad_kernel<2>);
    if (e != hipSuccess) return e;
    const int blocks = (int)ceil_div64((int64_t)d_in * kBwdNP, 256) + 1;
    gate_bwd_reduce_kernel<<<blocks, 256, 0, stream>>>(wpart, bpart, slices, d_in, N, dW_gate, dbias);
    return hipGetLastError();
}

}  // namespace meteora
