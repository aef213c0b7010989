// The layer with fp32 storage: the base projection on fp32 MFMAs, and everything else of Eq. 2 per token.
#include <type_traits>
#include "common.hpp"
#include "gate_row.hpp"
#include "kernels.hpp"
#include "topk_key.hpp"

namespace meteora {

// ------------------------------------------------------------------------------------------
// out[T, d_out] = x[T, d_in] * W[d_out, d_in]^T in fp32.
//
// v_mfma_f32_16x16x4_f32 takes one K value per lane, 16 rows x 4 K values per operand.  A lane loads 16 bytes, the K
// values 4c..4c+3 of its row (c = lane / 16), and feeds them to four MFMAs: the j-th multiplies K values 4c + j of
// both operands, which is the same set.  The matrix cores take 32 cycles for what two such loads of 1 KB feed to one
// block, so operands come straight from L2 into registers, one step of 16 K values ahead (four with the split), without
// LDS.
// A wavefront owns MB x NB blocks of 16 x 16; the four of a workgroup either share one such tile, each taking a
// quarter of K (small outputs: latency counts, and tiles are few), or are 2 x 2 tiles next to each other.
// Rows of all three matrices are whole 32-byte pieces.
//
// Measured against 64 x 64 tiles of plain FMAs through LDS, call by call: 64 x 256 -> 256 29.7 -> 9.7 us, 1024 x 768 ->
// 768 84 -> 27, 4096 x 4096 -> 4096 3.57 -> 1.36 ms.
// ------------------------------------------------------------------------------------------
template <int MB, int NB, bool SPLIT>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ x, const float* __restrict__ W, int T,
                                                       int d_in, int d_out, float* __restrict__ out) {
    constexpr int TM = MB * 16, TN = NB * 16;                       // a wavefront's tile
    constexpr int AHEAD = SPLIT ? 4 : 1;                            // K steps whose loads are in flight
    __shared__ __attribute__((aligned(16))) float red[SPLIT ? 4 : 1][SPLIT ? TM : 1][SPLIT ? TN + 4 : 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l15 = lane & 15, kc = (lane >> 4) * 4;
    const int tiles_n = ceil_div(d_out, SPLIT ? TN : 2 * TN);
    const int tile_m = blockIdx.x / tiles_n, tile_n = blockIdx.x - tile_m * tiles_n;
    const int m0 = SPLIT ? tile_m * TM : tile_m * 2 * TM + (wave >> 1) * TM;
    const int n0 = SPLIT ? tile_n * TN : tile_n * 2 * TN + (wave & 1) * TN;
    const int steps = ceil_div(d_in, 16);
    const int s0 = SPLIT ? wave * steps / 4 : 0, s1 = SPLIT ? (wave + 1) * steps / 4 : steps;

    // rows past the edge repeat the last one (computed, never stored); K values past d_in count as zeros
    const float* xp[MB];
    const float* wp[NB];
#pragma unroll
    for (int i = 0; i < MB; ++i) xp[i] = x + (size_t)min(m0 + i * 16 + l15, T - 1) * d_in;
#pragma unroll
    for (int i = 0; i < NB; ++i) wp[i] = W + (size_t)min(n0 + i * 16 + l15, d_out - 1) * d_in;
    struct Step { f32x4 x[MB], w[NB]; };
    auto load4 = [&](const float* row, int k) -> f32x4 {   // values k..k+3 of a row, zeros past its end
        const f32x4 v = *reinterpret_cast<const f32x4*>(row + min(k, d_in - 4));
        return k < d_in ? v : f32x4{0.f, 0.f, 0.f, 0.f};
    };
    auto load = [&](Step& f, int s) {
        const int k = s * 16 + kc;
#pragma unroll
        for (int i = 0; i < MB; ++i) f.x[i] = load4(xp[i], k);
#pragma unroll
        for (int i = 0; i < NB; ++i) f.w[i] = load4(wp[i], k);
    };
    f32x4 acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    Step f[AHEAD + 1];
#pragma unroll
    for (int a = 0; a < AHEAD; ++a)
        if (s0 + a < s1) load(f[a], s0 + a);
    for (int s = s0; s < s1; s += AHEAD + 1) {
#pragma unroll
        for (int u = 0; u <= AHEAD; ++u) {   // register sets have fixed numbers
            if (s + u >= s1) break;          // uniform per wavefront
            if (s + u + AHEAD < s1) load(f[(u + AHEAD) % (AHEAD + 1)], s + u + AHEAD);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int mi = 0; mi < MB; ++mi)
#pragma unroll
                    for (int ni = 0; ni < NB; ++ni)
                        acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x4f32(f[u].w[ni][j], f[u].x[mi][j], acc[mi][ni], 0, 0, 0);
        }
    }
    // a lane holds columns 4 * (lane / 16) .. + 3 of token lane % 16 of every block
    auto store = [&](int row, int col, f32x4 v) {
        if (row < T && col < d_out) *reinterpret_cast<f32x4*>(out + (size_t)row * d_out + col) = v;
    };
    if constexpr (SPLIT) {
#pragma unroll
        for (int mi = 0; mi < MB; ++mi)
#pragma unroll
            for (int ni = 0; ni < NB; ++ni)
                *reinterpret_cast<f32x4*>(&red[wave][mi * 16 + l15][ni * 16 + kc]) = acc[mi][ni];
        __syncthreads();
        for (int e = threadIdx.x; e < TM * TN / 4; e += 256) {
            const int r = e / (TN / 4), c = (e % (TN / 4)) * 4;
            f32x4 v[4];
#pragma unroll
            for (int w = 0; w < 4; ++w) v[w] = *reinterpret_cast<const f32x4*>(&red[w][r][c]);
            store(m0 + r, n0 + c, (v[0] + v[1]) + (v[2] + v[3]));
        }
    } else {
#pragma unroll
        for (int mi = 0; mi < MB; ++mi)
#pragma unroll
            for (int ni = 0; ni < NB; ++ni) store(m0 + mi * 16 + l15, n0 + ni * 16 + kc, acc[mi][ni]);
    }
}

// 16 x 16 tiles up to 1024 of them (a latency-bound call: 64 x 256 -> 256 is 64 workgroups of four steps of loads), 32 x
// 32 until 128 x 128 tiles would occupy three quarters of the CUs.
hipError_t launch_gemm_f32(const float* x, const float* W, int T, int d_in, int d_out, float* out, hipStream_t stream) {
    if (d_in % 8 != 0 || d_out % 8 != 0) return hipErrorInvalidValue;
    auto go = [&](auto kern, int tm, int tn) {
        const int64_t tiles = ceil_div64(T, tm) * ceil_div64(d_out, tn);
        if (tiles > INT32_MAX) return hipErrorInvalidValue;
        kern<<<(unsigned)tiles, 256, 0, stream>>>(x, W, T, d_in, d_out, out);
        return hipGetLastError();
    };
    if (ceil_div64(T, 16) * ceil_div64(d_out, 16) <= 1024) return go(gemm_f32_kernel<1, 1, true>, 16, 16);
    if (ceil_div64(T, 128) * ceil_div64(d_out, 128) < 192) return go(gemm_f32_kernel<2, 2, true>, 32, 32);
    return go(gemm_f32_kernel<4, 4, false>, 128, 128);
}

// ------------------------------------------------------------------------------------------
// The rest of the layer, a workgroup per token: gate logits, top-k, softmax (Eq. 3), the shrink of the selected
// adapters and their expand onto the base projection that `out` already holds.  At the sizes fp32 storage is used at
// (a few hundred inputs and outputs) each of these steps is a microsecond of memory latency; as launches of their own
// (gate logits, top-k, bucket scatter, shrink, expand) they took 4 to 7 us each.  Measured, whole layer, 28 adapters of
// rank 8, top-2: 64 x 256 -> 256 (4 adapters) 52.4 -> 15.5 us, 300 x 512 -> 768 91 -> 24, 4096 x 4096 -> 4096 without the
// projection 745 -> 360.  Wide outputs get the expand as a launch of its own, see below.
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kRowThreads) void route_lora_f32_kernel(
    const float* __restrict__ x, const float* __restrict__ W_gate, const float* __restrict__ bias,
    const float* __restrict__ A, const float* __restrict__ B, int d_in, int d_out, int N, int gate_cols, int r, int k,
    int h_cols, float inv_temperature, float scale, int32_t* __restrict__ topk_idx, float* __restrict__ topk_w,
    float* __restrict__ out, float* __restrict__ h_out) {
    __shared__ float red[4][kMaxAdapters];
    __shared__ int sel_idx[kMaxTopK];
    __shared__ float sel_w[kMaxTopK];
    __shared__ float hs[kMaxTopK * kMaxRank];   // scale * w * h of the k slots
    const int t = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const float* xt = x + (size_t)t * d_in;
    gate_row(xt, W_gate, d_in, N, gate_cols, red);
    if (wave == 0) {   // lane = adapter
        float g[1] = {0.f};
        if (lane < N) {
            g[0] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
            g[0] += bias != nullptr ? bias[lane] : 0.f;
            if (g[0] == 0.f) g[0] = 0.f;   // -0 -> +0 so equal logits have equal keys
        }
        int my_i[1];
        float my_w[1];
        wave_topk_softmax<64, 1>(g, lane, N, k, inv_temperature, my_i, my_w);
        if (lane < k) {
            sel_idx[lane] = my_i[0];
            sel_w[lane] = my_w[0];
            topk_idx[(size_t)t * k + lane] = my_i[0];
            topk_w[(size_t)t * k + lane] = my_w[0];
        }
    }
    __syncthreads();
    // shrink: h_cols (a power of two, at most 64) of the k * r products at a time
    const int kr = k * r;
    for (int c0 = 0; c0 < kr; c0 += h_cols) {
        const int c = threadIdx.x & (h_cols - 1), e = c0 + c;
        float v = 0.f;
        if (e < kr) {
            const int slot = e / r, q = e - slot * r;
            v = row_dot(xt, A + (size_t)sel_idx[slot] * d_in * r + q, r, d_in, threadIdx.x / h_cols, kRowThreads / h_cols);
        }
        v = sum_columns(v, h_cols);
        if (lane < h_cols) red[wave][c] = v;
        __syncthreads();
        if (wave == 0 && lane < h_cols && c0 + lane < kr) {
            const float h = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
            hs[c0 + lane] = scale * sel_w[(c0 + lane) / r] * h;
        }
        __syncthreads();
    }
    if (h_out != nullptr) {   // expand_f32_kernel follows
        for (int i = threadIdx.x; i < kr; i += kRowThreads) h_out[(size_t)t * kr + i] = hs[i];
        return;
    }
    for (int c = threadIdx.x; c < d_out; c += kRowThreads) {
        float acc = out[(size_t)t * d_out + c];
        for (int slot = 0; slot < k; ++slot) {
            const float* Ba = B + (size_t)sel_idx[slot] * r * d_out + c;
            float d = 0.f;
            for (int q0 = 0; q0 < r; q0 += 8) {   // 8 rows of B in flight
                float b[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) b[u] = Ba[(size_t)min(q0 + u, r - 1) * d_out];
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (q0 + u < r) d = fmaf(hs[slot * r + q0 + u], b[u], d);
            }
            acc += d;
        }
        out[(size_t)t * d_out + c] = acc;
    }
}

// The expand of the same as a launch of its own: a wavefront adds to 256 columns of a token, and the tokens of one stretch
// of columns come before the next stretch, so that the workgroups under way share the N * r KB of B that belong to one.
__global__ __launch_bounds__(256) void expand_f32_kernel(const float* __restrict__ h, const float* __restrict__ B,
                                                         const int32_t* __restrict__ topk_idx, int T, int d_out, int r,
                                                         int k, float* __restrict__ out) {
    __shared__ __attribute__((aligned(16))) float hs[4][kMaxTopK * kMaxRank];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, blocks = ceil_div(T, 4);
    const int stretch = blockIdx.x / blocks;
    const int t = min((int)(blockIdx.x - stretch * blocks) * 4 + wave, T - 1);   // the last token again past the end
    const int c = stretch * 256 + lane * 4, kr = k * r;
    for (int i = lane; i < kr; i += 64) hs[wave][i] = h[(size_t)t * kr + i];
    __syncthreads();
    if (c >= d_out || (int)(blockIdx.x - stretch * blocks) * 4 + wave >= T) return;
    f32x4* o = reinterpret_cast<f32x4*>(out + (size_t)t * d_out + c);
    f32x4 acc = *o;
    for (int slot = 0; slot < k; ++slot) {
        const int a = __builtin_amdgcn_readfirstlane(topk_idx[(size_t)t * k + slot]);
        const float* Ba = B + (size_t)a * r * d_out + c;
        f32x4 d = {0.f, 0.f, 0.f, 0.f};
        for (int q0 = 0; q0 < r; q0 += 8) {   // 8 rows of B in flight
            f32x4 b[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) b[u] = *reinterpret_cast<const f32x4*>(Ba + (size_t)min(q0 + u, r - 1) * d_out);
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (q0 + u < r) {
                    const float hv = hs[wave][slot * r + q0 + u];
#pragma unroll
                    for (int j = 0; j < 4; ++j) d[j] = fmaf(hv, b[u][j], d[j]);
                }
        }
        acc += d;
    }
    *o = acc;
}

// Bound by B from L2.  In the launch of everything a workgroup walks the k * r rows of its token at columns of its own, so
// that with many tokens the whole of B is in use at a time; where a thread of it has a single column, or few rows to
// walk, the second launch costs more than it saves.  Whole layer, without and with it: 28 adapters of rank 64, top-8, 256
// -> 4096 64 tokens 816 -> 119 us, 1024 1032 -> 627, 4096 3344 -> 1408 (bucketed: 2546); rank 8, top-2, 256 -> 4096 64 tokens
// 43 -> 19, 4096 213 -> 177; 512 -> 768 (6 groups of 8 rows per thread) 64 tokens 20.2 against 18.7, 4096 103.4 against
// 104.8; 256 -> 264, 12 adapters of rank 16, top-3 (6.2 groups) 5000 tokens 75.2 against 78.0; 256 -> 256 64 tokens 10.5
// against 13.8, with 64 adapters of rank 32, top-4, 31.2 against 34.5.
bool f32_expand_apart(int d_out, int r, int k) {
    return d_out > kRowThreads && (int64_t)d_out * k * ceil_div(r, 8) >= 8 * kRowThreads;
}

hipError_t launch_route_lora_f32(const float* x, const float* W_gate, const float* bias, const float* A, const float* B,
                                 int T, int d_in, int d_out, int N, int r, int k, float inv_temperature, float scale,
                                 int32_t* topk_idx, float* topk_w, float* out, float* h, hipStream_t stream) {
    const bool apart = f32_expand_apart(d_out, r, k);
    const int64_t blocks = ceil_div64(d_out, 256) * ceil_div64(T, 4);
    if (apart && (h == nullptr || blocks > INT32_MAX)) return hipErrorInvalidValue;
    const int h_cols = k * r >= 64 ? 64 : pow2_at_least(k * r);
    route_lora_f32_kernel<<<T, kRowThreads, 0, stream>>>(x, W_gate, bias, A, B, d_in, d_out, N, pow2_at_least(N), r, k,
                                                         h_cols, inv_temperature, scale, topk_idx, topk_w, out,
                                                         apart ? h : nullptr);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !apart) return e;
    expand_f32_kernel<<<(unsigned)blocks, 256, 0, stream>>>(h, B, topk_idx, T, d_out, r, k, out);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// The whole layer in one launch, for few adapters: a workgroup computes 16 columns for 16 tokens, and on the
// way the tokens' gate logits and x * A_i of every adapter (EB blocks of 16 columns in all) instead of waiting for a launch
// that does so once.  Four wavefronts take a quarter of K each of the two products on the matrix cores, four others the
// logits; what is left is one round through LDS, the ranking, and the rows of B of the chosen adapters.  A layer of this
// size is latency and launches: 64 x 256 -> 256 with 4 adapters of rank 8 is two rounds of loads instead of six.
// ------------------------------------------------------------------------------------------
constexpr int kF32LayerThreads = 512, kF32LayerInputs = 512, kF32LayerAdapters = 16;
constexpr int kF32LayerGate = 2048;   // most values of W_gate, four columns at least

// Where gate_row's 256 threads are (part, column), its wavefront w has the parts from w * mine, and the rows m * 4 * mine
// + part of a part are its m-th, M of them for every part (past d_in: zeros).
struct GateRows {
    int mine, mine_log2, stride, stride_log2, M, x_row;   // stride: values per row of W_gate in LDS; x_row: x per token
    __host__ __device__ GateRows(int d_in, int N) {
        const int cols_log2 = N > 8 ? 4 : N > 4 ? 3 : N > 2 ? 2 : N > 1 ? 1 : 0;   // columns: N to a power of two
        stride_log2 = cols_log2 < 2 ? 2 : cols_log2;
        stride = 1 << stride_log2;
        mine_log2 = 6 - cols_log2;
        mine = 1 << mine_log2;
        M = ceil_div(d_in, 4 * mine);
        x_row = M * mine + 4;           // rows four banks apart
    }
    __host__ __device__ int wave_floats() const { return 16 * x_row + M * mine * stride; }
};

// gate_row of 16 tokens, the part of its wavefront w, bit for bit: the same products in the same four chains per part, added
// as there, so that a token's routing is the same in gate_topk, in the launches of the larger layers and here.  The rows
// of x and W_gate that belong to w's parts pass through LDS (`staged`, this wavefront's own: no barrier); a lane takes a part
// (two or four adjacent ones where N leaves fewer than 4 columns) of 4 tokens and 4 columns.
// TOK tokens at a time: four take more than 128 registers.
template <int TOK>
__device__ __forceinline__ void gate_rows_f32(const __amdgpu_buffer_rsrc_t xr, const __amdgpu_buffer_rsrc_t gr, int m0, int T,
                                              int d_in, int N, int w, int lane, float* staged,
                                              float (&gate)[16][kF32LayerAdapters + 4]) {
    constexpr uint32_t kOutside = 0x80000000u;
    constexpr int XP = kF32LayerInputs / 64, WP = kF32LayerGate / 256;
    const GateRows g(d_in, N);
    const int rows = g.M * g.mine;
    // row of x and W_gate that is the l-th of this wavefront
    auto row = [&](int l) { return (((l >> g.mine_log2) * 4 + w) << g.mine_log2) + (l & (g.mine - 1)); };
    float* const xs = staged;
    float* const ws = staged + 16 * g.x_row;
    // a token's x: 16-byte pieces, four lanes to a token;  W_gate: 64 / stride rows at a time
    const int tok = lane >> 2, sub = lane & 3;
    const uint32_t xo = (uint32_t)min(m0 + tok, T - 1) * (uint32_t)d_in;
    u32x4 xv[XP];
    float wv[WP];
#pragma unroll
    for (int p = 0; p < XP; ++p) {
        const int i = row((p * 4 + sub) * 4);
        if (p * 16 < rows) xv[p] = __builtin_amdgcn_raw_buffer_load_b128(xr, i < d_in ? (xo + i) * 4 : kOutside, 0, 0);
    }
    const int wrows = 64 >> g.stride_log2, lr = lane >> g.stride_log2, c = lane & (g.stride - 1);
#pragma unroll
    for (int p = 0; p < WP; ++p) {
        const int i = row(p * wrows + lr);
        if (p * wrows < rows)
            wv[p] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                                  gr, c < N && i < d_in ? (uint32_t)(i * N + c) * 4 : kOutside, 0, 0));
    }
#pragma unroll
    for (int p = 0; p < XP; ++p)
        if ((p * 4 + sub) * 4 < rows) *reinterpret_cast<u32x4*>(&xs[tok * g.x_row + (p * 4 + sub) * 4]) = xv[p];
#pragma unroll
    for (int p = 0; p < WP; ++p)
        if (p * wrows + lr < rows) ws[p * 64 + lane] = wv[p];
    __builtin_amdgcn_wave_barrier();

    const int pl = lane & 15;
    const int local = g.mine > 16 ? g.mine >> 4 : 1;                      // parts of a lane
    const int first = g.mine > 16 ? pl * local : pl & (g.mine - 1);
    const int c0 = (pl >> g.mine_log2) * 4;
#pragma unroll 1
    for (int t0 = (lane >> 4) * 4, left = 4; left > 0; left -= TOK, t0 += TOK) {
        f32x4 sum[TOK], held[TOK];
#pragma unroll 1
        for (int n = 0; n < local; ++n) {
            f32x4 a[4][TOK];   // [chain][token]
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int t = 0; t < TOK; ++t) a[u][t] = f32x4{0.f, 0.f, 0.f, 0.f};
            const float* xl = xs + t0 * g.x_row + first + n;
            const float* wl = ws + (first + n) * g.stride + c0;
            for (int m = 0; m < g.M; m += 4) {
                f32x4 wq[4];
                float xq[4][TOK];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int at = min(m + u, g.M - 1) << g.mine_log2;
                    wq[u] = *reinterpret_cast<const f32x4*>(wl + (at << g.stride_log2));
#pragma unroll
                    for (int t = 0; t < TOK; ++t) xq[u][t] = xl[t * g.x_row + at];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (m + u >= g.M) break;   // uniform
#pragma unroll
                    for (int t = 0; t < TOK; ++t)
#pragma unroll
                        for (int j = 0; j < 4; ++j) a[u][t][j] = fmaf(xq[u][t], wq[u][j], a[u][t][j]);
                }
            }
#pragma unroll
            for (int t = 0; t < TOK; ++t) {   // the lane's parts in pairs, then pairs of pairs
                const f32x4 v = (a[0][t] + a[1][t]) + (a[2][t] + a[3][t]);
                if (n == 0) sum[t] = v;
                else if (n == 1) sum[t] = sum[t] + v;
                else if (n == 2) held[t] = v;
                else sum[t] = sum[t] + (held[t] + v);
            }
        }
        // the other parts are in the lanes beside this one: quads, then the quads of 8 and of 16 lanes (each level leaves
        // its sum in all lanes of a group, so that a mirrored lane is as good as the one across)
        auto across = [&](auto ctrl) {
#pragma unroll
            for (int t = 0; t < TOK; ++t)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    sum[t][j] += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, (float)sum[t][j]),
                                                                                    decltype(ctrl)::value, 0xf, 0xf, true));
        };
        across(std::integral_constant<int, 0xB1>{});   // quad_perm 1,0,3,2
        across(std::integral_constant<int, 0x4E>{});   // quad_perm 2,3,0,1
        if (g.mine >= 8) across(std::integral_constant<int, 0x141>{});    // row_half_mirror
        if (g.mine >= 16) across(std::integral_constant<int, 0x140>{});   // row_mirror
        if ((pl & (g.mine - 1)) == 0) {
#pragma unroll
            for (int t = 0; t < TOK; ++t) *reinterpret_cast<f32x4*>(&gate[t0 + t][c0]) = sum[t];
        }
    }
}

// ALONE: at most one workgroup per CU (256 tiles, and always with four blocks of adapter columns, see layer_f32_applies), which then
// has twice the registers: a fourth K step in flight and four tokens of the gate at a time.  GPU alone, two tokens and 128 registers as for
// two workgroups, and so: 64 x 256 -> 256, 4 adapters of rank 8 8.06 and 7.99 us, 64 x 512 -> 512 10.07 and 9.81, 8 adapters 64 x 168
// -> 256 8.36 and 8.03, 13 of rank 4 64 x 128 -> 256 9.78 and 9.17.
template <int EB, bool ALONE>
__global__ __launch_bounds__(kF32LayerThreads, EB == 2 && !ALONE ? 4 : 2) void layer_f32_kernel(
    const float* __restrict__ x, const float* __restrict__ W, const float* __restrict__ W_gate,
    const float* __restrict__ bias, const float* __restrict__ A, const float* __restrict__ B, int T, int d_in, int d_out,
    int N, int r, int k, float inv_temperature, float scale, int32_t* __restrict__ topk_idx, float* __restrict__ topk_w,
    float* __restrict__ out) {
    constexpr int TN = 16, C = (1 + EB) * 16, AHEAD = EB == 2 && !ALONE ? 3 : 4;
    __shared__ __attribute__((aligned(16))) float red[4][16][C + 4];
    __shared__ __attribute__((aligned(16))) float gate[4][16][kF32LayerAdapters + 4];   // gate_row's sums per wavefront
    __shared__ int sel_idx[16][kMaxTopK];
    __shared__ float sel_sw[16][kMaxTopK];   // scale * w
    extern __shared__ __attribute__((aligned(16))) float staged[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l15 = lane & 15, kc = (lane >> 4) * 4;
    const int tiles_n = ceil_div(d_out, TN);
    const int tile_m = blockIdx.x / tiles_n, tile_n = blockIdx.x - tile_m * tiles_n;
    const int m0 = tile_m * 16, n0 = tile_n * TN, NR = N * r;
    const int steps = ceil_div(d_in, 16);

    // Loads through buffer resources: offsets of a lane that never change and a uniform K offset, so that no address
    // arithmetic stands between the loads of a step.  Rows past the edge repeat the last one (computed, never stored);
    // columns past the last and K values past d_in are outside for the hardware and count as zeros.
    constexpr uint32_t kOutside = 0x80000000u;
    auto resource = [](const float* p, uint32_t floats) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, floats * 4u, 0x00020000);
    };
    const uint32_t ld = (uint32_t)d_in;
    const __amdgpu_buffer_rsrc_t xr = resource(x, T * ld), wr = resource(W, d_out * ld), gr = resource(W_gate, ld * N),
                                 ar = resource(A, (uint32_t)NR * ld);
    if (wave >= 4) {
        gate_rows_f32<ALONE ? 4 : 2>(xr, gr, m0, T, d_in, N, wave - 4, lane, staged + (wave - 4) * GateRows(d_in, N).wave_floats(),
                      gate[wave - 4]);
    } else {
        const int s0 = wave * steps / 4, s1 = (wave + 1) * steps / 4;
        const uint32_t xo = (uint32_t)min(m0 + l15, T - 1) * ld * 4;
        const uint32_t wo = (uint32_t)min(n0 + l15, d_out - 1) * ld * 4;
        // component q of adapter a is column a * r + q
        uint32_t eo[EB];
#pragma unroll
        for (int e = 0; e < EB; ++e) {
            const int c = e * 16 + l15;
            eo[e] = c < NR ? (uint32_t)((c / r) * d_in * r + kc * r + c % r) * 4 : kOutside;
        }
        struct Step { f32x4 x, w, e[EB]; };
        auto load = [&](Step& f, int s) {
            const bool inside = s * 16 + kc < d_in;   // d_in % 8 == 0: all four values or none
            const uint32_t xk = inside ? xo + kc * 4 : kOutside, wk = inside ? wo + kc * 4 : kOutside;
            f.x = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(xr, xk, s * 64, 0));
            f.w = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(wr, wk, s * 64, 0));
#pragma unroll
            for (int e = 0; e < EB; ++e) {
                const uint32_t off = inside ? eo[e] : kOutside;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    f.e[e][j] = __builtin_bit_cast(
                        float, __builtin_amdgcn_raw_buffer_load_b32(ar, off, (s * 16 + j) * r * 4, 0));
            }
        };
        // a chain for each of a lane's four K values: less latency and a smaller rounding error than one
        f32x4 acc[1 + EB][4];
#pragma unroll
        for (int i = 0; i < 1 + EB; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        Step f[AHEAD + 1];
#pragma unroll
        for (int a = 0; a < AHEAD; ++a)
            if (s0 + a < s1) load(f[a], s0 + a);
        for (int s = s0; s < s1; s += AHEAD + 1) {
#pragma unroll
            for (int u = 0; u <= AHEAD; ++u) {   // register sets have fixed numbers
                if (s + u >= s1) break;          // uniform per wavefront
                if (s + u + AHEAD < s1) load(f[(u + AHEAD) % (AHEAD + 1)], s + u + AHEAD);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    acc[0][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(f[u].w[j], f[u].x[j], acc[0][j], 0, 0, 0);
#pragma unroll
                    for (int e = 0; e < EB; ++e)
                        acc[1 + e][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(f[u].e[e][j], f[u].x[j], acc[1 + e][j], 0, 0, 0);
                }
            }
        }
        // a lane holds columns 4 * (lane / 16) .. + 3 of token lane % 16 of every block
#pragma unroll
        for (int i = 0; i < 1 + EB; ++i)
            *reinterpret_cast<f32x4*>(&red[wave][l15][i * 16 + kc]) = (acc[i][0] + acc[i][1]) + (acc[i][2] + acc[i][3]);
    }
    __syncthreads();
    if (wave < 4) {
        for (int e = threadIdx.x; e < 16 * C / 4; e += 256) {
            const int t = e / (C / 4), c = (e % (C / 4)) * 4;
            f32x4 v[4];
#pragma unroll
            for (int w = 0; w < 4; ++w) v[w] = *reinterpret_cast<const f32x4*>(&red[w][t][c]);
            *reinterpret_cast<f32x4*>(&red[0][t][c]) = (v[0] + v[1]) + (v[2] + v[3]);
        }
    } else {   // a wavefront ranks four tokens, two at a time
        constexpr int NP = 32, G = 2;
        const int col = lane & (NP - 1), sub = lane / NP;
        float g[G];
        int si[G];
        float sw[G];
#pragma unroll
        for (int i = 0; i < G; ++i) {
            g[i] = 0.f;
            if (col < N) {
                const int t = (wave - 4) * 4 + i * 2 + sub;
                g[i] = (gate[0][t][col] + gate[1][t][col]) + (gate[2][t][col] + gate[3][t][col]);
                g[i] += bias != nullptr ? bias[col] : 0.f;
                if (g[i] == 0.f) g[i] = 0.f;   // -0 -> +0 so equal logits have equal keys
            }
        }
        wave_topk_softmax<NP, G>(g, lane, N, k, inv_temperature, si, sw);
#pragma unroll
        for (int i = 0; i < G; ++i) {
            const int t = (wave - 4) * 4 + i * 2 + sub;
            if (col < k) {
                sel_idx[t][col] = si[i];
                sel_sw[t][col] = scale * sw[i];
                if (tile_n == 0 && m0 + t < T) {
                    topk_idx[(size_t)(m0 + t) * k + col] = si[i];
                    topk_w[(size_t)(m0 + t) * k + col] = sw[i];
                }
            }
        }
    }
    __syncthreads();
    const int t = threadIdx.x / TN, c = n0 + threadIdx.x % TN;
    if (wave >= 4 || m0 + t >= T || c >= d_out) return;
    float v = red[0][t][c - n0];
    const int R8 = ceil_div(r, 8), groups = k * R8;   // (slot, 8 rows of B): the rows of two groups in flight
    for (int g0 = 0; g0 < groups; g0 += 2) {
        float b[2][8], d[2] = {0.f, 0.f};
        int at[2], q0[2], slot[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int g = min(g0 + i, groups - 1);
            slot[i] = g / R8;
            q0[i] = (g - slot[i] * R8) * 8;
            const int a = sel_idx[t][slot[i]];
            at[i] = TN + a * r;
#pragma unroll
            for (int u = 0; u < 8; ++u) b[i][u] = B[((size_t)a * r + min(q0[i] + u, r - 1)) * d_out + c];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if (g0 + i >= groups) break;
            const float sw = sel_sw[t][slot[i]];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (q0[i] + u < r) d[i] = fmaf(sw * red[0][t][at[i] + q0[i] + u], b[i][u], d[i]);
            v += d[i];
        }
    }
    out[(size_t)(m0 + t) * d_out + c] = v;
}

// Every workgroup reads the whole of W_gate and A, so this is for what one round or two of workgroups finish: the product
// of rounds, inputs and 16-column blocks is what the time goes with.  Against two launches, whole calls (the host takes 7.9
// us to issue one launch and 10.3 to 11 for two), 4 adapters of rank 8, top-2: 64 x 256 -> 256 11.1 and 8.1 us, 8 x 256 -> 4096
// 13.7 and 8.2, 64 x 384 -> 384 11.1 and 9.3, 64 x 512 -> 512 11.6 and 10.4, 512 workgroups (128 x 256 -> 1024) 13.8 and
// 10.4; 8 of rank 8: 64 x 168 -> 256 11.2 and 8.2.  Not taken, the line as it lies where the second figure is the larger one:
// more adapters and inputs, the logits take the longest (16 of rank 2, 64 x 256 -> 256 10.9 and 12.9, 128 -> 256 11.1 and
// 8.7; one adapter, whose columns fill a quarter of the lanes, 64 x 512 -> 256 12.2 and 12.8, of rank 64 12.1 and 13.8); two
// workgroups per CU with many adapter columns (4 of rank 16, 128 x 80 -> 1024 13.9 and 15.7); top-8 of many (8 of rank 4,
// 64 x 256 -> 256 12.6 and 13.4; of 4 adapters top-4 10.7 and 9.8).
bool layer_f32_applies(int T, int d_in, int d_out, int N, int r, int k) {
    if (N > kF32LayerAdapters || N * r > 64 || d_in > kF32LayerInputs) return false;
    if ((d_in << GateRows(d_in, N).stride_log2) > kF32LayerGate) return false;
    if ((N == 1 && (r > 32 || d_in > 256)) || (N > 4 && k > 4)) return false;
    const int64_t tiles = ceil_div64(T, 16) * ceil_div64(d_out, 16);
    const int blocks = N * r <= 32 ? 4 : 6;
    return tiles <= (N <= 8 && N * r <= 32 ? 512 : 256) &&
           ceil_div64(tiles, 256) * d_in * blocks <= (blocks == 4 && r >= 8 ? 2048 : 1024);
}

hipError_t launch_layer_f32(const float* x, const float* W, const float* W_gate, const float* bias, const float* A,
                            const float* B, int T, int d_in, int d_out, int N, int r, int k, float inv_temperature,
                            float scale, int32_t* topk_idx, float* topk_w, float* out, hipStream_t stream) {
    if (d_in % 8 != 0 || d_out % 8 != 0 || !layer_f32_applies(T, d_in, d_out, N, r, k) || k < 1 || k > N || k > kMaxTopK)
        return hipErrorInvalidValue;
    const int64_t tiles = ceil_div64(T, 16) * ceil_div64(d_out, 16);
    const size_t lds = (size_t)4 * GateRows(d_in, N).wave_floats() * sizeof(float);
    auto go = [&](auto kern) {
        kern<<<(unsigned)tiles, kF32LayerThreads, lds, stream>>>(x, W, W_gate, bias, A, B, T, d_in, d_out, N, r, k,
                                                                 inv_temperature, scale, topk_idx, topk_w, out);
        return hipGetLastError();
    };
    if (N * r > 32) return go(layer_f32_kernel<4, true>);
    return tiles <= 256 ? go(layer_f32_kernel<2, true>) : go(layer_f32_kernel<2, false>);
}

}  // namespace meteora
