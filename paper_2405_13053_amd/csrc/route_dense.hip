// Mid-sized batches (a few hundred to a few thousand tokens): routing and LoRA shrink without bucket lists.
//
// At these sizes the gate logits, top-k, bucketing, grouped shrink and its finalize are five short launches
// that each read little and sit on launch and fill/drain time.  Here one MFMA launch computes, for every
// token, the split-bf16 gate logits (Sec. 3.1) AND x * A_i for EVERY adapter i (the shrink of Eq. 2 before
// the selection): x[T, d_in] times Wcat[3*NP + N*r, d_in]^T, a 320-column GEMM at N = 28, r = 8, whose
// extra flops (N/k times the selected adapters') are cheap next to a second gathered pass over x.
// This file's kernel then, per token, adds the K-splits in a fixed order, picks the top-k (ties to the lowest
// index), takes the softmax over the k selected (Eq. 3) and writes the token's row of the dense expand
// operand: hdense[t, a*r + q] = bf16(scale * w * h) for the selected adapters a, zero elsewhere.
// The values are those of the bucketed path up to fp32 summation order; the ranking routine is the same.
#include <type_traits>
#include "common.hpp"
#include "kernels.hpp"
#include "topk_key.hpp"
#include "dense_logits.hpp"

namespace meteora {

// Independent wavefronts, no LDS and no barrier: a wavefront ranks two tokens (one per half, NP = 32 lanes each; one of
// more than 32 adapters) and writes their rows, a 16-byte piece (8 columns: of one adapter with R8, r % 8 == 0) per lane and
// round.  Two rounds of
// loads: the gate terms of every K split, then the selected adapters' shrink columns.  (A workgroup form of it — 16
// tokens per workgroup, the choices handed from the ranking wavefront to the row writers through LDS behind a
// barrier — took 7.9 us at config 2 and 9.3 us at T = 1024 where this one takes 5.6 and 5.3.)
// WIDE (more than 4 K splits): twice as many splits' loads in flight
constexpr int kSelThreads = 256;
template <bool WIDE, int NP, bool R8>
__global__ __launch_bounds__(kSelThreads) void route_dense_select_kernel(const float* __restrict__ part,   // [S][T][CR]
                                                                         const float* __restrict__ bias, int S, int CR, int T,
                                                                         int N, int r, int k, float inv_temperature,
                                                                         float scale, int32_t* __restrict__ topk_idx,
                                                                         float* __restrict__ topk_w, bf16_t* __restrict__ hdense,
                                                                         int ext_stride) {
    constexpr int TPW = 64 / NP;   // tokens per wavefront
    const int lane = threadIdx.x & 63, col = lane & (NP - 1), sub = lane / NP;
    const int t0 = (blockIdx.x * (kSelThreads / 64) + (threadIdx.x >> 6)) * TPW;
    if (t0 >= T) return;   // the whole wavefront
    float g[1];
    const int lt[1] = {sub};
    dense_logits<NP, 1, WIDE ? 8 : 4>(part, S, CR, bias, T, N, t0, lt, col, g);
    int sel_i[1];
    float sel_w[1];
    wave_topk_softmax<NP, 1>(g, lane, N, k, inv_temperature, sel_i, sel_w);   // lane col = s < k: the s-th choice
    if (col < k && t0 + sub < T) {
        topk_idx[(size_t)(t0 + sub) * k + col] = sel_i[0];
        topk_w[(size_t)(t0 + sub) * k + col] = sel_w[0];
    }
    const int C8 = ext_stride / 8;
    constexpr int HU = WIDE ? 8 : 4;   // splits whose loads are in flight
    for (int e0 = 0; e0 < TPW * C8; e0 += 64) {   // uniform trip count: every lane takes part in the exchanges
        const int e = e0 + lane;
        const bool active = e < TPW * C8;
        const int th = active ? e / C8 : 0, c0 = active ? (e - th * C8) * 8 : 0;
        const int t = active ? t0 + th : T;
        u32x4 pk = {0u, 0u, 0u, 0u};
        if constexpr (!R8) {   // the columns of a piece may belong to several adapters
            const int RP = wcat_rank(r);
            int at[8];         // column of the products
            float sw[8];       // scale * w, 0 in columns of other adapters
#pragma unroll
            for (int j = 0; j < 8; ++j) { at[j] = 0; sw[j] = 0.f; }
            bool any = false;
            for (int s = 0; s < k; ++s) {
                const int q0 = c0 - __shfl(sel_i[0], th * NP + s) * r;   // the piece's first column as one of this adapter's
                const float wi = __shfl(sel_w[0], th * NP + s);
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (q0 + j >= 0 && q0 + j < r) {
                        at[j] = 3 * NP + (c0 - q0) / r * RP + q0 + j;
                        sw[j] = scale * wi;
                        any = true;
                    }
            }
            if (any && t < T) {
                float h[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                const float* src = part + (size_t)t * CR;
                for (int s0 = 0; s0 < S; s0 += 4) {   // splits in order
                    float v[4][8];
#pragma unroll
                    for (int u = 0; u < 4; ++u)
#pragma unroll
                        for (int j = 0; j < 8; ++j) v[u][j] = src[(size_t)min(s0 + u, S - 1) * T * CR + at[j]];
#pragma unroll
                    for (int u = 0; u < 4; ++u)
#pragma unroll
                        for (int j = 0; j < 8; ++j)
                            if (s0 + u < S) h[j] += v[u][j];
                }
#pragma unroll
                for (int j = 0; j < 8; ++j) h[j] = at[j] > 0 ? sw[j] * h[j] : 0.f;   // products of columns not chosen may be anything
#pragma unroll
                for (int j = 0; j < 4; ++j) pk[j] = pack_bf16x2(h[2 * j], h[2 * j + 1]);
            }
            if (t < T) *reinterpret_cast<u32x4*>(hdense + (size_t)t * ext_stride + c0) = pk;
            continue;
        }
        const int a = c0 / r;
        bool hit = false;
        float sw = 0.f;
        for (int s = 0; s < k; ++s) {
            const int ai = __shfl(sel_i[0], th * NP + s);
            const float wi = __shfl(sel_w[0], th * NP + s);
            if (c0 < N * r && ai == a) { hit = true; sw = scale * wi; }
        }
        if (hit && t < T) {
            f32x4 h0 = {0.f, 0.f, 0.f, 0.f}, h1 = {0.f, 0.f, 0.f, 0.f};
            const float* src = part + (size_t)t * CR + 3 * NP + c0;
            for (int s0 = 0; s0 < S; s0 += HU) {   // splits in order, 2 * HU loads in flight
                f32x4 v0[HU], v1[HU];
#pragma unroll
                for (int u = 0; u < HU; ++u) {
                    const float* p = src + (size_t)min(s0 + u, S - 1) * T * CR;
                    v0[u] = *reinterpret_cast<const f32x4*>(p);
                    v1[u] = *reinterpret_cast<const f32x4*>(p + 4);
                }
#pragma unroll
                for (int u = 0; u < HU; ++u)
                    if (s0 + u < S) { h0 += v0[u]; h1 += v1[u]; }
            }
            pk[0] = pack_bf16x2(sw * h0[0], sw * h0[1]); pk[1] = pack_bf16x2(sw * h0[2], sw * h0[3]);
            pk[2] = pack_bf16x2(sw * h1[0], sw * h1[1]); pk[3] = pack_bf16x2(sw * h1[2], sw * h1[3]);
        }
        if (t < T) *reinterpret_cast<u32x4*>(hdense + (size_t)t * ext_stride + c0) = pk;
    }
}

// Rows of hdense for a routing the caller holds, from the products of every adapter (no gate columns in `part`): a thread
// owns a 16-byte piece, 8 columns of one adapter.  An adapter named twice by a token counts in its last slot, ids outside
// [0, N) nowhere, as in the bucketed path.
__global__ __launch_bounds__(256) void dense_expand_operand_kernel(const float* __restrict__ part, int S,
                                                                   const int32_t* __restrict__ topk_idx,
                                                                   const float* __restrict__ topk_w, int T, int N,
                                                                   int r, int k, float scale,
                                                                   bf16_t* __restrict__ hdense, int ext_stride) {
    const int C8 = ext_stride / 8;
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (gid >= (int64_t)T * C8) return;
    const int t = (int)(gid / C8), c0 = (int)(gid - (int64_t)t * C8) * 8, NR = N * r;
    u32x4 pk = {0u, 0u, 0u, 0u};
    if (c0 < NR) {
        const int a = c0 / r;
        int slot = -1;
        for (int s = 0; s < k; ++s)
            if (topk_idx[(size_t)t * k + s] == a) slot = s;
        if (slot >= 0) {
            f32x4 h0 = {0.f, 0.f, 0.f, 0.f}, h1 = {0.f, 0.f, 0.f, 0.f};
            const float* src = part + (size_t)t * NR + c0;
            const float sw = scale * topk_w[(size_t)t * k + slot];
            f32x4 v0[8], v1[8];   // at most 8 splits, added in order
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const float* p = src + (size_t)min(u, S - 1) * T * NR;
                v0[u] = *reinterpret_cast<const f32x4*>(p);
                v1[u] = *reinterpret_cast<const f32x4*>(p + 4);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (u < S) { h0 += v0[u]; h1 += v1[u]; }
            pk[0] = pack_bf16x2(sw * h0[0], sw * h0[1]); pk[1] = pack_bf16x2(sw * h0[2], sw * h0[3]);
            pk[2] = pack_bf16x2(sw * h1[0], sw * h1[1]); pk[3] = pack_bf16x2(sw * h1[2], sw * h1[3]);
        }
    }
    *reinterpret_cast<u32x4*>(hdense + (size_t)t * ext_stride + c0) = pk;
}

hipError_t launch_dense_expand_operand(const float* part, int S, const int32_t* topk_idx, const float* topk_w, int T,
                                       int N, int r, int k, float scale, void* hdense, int ext_stride,
                                       hipStream_t stream) {
    if (S < 1 || S > 8 || r % 8 != 0 || ext_stride < N * r) return hipErrorInvalidValue;
    const int64_t pieces = (int64_t)T * (ext_stride / 8);
    dense_expand_operand_kernel<<<(unsigned)ceil_div64(pieces, 256), 256, 0, stream>>>(
        part, S, topk_idx, topk_w, T, N, r, k, scale, (bf16_t*)hdense, ext_stride);
    return hipGetLastError();
}

// Widths off 64 gain as much from the dense forms as the others: 200 x 4104 -> 4096 bucketed 55.8 us, dense 24.9, 512 61.5 and
// 39.5, 2000 96.3 and 87.4, 8192 277 and 261.  Up to 640 rows of Wcat (28 adapters of rank 16: 544): measured against the bucketed
// sequence on 4096 -> 4096, rank 16, the dense forms are faster or equal from T = 8 to 8192 (T = 128: 35 against 55 us).  Ranks
// that are no multiple of 8 gain too, padding included: rank 12 2000 x 4096 -> 4096 91.8 and 75.9, 4000 140 and 123, 9000 315 and
// 311; rank 4 88.0 and 70.7, 135 and 113, 309 and 282.
// Measured against the bucketed sequence (gate logits, top-k, scatter, whole-K shrink) on 4096 -> 4096 and
// 14336 -> 4096 at T = 12000 ... 65536: with 320 rows of Wcat (28 adapters of rank 8) the dense form wins at every
// size (whole call: 357.6 against 377.0 us at T = 12000, 918.9 against 984.8 at 32768, 1830 against 1985 at 65536);
// with 544 rows (rank 16) it wins by 0.3-8% where the products' 128 x 320 tiles fill the CUs (T = 16384: 496.7 against
// 515.2 us, 1631 against 1680 with d_in = 14336) and loses where they do not (T = 12000, d_in = 14336: 188 workgroups
// of a full K sweep each, 1269 against 1231 us).
bool route_dense_applies(int T, int d_in, int N, int r, bool bf16) {
    const int CR = prep_wcat_rows(N, r);
    if (!bf16 || CR > kWcatMaxRows || T <= 64 || !gemm_dense_splitk_ok(T, d_in, CR)) return false;
    if (T <= kRouteDenseMaxTokens || CR <= 320) return true;
    const int64_t wgs = (int64_t)ceil_div(T, 128) * ceil_div(CR, 320) * gemm_dense_splits(T, d_in, CR);
    return wgs * 10 >= (wgs + 255) / 256 * 256 * 9;   // at least 90% of the CUs' slots over the launch
}

// The LoRA term alone on a given routing: the products of every adapter cost T * N * r, the bucketed sequence (histogram,
// scatter, grouped shrink, finalize) about 25 us and T * k * r.  Whole lora_forward calls, dense against bucketed: N * r =
// 224, d_in = 4096: top-1 T = 500 20.4 against 26.6 us, 4096 30.3 against 32.3, 8192 44.1 against 43.2; top-2 T = 500 20.5
// against 27.3, 10000 53.1 against 65.7, 12000 97.8 against 97.1 (4096 outputs), 16384 x 14336 174 against 225; N * r = 448:
// top-1 T = 1000 27.7 against 29.1, 2000 34.0 against 32.1; top-2 3000 x 14336 71.3 against 69.8.
bool lora_dense_applies(int T, int d_in, int N, int r, int k, bool bf16) {
    return r % 8 == 0 && route_dense_applies(T, d_in, N, r, bf16) && (N * r <= 256 ? T <= 4096 || k >= 2 : T <= 1024);
}

hipError_t launch_route_dense_products(const void* x, const void* wcat, int T, int d_in, int N, int r, float* part,
                                       hipStream_t stream) {
    return launch_gemm_dense_splitk(x, wcat, T, d_in, prep_wcat_rows(N, r), part, stream);
}

hipError_t launch_route_dense_select(const float* part, const float* bias, int T, int d_in, int N, int r, int k,
                                     float inv_temperature, float scale, int32_t* topk_idx, float* topk_w,
                                     void* hdense, int ext_stride, hipStream_t stream) {
    const int CR = prep_wcat_rows(N, r), S = gemm_dense_splits(T, d_in, CR), NP = padded_adapters(N);
    const int grid = ceil_div(T, 64 / NP * (kSelThreads / 64));
    auto go = [&](auto kern) {
        kern<<<grid, kSelThreads, 0, stream>>>(part, bias, S, CR, T, N, r, k, inv_temperature, scale, topk_idx, topk_w,
                                               (bf16_t*)hdense, ext_stride);
        return hipGetLastError();
    };
    auto by_rank = [&](auto np) {
        constexpr int P = decltype(np)::value;
        if (r % 8 != 0) return go(route_dense_select_kernel<false, P, false>);
        return S > 4 ? go(route_dense_select_kernel<true, P, true>) : go(route_dense_select_kernel<false, P, true>);
    };
    return NP == 32 ? by_rank(std::integral_constant<int, 32>{}) : by_rank(std::integral_constant<int, 64>{});
}

}  // namespace meteora
