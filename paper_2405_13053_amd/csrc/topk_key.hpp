// Wavefront top-k of the gate (Sec. 3.1: I(x) = top-k of G(x), ties to the lowest index) and the softmax over
// the k selected logits (Eq. 3), shared by the routing kernels so that every path ranks identically.
//
// A logit is ranked by an order-preserving unsigned image of its bits; among equal logits the lowest index wins.
#pragma once
#include "common.hpp"

namespace meteora {

__device__ __forceinline__ uint32_t logit_key(float g) {
    const uint32_t u = __float_as_uint(g);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);   // monotonic; 0 is the image of no float but one NaN
}
__device__ __forceinline__ float key_logit(uint32_t u) {
    return __uint_as_float((u & 0x80000000u) ? (u & 0x7fffffffu) : ~u);
}

// The value of another lane of the same row of 16, or of the row before (DPP controls; no trip through LDS as a
// shuffle would take, about 60 cycles each).  Lanes without a source read 0.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, false);
}
constexpr int kDppQuad1032 = 0xb1, kDppQuad2301 = 0x4e, kDppRowShr = 0x110, kDppHalfMirror = 0x141, kDppBcast15 = 0x142,
              kDppBcast31 = 0x143;
static_assert(kMaxTopK == 8, "the softmax sums eight lanes");

// Unsigned maximum over the NP (32 or 64) lanes of each group, known to all of them.
template <int NP>
__device__ __forceinline__ uint32_t group_max(uint32_t v, int lane) {
    v = max(v, dpp<kDppRowShr + 1>(v));
    v = max(v, dpp<kDppRowShr + 2>(v));
    v = max(v, dpp<kDppRowShr + 4>(v));
    v = max(v, dpp<kDppRowShr + 8>(v));          // lane 15 of a row: the row's maximum
    v = max(v, dpp<kDppBcast15>(v));             // lanes 31 and 63: of two rows
    if constexpr (NP == 64) {
        v = max(v, dpp<kDppBcast31>(v));
        return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
    } else {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)v, 31);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
        return lane < 32 ? lo : hi;
    }
}

// Bitwise or over the lanes of a wavefront, known to all of them.
__device__ __forceinline__ uint32_t wave_or(uint32_t v) {
    v |= dpp<kDppRowShr + 1>(v);
    v |= dpp<kDppRowShr + 2>(v);
    v |= dpp<kDppRowShr + 4>(v);
    v |= dpp<kDppRowShr + 8>(v);
    v |= dpp<kDppBcast15>(v);
    v |= dpp<kDppBcast31>(v);
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// A token's NP (32 or 64) logit columns sit in NP adjacent lanes (col = lane % NP), so a wavefront ranks
// 64/NP tokens per group and G interleaved groups (their latencies overlap).  g[i] is this lane's
// logit of group i (lanes col >= N are padding; -0 must already be +0).  Selecting k adapters is k maxima over the NP
// lanes, each followed by the lowest lane that holds it; padding and selected lanes stand out.
// On return lane col = s < k of each token holds its s-th choice: sel_i[i] = adapter, sel_w[i] = Eq. 3 weight.
// 2000 tokens, 64 adapters, top-4, 8 K slices: the kernel around it takes 7.5 us against 13.2 with 64-bit keys (value
// and index) in shuffles.
template <int NP, int G>
__device__ __forceinline__ void wave_topk_softmax(const float (&g)[G], int lane, int N, int k, float inv_temperature,
                                                  int (&sel_i)[G], float (&sel_w)[G]) {
    const int col = lane & (NP - 1);
    uint32_t key[G];
    bool open[G];
    float sel_g[G], gmax[G];
#pragma unroll
    for (int i = 0; i < G; ++i) { key[i] = logit_key(g[i]); open[i] = col < N; sel_g[i] = 0.f; sel_i[i] = 0; }
    for (int s = 0; s < k; ++s) {
#pragma unroll
        for (int i = 0; i < G; ++i) {
            const uint32_t best = group_max<NP>(open[i] ? key[i] : 0u, lane);
            unsigned long long m = __ballot(open[i] && key[i] == best);
            int win;
            if constexpr (NP == 64) win = __ffsll(m) - 1;
            else win = __ffs(lane < 32 ? (uint32_t)m : (uint32_t)(m >> 32)) - 1;
            if (col == win) open[i] = false;
            if (s == 0) gmax[i] = key_logit(best);
            if (col == s) { sel_g[i] = key_logit(best); sel_i[i] = win; }
        }
    }
    if (k == 1) {
        // Top-1 strategy (App. A.1): the softmax over a single logit is exactly 1 whatever the logit and the
        // temperature, so neither the exponential nor the normalising sum is evaluated
#pragma unroll
        for (int i = 0; i < G; ++i) sel_w[i] = col == 0 ? 1.f : 0.f;
        return;
    }
#pragma unroll
    for (int i = 0; i < G; ++i) {
        const float e = (col < k) ? expf((sel_g[i] - gmax[i]) * inv_temperature) : 0.f;
        float sum = e;   // lanes 0..7 of a group: neighbours, pairs, fours
        sum += __uint_as_float(dpp<kDppQuad1032>(__float_as_uint(sum)));
        sum += __uint_as_float(dpp<kDppQuad2301>(__float_as_uint(sum)));
        sum += __uint_as_float(dpp<kDppHalfMirror>(__float_as_uint(sum)));
        sel_w[i] = e / sum;
    }
}

}  // namespace meteora
