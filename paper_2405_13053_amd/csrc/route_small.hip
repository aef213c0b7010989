// The second of the two launches of a decode-sized layer call, and of the few-tile form of a few hundred tokens: routing, the
// sum of the K splits and the LoRA expand in one kernel.
#include <type_traits>
#include "common.hpp"
#include "kernels.hpp"
#include "topk_key.hpp"
#include "dense_logits.hpp"

namespace meteora {

// A group of layers that share x (same T, N, r, k, number of K splits): the operands of the decode tail per member.
struct RouteGroup {
    struct Member {
        const float* gpart;   // [S][T][rows of Wcat]
        const float* bias;
        int32_t* idx;
        float* w;
    } m[kMaxDecodeGroup];
};
struct FinishGroup {
    struct Member {
        const float* partial;   // [S][T][d_out]
        const bf16_t* B;        // [N, r, d_out]
        bf16_t* out;            // [T, d_out]
        int d_out;
        int tile0, gate_tile0;  // first row tile of its W and of its Wcat in the launch that wrote the K splits
        int chunk0;             // first of its stretches of kTailThreads * 8 columns; of members not there: past the last one
    } m[kMaxDecodeGroup];
    SplitPlan plan;
    int chunks;                 // per_xcd: stretches of all members; else those of the widest
    int per_xcd;                // (stretch, token) pairs of an XCD, 0: member by member, the stretches of a token side by side
};

// K splits of row tile g of the launch (see SplitPlan)
__device__ __forceinline__ int split_count(const SplitPlan& p, int g) {
    if (p.per_wg == 0) return p.S;   // uniform
    const uint32_t first = (uint32_t)(g * p.nk) / (uint32_t)p.per_wg;
    return (int)((uint32_t)(g * p.nk + p.nk - 1) / (uint32_t)p.per_wg - first) + 1;
}

// ------------------------------------------------------------------------------------------------------------
// Decode tail: everything of a decode-sized layer call after the one launch that streams W.  That launch computes,
// as fp32 K-split tiles, x * W^T and x * Wcat^T, the latter being the gate terms (Sec. 3.1) AND the shrink x * A_i
// of EVERY adapter (N * r columns: 4% more rows to stream than W alone at N = 28, r = 8, 5120 -> 5120; half as many again at N = 64, r = 32, 4096 ->
// 4096, which still beats a gathered shrink, see decode_fused_applies).  What is
// left per token is a chain of two memory round trips, taken here by independent wavefronts with no LDS and no
// barrier: (1) the gate tiles -> logits, top-k, softmax (Eq. 3); (2) the selected adapters' shrink tiles and rows
// of B -> out = bf16( sum of the projection's split tiles + sum_slot sum_q (scale * w * h) * B ), Eq. 2 with one
// rounding.  A wavefront owns 64 x 8 consecutive output columns of one token and repeats the token's routing
// (a few hundred bytes) instead of waiting for another wavefront.  The routing is the routine every path shares.
// ------------------------------------------------------------------------------------------------------------

// one wavefront per workgroup (measured: 64, 128 and 256 threads per workgroup time the same)
constexpr int kTailThreads = 64;

// A wavefront reads its stretch of k * r rows of B.  Workgroup ids are dealt round-robin to the XCDs, so with a token's stretches side
// by side every XCD reads all of B where their number is odd, a half or a quarter where it is even: where that is more than
// an XCD's L2 holds, and where members of a group differ in width, an XCD gets stretches of its own instead, one after the other
// for all tokens.  Whole calls, side by side and so, us: 64 adapters of rank 32, top-4, 190 x 5120 -> 13824 142 and 96, twice 286
// and 194, 300 x 2048 -> 5504 twice 146 and 98; 28 of rank 8 64 x 5120 -> 13824 36.0 and 34.6; q, k, v of 300 tokens 4096 inputs 37.5
// and 33.5.  With less (1368 -> 1072, three stretches of which the last is short) 300 to 1000 tokens lose 2 to 4%.
constexpr int64_t kTailL2Bytes = 4 << 20;

// U: K splits whose loads are in flight.  The loads of a round are unconditional, those past the last split repeat it, so U
// follows the number of splits of the launch.  Whole calls with eight always, and so: 300 x 4096 -> 4096 (three splits) 26.6
// and 26.1 us, 1531 x 4096 -> 1024 rank 16 (three) 38.4 and 37.7, 64 x 5120 -> 13824 (two) 36.6 and 36.2.
// Ranks off 8, 16, 32 and 64 have two of them, since one and two splits with four in flight lose 0.1 to 0.3 us: rank 12, four always and
// so, 1 x 4096 -> 1024 (eight splits) 12.6 and 11.9, 8384 -> 264 (16) 15.5 and 14.2, 200 x 4096 -> 4096 top-8 (six) 37.1 and 36.2.
// R8: a slot's shrink values take 8 * R8 lanes.  NP: N padded to 32 or 64.  WHOLE: the rank is 8 * R8; otherwise it is less, and
// the rows of B past it are left out.
template <int R8, int U, int NP, bool WHOLE>
__global__ __launch_bounds__(kTailThreads) void decode_tail_kernel(int T, int N, int CR, int k, int rank, float inv_temperature,
                                                                   float scale, const RouteGroup rg,
                                                                   const FinishGroup fg) {
    constexpr int RL = R8 * 8;       // lanes per slot
    constexpr int SLOTS = 64 / RL;   // slots whose shrink values a wavefront holds at a time, one value per lane
    const int r = WHOLE ? RL : rank, groups = WHOLE ? R8 : (r + 7) / 8;   // groups of 8 rows of B per slot
    const int lane = threadIdx.x & 63;
    int chunk, t, member = 0;
    if (__builtin_expect(fg.per_xcd == 0, 1)) {   // uniform
        chunk = blockIdx.x % fg.chunks;
        t = blockIdx.x / fg.chunks;
        if (t >= T) {
            member = t / T;
            t -= member * T;
        }
    } else {   // the token runs fastest, in eight equal parts
        const int pair = (int)(blockIdx.x % 8) * fg.per_xcd + (int)(blockIdx.x / 8);
        if (pair >= fg.chunks * T) return;
        chunk = pair / T;
        t = pair - chunk * T;
#pragma unroll
        for (int g = 1; g < kMaxDecodeGroup; ++g) member += chunk >= fg.m[g].chunk0 ? 1 : 0;
        chunk -= fg.m[member].chunk0;
    }
    const int d_out = fg.m[member].d_out, c8 = d_out / 8, S = fg.plan.S;
    const int gi = chunk * kTailThreads + threadIdx.x;
    const bool active = gi < c8;              // lanes past the row's end work on its last columns and do not store
    const int c = (active ? gi : c8 - 1) * 8;
    const float* __restrict__ gpart = rg.m[member].gpart;
    const bf16_t* __restrict__ B = fg.m[member].B;
    const float* partial = fg.m[member].partial + (size_t)t * d_out + c;
    const size_t pstride = (size_t)T * d_out;

    const int tile = c / kSplitRows, nsplit = split_count(fg.plan, fg.m[member].tile0 + tile);

    // the projection's split tiles do not depend on the routing: the first U go out first
    f32x4 pre0[U], pre1[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const float* src = partial + (size_t)min(u, nsplit - 1) * pstride;
        pre0[u] = *reinterpret_cast<const f32x4*>(src);
        pre1[u] = *reinterpret_cast<const f32x4*>(src + 4);
    }
    float g[1];
    const int lt[1] = {0};
    static_assert(2 * NP <= kSplitRows, "the hi and mid terms are rows of Wcat's first row tile");
    const int gate_tile0 = fg.m[member].gate_tile0;
    dense_logits<NP, 1, U>(gpart, split_count(fg.plan, gate_tile0), CR, rg.m[member].bias, T, N, t, lt, lane & (NP - 1), g,
                           split_count(fg.plan, gate_tile0 + 2 * NP / kSplitRows));
    int sel_i[1];
    float sel_w[1];
    wave_topk_softmax<NP, 1>(g, lane, N, k, inv_temperature, sel_i, sel_w);   // lane s < k: the s-th choice
    if (chunk == 0 && threadIdx.x < k) {   // the wavefronts of a token compute the same routing: one reports it
        rg.m[member].idx[(size_t)t * k + lane] = sel_i[0];
        rg.m[member].w[(size_t)t * k + lane] = sel_w[0];
    }
    f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (u < nsplit) { lo += pre0[u]; hi += pre1[u]; }
    for (int s0 = U; s0 < S; s0 += U) {   // tiles in order, U tiles' loads in flight
        f32x4 v0[U], v1[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float* src = partial + (size_t)min(s0 + u, nsplit - 1) * pstride;
            v0[u] = *reinterpret_cast<const f32x4*>(src);
            v1[u] = *reinterpret_cast<const f32x4*>(src + 4);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (s0 + u < nsplit) { lo += v0[u]; hi += v1[u]; }
    }

    auto load_rows = [&](int slot, int q0, u32x4 (&b)[8]) {   // 8 rows of B of the slot's adapter, this lane's columns
        const int a = __builtin_amdgcn_readlane(sel_i[0], slot);
        const bf16_t* Ba = B + ((size_t)a * r + q0) * d_out + c;
#pragma unroll
        for (int u = 0; u < 8; ++u) b[u] = *reinterpret_cast<const u32x4*>(Ba + (size_t)(WHOLE ? u : min(u, r - 1 - q0)) * d_out);
    };
    for (int s0 = 0; s0 < k; s0 += SLOTS) {
        const int ns = min(SLOTS, k - s0);
        // lane e holds scale * w * h of slot s0 + e / RL, component e % RL: the shrink tiles of that adapter's columns
        // of Wcat, added in split order
        const int my_slot = min(s0 + lane / RL, k - 1);
        const int a_e = __shfl(sel_i[0], my_slot);
        const float w_e = __shfl(sel_w[0], my_slot);
        const int q_e = lane & (RL - 1);
        const int hcol = 3 * NP + a_e * (WHOLE ? r : groups * 8) + (WHOLE ? q_e : min(q_e, r - 1));
        const float* hsrc = gpart + (size_t)t * CR + hcol;
        const int hsplit = split_count(fg.plan, gate_tile0 + hcol / kSplitRows);
        float hvs[U];
#pragma unroll
        for (int u = 0; u < U; ++u) hvs[u] = hsrc[(size_t)min(u, hsplit - 1) * T * CR];
        u32x4 bcur[8];
        load_rows(s0, 0, bcur);   // the first rows of B are under way while the shrink tiles arrive
        float h = 0.f;
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (u < hsplit) h += hvs[u];
        for (int p0 = U; p0 < S; p0 += U) {
            float v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = hsrc[(size_t)min(p0 + u, hsplit - 1) * T * CR];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (p0 + u < hsplit) h += v[u];
        }
        const float hv = scale * w_e * h;
        const int ngroups = ns * groups;
        int slot = 0, q0 = 0;
        for (int j = 0; j < ngroups; ++j) {   // (slot, 8 rows) pieces; the next piece's loads go out before this one's FMAs
            u32x4 bnext[8];
            const bool more = j + 1 < ngroups;
            const int e0 = WHOLE ? j * 8 : slot * RL + q0, rows = WHOLE ? 8 : r - q0;
            if constexpr (WHOLE) {
                slot = (j + 1) / R8;
                q0 = (j + 1) % R8 * 8;
            } else {
                q0 += 8;
                if (q0 >= r) { q0 = 0; ++slot; }
            }
            if (more) load_rows(s0 + slot, q0, bnext);
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (!WHOLE && u >= rows) break;   // uniform
                const float hq = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(hv), e0 + u));
                lo[0] = fmaf(hq, bf16_bits_to_float(bcur[u][0] & 0xffffu), lo[0]);
                lo[1] = fmaf(hq, bf16_bits_to_float(bcur[u][0] >> 16), lo[1]);
                lo[2] = fmaf(hq, bf16_bits_to_float(bcur[u][1] & 0xffffu), lo[2]);
                lo[3] = fmaf(hq, bf16_bits_to_float(bcur[u][1] >> 16), lo[3]);
                hi[0] = fmaf(hq, bf16_bits_to_float(bcur[u][2] & 0xffffu), hi[0]);
                hi[1] = fmaf(hq, bf16_bits_to_float(bcur[u][2] >> 16), hi[1]);
                hi[2] = fmaf(hq, bf16_bits_to_float(bcur[u][3] & 0xffffu), hi[2]);
                hi[3] = fmaf(hq, bf16_bits_to_float(bcur[u][3] >> 16), hi[3]);
            }
            if (more) {
#pragma unroll
                for (int u = 0; u < 8; ++u) bcur[u] = bnext[u];
            }
        }
    }
    if (active) {
        u32x4 pk;
        pk[0] = pack_bf16x2(lo[0], lo[1]); pk[1] = pack_bf16x2(lo[2], lo[3]);
        pk[2] = pack_bf16x2(hi[0], hi[1]); pk[3] = pack_bf16x2(hi[2], hi[3]);
        *reinterpret_cast<u32x4*>(fg.m[member].out + (size_t)t * d_out + c) = pk;
    }
}

// gate_rows = every row of Wcat: the split tiles mem[g].gpartial hold the gate terms and all adapters' shrink.
hipError_t launch_decode_tail_group(const DecodeMember* mem, int G, const SplitPlan& plan, int T, int N, int r, int k, int gate_rows,
                                    float inv_temperature, float scale, hipStream_t stream) {
    if (G < 1 || G > kMaxDecodeGroup || plan.S < 1 || r < 1 || r > kMaxRank || gate_rows != prep_wcat_rows(N, r))
        return hipErrorInvalidValue;
    RouteGroup rg{};
    FinishGroup fg{};
    int tiles = 0, chunks = 0, widest = 0;
    for (int g = 0; g < G; ++g) {
        if (mem[g].d_out % 8 != 0 || mem[g].d_out < 8) return hipErrorInvalidValue;
        rg.m[g] = {mem[g].gpartial, mem[g].bias, mem[g].idx, mem[g].w};
        fg.m[g] = {mem[g].partial, (const bf16_t*)mem[g].B, (bf16_t*)mem[g].out, mem[g].d_out, tiles,
                   tiles + ceil_div(mem[g].d_out, kSplitRows), chunks};
        tiles += ceil_div(mem[g].d_out, kSplitRows) + ceil_div(gate_rows, kSplitRows);
        const int stretches = ceil_div(mem[g].d_out / 8, kTailThreads);
        chunks += stretches;
        widest = stretches > widest ? stretches : widest;
    }
    for (int g = G; g < kMaxDecodeGroup; ++g) fg.m[g].chunk0 = chunks;
    fg.plan = plan;
    const bool apart = chunks != G * widest || (int64_t)chunks * kTailThreads * 8 * N * r * 2 > kTailL2Bytes;
    fg.per_xcd = apart ? ceil_div(chunks * T, 8) : 0;
    fg.chunks = fg.per_xcd > 0 ? chunks : widest;
    const unsigned grid = fg.per_xcd > 0 ? (unsigned)fg.per_xcd * 8 : (unsigned)G * T * widest;
    auto go = [&](auto kern) {
        kern<<<grid, kTailThreads, 0, stream>>>(T, N, gate_rows, k, r, inv_temperature, scale, rg, fg);
        return hipGetLastError();
    };
    auto by_splits = [&](auto r8, auto np) {
        constexpr int R8 = decltype(r8)::value, NP = decltype(np)::value;
        if (r != 8 * R8) return plan.S <= 4 ? go(decode_tail_kernel<R8, 4, NP, false>) : go(decode_tail_kernel<R8, 8, NP, false>);
        if (plan.S == 1) return go(decode_tail_kernel<R8, 1, NP, true>);
        if (plan.S == 2) return go(decode_tail_kernel<R8, 2, NP, true>);
        if (plan.S <= 4) return go(decode_tail_kernel<R8, 4, NP, true>);
        return go(decode_tail_kernel<R8, 8, NP, true>);
    };
    auto by_rank = [&](auto np) {
        if (r <= 8) return by_splits(std::integral_constant<int, 1>{}, np);
        if (r <= 16) return by_splits(std::integral_constant<int, 2>{}, np);
        if (r <= 32) return by_splits(std::integral_constant<int, 4>{}, np);
        return by_splits(std::integral_constant<int, 8>{}, np);
    };
    return padded_adapters(N) == 32 ? by_rank(std::integral_constant<int, 32>{}) : by_rank(std::integral_constant<int, 64>{});
}

}  // namespace meteora
