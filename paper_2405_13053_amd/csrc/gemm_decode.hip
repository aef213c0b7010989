// Decode (at most 64 tokens): the first of the two launches of a layer call, x * [W; Wcat]^T of every layer of a
// group as fp32 K-split tiles; decode_tail_kernel is the second.
//
// Bound by streaming W from HBM (64 tokens use each weight for 64 multiply-adds, a tenth of what the matrix cores do
// in the time the weight takes to arrive), next by what else has to move: x from L2 for every row tile, the fp32
// tiles out and in again.
//   - A row tile is 128 rows of W: the x columns that come along with it are half its bytes (64 rows: as many; a load
//     and multiply loop without the output ran at 4.2 against 4.7 TB/s on 14144 x 5120 weights, 64 tokens).
//   - K advances 128 columns at a time through a ring of LDS slots filled by 16-byte global->LDS loads, two slots
//     (64 KB of W) in flight per CU, one workgroup per CU.  A wavefront multiplies 16 rows of W with all tokens.
//   - As few K splits as give every CU a workgroup, since each costs an fp32 tile written and read: all workgroups
//     are resident together and share the bandwidth evenly, so CUs left over cost nothing (SplitPlan).
//
// Measured at 64 tokens, kernel alone, W not in any cache, against 64 x 64 tiles with a two-slot ring and about 512
// workgroups: 4096 -> 14336 twice 64.9 -> 43.9 us (5.5 TB/s; a loop of the same loads alone takes 44), 14336 -> 4096
// 37 -> 26.4, 5120 -> 13824 40.1 -> 30.1.  Of the first, without the staggered K walk 49.6, with W's loads cached 54.6.
// Stores of a run that ends its tile: with "nt" 4096 -> 4096 11.4 us against 12.4; of runs cut at any step, which stream
// W on behind their stores, without: 5120 -> 5120 three times 35.8 against 39.4.
#include "common.hpp"
#include "gemm_mfma.hpp"
#include "kernels.hpp"

namespace meteora {

constexpr int kStreamRows = kSplitRows, kStreamK = 128, kStreamThreads = 512, kStreamSlots = 3;
constexpr int kStageStride = kStreamRows * 4 + 16;   // bytes per token of the output stage, 16 tokens at a time

struct StreamArgs {
    const bf16_t* x;   // [T, d_in]
    int T, d_in, nk, tiles, nseg;
    SplitPlan plan;
    struct Segment {
        const bf16_t* W;   // [rows, d_in]
        float* partial;    // [splits of the row tile][T][rows]
        int rows, tile0;   // first row tile
    } seg[2 * kMaxDecodeGroup];
};

// token blocks of 16; the x slot is at least 32 rows, one load instruction per wavefront
template <int TB> constexpr int stream_x_rows() { return TB < 2 ? 32 : TB * 16; }
template <int TB> constexpr int stream_slot_bytes() { return (stream_x_rows<TB>() + kStreamRows) * kStreamK * 2; }
template <int TB> constexpr int stream_lds_bytes() { return kStreamSlots * stream_slot_bytes<TB>() + 16 * kStageStride; }

struct StreamOperand { __amdgpu_buffer_rsrc_t rsrc; };

__device__ __forceinline__ StreamOperand stream_operand(const bf16_t* base, int rows, uint32_t ld) {
    return {__builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(base), 0, (uint32_t)rows * ld, 0x00020000)};
}

// Cache policy of a load: the default, or "nt".  W is read "nt": a decode step streams the weights of a whole model, and
// what a call reads is gone before its next.  A caller who does come back to the same weights finds them in the Infinity
// Cache with ordinary loads only (64 tokens, 4096 -> 4096 over and over 16.1 against 17.8 us, 4096 -> 14336 27.7 against
// 32.8; out of cache 17.7 against 18.0 and 34.9 against 33.1); ordinary loads for launches of up to 56 MB alone made the
// seven linears of a block 128.5 us instead of 121.1.
constexpr int kReused = 0, kReadOnce = 2;
template <int POLICY>
__device__ __forceinline__ void stream_load(const StreamOperand& o, unsigned char* dst, uint32_t voff, int soff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(o.rsrc, (__attribute__((address_space(3))) void*)dst, 16, voff, soff, 0,
                                             POLICY);
}

template <int TB>
__global__ __launch_bounds__(kStreamThreads) void gemm_decode_stream_kernel(const StreamArgs a) {
    constexpr int ROW = kStreamK * 2;                                      // bytes per LDS row: 16 chunks
    constexpr int PX = stream_x_rows<TB>() / 32, PW = kStreamRows / 32;    // loads per wavefront and slot: 4 rows each
    constexpr int NS = kStreamSlots;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned char* stage = smem + NS * stream_slot_bytes<TB>();
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l15 = lane & 15, kq = lane >> 4;
    const uint32_t ld = (uint32_t)a.d_in * 2;

    // this workgroup's run of (row tile, K step) units; a split of a tile is walked from a step of its own on and around,
    // or the workgroups would all read the same columns of their rows together, which lie a power of two apart and
    // meet in few memory channels
    int u0, n, first = 0;
    if (a.plan.per_wg == 0) {   // split s of a tile: an equal share of its K steps
        const int t = blockIdx.x / a.plan.S, s = blockIdx.x - t * a.plan.S;
        const int k0 = s * a.nk / a.plan.S;
        u0 = t * a.nk + k0;
        n = (s + 1) * a.nk / a.plan.S - k0;
        first = blockIdx.x % n;
    } else {
        u0 = blockIdx.x * a.plan.per_wg;
        n = min(a.plan.per_wg, a.tiles * a.nk - u0);
    }
    auto segment_of = [&](int tile) {
        int e = 0;
        for (int i = 1; i < a.nseg; ++i)
            if (tile >= a.seg[i].tile0) e = i;
        return e;
    };
    // A load instruction moves 4 rows x 256 bytes; the 16-byte chunks of row r are XOR-swizzled with r & 15, so that a
    // ds_read_b128 of 16 rows of one chunk touches every bank once.  Rows and columns outside the matrix load zeros.
    const int rsub = lane >> 4;
    constexpr uint32_t kOutside = 0x80000000u;   // past every resource here, also after the K offset is added
    auto voffset = [&](int row, int kstep) {   // row of the LDS tile (its swizzle), as an offset from the tile's first row
        const int chunk = l15 ^ (row & 15);
        return kstep * kStreamK + chunk * 8 < a.d_in ? (uint32_t)row * ld + (uint32_t)chunk * 16 : kOutside;
    };
    const StreamOperand xr = stream_operand(a.x, a.T, ld);
    auto w_resource = [&](int tile) {
        const int e = segment_of(tile), row0 = (tile - a.seg[e].tile0) * kStreamRows;
        return stream_operand(a.seg[e].W + (size_t)row0 * a.d_in, min(a.seg[e].rows - row0, kStreamRows), ld);
    };
    int rq_tile = u0 / a.nk, rq_left = n;
    const int k_begin = u0 - rq_tile * a.nk, k_end = min(a.nk, k_begin + n);
    int rq_k = k_begin + first;
    StreamOperand wr = w_resource(rq_tile);
    auto request = [&](int slot) {   // the run's next unit
        unsigned char* ws = smem + slot * stream_slot_bytes<TB>();
        unsigned char* xs = ws + kStreamRows * ROW;
#pragma unroll
        for (int j = 0; j < PW; ++j)
            stream_load<kReadOnce>(wr, ws + (j * 8 + wave) * 1024, voffset((j * 8 + wave) * 4 + rsub, rq_k), rq_k * ROW);
#pragma unroll
        for (int j = 0; j < PX; ++j)
            stream_load<kReused>(xr, xs + (j * 8 + wave) * 1024, voffset((j * 8 + wave) * 4 + rsub, rq_k), rq_k * ROW);
        --rq_left;
        if (a.plan.per_wg == 0) {
            if (++rq_k == k_end) rq_k = k_begin;
        } else if (++rq_k == a.nk) {
            rq_k = 0;
            if (rq_left > 0) wr = w_resource(++rq_tile);
        }
    };
    for (int s = 0; s < NS - 1 && s < n; ++s) request(s);

    f32x4 acc[TB];
#pragma unroll
    for (int b = 0; b < TB; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    int tile = u0 / a.nk, k = u0 - tile * a.nk, slot = 0, free_slot = NS - 1;
    for (int i = 0; i < n; ++i) {
        // unit i has landed when only the younger units' loads are outstanding (stores of a finished tile may be among
        // them, which only makes the wait longer); every wavefront's reads of unit i-1 are complete
        if (n - i >= NS - 1)
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NS - 2) * (PX + PW)) : "memory");
        else
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (rq_left > 0) request(free_slot);
        const unsigned char* ws = smem + slot * stream_slot_bytes<TB>() + wave * 16 * ROW;
        const unsigned char* xs = smem + slot * stream_slot_bytes<TB>() + kStreamRows * ROW;
#pragma unroll
        for (int ks = 0; ks < kStreamK / 32; ++ks) {
            const int at = l15 * ROW + (((ks * 4 + kq) ^ l15) << 4);   // row l15 of a block of 16
            const bf16x8 wf = *reinterpret_cast<const bf16x8*>(ws + at);
#pragma unroll
            for (int b = 0; b < TB; ++b) {
                const bf16x8 xf = *reinterpret_cast<const bf16x8*>(xs + b * 16 * ROW + at);
                acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, xf, acc[b], 0, 0, 0);
            }
        }
        free_slot = slot;
        slot = slot + 1 == NS ? 0 : slot + 1;
        if (++k < a.nk && i + 1 < n) continue;
        // the run leaves this row tile: a lane holds 4 consecutive columns of a token per block; staged, so that the
        // stores are whole lines of 512 bytes per token
        const int e = segment_of(tile), rows = a.seg[e].rows, col0 = (tile - a.seg[e].tile0) * kStreamRows;
        const int part = a.plan.per_wg == 0 ? (int)blockIdx.x - tile * a.plan.S
                                            : (int)blockIdx.x - tile * a.nk / a.plan.per_wg;
        float* dst = a.seg[e].partial + (size_t)part * a.T * rows;
        const int st = tid >> 5, sc = (tid & 31) * 4;   // token and column of this thread's 16-byte piece
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            *reinterpret_cast<f32x4*>(stage + l15 * kStageStride + (wave * 16 + kq * 4) * 4) = acc[b];
            acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            const f32x4 v = *reinterpret_cast<const f32x4*>(stage + st * kStageStride + sc * 4);
            if (b * 16 + st < a.T && col0 + sc < rows) {
                f32x4* p = reinterpret_cast<f32x4*>(dst + (size_t)(b * 16 + st) * rows + col0 + sc);
                if (a.plan.per_wg == 0) __builtin_nontemporal_store(v, p);
                else *p = v;
            }
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        }
        k = 0;
        ++tile;
    }
}

// S equal K splits per row tile where that occupies at least three quarters of the 256 CUs with one workgroup each;
// otherwise (86 to 95 or 129 to 191 row tiles, or more than 256) 256 runs of equal length over all units of the launch,
// which cut row tiles where they fall.  A split is two K steps or more.  Whole layers of 89 row tiles (11008 outputs), two
// equal splits against runs, 1, 16 and 64 tokens: 4096 inputs 23.5, 24.4, 29.3 against 21.7, 22.8, 28.6 us, 8192 36.9,
// 38.1, 46.0 against 35.7, 36.9, 45.0, 2048 14.9, 15.9, 20.4 against 15.0, 16.1, 21.3.
SplitPlan gemm_decode_plan(int d_in, const int* d_out, int G, int gate_rows) {
    SplitPlan p{};
    p.nk = ceil_div(d_in, kStreamK);
    int tiles = 0;
    for (int g = 0; g < G; ++g) tiles += ceil_div(d_out[g], kStreamRows) + ceil_div(gate_rows, kStreamRows);
    p.S = 256 / tiles;
    const int most = p.nk / 2 > 1 ? p.nk / 2 : 1;
    if (p.S > most) p.S = most;
    else if (p.S * tiles < 192) {
        p.per_wg = (int)ceil_div64((int64_t)tiles * p.nk, 256);
        p.S = ceil_div(p.nk - 1, p.per_wg) + 1;   // most runs that nk consecutive units can touch
    }
    // The tail adds the splits eight at a time, so of narrow outputs (up to 28 row tiles) one round unless its splits are longer
    // than 8 K steps, two at most.  Whole layers, as many splits as fit and so, 1, 16 and 64 tokens: 4096 -> 1024 (16 splits, 8)
    // 11.9, 12.7, 15.0 and 11.1, 11.8, 14.1 us; 4096 -> 2048 (13, 8) 13.0, 14.3, 17.8 and 11.5, 12.4, 15.0; 8192 -> 1024 (23, 8)
    // 15.4, 16.4, 19.2 and 13.8, 14.6, 17.0; 14336 -> 1024 (23, 16) 17.4, 18.8, 21.5 and 16.0, 16.8, 20.1, with 8 18.1, 19.1,
    // 23.2.  Where 12 to 16 splits fill the CUs and eight are longer than 6 K steps, few tokens are slower with eight, so as many
    // as fit: 7360 -> 1400 of rank 16 (16) 13.7, 14.8, 18.6 and with 8 14.6, 15.4, 18.2; 8128 -> 1808 (14) 13.5, 14.6, 19.8 and
    // 14.1, 14.5, 18.4; 6400 -> 2048 (13) 12.5, 14.3 and 13.3, 13.9; but 7168 -> 2560 (11) 13.8, 15.9 and 13.8, 14.4, 8192 -> 1400
    // (18) 14.5, 15.8 and 13.5, 14.4.  (The token count does not decide: a token's logits are the same at every decode batch.)
    if (p.per_wg == 0 && p.S > 8) {
        if (p.nk > 64) p.S = p.S > 16 ? 16 : p.S;
        else if (!(p.nk > 48 && p.S >= 12 && p.S <= 16)) p.S = 8;
    }
    return p;
}

// the offsets inside a row tile of W, and of the rows and columns outside it (kOutside), fit
bool gemm_decode_ok(int d_in) { return (uint64_t)kStreamRows * d_in * 2 < (1ull << 31); }

hipError_t launch_gemm_decode_main(const void* x, const DecodeMember* mem, int G, int gate_rows, const SplitPlan& plan,
                                   int T, int d_in, hipStream_t stream) {
    if (gate_rows % 8 != 0 || G < 1 || G > kMaxDecodeGroup || T < 1 || T > 64 || d_in % 8 != 0 || plan.S < 1 ||
        plan.nk != ceil_div(d_in, kStreamK) || !gemm_decode_ok(d_in))
        return hipErrorInvalidValue;
    StreamArgs a{};
    a.x = (const bf16_t*)x; a.T = T; a.d_in = d_in; a.nk = plan.nk; a.plan = plan;
    for (int g = 0; g < G; ++g) {
        if (mem[g].d_out % 8 != 0) return hipErrorInvalidValue;
        a.seg[2 * g] = {(const bf16_t*)mem[g].W, mem[g].partial, mem[g].d_out, a.tiles};
        a.tiles += ceil_div(mem[g].d_out, kStreamRows);
        a.seg[2 * g + 1] = {(const bf16_t*)mem[g].wg3, mem[g].gpartial, gate_rows, a.tiles};
        a.tiles += ceil_div(gate_rows, kStreamRows);
    }
    a.nseg = 2 * G;
    if ((int64_t)a.tiles * a.nk >= INT32_MAX) return hipErrorInvalidValue;
    const int grid = plan.per_wg == 0 ? a.tiles * plan.S : ceil_div(a.tiles * a.nk, plan.per_wg);
    auto go = [&](auto kern, int smem) {
        const hipError_t e = ensure_lds_limit(reinterpret_cast<const void*>(kern), smem);
        if (e != hipSuccess) return e;
        kern<<<grid, kStreamThreads, smem, stream>>>(a);
        return hipGetLastError();
    };
    if (T <= 16) return go(&gemm_decode_stream_kernel<1>, stream_lds_bytes<1>());
    if (T <= 32) return go(&gemm_decode_stream_kernel<2>, stream_lds_bytes<2>());
    return go(&gemm_decode_stream_kernel<4>, stream_lds_bytes<4>());
}

hipError_t gemm_decode_init_kernels() {
    hipError_t e = ensure_lds_limit(reinterpret_cast<const void*>(&gemm_decode_stream_kernel<1>), stream_lds_bytes<1>());
    if (e == hipSuccess)
        e = ensure_lds_limit(reinterpret_cast<const void*>(&gemm_decode_stream_kernel<2>), stream_lds_bytes<2>());
    if (e == hipSuccess)
        e = ensure_lds_limit(reinterpret_cast<const void*>(&gemm_decode_stream_kernel<4>), stream_lds_bytes<4>());
    return e;
}

}  // namespace meteora
