// C ABI of the library (declared in include/meteora.h): argument validation, workspace
// carving and the launch sequence of each entry point.  No device memory is allocated here
// and nothing synchronises with the host.
#include <math.h>
#include <string.h>

#include <algorithm>

#include "../../include/meteora.h"
#include "common.hpp"
#include "kernels.hpp"

using namespace meteora;

namespace {

struct WsLayout {
    size_t wsplit, partials, chunk_counts, counts, offsets, bucket_tok, bucket_slot, topk_idx, topk_w, h32,
        hdense, apack, hpart, splitk, btrans, wcat, dpart, gpart, spart, total;
    int ext_stride;   // columns of hdense: N*r rounded up to 64 (one K tile of the GEMM)
};

bool shape_ok(int T, int d_in, int d_out, int N, int r, int k) {
    return T >= 0 && d_in >= 1 && d_out >= 1 && N >= 1 && r >= 1 && k >= 1 && k <= N;
}

// The decode tail reads k * r rows of B for every token, from L2; beyond some 0.5 to 1.3 GB (the more, the
// more inputs the other sequences gather for their shrink) the dense operand of every adapter and MFMAs are cheaper.  Top-8 of
// 64 adapters, tail against bucketed, us: 4096 -> 14336 of rank 32 64 tokens (0.47 GB) 68 and 78, of rank 64 40 tokens (0.59) 96
// and 98, 64 (0.94) 124 and 102; 4096 -> 4096 of rank 64 128 tokens (0.54) 55.8 and 75.6, 256 (1.1) 79.2 and 77.6, of rank 32
// 300 tokens (0.63) 61.6 and 70.5, 512 (1.1) 83.0 and 68.7; 14336 -> 4096 of rank 32 512 tokens (1.1) 163 and 211.
bool expand_by_rows_applies(int T, int d_in, int d_out, int r, int k) {
    return 2.0 * T * k * r * d_out <= (T <= 64 ? 2.6e8 : 4e8) + 6e4 * d_in;
}
// the largest batch of more than 64 tokens it takes (or fewer: none)
int expand_by_rows_tokens(int d_in, int d_out, int r, int k) {
    return (int)std::min((4e8 + 6e4 * d_in) / (2.0 * k * r * d_out), 1e9);
}

// Decode in two launches (gate logits and every adapter's shrink inside the GEMM's launch, then routing + reduce +
// expand): whatever the widths (below 8 million inputs) and adapters.  Four launches (gate logits, top-k with the shrink, split GEMM, reduction), as
// widths off 64, fewer than 512 inputs and more than 32704 outputs had, and so: 1 token of 4104 -> 4096 24.0 and 15.1 us, 64 27.8
// and 20.1, 49 x 320 -> 2920 of rank 16 packed per call 21.6 and 16.9, 1 x 4096 -> 40960 89.5 and 60.5, 64 95.5 and 81.4.
// 64 adapters of rank 32, top-4 and top-8, 4096 -> 4096, 1 token 61.3 and 89.1 against 23.2 and 33.7, 64 tokens 66.5 and 95.4
// against 29.8 and 39.6, though 2240 more rows are streamed; 28 adapters of rank 12, 40.2 and 45.0 against 15.3 and 19.2.
// The token count does not decide, so that a token is routed by the same sums in every decode batch: the rows of B that 64 tokens
// read do (64 adapters of rank 64, top-8, 4096 -> 14336, tail and bucketed, 1 token 62 and 87, 30 tokens 82 and 95, 64 124 and 102).
// Layers whose projection the bucketed sequence would split along K too (whole K tiles, 512 inputs and more, up to 32704 outputs), with
// rank 8, 16 or 32 and up to 640 rows of Wcat, take the tail whatever they read: 28 adapters of rank 16, top-8, 64 tokens, bucketed
// and tail 512 -> 28672 39.0 and 37.3, 4096 -> 32704 105 and 83; 17 of rank 32 4096 -> 32704 32 tokens 101 and 79, 64 107 and 103, but
// 512 -> 32704 38.6 and 41.5, 44 and 63.  Wider ones lose more: 17 of rank 32, 64 tokens, 512 -> 65536 53 and 114.
bool decode_fused_applies(int T, int d_in, int d_out, int N, int r, int k, bool bf16) {
    if (!bf16 || T > 64 || !gemm_decode_ok(d_in)) return false;
    const bool split_too = d_in % 64 == 0 && d_in >= 512 && d_out <= 32704;
    return (split_too && (r == 8 || r == 16 || r == 32) && prep_wcat_rows(N, r) <= kWcatMaxRows) ||
           expand_by_rows_applies(64, d_in, d_out, r, k);
}

// Mid-sized batches whose 128 x 128 output tiles would leave most CUs idle (a few hundred tokens): the base
// projection is split along K over workgroups like the routing products (fp32 tiles), and the reduction adds the
// LoRA expand, as for decode.  Returns the number of K splits, 0 = the fused GEMM runs instead.
int dense_midsplit_splits(int T, int d_in, int d_out, int N, int r, int k, bool bf16) {
    // measured on 4096 -> 4096, 4096 -> 14336 and 14336 -> 4096, T = 65 ... 2048: the split form wins as long as the
    // projection can still be cut into at least two K splits (see gemm_multi_splits for how many) (19.0 against 56.1 us
    // at T = 65, 36.1 against 60.1 at T = 512, 45.6 against 48.7 at T = 704, 47.6 against 48.8 at T = 768 for
    // 4096 -> 4096; 43.3 against 47.6 at T = 160 for 4096 -> 14336; 107 against 131 at T = 704 for 14336 -> 4096)
    // Above 640 rows of Wcat the bucketed sequence is the other choice: 64 adapters of rank 32, top-4, 4096 -> 4096 T = 65 29.2
    // against 60.5, 200 36.6 against 61.7, 512 58.2 against 63.6; 14336 -> 4096 top-8 T = 300 123 against 170.  Two workgroups
    // per CU, which lost while every XCD read all of B (4096 -> 14336 T = 65 91.0 against 84.9, 128 143 against 95.7; now 59 and 78
    // against 82 and 92, top-8 76 and 108 against 84 and 94), are not taken.
    const int CR = prep_wcat_rows(N, r);
    if (!bf16 || T <= 64 || !gemm_multi_ok(T, d_in, CR) || !gemm_multi_ok(T, d_in, d_out)) return 0;
    const int col_tiles = ceil_div(d_out, 128) + ceil_div(CR, 128), fit = gemm_multi_fit(T, d_in, d_out);
    if (CR > kWcatMaxRows && (2 * ceil_div(T, 256) * col_tiles > 256 || !expand_by_rows_applies(T, d_in, d_out, r, k))) return 0;
    const int S = gemm_multi_splits(T, col_tiles, fit, ceil_div(d_in, 64), (int64_t)d_out + CR);
    return S >= 2 ? S : 0;
}

// Which sequence of launches a call of meteora_linear_forward runs.  S: its K splits (decode, few tiles, dense products).
enum class Form { kDecode, kFewTiles, kDense, kBucketed, kF32 };
struct LayerForm { Form form; int S; };

LayerForm layer_form(int T, int d_in, int d_out, int N, int r, int k, bool bf16) {
    if (!bf16) return {Form::kF32, 0};
    const int CR = prep_wcat_rows(N, r);
    if (decode_fused_applies(T, d_in, d_out, N, r, k, bf16)) return {Form::kDecode, gemm_decode_plan(d_in, &d_out, 1, CR).S};
    if (const int S = dense_midsplit_splits(T, d_in, d_out, N, r, k, bf16)) return {Form::kFewTiles, S};
    if (route_dense_applies(T, d_in, N, r, bf16)) return {Form::kDense, gemm_dense_splits(T, d_in, CR)};
    return {Form::kBucketed, 0};
}

bool shape_supported(int T, int d_in, int d_out, int N, int r, int k) {
    return N <= kMaxAdapters && k <= kMaxTopK && r <= kMaxRank && d_in % 8 == 0 && d_out % 8 == 0 &&
           (int64_t)T * k < (int64_t)INT32_MAX && (int64_t)T * (int64_t)(d_in > d_out ? d_in : d_out) < ((int64_t)1 << 40);
}

// The regions that one call writes, one behind the other; those of other forms are empty.  pairs: tokens times K splits.  For
// decode the bucketed sequence's have their places too, so that the K splits lie behind them, where a group that shares the workspace
// has written fewer of its own: the seven linears of a block, 64 tokens, 122.2 and 121.0 us.
WsLayout ws_carve(Form form, int64_t pairs, int T, int d_in, int d_out, int N, int r, int k, bool lora) {
    WsLayout L{};
    size_t off = 0;
    auto take = [&](bool used, size_t bytes) { size_t o = off; off = align_up(off + (used ? bytes : 0), 256); return o; };
    const bool bf16 = form != Form::kF32, routes = !lora;
    const bool decode = form == Form::kDecode, few = form == Form::kFewTiles, dense = form == Form::kDense;
    const bool bucketed = form == Form::kBucketed || decode, lists = bucketed || (lora && !bf16), expand = dense || bucketed;
    const size_t slots = (size_t)T * k, CR = lora ? (size_t)N * wcat_rank(r) : prep_wcat_rows(N, r);
    L.ext_stride = (int)align_up((size_t)N * r, 64);
    L.wsplit = take(bucketed && routes, gate_wsplit_bytes(d_in, N, bf16));
    L.partials = take(bucketed && routes, (size_t)gate_kslices(d_in, bf16) * T * padded_adapters(N) * sizeof(float));
    L.chunk_counts = take(lists, (size_t)(bucket_chunks(T) + routing_chunks_extra(T)) * N * sizeof(int32_t));
    L.counts = take(lists, (size_t)N * sizeof(int32_t));
    L.offsets = take(lists, (size_t)(N + 1) * sizeof(int32_t));
    L.bucket_tok = take(lists, slots * sizeof(int32_t));
    L.bucket_slot = take(lists, slots * sizeof(int32_t));
    L.topk_idx = take(routes, slots * sizeof(int32_t));
    L.topk_w = take(routes, slots * sizeof(float));
    L.h32 = take(!bf16, slots * r * sizeof(float));
    L.hdense = take(expand, (size_t)T * L.ext_stride * sizeof(uint16_t));
    // A packed for the bucketed sequence, or Wcat: a call reads the one or the other
    const size_t apack = bucketed ? shrink_apack_bytes(d_in, N, r, bf16) : 0;
    L.apack = L.wcat = take(bf16, form == Form::kBucketed ? apack : std::max(apack, CR * d_in * sizeof(uint16_t)));
    L.hpart = take(bucketed, shrink_hpart_bytes(T, d_in, r, k, bf16));
    L.splitk = take(decode || (bucketed && routes), decode ? (size_t)pairs * d_out * sizeof(float) : gemm_splitk_bytes(T, d_in, d_out, bf16));
    L.btrans = take(expand, prep_btrans_bytes(d_out, N, r, bf16));
    L.dpart = take(few || dense, (size_t)pairs * CR * sizeof(float));
    L.gpart = take(decode, (size_t)pairs * CR * sizeof(float));
    L.spart = take(few, (size_t)pairs * d_out * sizeof(float));
    L.total = off;
    return L;
}

WsLayout ws_layout(int T, int d_in, int d_out, int N, int r, int k, bool bf16) {   // of meteora_linear_forward
    const LayerForm f = layer_form(T, d_in, d_out, N, r, k, bf16);
    return ws_carve(f.form, (int64_t)f.S * T, T, d_in, d_out, N, r, k, false);
}

WsLayout lora_layout(int T, int d_in, int d_out, int N, int r, int k, bool bf16) {   // of meteora_lora_forward
    if (!bf16) return ws_carve(Form::kF32, 0, T, d_in, d_out, N, r, k, true);
    if (!lora_dense_applies(T, d_in, N, r, k, bf16)) return ws_carve(Form::kBucketed, 0, T, d_in, d_out, N, r, k, true);
    return ws_carve(Form::kDense, (int64_t)gemm_dense_splits(T, d_in, N * r) * T, T, d_in, d_out, N, r, k, true);
}

// meteora_gate_topk: the split gate weight, then the partial logits
size_t gate_ws_bytes(int T, int d_in, int N, bool bf16) {
    return align_up(gate_wsplit_bytes(d_in, N, bf16), 256) +
           align_up((size_t)gate_kslices(d_in, bf16) * T * padded_adapters(N) * sizeof(float), 256);
}

// What the entry points that share a workspace write of it, the largest of them, for a batch of T tokens.  linear: what
// meteora_linear_forward does (ws_layout)
size_t ws_written(size_t linear, int T, int d_in, int d_out, int N, int r, int k, bool bf16) {
    return std::max({linear, lora_layout(T, d_in, d_out, N, r, k, bf16).total, gate_ws_bytes(T, d_in, N, bf16),
                     (size_t)bucket_chunks(T) * N * sizeof(int32_t)});
}
size_t ws_written(int T, int d_in, int d_out, int N, int r, int k, bool bf16) {
    return ws_written(ws_layout(T, d_in, d_out, N, r, k, bf16).total, T, d_in, d_out, N, r, k, bf16);
}

// and for any batch of up to T, since a program allocates for its largest.  Every form as it is for the largest batch that takes it,
// with the most (token, K split) pairs that any smaller one has: the splits fall where the tokens grow.
size_t ws_reserved(int T, int d_in, int d_out, int N, int r, int k, bool bf16) {
    size_t need = std::max(ws_written(T, d_in, d_out, N, r, k, bf16), ws_written(std::min(T, 64), d_in, d_out, N, r, k, bf16));
    if (!bf16 || T <= 64) return need;
    auto add = [&](Form f, int64_t pairs, int t, bool lora) {
        need = std::max(need, ws_carve(f, pairs, t, d_in, d_out, N, r, k, lora).total);
    };
    const int CR = prep_wcat_rows(N, r), NR = N * r;
    // few tiles: the splits change downwards inside 32 tokens only; with more than 256 tiles of 128 rows there are none
    int last = std::min(T, 256 * 128 / (ceil_div(d_out, 128) + ceil_div(CR, 128)));
    if (CR > kWcatMaxRows) last = std::min(last, expand_by_rows_tokens(d_in, d_out, r, k));
    int64_t pairs = 0;
    int takes = 0;
    for (int t = 64; t < last; t += 32)
        if (const int S = dense_midsplit_splits(t + 1, d_in, d_out, N, r, k, bf16)) {
            takes = std::min(t + 32, last);
            pairs = std::max(pairs, (int64_t)S * takes);
        }
    if (takes > 0) add(Form::kFewTiles, pairs, takes, false);
    const bool products = CR <= kWcatMaxRows;
    if (products) add(Form::kDense, gemm_dense_pairs_reserved(T, d_in, CR), T, false);
    if (!products || T > kRouteDenseMaxTokens || !gemm_dense_splitk_ok(T, d_in, CR)) add(Form::kBucketed, 0, T, false);
    if (products && r % 8 == 0) {
        const int most = NR <= 256 ? (k >= 2 ? T : std::min(T, 4096)) : std::min(T, 1024);   // see lora_dense_applies
        add(Form::kDense, gemm_dense_pairs_reserved(most, d_in, NR), most, true);
    }
    add(Form::kBucketed, 0, T, true);
    return need;
}

// Packed weights (meteora_pack_weights): the three operand layouts, each 256-byte aligned.
// `least`: what a blob may hold at the least.  Wcat once belonged only to widths that are multiples of 64, ranks that are multiples
// of 8, up to 32 adapters and 640 rows: a blob without it, kept in a file, is still taken, and a call that reads Wcat packs that itself.
struct PackLayout { size_t wsplit, apack, btrans, wcat, total, least; };

PackLayout pack_layout(int d_in, int d_out, int N, int r, bool bf16) {
    PackLayout P{};
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
    P.wsplit = take(gate_wsplit_bytes(d_in, N, bf16));
    P.apack = take(shrink_apack_bytes(d_in, N, r, bf16));
    P.btrans = take(prep_btrans_bytes(d_out, N, r, bf16));
    P.wcat = take(prep_wcat_bytes(d_in, N, r, bf16));
    P.total = off;
    P.least = d_in % 64 == 0 && r % 8 == 0 && N <= 32 && prep_wcat_rows(N, r) <= kWcatMaxRows ? P.total : P.wcat;
    return P;
}

// Where the kernels find the packed operands: in the caller's blob, or in the workspace after a prep launch.
struct PackedPtrs { void* wsplit; void* apack; void* btrans; void* wcat; };

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline bool aligned4(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 3u) == 0; }
inline bool aligned256(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 255u) == 0; }
template <typename T> T* at(void* ws, size_t off) { return reinterpret_cast<T*>(static_cast<char*>(ws) + off); }

#define METEORA_HIP(expr)                              \
    do {                                               \
        if ((expr) != hipSuccess) return METEORA_ERR_HIP; \
    } while (0)

// ---- optional per-stage timing (off by default; hipEvents recorded between the launches) ----
enum Stage { ST_PREP = 0, ST_GATE_LOGITS, ST_GATE_TOPK, ST_BUCKET, ST_SHRINK, ST_GEMM, ST_EXPAND, ST_COUNT };
constexpr int kTimingRing = 256;
struct StageTiming {
    bool on = false;
    int calls = 0;
    hipEvent_t ev[kTimingRing][ST_COUNT][2];
    bool used[kTimingRing][ST_COUNT];
} g_timing;

struct StageScope {
    int stage;
    hipStream_t st;
    int slot;
    StageScope(int stage_, hipStream_t st_, int slot_) : stage(stage_), st(st_), slot(slot_) {
        if (slot >= 0) { (void)hipEventRecord(g_timing.ev[slot][stage][0], st); }
    }
    ~StageScope() {
        if (slot >= 0) { (void)hipEventRecord(g_timing.ev[slot][stage][1], st); g_timing.used[slot][stage] = true; }
    }
};

int timing_begin_call(hipStream_t) {
    if (!g_timing.on || g_timing.calls >= kTimingRing) return -1;
    return g_timing.calls++;
}

}  // namespace

extern "C" {

int meteora_stage_count(void) { return ST_COUNT; }

const char* meteora_stage_name(int stage) {
    static const char* names[ST_COUNT] = {"prep", "gate_logits", "gate_topk", "bucket", "shrink", "gemm", "expand"};
    return (stage >= 0 && stage < ST_COUNT) ? names[stage] : "";
}

meteora_status meteora_stage_timing_enable(int on) {
    if (on && !g_timing.on) {
        for (int c = 0; c < kTimingRing; ++c)
            for (int s = 0; s < ST_COUNT; ++s) {
                METEORA_HIP(hipEventCreate(&g_timing.ev[c][s][0]));
                METEORA_HIP(hipEventCreate(&g_timing.ev[c][s][1]));
                g_timing.used[c][s] = false;
            }
        g_timing.calls = 0;
        g_timing.on = true;
    } else if (!on && g_timing.on) {
        for (int c = 0; c < kTimingRing; ++c)
            for (int s = 0; s < ST_COUNT; ++s) {
                (void)hipEventDestroy(g_timing.ev[c][s][0]);
                (void)hipEventDestroy(g_timing.ev[c][s][1]);
            }
        g_timing.on = false;
    }
    return METEORA_OK;
}

meteora_status meteora_stage_timing_read(float* ms_sum, int* launches, int* calls) {
    if (!ms_sum || !launches || !calls) return METEORA_ERR_INVALID_ARG;
    if (!g_timing.on) return METEORA_ERR_INVALID_ARG;
    for (int s = 0; s < ST_COUNT; ++s) { ms_sum[s] = 0.f; launches[s] = 0; }
    for (int c = 0; c < g_timing.calls; ++c)
        for (int s = 0; s < ST_COUNT; ++s) {
            if (!g_timing.used[c][s]) continue;
            METEORA_HIP(hipEventSynchronize(g_timing.ev[c][s][1]));
            float ms = 0.f;
            METEORA_HIP(hipEventElapsedTime(&ms, g_timing.ev[c][s][0], g_timing.ev[c][s][1]));
            ms_sum[s] += ms;
            launches[s] += 1;
            g_timing.used[c][s] = false;
        }
    *calls = g_timing.calls;
    g_timing.calls = 0;
    return METEORA_OK;
}

int meteora_version(void) { return 200; }

meteora_status meteora_init(int device) {
    int cur = 0;
    if (hipGetDevice(&cur) != hipSuccess) return METEORA_ERR_HIP;
    const bool other = device >= 0 && device != cur;
    if (other && hipSetDevice(device) != hipSuccess) return METEORA_ERR_INVALID_ARG;
    const hipError_t e = init_kernels();
    if (other) (void)hipSetDevice(cur);
    return e == hipSuccess ? METEORA_OK : METEORA_ERR_HIP;
}

const char* meteora_status_string(meteora_status s) {
    switch (s) {
        case METEORA_OK: return "ok";
        case METEORA_ERR_INVALID_ARG: return "invalid argument";
        case METEORA_ERR_UNSUPPORTED: return "unsupported shape, dtype or alignment";
        case METEORA_ERR_WORKSPACE: return "workspace missing or too small";
        case METEORA_ERR_HIP: return "HIP launch error";
        case METEORA_ERR_TOO_LARGE: return "problem larger than the fixed scratch of a call that takes no workspace";
    }
    return "unknown status";
}

size_t meteora_workspace_bytes(int T, int d_in, int d_out, int N, int r, int k, meteora_dtype dt) {
    if (!shape_ok(T, d_in, d_out, N, r, k) || !shape_supported(T, d_in, d_out, N, r, k)) return 0;
    if (dt != METEORA_F32 && dt != METEORA_BF16) return 0;
    return ws_reserved(T, d_in, d_out, N, r, k, dt == METEORA_BF16) + 256;
}

// Host-only audit of the workspace carving of meteora_linear_forward(_packed): for every region, where it starts,
// how many bytes the layout reserves and how many bytes the launch sequence that this shape selects writes there.
// The written extents are derived from the launch decisions (which path, how many K splits), not from the layout's
// own size formulas, so that a region sized for another split count than the one that writes it shows up.
int meteora_workspace_regions(int T, int d_in, int d_out, int N, int r, int k, meteora_dtype dt, int with_packed,
                              const char** names, size_t* offset, size_t* reserved, size_t* written, int max_regions) {
    if (!shape_ok(T, d_in, d_out, N, r, k) || !shape_supported(T, d_in, d_out, N, r, k)) return -1;
    if (dt != METEORA_F32 && dt != METEORA_BF16) return -1;
    const bool bf16 = dt == METEORA_BF16;
    const WsLayout L = ws_layout(T, d_in, d_out, N, r, k, bf16);
    struct Region { const char* name; size_t off, written; };
    Region R[18] = {{"wsplit", L.wsplit, 0}, {"partials", L.partials, 0}, {"chunk_counts", L.chunk_counts, 0},
                    {"counts", L.counts, 0}, {"offsets", L.offsets, 0}, {"bucket_tok", L.bucket_tok, 0},
                    {"bucket_slot", L.bucket_slot, 0}, {"topk_idx", L.topk_idx, 0}, {"topk_w", L.topk_w, 0},
                    {"h32", L.h32, 0}, {"hdense", L.hdense, 0}, {"apack", L.apack, 0}, {"hpart", L.hpart, 0},
                    {"splitk", L.splitk, 0}, {"btrans", L.btrans, 0}, {"dpart", L.dpart, 0},
                    {"gpart", L.gpart, 0}, {"spart", L.spart, 0}};
    auto wr = [&](const char* name, size_t bytes) {
        for (Region& g : R)
            if (strcmp(g.name, name) == 0 && bytes > g.written) g.written = bytes;
    };
    const int NP = padded_adapters(N);
    const size_t pairs = (size_t)T * k;
    const int CR = prep_wcat_rows(N, r);
    const int S_mid = dense_midsplit_splits(T, d_in, d_out, N, r, k, bf16);
    const bool dense = S_mid > 0 || route_dense_applies(T, d_in, N, r, bf16);
    const bool decode3 = decode_fused_applies(T, d_in, d_out, N, r, k, bf16);
    wr("topk_idx", pairs * sizeof(int32_t));
    wr("topk_w", pairs * sizeof(float));
    if (!with_packed) {
        if (!dense && !decode3) { wr("wsplit", gate_wsplit_bytes(d_in, N, bf16)); wr("apack", shrink_apack_bytes(d_in, N, r, bf16)); }
        if (!decode3 && S_mid == 0) wr("btrans", prep_btrans_bytes(d_out, N, r, bf16));
        if (dense || decode3) wr("apack", prep_wcat_bytes(d_in, N, r, bf16));   // Wcat in its place
    }
    if (decode3) {
        const int S = gemm_decode_plan(d_in, &d_out, 1, CR).S;
        wr("splitk", (size_t)S * T * d_out * sizeof(float));
        wr("gpart", (size_t)S * T * CR * sizeof(float));
    } else if (dense) {
        if (S_mid > 0) {
            wr("spart", (size_t)S_mid * T * d_out * sizeof(float));
            wr("dpart", (size_t)S_mid * T * CR * sizeof(float));
        } else {
            wr("dpart", (size_t)gemm_dense_splits(T, d_in, CR) * T * CR * sizeof(float));
            wr("hdense", (size_t)T * L.ext_stride * sizeof(uint16_t));
        }
    } else if (!bf16) {
        wr("h32", !layer_f32_applies(T, d_in, d_out, N, r, k) && f32_expand_apart(d_out, r, k) ? pairs * r * sizeof(float) : 0);
    } else {
        wr("partials", (size_t)gate_kslices(d_in, bf16) * T * NP * sizeof(float));
        const bool fused = gemm_fuses_expand(bf16);
        if (fused) wr("hdense", (size_t)T * L.ext_stride * sizeof(uint16_t));
        wr("chunk_counts", (size_t)routing_chunks(T) * N * sizeof(int32_t));
        wr("counts", (size_t)N * sizeof(int32_t));
        wr("offsets", (size_t)(N + 1) * sizeof(int32_t));
        wr("bucket_tok", pairs * sizeof(int32_t));
        wr("bucket_slot", pairs * sizeof(int32_t));
        wr("hpart", shrink_hpart_bytes(T, d_in, r, k, bf16));
        if (!fused) wr("h32", pairs * r * sizeof(float));
        const int S = gemm_splitk_splits(T, d_in, d_out, bf16);
        if (fused && S > 0) wr("splitk", (size_t)(S + 1) * T * d_out * sizeof(float));
    }
    const int n = (int)(sizeof(R) / sizeof(R[0]));
    for (int i = 0; i < n && i < max_regions; ++i) {
        const size_t end = i + 1 < n ? R[i + 1].off : L.total;
        if (names) names[i] = R[i].name;
        if (offset) offset[i] = R[i].off;
        if (reserved) reserved[i] = end - R[i].off;
        if (written) written[i] = R[i].written;
    }
    return n;
}

meteora_status meteora_gate_topk(const void* x, const float* W_gate, const float* gate_bias, int T, int d_in,
                                 int N, int k, meteora_dtype dt, float inv_temperature, int32_t* topk_idx,
                                 float* topk_w, float* logits, void* ws, size_t ws_bytes,
                                 meteora_stream stream) {
    if (!x || !W_gate || !topk_idx || !topk_w) return METEORA_ERR_INVALID_ARG;
    if (!shape_ok(T, d_in, 8, N, 1, k) || !isfinite(inv_temperature)) return METEORA_ERR_INVALID_ARG;
    if (dt != METEORA_F32 && dt != METEORA_BF16) return METEORA_ERR_UNSUPPORTED;
    if (!shape_supported(T, d_in, 8, N, 1, k)) return METEORA_ERR_UNSUPPORTED;
    if (!aligned16(x) || !aligned16(W_gate) || !aligned16(topk_idx) || !aligned16(topk_w) ||
        (logits && !aligned16(logits)) || (gate_bias && !aligned4(gate_bias)))
        return METEORA_ERR_UNSUPPORTED;
    const bool bf16 = dt == METEORA_BF16;
    if (!ws || !aligned256(ws) || ws_bytes < gate_ws_bytes(T, d_in, N, bf16)) return METEORA_ERR_WORKSPACE;
    if (T == 0) return METEORA_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    float* partials = at<float>(ws, align_up(gate_wsplit_bytes(d_in, N, bf16), 256));
    if (gate_wsplit_bytes(d_in, N, bf16) > 0)
        METEORA_HIP(launch_prep(W_gate, ws, nullptr, nullptr, nullptr, nullptr, nullptr, d_in, 8, N, 1, st));
    METEORA_HIP(launch_gate_logits(x, W_gate, T, d_in, N, bf16, ws, partials, st));
    METEORA_HIP(launch_gate_topk(partials, gate_kslices(d_in, bf16), gate_bias, T, N, k, inv_temperature,
                                 topk_idx, topk_w, logits, nullptr, st));
    return METEORA_OK;
}

meteora_status meteora_bucket_tokens(const int32_t* topk_idx, int T, int k, int N, int32_t* counts,
                                     int32_t* offsets, int32_t* bucket_tok, int32_t* bucket_slot, void* ws,
                                     size_t ws_bytes, meteora_stream stream) {
    if (!topk_idx || !counts || !offsets || !bucket_tok || !bucket_slot) return METEORA_ERR_INVALID_ARG;
    if (!shape_ok(T, 8, 8, N, 1, k)) return METEORA_ERR_INVALID_ARG;
    if (!shape_supported(T, 8, 8, N, 1, k)) return METEORA_ERR_UNSUPPORTED;
    if (!aligned16(topk_idx) || !aligned4(counts) || !aligned4(offsets) || !aligned16(bucket_tok) ||
        !aligned16(bucket_slot))
        return METEORA_ERR_UNSUPPORTED;
    // only the chunk histograms live in the workspace; they sit at offset 0 for this entry point
    const size_t need = (size_t)bucket_chunks(T) * N * sizeof(int32_t);
    if (!ws || !aligned256(ws) || ws_bytes < need) return METEORA_ERR_WORKSPACE;
    if (T == 0) {
        // nothing to enqueue; counts/offsets of an empty batch are left to the caller
        return METEORA_OK;
    }
    METEORA_HIP(launch_bucket(topk_idx, T, k, N, static_cast<int32_t*>(ws), false, counts, offsets, bucket_tok,
                              bucket_slot, nullptr, 0, static_cast<hipStream_t>(stream)));
    return METEORA_OK;
}

meteora_status meteora_bucket_tokens_noalloc(const int32_t* topk_idx, int T, int k, int N, int32_t* counts,
                                             int32_t* offsets, int32_t* bucket_tok, int32_t* bucket_slot,
                                             meteora_stream stream) {
    if (!topk_idx || !counts || !offsets || !bucket_tok || !bucket_slot) return METEORA_ERR_INVALID_ARG;
    if (!shape_ok(T, 8, 8, N, 1, k)) return METEORA_ERR_INVALID_ARG;
    if (!shape_supported(T, 8, 8, N, 1, k)) return METEORA_ERR_UNSUPPORTED;
    if (T > kStaticBucketMaxTokens) return METEORA_ERR_TOO_LARGE;   // beyond the library's fixed scratch
    if (!aligned16(topk_idx) || !aligned4(counts) || !aligned4(offsets) || !aligned16(bucket_tok) ||
        !aligned16(bucket_slot))
        return METEORA_ERR_UNSUPPORTED;
    if (T == 0) return METEORA_OK;
    int32_t* chunk_counts = nullptr;   // the current device's copy of the library's scratch array
    METEORA_HIP(bucket_static_scratch(&chunk_counts));
    METEORA_HIP(launch_bucket(topk_idx, T, k, N, chunk_counts, false, counts, offsets, bucket_tok, bucket_slot, nullptr,
                              0, static_cast<hipStream_t>(stream)));
    return METEORA_OK;
}

static meteora_status check_lora_args(const void* x, const void* A, const void* B, int T, int d_in, int d_out,
                                      int N, int r, int k, float scale, meteora_dtype dt, const void* out) {
    if (!x || !A || !B || !out) return METEORA_ERR_INVALID_ARG;
    if (!shape_ok(T, d_in, d_out, N, r, k) || !isfinite(scale)) return METEORA_ERR_INVALID_ARG;
    if (dt != METEORA_F32 && dt != METEORA_BF16) return METEORA_ERR_UNSUPPORTED;
    if (!shape_supported(T, d_in, d_out, N, r, k)) return METEORA_ERR_UNSUPPORTED;
    if (!aligned16(x) || !aligned16(A) || !aligned16(B) || !aligned16(out)) return METEORA_ERR_UNSUPPORTED;
    return METEORA_OK;
}

// bucketing + shrink + (base projection if W != NULL: bf16 only) + expand on a given routing;
// shared by lora_forward (W == NULL) and linear_forward
static meteora_status run_lora(const void* x, const void* W, const void* A, const void* B, const int32_t* topk_idx,
                               const float* topk_w, int T, int d_in, int d_out, int N, int r, int k, float scale,
                               bool bf16, void* out, int accumulate, void* ws, const WsLayout& L,
                               const PackedPtrs& pk, hipStream_t st, int tslot, bool have_hist) {
    int32_t* offsets = at<int32_t>(ws, L.offsets);
    int32_t* btok = at<int32_t>(ws, L.bucket_tok);
    int32_t* bslot = at<int32_t>(ws, L.bucket_slot);
    float* h32 = at<float>(ws, L.h32);
    const bool fused = gemm_fuses_expand(bf16);
    {
        StageScope sc(ST_BUCKET, st, tslot);
        const bool clear = fused && !shrink_clears_hdense(bf16, r, T, k);
        METEORA_HIP(launch_bucket(topk_idx, T, k, N, at<int32_t>(ws, L.chunk_counts), have_hist,
                                  at<int32_t>(ws, L.counts), offsets, btok, bslot,
                                  clear ? at<void>(ws, L.hdense) : nullptr, L.ext_stride * (int)sizeof(uint16_t), st));
    }
    {
        StageScope sc(ST_SHRINK, st, tslot);
        METEORA_HIP(launch_shrink(x, A, topk_idx, topk_w, offsets, btok, bslot, T, d_in, N, r, k, scale, bf16,
                                  pk.apack, at<float>(ws, L.hpart), fused ? nullptr : h32,
                                  fused ? at<void>(ws, L.hdense) : nullptr, L.ext_stride, st));
    }
    if (fused) {
        // base projection (if W is given) and LoRA expand in one MFMA kernel, one rounding of the output
        StageScope sc(ST_GEMM, st, tslot);
        METEORA_HIP(launch_gemm(x, W, T, W ? d_in : 0, d_out, bf16, at<void>(ws, L.hdense), L.ext_stride,
                                pk.btrans, N * r, out, accumulate,
                                gemm_splitk_bytes(T, d_in, d_out, bf16) > 0 ? at<float>(ws, L.splitk) : nullptr, st,
                                topk_idx, k, r));
    } else {
        StageScope sc(ST_EXPAND, st, tslot);
        METEORA_HIP(launch_expand(h32, B, topk_idx, topk_w, T, d_out, N, r, k, scale, bf16, out,
                                  accumulate, st));
    }
    return METEORA_OK;
}

meteora_status meteora_lora_forward(const void* x, const void* A, const void* B, const int32_t* topk_idx,
                                    const float* topk_w, int T, int d_in, int d_out, int N, int r, int k,
                                    float scale, meteora_dtype dt, void* out, int accumulate, void* ws,
                                    size_t ws_bytes, meteora_stream stream) {
    if (!topk_idx || !topk_w) return METEORA_ERR_INVALID_ARG;
    if (accumulate != 0 && accumulate != 1) return METEORA_ERR_INVALID_ARG;
    meteora_status s = check_lora_args(x, A, B, T, d_in, d_out, N, r, k, scale, dt, out);
    if (s != METEORA_OK) return s;
    if (!aligned16(topk_idx) || !aligned16(topk_w)) return METEORA_ERR_UNSUPPORTED;
    const bool bf16 = dt == METEORA_BF16;
    const WsLayout L = lora_layout(T, d_in, d_out, N, r, k, bf16);
    if (!ws || !aligned256(ws) || ws_bytes < ws_written(T, d_in, d_out, N, r, k, bf16)) return METEORA_ERR_WORKSPACE;
    if (T == 0) return METEORA_OK;
    if (lora_dense_applies(T, d_in, N, r, k, bf16)) {
        // x * A_i of every adapter in one MFMA launch, then the selected columns as the expand operand: three short
        // launches fewer than bucket lists and grouped shrink, and x is read in order
        hipStream_t st = static_cast<hipStream_t>(stream);
        const int tslot = timing_begin_call(st);
        float* part = at<float>(ws, L.dpart);
        METEORA_HIP(launch_prep(nullptr, nullptr, A, nullptr, B, at<void>(ws, L.btrans), at<void>(ws, L.wcat), d_in, d_out,
                                N, r, st));
        {
            StageScope sc(ST_SHRINK, st, tslot);
            METEORA_HIP(launch_gemm_dense_splitk(x, at<void>(ws, L.wcat), T, d_in, N * r, part, st));
            METEORA_HIP(launch_dense_expand_operand(part, gemm_dense_splits(T, d_in, N * r), topk_idx, topk_w, T, N, r, k,
                                                    scale, at<void>(ws, L.hdense), L.ext_stride, st));
        }
        StageScope sc(ST_GEMM, st, tslot);
        METEORA_HIP(launch_gemm(x, nullptr, T, 0, d_out, bf16, at<void>(ws, L.hdense), L.ext_stride, at<void>(ws, L.btrans),
                                N * r, out, accumulate, nullptr, st, topk_idx, k, r));
        return METEORA_OK;
    }
    {
        const bool pa = shrink_apack_bytes(d_in, N, r, bf16) > 0, pb = prep_btrans_bytes(d_out, N, r, bf16) > 0;
        METEORA_HIP(launch_prep(nullptr, nullptr, pa ? A : nullptr, pa ? at<void>(ws, L.apack) : nullptr,
                                pb ? B : nullptr, pb ? at<void>(ws, L.btrans) : nullptr, nullptr, d_in, d_out, N, r,
                                static_cast<hipStream_t>(stream)));
    }
    const PackedPtrs pk{nullptr, at<void>(ws, L.apack), at<void>(ws, L.btrans), nullptr};
    return run_lora(x, nullptr, A, B, topk_idx, topk_w, T, d_in, d_out, N, r, k, scale, bf16, out, accumulate, ws, L,
                    pk, static_cast<hipStream_t>(stream), timing_begin_call(static_cast<hipStream_t>(stream)), false);
}

meteora_status meteora_base_gemm(const void* x, const void* W, int T, int d_in, int d_out, meteora_dtype dt,
                                 void* out, meteora_stream stream) {
    if (!x || !W || !out) return METEORA_ERR_INVALID_ARG;
    if (!shape_ok(T, d_in, d_out, 1, 1, 1)) return METEORA_ERR_INVALID_ARG;
    if (dt != METEORA_F32 && dt != METEORA_BF16) return METEORA_ERR_UNSUPPORTED;
    if (!shape_supported(T, d_in, d_out, 1, 1, 1)) return METEORA_ERR_UNSUPPORTED;
    if (!aligned16(x) || !aligned16(W) || !aligned16(out)) return METEORA_ERR_UNSUPPORTED;
    if (T == 0) return METEORA_OK;
    METEORA_HIP(launch_gemm(x, W, T, d_in, d_out, dt == METEORA_BF16, nullptr, 0, nullptr, 0, out, 0, nullptr,
                            static_cast<hipStream_t>(stream)));
    return METEORA_OK;
}

size_t meteora_packed_bytes(int d_in, int d_out, int N, int r, meteora_dtype dt) {
    if (!shape_ok(0, d_in, d_out, N, r, 1) || !shape_supported(0, d_in, d_out, N, r, 1)) return 0;
    if (dt != METEORA_F32 && dt != METEORA_BF16) return 0;
    return pack_layout(d_in, d_out, N, r, dt == METEORA_BF16).total;
}

meteora_status meteora_pack_weights(const float* W_gate, const void* A, const void* B, int d_in, int d_out, int N,
                                    int r, meteora_dtype dt, void* packed, size_t packed_bytes,
                                    meteora_stream stream) {
    if (!W_gate || !A || !B) return METEORA_ERR_INVALID_ARG;
    if (!shape_ok(0, d_in, d_out, N, r, 1)) return METEORA_ERR_INVALID_ARG;
    if (dt != METEORA_F32 && dt != METEORA_BF16) return METEORA_ERR_UNSUPPORTED;
    if (!shape_supported(0, d_in, d_out, N, r, 1)) return METEORA_ERR_UNSUPPORTED;
    if (!aligned16(W_gate) || !aligned16(A) || !aligned16(B)) return METEORA_ERR_UNSUPPORTED;
    const bool bf16 = dt == METEORA_BF16;
    const PackLayout P = pack_layout(d_in, d_out, N, r, bf16);
    if (P.total == 0) return METEORA_OK;   // this dtype reads the tensors as they are
    if (!packed || !aligned256(packed) || packed_bytes < P.total) return METEORA_ERR_WORKSPACE;
    const bool pw = gate_wsplit_bytes(d_in, N, bf16) > 0, pa = shrink_apack_bytes(d_in, N, r, bf16) > 0;
    const bool pb = prep_btrans_bytes(d_out, N, r, bf16) > 0, pc = prep_wcat_bytes(d_in, N, r, bf16) > 0;
    METEORA_HIP(launch_prep(W_gate, pw ? at<void>(packed, P.wsplit) : nullptr, A,
                            pa ? at<void>(packed, P.apack) : nullptr, pb ? B : nullptr,
                            pb ? at<void>(packed, P.btrans) : nullptr, pc ? at<void>(packed, P.wcat) : nullptr, d_in,
                            d_out, N, r, static_cast<hipStream_t>(stream)));
    return METEORA_OK;
}

meteora_status meteora_linear_forward_packed(const void* x, const void* W, const float* W_gate,
                                             const float* gate_bias, const void* A, const void* B,
                                             const void* packed, size_t packed_bytes, int T, int d_in, int d_out,
                                             int N, int r, int k, float scale, float inv_temperature,
                                             meteora_dtype dt, void* out, int32_t* topk_idx_out, float* topk_w_out,
                                             void* ws, size_t ws_bytes, meteora_stream stream) {
    if (!W || !W_gate || !isfinite(inv_temperature)) return METEORA_ERR_INVALID_ARG;
    meteora_status s = check_lora_args(x, A, B, T, d_in, d_out, N, r, k, scale, dt, out);
    if (s != METEORA_OK) return s;
    if (!aligned16(W) || !aligned16(W_gate) || (gate_bias && !aligned4(gate_bias)) ||
        (topk_idx_out && !aligned16(topk_idx_out)) || (topk_w_out && !aligned16(topk_w_out)))
        return METEORA_ERR_UNSUPPORTED;
    const bool bf16 = dt == METEORA_BF16;
    const LayerForm form = layer_form(T, d_in, d_out, N, r, k, bf16);
    const WsLayout L = ws_carve(form.form, (int64_t)form.S * T, T, d_in, d_out, N, r, k, false);
    if (!ws || !aligned256(ws) || ws_bytes < ws_written(L.total, T, d_in, d_out, N, r, k, bf16)) return METEORA_ERR_WORKSPACE;
    const PackLayout P = pack_layout(d_in, d_out, N, r, bf16);
    if (packed != nullptr && P.total > 0 && (!aligned256(packed) || packed_bytes < P.least)) return METEORA_ERR_WORKSPACE;
    const bool use_packed = packed != nullptr && P.total > 0, has_wcat = use_packed && packed_bytes >= P.total;
    if (T == 0) return METEORA_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    int32_t* idx = topk_idx_out ? topk_idx_out : at<int32_t>(ws, L.topk_idx);
    float* w = topk_w_out ? topk_w_out : at<float>(ws, L.topk_w);
    float* partials = at<float>(ws, L.partials);
    const int tslot = timing_begin_call(st);
    // mid-sized batch: gate logits and the shrink of every adapter in one MFMA launch, selection afterwards
    const int S_mid = form.form == Form::kFewTiles ? form.S : 0;
    const bool dense = S_mid > 0 || form.form == Form::kDense, decode3 = form.form == Form::kDecode;
    PackedPtrs pk{at<void>(ws, L.wsplit), at<void>(ws, L.apack), at<void>(ws, L.btrans), at<void>(ws, L.wcat)};
    if (use_packed) {
        void* blob = const_cast<void*>(packed);   // read only from here on
        pk = PackedPtrs{at<void>(blob, P.wsplit), at<void>(blob, P.apack), at<void>(blob, P.btrans),
                        has_wcat ? at<void>(blob, P.wcat) : pk.wcat};
    }
    // only the operands that this batch size reads and the blob does not hold are packed (a few hundred tokens and decode read B
    // as it is)
    const bool pw = !use_packed && !dense && !decode3 && gate_wsplit_bytes(d_in, N, bf16) > 0;
    const bool pa = !use_packed && !dense && !decode3 && shrink_apack_bytes(d_in, N, r, bf16) > 0;
    const bool pb = !use_packed && !decode3 && S_mid == 0 && prep_btrans_bytes(d_out, N, r, bf16) > 0;
    const bool pc = !has_wcat && (dense || decode3);
    if (!use_packed || pc) {
        StageScope sc(ST_PREP, st, tslot);
        METEORA_HIP(launch_prep(W_gate, pw ? pk.wsplit : nullptr, A, pa ? pk.apack : nullptr, pb ? B : nullptr,
                                pb ? pk.btrans : nullptr, pc ? pk.wcat : nullptr, d_in, d_out, N, r, st));
    }
    if (decode3) {
        // decode-sized batch: the launch that streams W also computes the gate logits; then top-k, softmax and the
        // shrink of the selected adapters token by token; then the split-K reduction, which adds the expand
        const DecodeMember mem{W, pk.wcat, gate_bias, B, d_out, at<float>(ws, L.splitk), at<float>(ws, L.gpart), idx, w, out};
        const int gate_rows = prep_wcat_rows(N, r);   // the gate terms and every adapter's shrink columns
        const SplitPlan plan = gemm_decode_plan(d_in, &d_out, 1, gate_rows);
        {
            StageScope sc(ST_GEMM, st, tslot);
            METEORA_HIP(launch_gemm_decode_main(x, &mem, 1, gate_rows, plan, T, d_in, st));
        }
        // top-k, softmax, then the split-K reduction with the expand from the selected adapters' shrink tiles: one launch
        StageScope sc(ST_SHRINK, st, tslot);
        METEORA_HIP(launch_decode_tail_group(&mem, 1, plan, T, N, r, k, gate_rows, inv_temperature, scale, st));
        return METEORA_OK;
    }
    if (dense) {
        float* dpart = at<float>(ws, L.dpart);
        if (S_mid > 0) {
            // few output tiles: x * W^T and x * Wcat^T as fp32 K-split tiles of one launch, then selection, reduction and expand
            // in another, as for decode
            const DecodeMember mem{W, nullptr, gate_bias, B, d_out, at<float>(ws, L.spart), dpart, idx, w, out};
            {
                StageScope sc(ST_GEMM, st, tslot);
                const DenseOperand two[2] = {{W, d_out, mem.partial}, {pk.wcat, prep_wcat_rows(N, r), dpart}};
                METEORA_HIP(launch_gemm_dense_splitk_multi(x, two, 2, S_mid, T, d_in, st));
            }
            StageScope sc(ST_SHRINK, st, tslot);
            METEORA_HIP(launch_decode_tail_group(&mem, 1, SplitPlan{S_mid, 0, 0}, T, N, r, k, prep_wcat_rows(N, r), inv_temperature,
                                                 scale, st));
            return METEORA_OK;
        }
        {
            StageScope sc(ST_GATE_LOGITS, st, tslot);
            METEORA_HIP(launch_route_dense_products(x, pk.wcat, T, d_in, N, r, dpart, st));
        }
        {
            StageScope sc(ST_GATE_TOPK, st, tslot);
            METEORA_HIP(launch_route_dense_select(dpart, gate_bias, T, d_in, N, r, k, inv_temperature, scale, idx, w,
                                                  at<void>(ws, L.hdense), L.ext_stride, st));
        }
        StageScope sc(ST_GEMM, st, tslot);
        METEORA_HIP(launch_gemm(x, W, T, d_in, d_out, bf16, at<void>(ws, L.hdense), L.ext_stride, pk.btrans, N * r,
                                out, 0, nullptr, st, idx, k, r));
        return METEORA_OK;
    }
    if (!bf16) {
        if (layer_f32_applies(T, d_in, d_out, N, r, k)) {
            StageScope sc(ST_GEMM, st, tslot);
            METEORA_HIP(launch_layer_f32((const float*)x, (const float*)W, W_gate, gate_bias, (const float*)A, (const float*)B,
                                         T, d_in, d_out, N, r, k, inv_temperature, scale, idx, w, (float*)out, st));
            return METEORA_OK;
        }
        {
            StageScope sc(ST_GEMM, st, tslot);
            METEORA_HIP(launch_gemm(x, W, T, d_in, d_out, false, nullptr, 0, nullptr, 0, out, 0, nullptr, st));
        }
        StageScope sc(ST_EXPAND, st, tslot);
        METEORA_HIP(launch_route_lora_f32((const float*)x, W_gate, gate_bias, (const float*)A, (const float*)B, T, d_in,
                                          d_out, N, r, k, inv_temperature, scale, idx, w, (float*)out,
                                          at<float>(ws, L.h32), st));
        return METEORA_OK;
    }
    {
        StageScope sc(ST_GATE_LOGITS, st, tslot);
        METEORA_HIP(launch_gate_logits(x, W_gate, T, d_in, N, bf16, pk.wsplit, partials, st));
    }
    {
        StageScope sc(ST_GATE_TOPK, st, tslot);
        METEORA_HIP(launch_gate_topk(partials, gate_kslices(d_in, bf16), gate_bias, T, N, k, inv_temperature, idx, w,
                                     nullptr, at<int32_t>(ws, L.chunk_counts), st));
    }
    return run_lora(x, W, A, B, idx, w, T, d_in, d_out, N, r, k, scale, bf16, out, 0, ws, L, pk, st, tslot, true);
}

}  // extern "C"

// ---- a group of layers that share x ----------------------------------------------------------------------------
namespace {

// Fused form: decode-sized batch, every member with packed weights.
bool group_fused(const int* d_out, const bool* packed, int G, int T, int d_in, int N, int r, int k, bool bf16) {
    if (G < 2 || G > kMaxDecodeGroup) return false;
    for (int g = 0; g < G; ++g)
        if (!packed[g] || !decode_fused_applies(T, d_in, d_out[g], N, r, k, bf16)) return false;
    return true;
}

// Second fused form: a few hundred tokens, every member with packed weights, few output tiles in all: the projections and
// routing products of all members as K-split tiles of one launch, one launch with the selections and expands.  Returns the
// number of K splits, 0 = not this form.
int group_mid_splits(const int* d_out, const bool* packed, int G, int T, int d_in, int N, int r, int k, bool bf16) {
    const int cat_rows = prep_wcat_rows(N, r);
    if (G < 2 || G > kMaxDecodeGroup || !bf16 || T <= 64 || !gemm_multi_ok(T, d_in, cat_rows)) return 0;
    int64_t tiles = 0;
    for (int g = 0; g < G; ++g) {
        if (!packed[g] || d_out[g] % 8 != 0 || !gemm_multi_ok(T, d_in, d_out[g])) return 0;
        if (cat_rows > kWcatMaxRows && !expand_by_rows_applies(T, d_in, d_out[g], r, k)) return 0;
        tiles += (int64_t)ceil_div(T, 128) * (ceil_div(d_out[g], 128) + ceil_div(cat_rows, 128));
    }
    if (tiles > 320) return 0;   // beyond: member by member (each on the path its own size selects)
    const int nk = ceil_div(d_in, 64);
    int S = (int)((384 + tiles / 2) / tiles);
    if (S > nk / 4) S = nk / 4;
    if (S > 8) S = 8;
    int col_tiles = 0;
    int64_t rows = 0;
    for (int g = 0; g < G; ++g) {
        col_tiles += ceil_div(d_out[g], 128) + ceil_div(cat_rows, 128);
        rows += d_out[g] + cat_rows;
    }
    // With many rows of B per token the tail does not make up for a second round of tiles as long as all of K: 64 adapters, 4096 -> 14336
    // twice (260 column tiles), in two launches and member by member, top-8 of rank 32 65 tokens 175 and 169, 80 187 and 173; top-4
    // 80 136 and 172, 128 159 and 188; top-2 of rank 64 128 171 and 230.
    if (cat_rows > kWcatMaxRows && k * r > 128 && col_tiles > 256) return 0;
    S = gemm_multi_splits(T, col_tiles, S, nk, rows);
    return S < 1 ? 1 : S;
}

struct GroupLayout { size_t partial[kMaxDecodeGroup], gpart[kMaxDecodeGroup], idx[kMaxDecodeGroup], w[kMaxDecodeGroup], total; int S; };

// gate_rows: columns of gpart per member, every row of Wcat
GroupLayout group_layout(const int* d_out, int G, int T, int d_in, int N, int r, int k, int S, int gate_rows) {
    GroupLayout L{};
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
    L.S = S;
    for (int g = 0; g < G; ++g) {
        L.partial[g] = take((size_t)L.S * T * d_out[g] * sizeof(float));
        L.gpart[g] = take((size_t)L.S * T * gate_rows * sizeof(float));
        L.idx[g] = take((size_t)T * k * sizeof(int32_t));
        L.w[g] = take((size_t)T * k * sizeof(float));
    }
    L.total = off;
    return L;
}

}  // namespace

extern "C" size_t meteora_group_workspace_bytes(const int* d_out, int G, int T, int d_in, int N, int r, int k,
                                                meteora_dtype dt) {
    if (!d_out || G < 1 || G > 64) return 0;
    if (dt != METEORA_F32 && dt != METEORA_BF16) return 0;
    const bool bf16 = dt == METEORA_BF16;
    size_t need = 0;
    for (int g = 0; g < G; ++g) {
        const size_t one = meteora_workspace_bytes(T, d_in, d_out[g], N, r, k, dt);
        if (one == 0) return 0;
        need = one > need ? one : need;
    }
    if (bf16 && G >= 2 && G <= kMaxDecodeGroup) {   // sized as if packed, the larger need, and for every smaller batch
        const int gate_rows = prep_wcat_rows(N, r), Td = T < 64 ? T : 64;
        auto fused = [&](int t, int S) {
            const size_t f = group_layout(d_out, G, t, d_in, N, r, k, S, gate_rows).total + 256;
            need = f > need ? f : need;
        };
        const bool all_packed[kMaxDecodeGroup] = {true, true, true, true};
        if (group_fused(d_out, all_packed, G, Td, d_in, N, r, k, bf16)) fused(Td, gemm_decode_plan(d_in, d_out, G, gate_rows).S);
        // at most 320 tiles of 128 rows; the splits change downwards inside 32 tokens only
        int last = std::min(T, 128 * 320 / (2 * G));
        for (int g = 0; g < G && gate_rows > kWcatMaxRows; ++g) last = std::min(last, expand_by_rows_tokens(d_in, d_out[g], r, k));
        for (int t = 64; t < last; t += 32) {
            const int S = group_mid_splits(d_out, all_packed, G, t + 1, d_in, N, r, k, bf16);
            if (S == 0) break;
            fused(std::min(t + 32, last), S);
        }
    }
    return need;
}

extern "C" meteora_status meteora_linear_forward_group(const void* x, const meteora_group_member* members, int G, int T,
                                                       int d_in, int N, int r, int k, float scale,
                                                       float inv_temperature, meteora_dtype dt, void* ws,
                                                       size_t ws_bytes, meteora_stream stream) {
    if (!members || G < 1 || G > 64 || !isfinite(inv_temperature)) return METEORA_ERR_INVALID_ARG;
    if (dt != METEORA_F32 && dt != METEORA_BF16) return METEORA_ERR_UNSUPPORTED;
    const bool bf16 = dt == METEORA_BF16;
    int d_outs[64];
    for (int g = 0; g < G; ++g) {
        const meteora_group_member& m = members[g];
        if (!m.W || !m.W_gate) return METEORA_ERR_INVALID_ARG;
        const meteora_status s = check_lora_args(x, m.A, m.B, T, d_in, m.d_out, N, r, k, scale, dt, m.out);
        if (s != METEORA_OK) return s;
        if (!aligned16(m.W) || !aligned16(m.W_gate) || (m.gate_bias && !aligned4(m.gate_bias)) ||
            (m.topk_idx_out && !aligned16(m.topk_idx_out)) || (m.topk_w_out && !aligned16(m.topk_w_out)))
            return METEORA_ERR_UNSUPPORTED;
        if (m.packed && (!aligned256(m.packed) ||
                         m.packed_bytes < pack_layout(d_in, m.d_out, N, r, bf16).least))
            return METEORA_ERR_WORKSPACE;
        d_outs[g] = m.d_out;
    }
    bool is_packed[64];
    for (int g = 0; g < G; ++g)
        is_packed[g] = members[g].packed != nullptr &&
                       members[g].packed_bytes >= pack_layout(d_in, members[g].d_out, N, r, bf16).total;
    const int gate_rows = prep_wcat_rows(N, r);
    const int S_mid = T > 0 ? group_mid_splits(d_outs, is_packed, G, T, d_in, N, r, k, bf16) : 0;
    const bool decode = S_mid == 0 && T > 0 && group_fused(d_outs, is_packed, G, T, d_in, N, r, k, bf16);
    const SplitPlan plan = decode ? gemm_decode_plan(d_in, d_outs, G, gate_rows) : SplitPlan{S_mid, 0, 0};
    const GroupLayout L = S_mid > 0 || decode ? group_layout(d_outs, G, T, d_in, N, r, k, plan.S, gate_rows) : GroupLayout{};
    size_t need = L.total;
    for (int g = 0; g < G && !decode && S_mid == 0; ++g) need = std::max(need, ws_written(T, d_in, d_outs[g], N, r, k, bf16));
    if (!ws || !aligned256(ws) || ws_bytes < need) return METEORA_ERR_WORKSPACE;
    if (T == 0) return METEORA_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (S_mid > 0) {
        DecodeMember mem[kMaxDecodeGroup];
        DenseOperand ops[2 * kMaxDecodeGroup];
        for (int g = 0; g < G; ++g) {
            const meteora_group_member& m = members[g];
            const PackLayout P = pack_layout(d_in, m.d_out, N, r, bf16);
            mem[g] = DecodeMember{m.W, at<void>(const_cast<void*>(m.packed), P.wcat), m.gate_bias, m.B, m.d_out,
                                  at<float>(ws, L.partial[g]), at<float>(ws, L.gpart[g]),
                                  m.topk_idx_out ? m.topk_idx_out : at<int32_t>(ws, L.idx[g]),
                                  m.topk_w_out ? m.topk_w_out : at<float>(ws, L.w[g]), m.out};
            ops[2 * g] = {mem[g].W, m.d_out, mem[g].partial};
            ops[2 * g + 1] = {mem[g].wg3, gate_rows, mem[g].gpartial};
        }
        const int tslot = timing_begin_call(st);
        {
            StageScope sc(ST_GEMM, st, tslot);
            METEORA_HIP(launch_gemm_dense_splitk_multi(x, ops, 2 * G, S_mid, T, d_in, st));
        }
        StageScope sc(ST_SHRINK, st, tslot);
        METEORA_HIP(launch_decode_tail_group(mem, G, plan, T, N, r, k, gate_rows, inv_temperature, scale, st));
        return METEORA_OK;
    }
    if (!decode) {
        // the same result one layer after the other (they share the workspace, which the stream order allows)
        for (int g = 0; g < G; ++g) {
            const meteora_group_member& m = members[g];
            const meteora_status s = meteora_linear_forward_packed(
                x, m.W, m.W_gate, m.gate_bias, m.A, m.B, m.packed, m.packed_bytes, T, d_in, m.d_out, N, r, k, scale,
                inv_temperature, dt, m.out, m.topk_idx_out, m.topk_w_out, ws, ws_bytes, stream);
            if (s != METEORA_OK) return s;
        }
        return METEORA_OK;
    }
    DecodeMember mem[kMaxDecodeGroup];
    for (int g = 0; g < G; ++g) {
        const meteora_group_member& m = members[g];
        const PackLayout P = pack_layout(d_in, m.d_out, N, r, bf16);
        mem[g] = DecodeMember{m.W, at<void>(const_cast<void*>(m.packed), P.wcat), m.gate_bias, m.B, m.d_out,
                              at<float>(ws, L.partial[g]), at<float>(ws, L.gpart[g]),
                              m.topk_idx_out ? m.topk_idx_out : at<int32_t>(ws, L.idx[g]),
                              m.topk_w_out ? m.topk_w_out : at<float>(ws, L.w[g]), m.out};
    }
    const int tslot = timing_begin_call(st);
    {
        StageScope sc(ST_GEMM, st, tslot);
        METEORA_HIP(launch_gemm_decode_main(x, mem, G, gate_rows, plan, T, d_in, st));
    }
    StageScope sc(ST_SHRINK, st, tslot);
    METEORA_HIP(launch_decode_tail_group(mem, G, plan, T, N, r, k, gate_rows, inv_temperature, scale, st));
    return METEORA_OK;
}

extern "C" {

meteora_status meteora_linear_forward(const void* x, const void* W, const float* W_gate, const float* gate_bias,
                                      const void* A, const void* B, int T, int d_in, int d_out, int N, int r,
                                      int k, float scale, float inv_temperature, meteora_dtype dt, void* out,
                                      int32_t* topk_idx_out, float* topk_w_out, void* ws, size_t ws_bytes,
                                      meteora_stream stream) {
    return meteora_linear_forward_packed(x, W, W_gate, gate_bias, A, B, nullptr, 0, T, d_in, d_out, N, r, k, scale,
                                         inv_temperature, dt, out, topk_idx_out, topk_w_out, ws, ws_bytes, stream);
}

size_t meteora_gate_backward_workspace_bytes(int T, int d_in, int d_out, int N, int r, int k, meteora_dtype dt) {
    if (!shape_ok(T, d_in, d_out, N, r, k) || !shape_supported(T, d_in, d_out, N, r, k) || T < 1) return 0;
    if (!gate_backward_applies(T, d_in, d_out, N, r, dt == METEORA_BF16)) return 0;
    return gate_backward_layout(T, d_in, d_out, N, r, true, true).total;
}

meteora_status meteora_gate_backward(const void* x, const void* dy, const float* gate_bias, const void* B,
                                     const void* packed, size_t packed_bytes, const int32_t* topk_idx,
                                     const float* topk_w, const int32_t* labels, float beta, int T, int d_in,
                                     int d_out, int N, int r, int k, float scale, meteora_dtype dt, float* dW_gate,
                                     float* dbias, float* d_logits, const void* A, const float* W_gate,
                                     const void* W_t, void* dx, const void* forward_ws, size_t forward_ws_bytes,
                                     void* ws, size_t ws_bytes, meteora_stream stream) {
    if (!x || !dy || !B || !packed || !dW_gate || (topk_idx == nullptr) != (topk_w == nullptr))
        return METEORA_ERR_INVALID_ARG;
    if (dx != nullptr && (!A || !W_gate || !W_t)) return METEORA_ERR_INVALID_ARG;
    if (!shape_ok(T, d_in, d_out, N, r, k) || !isfinite(scale) || !isfinite(beta)) return METEORA_ERR_INVALID_ARG;
    if (dt != METEORA_BF16 && dt != METEORA_F32) return METEORA_ERR_INVALID_ARG;
    if (T == 0) return METEORA_OK;
    const bool bf16 = dt == METEORA_BF16;
    if (!shape_supported(T, d_in, d_out, N, r, k) || !gate_backward_applies(T, d_in, d_out, N, r, bf16))
        return METEORA_ERR_UNSUPPORTED;
    if (!aligned16(x) || !aligned16(dy) || !aligned16(B) || !aligned16(dW_gate) || (gate_bias && !aligned4(gate_bias)) ||
        (dbias && !aligned4(dbias)) || (d_logits && !aligned4(d_logits)) || (labels && !aligned4(labels)) ||
        (topk_idx && (!aligned4(topk_idx) || !aligned4(topk_w))) ||
        (dx && (!aligned16(dx) || !aligned16(A) || !aligned16(W_gate) || !aligned16(W_t))))
        return METEORA_ERR_UNSUPPORTED;
    const PackLayout P = pack_layout(d_in, d_out, N, r, bf16);
    if (!aligned256(packed) || packed_bytes < P.total) return METEORA_ERR_WORKSPACE;
    const GateBackwardLayout L = gate_backward_layout(T, d_in, d_out, N, r, dx != nullptr, false);
    if (!ws || !aligned256(ws) || ws_bytes < L.total) return METEORA_ERR_WORKSPACE;
    const void* wcat = static_cast<const char*>(packed) + P.wcat;
    // the forward call of a mid-sized batch leaves x * Wcat^T in its workspace: take it instead of computing it again
    const float* part_x = nullptr;
    int part_x_splits = 0;
    if (forward_ws != nullptr && route_dense_applies(T, d_in, N, r, bf16)) {
        const WsLayout F = ws_layout(T, d_in, d_out, N, r, k, bf16);
        if (!aligned256(forward_ws) || forward_ws_bytes < F.total) return METEORA_ERR_WORKSPACE;
        part_x = reinterpret_cast<const float*>(static_cast<const char*>(forward_ws) + F.dpart);
        part_x_splits = dense_midsplit_splits(T, d_in, d_out, N, r, k, bf16);   // 0: the products launch's own split count
    }
    const hipError_t e = launch_gate_backward(x, dy, wcat, B, gate_bias, topk_idx, topk_w, labels, beta, T, d_in, d_out,
                                              N, r, k, scale, dW_gate, dbias, d_logits, part_x, part_x_splits, A, W_gate, W_t, dx,
                                              static_cast<char*>(ws),
                                              static_cast<hipStream_t>(stream));
    return e == hipSuccess ? METEORA_OK : METEORA_ERR_HIP;
}

}  // extern "C"
