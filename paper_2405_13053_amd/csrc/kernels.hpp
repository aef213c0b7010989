// Host-side launchers of the gfx950 kernels.  Every launcher only enqueues work
// on `stream`; none allocates or synchronises.  Shapes have been validated by
// the C-ABI layer before a launcher is called.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace meteora {

// ---- process state (runtime.hip): raise a kernel's dynamic-LDS limit once per device (thread-safe), and the
// set-up of every kernel of the library ahead of its first launch, for the current device (meteora_init)
hipError_t ensure_lds_limit(const void* kernel, int bytes);
hipError_t init_kernels();
hipError_t gemm_init_kernels();
hipError_t gemm_decode_init_kernels();
hipError_t gate_init_kernels();
hipError_t shrink_init_kernels();
hipError_t gate_bwd_init_kernels();
hipError_t bucket_init_scratch();

// ---- weight repacking, one launch: W_gate -> split bf16 fragments (bf16 gate), A -> MFMA fragments,
// stacked B -> its transpose Bt[d_out, N*r rounded up to 64] (zero-padded) for the GEMM's K-extension.
// Any pair (W_gate, wsplit) / (A, apack) / (B, btrans) may be NULL to skip it; sizes are gate_wsplit_bytes,
// shrink_apack_bytes and prep_btrans_bytes (0 = that operand is not packed for this dtype/rank: pass NULL).
// wcat (optional, needs A): Wcat[prep_wcat_rows, d_in] bf16 for the dense routing path,
// rows = hi | mid | lo terms of the gate columns (padded_adapters(N) rows each), then column q of A_a as row
// a*wcat_rank(r)+q (rows q >= r zero).
// Without W_gate: the rows of A alone.
size_t prep_btrans_bytes(int d_out, int N, int r, bool bf16);
int prep_wcat_rows(int N, int r);
size_t prep_wcat_bytes(int d_in, int N, int r, bool bf16);
hipError_t launch_prep(const float* W_gate, void* wsplit, const void* A, void* apack, const void* B, void* btrans,
                       void* wcat, int d_in, int d_out, int N, int r, hipStream_t stream);

// ---- gate (Sec. 3.1: G(x), I(x), Eq. 3) ------------------------------------------------
// Number of K-slices the logit kernel splits d_in into (partials[KS][T][NP]).
int gate_kslices(int d_in, bool bf16);
// bytes of the split-bf16 copy of W_gate the MFMA logit kernel reads (0 for fp32 inputs)
size_t gate_wsplit_bytes(int d_in, int N, bool bf16);
hipError_t launch_gate_logits(const void* x, const float* W_gate, int T, int d_in, int N, bool bf16,
                              void* wsplit, float* partials, hipStream_t stream);
// chunk_counts (optional): per-chunk adapter histograms [routing_chunks(T)][N] for launch_bucket_scatter
hipError_t launch_gate_topk(const float* partials, int KS, const float* bias, int T, int N, int k,
                            float inv_temperature, int32_t* topk_idx, float* topk_w, float* logits,
                            int32_t* chunk_counts, hipStream_t stream);

// ---- batches of more than 64 tokens (bf16, at most 640 rows of Wcat): one MFMA launch
// computes the split-bf16 gate logits and x * A_i of every adapter as fp32 K-split partials
// part[splits][T][prep_wcat_rows], then a launch of independent wavefronts adds the splits, ranks (Sec. 3.1, Eq. 3)
// and writes topk_idx, topk_w and every column of the tokens' rows of hdense.  Replaces launch_gate_logits,
// launch_gate_topk, launch_bucket and launch_shrink for the whole-layer call.  Up to kRouteDenseMaxTokens always;
// beyond, with up to 320 rows of Wcat always, with more where the products' tiles fill the CUs
// (route_dense_applies).
constexpr int kRouteDenseMaxTokens = 8192, kWcatMaxRows = 640;
bool route_dense_applies(int T, int d_in, int N, int r, bool bf16);
bool lora_dense_applies(int T, int d_in, int N, int r, int k, bool bf16);   // lora_forward, whose routing is given
hipError_t launch_route_dense_products(const void* x, const void* wcat, int T, int d_in, int N, int r, float* part,
                                       hipStream_t stream);
// the expand operand for a routing that is given (r % 8 == 0): part[S][T][N*r] = x * A_i of every adapter
hipError_t launch_dense_expand_operand(const float* part, int S, const int32_t* topk_idx, const float* topk_w, int T,
                                       int N, int r, int k, float scale, void* hdense, int ext_stride,
                                       hipStream_t stream);
hipError_t launch_route_dense_select(const float* part, const float* bias, int T, int d_in, int N, int r, int k,
                                     float inv_temperature, float scale, int32_t* topk_idx, float* topk_w,
                                     void* hdense, int ext_stride, hipStream_t stream);
// the GEMM behind launch_route_dense_products: partial[split][T][rows] = x * Wcat^T over the split's K range
bool gemm_dense_splitk_ok(int T, int d_in, int rows);
bool gemm_multi_ok(int T, int d_in, int rows);
int gemm_dense_splits(int T, int d_in, int rows);
int gemm_multi_fit(int T, int d_in, int rows);
// few-tile split-K launches over several matrices (col_tiles: the 128-column tiles of all of them, rows: their rows): S
// capped to one workgroup per CU, or for few tokens to two, and of what that leaves the number that costs the least
int gemm_multi_splits(int T, int col_tiles, int S, int nk, int64_t rows);
// What a workspace reserves: the splits come and go with the token count, and a workspace for the largest batch holds the smaller
// ones.  The most tokens times splits that the products of any batch of up to T tokens have.
int64_t gemm_dense_pairs_reserved(int T, int d_in, int rows);
hipError_t launch_gemm_dense_splitk(const void* x, const void* Wcat, int T, int d_in, int rows, float* partial,
                                    hipStream_t stream);

// the same for several matrices in one launch (tiles of 128 columns and 96 to 256 rows), all with S splits (at most 8
// matrices)
struct DenseOperand { const void* W; int rows; float* partial; };
hipError_t launch_gemm_dense_splitk_multi(const void* x, const DenseOperand* ops, int n_ops, int S, int T, int d_in,
                                          hipStream_t stream);

// ---- bucketing (Sec. 3.3: per-adapter token sets as index lists) --------------------------
constexpr int kBucketChunkTokens = 64;   // tokens (k pairs each) whose pairs one workgroup histograms and scatters
// The chunks of the histograms that the ranking kernel leaves for the scatter pass.  With 64 tokens a ranking of 2000 tokens
// runs on 32 CUs; up to 128 chunks the scatter pass reads every histogram in one round of loads.  Whole layers, 64 and 16
// tokens to a chunk (and loads of 8 K slices instead of 16 where there are no more): 64 adapters of rank 32, top-4, 4096 ->
// 4096, 300 tokens 66.3 and 62.8 us, 2000 101.6 and 96.6; 28 of rank 12, top-2, 2000 95.4 and 92.3.
constexpr int kFineChunkTokens = 16;
inline int routing_chunk_tokens(int T) { return T <= 2048 ? kFineChunkTokens : kBucketChunkTokens; }
inline int routing_chunks(int T) { return (T + routing_chunk_tokens(T) - 1) / routing_chunk_tokens(T); }
inline int bucket_chunks(int T) { return (T + kBucketChunkTokens - 1) / kBucketChunkTokens; }
// Beyond bucket_chunks, for batches of up to T tokens: a workspace for 3000 tokens (47 chunks) holds 2048 (128 chunks) too.
inline int routing_chunks_extra(int T) {
    const int most = T <= 2048 ? T : 2048;
    return routing_chunks(most) - bucket_chunks(most);
}
// The library's own histogram scratch (a file-scope device array, one copy per GPU) for the entry point that takes
// no workspace: room for kStaticBucketMaxTokens tokens and any supported N; the pointer is the current device's.
constexpr int kStaticBucketMaxTokens = 65536;
hipError_t bucket_static_scratch(int32_t** ptr);
// have_hist: chunk_counts already holds the histograms (written by launch_gate_topk)
// clear_rows (optional): a [T][clear_row_bytes] array (row bytes a multiple of 16) that the scatter zeroes,
// every chunk its own rows: the dense expand operand that launch_shrink then fills in (shrink_clears_hdense)
hipError_t launch_bucket(const int32_t* topk_idx, int T, int k, int N, int32_t* chunk_counts, bool have_hist,
                         int32_t* counts, int32_t* offsets, int32_t* bucket_tok, int32_t* bucket_slot,
                         void* clear_rows, int clear_row_bytes, hipStream_t stream);

// ---- grouped LoRA shrink: h[t,slot,:] = x[t,:] * A[idx[t,slot]] ---------------------------
// h32 ([T,k,r] fp32) and/or hdense (bf16 [T, ext_stride], column idx*r+q = scale*w*h, other
// columns zero) are written; either may be NULL.
// apack / hpart: scratch of shrink_apack_bytes / shrink_hpart_bytes (A in MFMA operand order,
// per-K-slice partial sums); both sizes are 0 when the plain-FMA kernel is used.
// false: launch_shrink writes only the selected columns of hdense, so the caller has its rows cleared
// first (launch_bucket's clear_rows); true: launch_shrink writes every column itself
bool shrink_clears_hdense(bool bf16, int r, int T, int k);
size_t shrink_apack_bytes(int d_in, int N, int r, bool bf16);
size_t shrink_hpart_bytes(int T, int d_in, int r, int k, bool bf16);
hipError_t launch_shrink(const void* x, const void* A, const int32_t* topk_idx, const float* topk_w,
                         const int32_t* offsets, const int32_t* bucket_tok, const int32_t* bucket_slot,
                         int T, int d_in, int N, int r, int k, float scale, bool bf16,
                         void* apack, float* hpart, float* h32, void* hdense, int ext_stride,
                         hipStream_t stream);

// ---- grouped LoRA expand: out (+)= scale * sum_slot w * h[t,slot,:] * B[idx[t,slot]] ------
hipError_t launch_expand(const float* h32, const void* B, const int32_t* topk_idx, const float* topk_w,
                         int T, int d_out, int N, int r, int k, float scale, bool bf16, void* out,
                         int accumulate, hipStream_t stream);

// ---- fp32 storage (layer_f32.hip): the base projection, and the rest of the layer onto it
hipError_t launch_gemm_f32(const float* x, const float* W, int T, int d_in, int d_out, float* out, hipStream_t stream);
hipError_t launch_route_lora_f32(const float* x, const float* W_gate, const float* bias, const float* A, const float* B,
                                 int T, int d_in, int d_out, int N, int r, int k, float inv_temperature, float scale,
                                 int32_t* topk_idx, float* topk_w, float* out, float* h /*[T,k,r], if apart*/,
                                 hipStream_t stream);
bool layer_f32_applies(int T, int d_in, int d_out, int N, int r, int k);   // everything in one launch
hipError_t launch_layer_f32(const float* x, const float* W, const float* W_gate, const float* bias, const float* A,
                            const float* B, int T, int d_in, int d_out, int N, int r, int k, float inv_temperature,
                            float scale, int32_t* topk_idx, float* topk_w, float* out, hipStream_t stream);
bool f32_expand_apart(int d_out, int r, int k);   // the expand is a launch of its own and h is used

// ---- decode-sized batches in two launches (T <= 64, bf16, Wcat packed), for one layer or for a group of up to
// kMaxDecodeGroup layers that share x (q/k/v, gate/up):
// launch_gemm_decode_main: the main K splits of x * W_g^T as fp32 tiles partial_g[S][T][d_out_g], and in the same
//   launch x * Wcat_g^T (gate_rows = prep_wcat_rows(N, r): the gate terms and every adapter's shrink columns) as
//   gpartial_g[S][T][gate_rows]; S and the splits of every row tile follow from gemm_decode_plan(...);
// launch_decode_tail_group (route_small.hip): top-k, softmax -> idx_g, w_g, and
//   out_g = bf16(sum of the S tiles in order + sum_slot (scale * w * h from the shrink tiles) * B_g[idx_g]).
// Batches of a few hundred tokens with few output tiles end in the same tail, behind launch_gemm_dense_splitk_multi over every
// W_g and Wcat_g.
constexpr int kMaxDecodeGroup = 4;
struct DecodeMember {
    const void* W;        // [d_out, d_in]
    const void* wg3;      // Wcat
    const float* bias;    // gate bias or NULL
    const void* B;        // [N, r, d_out]
    int d_out;
    float* partial;       // [S][T][d_out]
    float* gpartial;      // [S][T][gate_rows]
    int32_t* idx;         // [T,k]
    float* w;             // [T,k]
    void* out;            // [T,d_out]
};
int gemm_splitk_splits(int T, int d_in, int d_out, bool bf16);
// How the K splits of a launch's row tiles (kSplitRows rows each, nk K steps) are cut.  per_wg = 0: every tile has S
// splits.  Otherwise the K steps of tile g are the units [g * nk, (g + 1) * nk) of the launch, cut into runs of per_wg
// units; the runs that touch a tile are its splits, at most S.
constexpr int kSplitRows = 128;
struct SplitPlan {
    int S, nk, per_wg;
};
bool gemm_decode_ok(int d_in);
SplitPlan gemm_decode_plan(int d_in, const int* d_out, int G, int gate_rows);
hipError_t launch_gemm_decode_main(const void* x, const DecodeMember* mem, int G, int gate_rows, const SplitPlan& plan,
                                   int T, int d_in, hipStream_t stream);
hipError_t launch_decode_tail_group(const DecodeMember* mem, int G, const SplitPlan& plan, int T, int N, int r, int k, int gate_rows,
                                    float inv_temperature, float scale, hipStream_t stream);

// ---- gate gradients (Sec. 3.2, Eq. 4): dW_gate[d_in,N], dbias[N] (optional) and d_logits[T,N] (optional) from
// x, dy = dL/do, the packed Wcat and B; bf16, N <= 32, r % 8 == 0, at most 640 rows of Wcat, d_in and d_out multiples of 64.
// idx_in / w_in (optional, both or neither): the routing of the forward call; NULL ranks again from the same
// logits.  labels (optional): per-token adapter label of the classification loss, weight beta; values outside
// [0, N) give that token no classification part.  ws: gate_backward_layout(...).total bytes.
// part_x_given (optional): the K-split products x * Wcat^T that launch_route_dense_products left for this x
// (same T, d_in, N, r) in part_x_splits K splits (0 = that launcher's own count); NULL computes them here.
// dx (optional, bf16 [T, d_in]): the input gradient; needs A, W_gate and W_t = the base weight transposed,
// [d_in, d_out].
constexpr int kGateBackwardMaxTokens = 65536;
struct GateBackwardLayout { size_t part_x, part_dy, dgs, wpart, bpart, hx, xt, dxpart, total; int ext; };
bool gate_backward_applies(int T, int d_in, int d_out, int N, int r, bool bf16);
GateBackwardLayout gate_backward_layout(int T, int d_in, int d_out, int N, int r, bool dx, bool reserve);
hipError_t launch_gate_backward(const void* x, const void* dy, const void* wcat, const void* B, const float* bias,
                                const int32_t* idx_in, const float* w_in, const int32_t* labels, float beta, int T,
                                int d_in, int d_out, int N, int r, int k, float scale, float* dW_gate, float* dbias,
                                float* d_logits, const float* part_x_given, int part_x_splits, const void* A,
                                const float* W_gate, const void* W_t, void* dx, char* ws, hipStream_t stream);

// ---- base projection out = x * W^T (W stored [d_out, d_in]), optional fused LoRA expand ---
// If hdense != NULL the contraction is extended by the columns of hdense against the stacked B
// (out += hdense * B viewed as [N*r, d_out]), i.e. the LoRA expand runs in the same accumulators;
// the kernel takes B transposed and zero-padded, Bt[d_out, ext_stride] as launch_prep writes it,
// and ext_stride must be a multiple of 64.
// d_in may be 0 (expand only); accumulate=1 adds the previous contents of out.
// true if launch_gemm applies the hdense/B extension for this dtype (else run launch_expand after it)
bool gemm_fuses_expand(bool bf16);
// splitk_ws: scratch of gemm_splitk_bytes (0 = this shape is not split) or NULL to forbid splitting.
// topk_idx[T,k], r (optional): the routing that hdense was made from; K tiles of the extension that are zero for all
// tokens of an output tile are left out.
size_t gemm_splitk_bytes(int T, int d_in, int d_out, bool bf16);
// bf16, more than 64 tokens with few output tiles: K splits of a launch of fp32 tiles and one that adds them (0: launch_gemm), and
// the scratch that any batch of up to T tokens takes (launch_gemm's splitk_ws up to 64)
int gemm_few_tile_splits(int T, int d_in, int d_out);
size_t gemm_few_tile_bytes(int T, int d_in, int d_out);
hipError_t launch_gemm_few_tiles(const void* x, const void* W, int T, int d_in, int d_out, const void* hdense, int ext_stride,
                                 const void* Bt, int ext_k, void* out, float* partial, hipStream_t stream);
hipError_t launch_gemm(const void* x, const void* W, int T, int d_in, int d_out, bool bf16,
                       const void* hdense, int ext_stride, const void* Bt, int ext_k,
                       void* out, int accumulate, float* splitk_ws, hipStream_t stream,
                       const int32_t* topk_idx = nullptr, int k = 0, int r = 0);

}  // namespace meteora
