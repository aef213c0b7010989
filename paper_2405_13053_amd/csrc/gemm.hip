// Base projection of the layer, first term of Eq. 1 / Eq. 2:  out = x * W_base, with W stored
// [d_out, d_in] so both operands are contiguous along the contraction.
#include <stdlib.h>
#include "common.hpp"
#include "gemm_mfma.hpp"
#include "kernels.hpp"

namespace meteora {

// Sum the fp32 split-K tiles in a fixed order (deterministic), add the old output if asked, round once.
__global__ __launch_bounds__(256) void gemm_splitk_reduce_kernel(const float* __restrict__ partial, int nsplit,
                                                                 int T, int d_out, bf16_t* __restrict__ out,
                                                                 int accumulate) {
    const size_t n8 = (size_t)T * d_out / 8;
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n8) return;
    f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < nsplit; s0 += 4) {   // tiles in order, four tiles' loads in flight
        f32x4 v0[4], v1[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float* src = partial + (size_t)min(s0 + u, nsplit - 1) * T * d_out + i * 8;
            v0[u] = *reinterpret_cast<const f32x4*>(src);
            v1[u] = *reinterpret_cast<const f32x4*>(src + 4);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (s0 + u < nsplit) { lo += v0[u]; hi += v1[u]; }
    }
    u32x4* dst = reinterpret_cast<u32x4*>(out) + i;
    if (accumulate) {
        const u32x4 old = *dst;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            lo[2 * e] += bf16_bits_to_float(old[e] & 0xffffu);
            lo[2 * e + 1] += bf16_bits_to_float(old[e] >> 16);
            hi[2 * e] += bf16_bits_to_float(old[2 + e] & 0xffffu);
            hi[2 * e + 1] += bf16_bits_to_float(old[2 + e] >> 16);
        }
    }
    u32x4 pk;
    pk[0] = pack_bf16x2(lo[0], lo[1]); pk[1] = pack_bf16x2(lo[2], lo[3]);
    pk[2] = pack_bf16x2(hi[0], hi[1]); pk[3] = pack_bf16x2(hi[2], hi[3]);
    *dst = pk;
}

// Skinny batches (decode): one 64-row tile per 64 output columns leaves most CUs idle while W streams
// from HBM, so K is split over workgroups.  Returns the number of main-K splits (0 = do not split).
int gemm_splitk_splits(int T, int d_in, int d_out, bool bf16) {
    if (!bf16 || T < 1 || T > 64) return 0;
    const int tiles = ceil_div(T, 64) * ceil_div(d_out, 64), nk = ceil_div(d_in, kGemmBK);
    if (tiles >= 512 || nk < 8) return 0;
    int S = ceil_div(512, tiles);   // about two workgroups per CU (measured: 384 to 1536 tried)
    if (S > nk / 4) S = nk / 4;
    return S >= 2 ? S : 0;
}

size_t gemm_splitk_bytes(int T, int d_in, int d_out, bool bf16) {
    const int S = gemm_splitk_splits(T, d_in, d_out, bf16);
    return S == 0 ? 0 : (size_t)(S + 1) * T * d_out * sizeof(float);   // +1: the expand extension
}

// The pipelined kernels need byte offsets inside x, W and the extension operands that fit 32 bits, and for their staged
// epilogue an output tile (256 rows at most, fp32 at the widest) whose offsets do too.
static bool dma_ok(const GemmArgs& a, int BM, int BN) {
    const uint64_t widest = (uint64_t)(a.d_in > a.ext_stride ? a.d_in : a.ext_stride) * 2;
    return ((uint64_t)a.T + BM) * widest < (1ull << 32) &&
           ((uint64_t)a.d_out + BN) * widest < (1ull << 32) && (uint64_t)a.d_out * 4 * 256 < (1ull << 32);
}

template <typename K>
static hipError_t launch_ring(K kern, const GemmArgs& a, int lds_bytes, int splits, hipStream_t stream) {
    const hipError_t e = ensure_lds_limit(reinterpret_cast<const void*>(kern), lds_bytes);
    if (e != hipSuccess) return e;
    kern<<<dim3(a.tiles_m * a.tiles_n, splits), 256, lds_bytes, stream>>>(a);
    return hipGetLastError();
}

static bool ragged(const GemmArgs& a) { return a.d_in % kGemmBK != 0; }
// Nothing behind the whole K tiles: kBehindNone.  Splits of K share one kernel, also where only the last of them has more.
static bool whole_tiles(const GemmArgs& a) { return !ragged(a) && a.ext_k == 0; }

// One workgroup per (MB*32) x (NB*32) output tile; the output is written, or added to, by the kernel itself.
template <int MB, int NB, int D>
static hipError_t launch_tiles(GemmArgs a, hipStream_t stream) {
    a.tiles_m = ceil_div(a.T, MB * 32);
    a.tiles_n = ceil_div(a.d_out, NB * 32);
    constexpr int smem = gemm_ring_lds_bytes<MB, NB, D>();
    if (a.accumulate) {   // an expand alone
        if (ragged(a)) return hipErrorInvalidValue;
        return launch_ring(&gemm_mfma_ring_kernel<MB, NB, D, kEpiAccumulate, kBehindExtLook>, a, smem, 1, stream);
    }
    if (a.ext_k == 0)
        return ragged(a) ? launch_ring(&gemm_mfma_ring_kernel<MB, NB, D, kEpiStore, kBehindPart>, a, smem, 1, stream)
                         : launch_ring(&gemm_mfma_ring_kernel<MB, NB, D, kEpiStore, kBehindNone>, a, smem, 1, stream);
    if (ragged(a)) return launch_ring(&gemm_mfma_ring_kernel<MB, NB, D, kEpiStore, kBehindAnyLook>, a, smem, 1, stream);
    return a.topk_idx != nullptr ? launch_ring(&gemm_mfma_ring_kernel<MB, NB, D, kEpiStore, kBehindExtLook>, a, smem, 1, stream)
                                 : launch_ring(&gemm_mfma_ring_kernel<MB, NB, D, kEpiStore, kBehindExt>, a, smem, 1, stream);
}

// Few tiles and no extension: base projections of few tokens.
template <int MB, int NB, int D>
static hipError_t launch_small_tiles(GemmArgs a, hipStream_t stream) {
    a.tiles_m = ceil_div(a.T, MB * 32);
    a.tiles_n = ceil_div(a.d_out, NB * 32);
    constexpr int smem = gemm_ring_lds_bytes<MB, NB, D>();
    return ragged(a) ? launch_ring(&gemm_mfma_ring_kernel<MB, NB, D, kEpiStore, kBehindPart>, a, smem, 1, stream)
                     : launch_ring(&gemm_mfma_ring_kernel<MB, NB, D, kEpiStore, kBehindNone>, a, smem, 1, stream);
}

// The same without the ring: any size.
template <int M>
static hipError_t launch_plain(GemmArgs a, hipStream_t stream) {
    constexpr int smem = gemm_lds_bytes<M, M>();
    const hipError_t e = ensure_lds_limit(reinterpret_cast<const void*>(&gemm_mfma_kernel<M, M>), smem);
    if (e != hipSuccess) return e;
    a.tiles_m = ceil_div(a.T, M * 64);
    a.tiles_n = ceil_div(a.d_out, M * 64);
    gemm_mfma_kernel<M, M><<<a.tiles_m * a.tiles_n, 256, smem, stream>>>(a);
    return hipGetLastError();
}

// At most 64 tokens: 64 x 64 tiles, split along K where the caller has room for the fp32 tiles (a.partial).
static hipError_t launch_skinny(GemmArgs a, hipStream_t stream) {
    constexpr int smem = gemm_lds_bytes<1, 1>();
    hipError_t e = ensure_lds_limit(reinterpret_cast<const void*>(&gemm_mfma_kernel<1, 1>), smem);
    const auto dma_kernel = ragged(a) ? &gemm_mfma_dma_kernel<1, 1, true> : &gemm_mfma_dma_kernel<1, 1, false>;
    if (e == hipSuccess) e = ensure_lds_limit(reinterpret_cast<const void*>(dma_kernel), smem);
    if (e != hipSuccess) return e;
    a.tiles_m = ceil_div(a.T, 64);
    a.tiles_n = ceil_div(a.d_out, 64);
    const bool dma = dma_ok(a, 64, 64);
    if (dma && a.partial != nullptr) {
        const int nsplit = a.splits + (a.ext_k > 0 ? 1 : 0);
        dma_kernel<<<dim3(a.tiles_m * a.tiles_n, nsplit), 256, smem, stream>>>(a);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        const size_t n8 = (size_t)a.T * a.d_out / 8;
        gemm_splitk_reduce_kernel<<<(unsigned)((n8 + 255) / 256), 256, 0, stream>>>(a.partial, nsplit, a.T, a.d_out,
                                                                                   a.out, a.accumulate);
    } else if (dma) {
        dma_kernel<<<a.tiles_m * a.tiles_n, 256, smem, stream>>>(a);
    } else {
        gemm_mfma_kernel<1, 1><<<a.tiles_m * a.tiles_n, 256, smem, stream>>>(a);
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Dense routing operand: partial[split][T][rows] = x[T, K-range of split] * Wcat[rows, same K]^T in fp32,
// no reduction (the select kernel adds the splits in order).
// ------------------------------------------------------------------------------------------
// Bound by the CU's port to L2 (a K tile of 128 x 160 is 37 KB and 640 cycles of MFMAs) and by the fp32 tiles.  One workgroup per CU:
//   - 128 x 160 tiles, a ring of three: 320 and 544 rows of Wcat fill them, and they are dealt evenly, where 128 x 128 tiles, two
//     to a CU, left half of the CUs with one of the 384 workgroups (and half of the third column tile of 320 rows empty).
//     While they make two K splits or more.
//   - beyond 2048 tokens, where x is read again for every column tile: the narrowest tile of up to 320 columns that takes the
//     rows in as few column tiles as 320 does (544 rows: 288).
// and otherwise, as where K ends the splits before the CUs are full, 128 x 128 tiles, two workgroups per CU.  So also while those are few
// (up to 176, or 256 of up to four K tiles) and their splits are shorter than 16 K tiles: a narrower tile is through its K tiles sooner, and
// more CUs work on it.  Gradients of the gate alone, 320 rows, 128 x 128 and 128 x 160: 2048 inputs 450 tokens 23.2 and 25.3, 1200 28.3 and
// 29.7, 1500 31.1 and 28.8; 4096 inputs 300 tokens 25.0 and 25.6, 1200 31.7 and 30.6; 6144 inputs 800 31.4 and 32.0, 1000 33.2 and 31.4;
// 14336 inputs 65 tokens 34.3 and 33.2.
// Whole calls, 128 x 128 up to 4096 tokens and 128 x 320 above with ordinary stores, as it was, and so (written through, see kWriteThrough;
// with ordinary stores), us: layers of rank 8, 4096 -> 4096 1000 tokens 49.3, 48.4 (48.0), 4096 117.6, 116.0 (117.9), 5000 181.6,
// 176.4 (176.3), 8192 227.2, 221.8 (223.1); 3000 x 5120 -> 5120 144.1, 136.0 (137.5), 4096 x 14336 -> 1024 193.7, 183.0
// (183.0); of rank 16 4096 x 4096 -> 4096 132.2, 127.1 (127.0), 16384 x 14336 -> 1024 584.6, 567.2 (567.3); lora_forward of rank 8
// 3000 x 5120 -> 1024 32.2, 29.8 (31.1), 8000 x 4096 -> 1024 42.7, 40.0 (40.9); a training step of 4096 x 4096 -> 4096 266.9,
// 262.1 (263.9).  128 x 160 with one split loses: 6000 tokens of rank 16 215 against 211; and where the contraction is long beside the
// fp32 tiles that 320 columns need for their extra splits: 5000 x 14336 -> 1024 198 against 195, 8192 x 14336 -> 4096 696 against 692;
// with 6144 inputs 8192 tokens 130 against 137.
struct DenseTile { int nb, splits; };   // columns in blocks of 32

static int dense_split_bounds(int S, int nk) {
    if (S > nk / 4) S = nk / 4;                // at least 4 K tiles per split
    if (S > 8) S = 8;                          // more splits cost the kernel that adds them more than they save here
    return S < 1 ? 1 : S;
}

static int dense_wide_blocks(int rows) { return ceil_div(ceil_div(rows, ceil_div(rows, 320)), 32); }

static DenseTile dense_tile(int T, int d_in, int rows) {
    const int nk = ceil_div(d_in, kGemmBK), row_tiles = ceil_div(T, 128), four = ceil_div(rows, 128), five = ceil_div(rows, 160);
    const DenseTile narrow = {4, dense_split_bounds((384 + row_tiles * four / 2) / (row_tiles * four), nk)};
    const int part = ceil_div(nk, narrow.splits);
    if (part < 16 && row_tiles * four * narrow.splits <= (part <= 4 ? 256 : 176)) return narrow;
    auto fits = [&](int tiles) { return dense_split_bounds(256 / tiles, nk) == dense_split_bounds(256 / tiles, 32); };   // K does not bind
    if (five * 160 <= four * 128 && 2 * row_tiles * five <= 256 && (T <= 4096 || nk <= 96) && fits(row_tiles * five))
        return {5, dense_split_bounds(256 / (row_tiles * five), nk)};
    const int nb = dense_wide_blocks(rows), tiles = row_tiles * ceil_div(rows, 32 * nb);
    if (nb > 4 && (T > 4096 || (T > 2048 && fits(tiles)))) return {nb, dense_split_bounds(256 / tiles, nk)};
    return narrow;
}

bool gemm_dense_splitk_ok(int T, int d_in, int rows) {
    const uint64_t widest = (uint64_t)d_in * 2;
    return d_in % 8 == 0 && rows % 8 == 0 && ((uint64_t)T + 2 * 64) * widest < (1ull << 32) &&
           ((uint64_t)rows + 5 * 64) * widest < (1ull << 32) && (uint64_t)rows * 4 * 256 < (1ull << 32);
}

// the same for tiles of up to 256 rows (launch_gemm_dense_splitk_multi, launch_gemm_few_tiles)
bool gemm_multi_ok(int T, int d_in, int rows) {
    return gemm_dense_splitk_ok(T, d_in, rows) && ((uint64_t)T + 256) * ((uint64_t)d_in * 2) < (1ull << 32);
}

int gemm_dense_splits(int T, int d_in, int rows) { return dense_tile(T, d_in, rows).splits; }

// The K splits that few-tile launches start from (see gemm_multi_splits)
int gemm_multi_fit(int T, int d_in, int rows) {
    const int tiles = ceil_div(T, 128) * ceil_div(rows, T <= 4096 ? 128 : 320);
    return dense_split_bounds(T <= 4096 ? (384 + tiles / 2) / tiles : 256 / tiles, ceil_div(d_in, kGemmBK));
}

int64_t gemm_dense_pairs_reserved(int T, int d_in, int rows) {
    // the splits change at multiples of 128 tokens; above 384 row tiles there is one
    int64_t pairs = (int64_t)gemm_dense_splits(T, d_in, rows) * T;
    for (int t = 128; t < T && t <= 384 * 128; t += 128) {
        const int64_t p = (int64_t)gemm_dense_splits(t, d_in, rows) * t;
        if (p > pairs) pairs = p;
    }
    return pairs;
}

// fp32 split-K tiles; tiles_n is the caller's.  MORE: what there may be behind the whole K tiles
template <int MB, int NB, int D, int EPI, int MORE = kBehindPart>
static hipError_t launch_dense(GemmArgs a, hipStream_t stream) {
    a.tiles_m = ceil_div(a.T, MB * 32);
    if (a.tiles_n == 0) a.tiles_n = ceil_div(a.d_out, NB * 32);
    constexpr int smem = gemm_ring_lds_bytes<MB, NB, D>();
    return whole_tiles(a) ? launch_ring(&gemm_mfma_ring_kernel<MB, NB, D, EPI, kBehindNone>, a, smem, a.splits, stream)
                          : launch_ring(&gemm_mfma_ring_kernel<MB, NB, D, EPI, MORE>, a, smem, a.splits, stream);
}

hipError_t launch_gemm_dense_splitk(const void* x, const void* Wcat, int T, int d_in, int rows, float* partial,
                                    hipStream_t stream) {
    if (!gemm_dense_splitk_ok(T, d_in, rows)) return hipErrorInvalidValue;
    GemmArgs a{};
    a.x = (const bf16_t*)x; a.W = (const bf16_t*)Wcat; a.T = T; a.d_in = d_in; a.d_out = rows;
    a.partial = partial;
    const DenseTile tile = dense_tile(T, d_in, rows);
    a.splits = tile.splits;
    a.tiles_per_split = ceil_div(ceil_div(d_in, kGemmBK), a.splits);
    switch (tile.nb) {
        case 4: return launch_dense<4, 4, 2, kEpiPartial, kBehindAny>(a, stream);   // one kernel with the few tiles of launch_multi_tiles
        case 5: return launch_dense<4, 5, 3, kEpiPartialThrough>(a, stream);
        case 6: return launch_dense<4, 6, 3, kEpiPartialThrough>(a, stream);
        case 7: return launch_dense<4, 7, 3, kEpiPartialThrough>(a, stream);
        case 8: return launch_dense<4, 8, 2, kEpiPartialThrough>(a, stream);
        case 9: return launch_dense<4, 9, 2, kEpiPartialThrough>(a, stream);
        default: return launch_dense<4, 10, 2, kEpiPartialThrough>(a, stream);
    }
}

// Several matrices in one split-K launch (few-tile batches): ops[i].partial[s][T][rows_i] = x * W_i^T over the K
// range of split s, the 128-column tiles of all of them in one grid, one workgroup per CU at most.  The tiles are up to
// 256 rows high (a wavefront's 128 x 64 piece needs 0.75 fragment reads per MFMA against 1.0 at 128 x 128), in steps
// of 32 so that the rows are dealt evenly: 300 tokens are two tiles of 160 rows.  Whole calls, against 256 rows above
// 128 tokens and 128 (two workgroups per CU) up to there, both with the two-deep ring, W not in any cache: 4096 -> 4096
// T = 80 23.6 -> 20.2 us, T = 300 40.7 -> 31.6, T = 512 43.0 -> 40.6; 14336 -> 4096 T = 128 58.7 -> 44.4, T = 300 102 -> 69.6.
static int gemm_multi_row_blocks(int T) {
    const int b = ceil_div(ceil_div(T, ceil_div(T, 256)), 32);
    return b < 3 ? 3 : b;
}
// One row tile, and so many columns that one workgroup per CU would mean a single split and half of the CUs without one:
// the splits stay as they are and two workgroups of the two-deep ring share a CU, if there are three splits or more (up
// to 153 column tiles; with two of them the second workgroup of most CUs is missing).  Whole calls, one against two per
// CU, at 65 and 128 tokens: 4096 -> 16384 (131 column tiles) 56.0 and 63.2 -> 43.0 and 50.5 us, 4096 -> 18432 56.7 and 64.2
// -> 45.8 and 55.2, 5120 -> 5120 three times (129) 67.4 and 80.6 -> 55.6 and 69.2, 4096 -> 9216 twice (150) 52.1 and 62.9 ->
// 47.4 and 58.8; with two splits 4096 -> 9728 twice (158) 55.6 and 66.5 against 57.8 and 69.2, 4096 -> 20480 (163) 59.0 and
// 65.2 against 58.0 and 66.0.
// Of the splits that leaves, the number at which the K tiles of a split and the fp32 tiles written and read again take the
// least: a K tile takes about 0.2 + 0.07 us for every 32 rows, a MB of fp32 tiles 0.45 us.  Whole calls, as many splits as
// fit and so: 512 x 2048 -> 2048 22.3 (6 splits) and 20.2 us (4), 700 x 4096 -> 1024 26.0 and 24.7, 900 x 1024 -> 1024 20.7 and
// 18.9, 200 x 1024 -> 4096 19.4 and 17.7, 96 x 4096 -> 4096 18.7 and 18.2; 1531 x 1024 -> 1024 20.1 and 21.1.
static int multi_cap(int T, int col_tiles) { return 256 / (ceil_div(T, 256) * (col_tiles > 0 ? col_tiles : 1)); }   // 256 CUs

int gemm_multi_splits(int T, int col_tiles, int S, int nk, int64_t rows) {
    const int cap = multi_cap(T, col_tiles);
    if (T <= 128 && cap < 2 && S >= 3) return S;
    if (S > cap) S = cap > 0 ? cap : 1;
    const float per_tile = 0.2f + 0.07f * (float)gemm_multi_row_blocks(T), per_split = 0.45e-6f * 4.f * (float)T * (float)rows;
    int best = S;
    float least = 0.f;
    for (int s = S; s >= 2; --s) {
        const float us = per_tile * (float)ceil_div(nk, s) + per_split * (float)s;
        if (s == S || us < least) { least = us; best = s; }
    }
    return best;
}

// The fp32 tiles go through the L2 (kWriteThrough) unless the launch streams many weights: those writes then share HBM with the
// stream.  Whole calls of 96, 144 and 256 tokens, weights not in the caches, ordinary and written through: 4096 -> 4096
// (36 MB) 19.5, 22.7, 28.1 and 18.6, 21.6, 26.8 us; 5120 -> 5120 (56 MB) 26.4, 31.6, 38.4 and 27.0, 32.2, 39.3; 14336 -> 4096
// (127 MB) 40.5, 45.0, 56.1 and 40.8, 45.8, 56.6.  The line is below the smallest size that loses: from 50 to 60 MB sizes differ
// (4096 -> 6144, 53 MB: 22.9, 25.7, 32.1 and 21.9, 24.5, 31.0), below it all of those tried gain 2 to 6%.
constexpr int64_t kWriteThroughWeights = 48 << 20;

template <int EPI>
static hipError_t launch_multi_tiles(const GemmArgs& a, bool two, hipStream_t stream) {
    if (two) return a.T <= 96 ? launch_dense<3, 4, 2, EPI, kBehindAny>(a, stream) : launch_dense<4, 4, 2, EPI, kBehindAny>(a, stream);
    switch (gemm_multi_row_blocks(a.T)) {
        case 3: return launch_dense<3, 4, 5, EPI, kBehindAny>(a, stream);
        case 4: return launch_dense<4, 4, 4, EPI, kBehindAny>(a, stream);
        case 5: return launch_dense<5, 4, 4, EPI, kBehindAny>(a, stream);
        case 6: return launch_dense<6, 4, 3, EPI, kBehindAny>(a, stream);
        case 7: return launch_dense<7, 4, 3, EPI, kBehindAny>(a, stream);
        default: return launch_dense<8, 4, 3, EPI, kBehindAny>(a, stream);
    }
}

hipError_t launch_gemm_dense_splitk_multi(const void* x, const DenseOperand* ops, int n_ops, int S, int T, int d_in,
                                          hipStream_t stream) {
    if (S < 1 || n_ops < 1 || n_ops > GemmArgs::kMaxSegments) return hipErrorInvalidValue;
    GemmArgs a{};
    a.x = (const bf16_t*)x; a.T = T; a.d_in = d_in;
    a.splits = S; a.tiles_per_split = ceil_div(ceil_div(d_in, kGemmBK), S);
    int tile0 = 0;
    int64_t rows = 0;
    for (int i = 0; i < n_ops; ++i) {
        if (!gemm_multi_ok(T, d_in, ops[i].rows)) return hipErrorInvalidValue;
        a.seg[i] = {(const bf16_t*)ops[i].W, ops[i].partial, ops[i].rows, tile0};
        tile0 += ceil_div(ops[i].rows, 128);
        rows += ops[i].rows;
    }
    a.nseg = n_ops;
    a.W = a.seg[0].W; a.d_out = a.seg[0].rows; a.partial = a.seg[0].partial;   // replaced per workgroup
    a.tiles_n = tile0;
    const bool two = T <= 128 && tile0 * S > 256;   // two per CU
    return rows * d_in * 2 <= kWriteThroughWeights ? launch_multi_tiles<kEpiPartialThrough>(a, two, stream)
                                                   : launch_multi_tiles<kEpiPartial>(a, two, stream);
}

bool gemm_fuses_expand(bool bf16) { return bf16; }

// The input gradient of a few hundred tokens: few output tiles and a long contraction, so K is split as in the few-tile layers,
// the extension going with the last split, and a second launch adds the tiles and rounds once.  Where the model of gemm_multi_splits
// says so, a launch being 4.5 us: a short contraction, or enough tiles for one sweep, lose (training steps, one sweep and
// split: 1000 x 4096 -> 1024 62 and 72 us, 800 x 4096 -> 4096 105 and 113).  Training steps with the input gradient, one sweep
// and so: 64 x 4096 -> 14336 220 and 105 us, 300 x 4096 -> 4096 78.5 and 70.2, 375 x 5120 -> 13824 267 and 208, 512 x 4096 ->
// 14336 250 and 191, 2000 x 1024 -> 14336 241 and 195.
int gemm_few_tile_splits(int T, int d_in, int d_out) {
    const int col_tiles = ceil_div(d_out, 128), nk = ceil_div(d_in, kGemmBK), row_tiles = 256 / col_tiles;
    if (T <= 64 || row_tiles < 1 || !gemm_multi_ok(T, d_in, d_out)) return 0;
    const int S = gemm_multi_splits(T, col_tiles, gemm_multi_fit(T, d_in, d_out), nk, d_out);
    if (S < 2) return 0;
    auto tile_us = [](int blocks) { return 0.2f + 0.07f * (float)(blocks < 4 ? 4 : blocks); };
    const float one = tile_us(ceil_div(ceil_div(T, row_tiles), 32)) * (float)nk;   // launch_gemm's tiles
    const float split = tile_us(gemm_multi_row_blocks(T)) * (float)ceil_div(nk, S) + 0.45e-6f * 4.f * (float)T * (float)d_out * (float)S;
    return split + 4.5f < one ? S : 0;
}

size_t gemm_few_tile_bytes(int T, int d_in, int d_out) {
    int64_t pairs = 0;   // tokens times splits of any batch of up to T tokens: the splits change downwards inside 32 tokens only
    const int col_tiles = ceil_div(d_out, 128), most = 256 * 128 / col_tiles, last = T < most ? T : most;
    for (int t = 64; t < last; t += 32) {
        const int S = gemm_multi_splits(t + 1, col_tiles, gemm_multi_fit(t + 1, d_in, d_out), ceil_div(d_in, kGemmBK), d_out);
        const int64_t p = S < 2 ? 0 : (int64_t)S * (t + 32 < last ? t + 32 : last);
        if (p > pairs) pairs = p;
    }
    const size_t few = gemm_splitk_bytes(T < 64 ? T : 64, d_in, d_out, true), many = (size_t)pairs * d_out * sizeof(float);
    return few > many ? few : many;
}

hipError_t launch_gemm_few_tiles(const void* x, const void* W, int T, int d_in, int d_out, const void* hdense, int ext_stride,
                                 const void* Bt, int ext_k, void* out, float* partial, hipStream_t stream) {
    const int S = gemm_few_tile_splits(T, d_in, d_out);
    GemmArgs a{};
    a.x = (const bf16_t*)x; a.W = (const bf16_t*)W; a.hd = (const bf16_t*)hdense; a.Bt = (const bf16_t*)Bt;
    a.T = T; a.d_in = d_in; a.d_out = d_out; a.ext_k = ext_k; a.ext_stride = ext_stride;
    a.partial = partial; a.splits = S; a.tiles_n = ceil_div(d_out, 128);
    if (S < 2 || ext_stride % kGemmBK != 0 || ext_stride < ext_k || !dma_ok(a, 256, 128)) return hipErrorInvalidValue;
    a.tiles_per_split = ceil_div(ceil_div(d_in, kGemmBK), S);
    const bool two = T <= 128 && a.tiles_n * S > 256;
    const hipError_t e = (int64_t)d_out * d_in * 2 <= kWriteThroughWeights ? launch_multi_tiles<kEpiPartialThrough>(a, two, stream)
                                                                           : launch_multi_tiles<kEpiPartial>(a, two, stream);
    if (e != hipSuccess) return e;
    const size_t n8 = (size_t)T * d_out / 8;
    gemm_splitk_reduce_kernel<<<(unsigned)((n8 + 255) / 256), 256, 0, stream>>>(partial, S, T, d_out, (bf16_t*)out, 0);
    return hipGetLastError();
}

// every kernel of this file that a launcher above may start with more than the default dynamic LDS
hipError_t gemm_init_kernels() {
    hipError_t e = hipSuccess;
    auto lim = [&](auto kern, int bytes) {
        if (e == hipSuccess) e = ensure_lds_limit(reinterpret_cast<const void*>(kern), bytes);
    };
    lim(&gemm_mfma_kernel<4, 4>, gemm_lds_bytes<4, 4>());
    lim(&gemm_mfma_kernel<2, 2>, gemm_lds_bytes<2, 2>());
    lim(&gemm_mfma_kernel<1, 1>, gemm_lds_bytes<1, 1>());
    lim(&gemm_mfma_dma_kernel<1, 1, false>, gemm_lds_bytes<1, 1>());
    lim(&gemm_mfma_dma_kernel<1, 1, true>, gemm_lds_bytes<1, 1>());
#define METEORA_RING(MB, NB, D, EPI, BEHIND) lim(&gemm_mfma_ring_kernel<MB, NB, D, EPI, BEHIND>, gemm_ring_lds_bytes<MB, NB, D>())
#define METEORA_BOTH(MB, NB, D, EPI)              \
    METEORA_RING(MB, NB, D, EPI, kBehindNone);    \
    METEORA_RING(MB, NB, D, EPI, kBehindPart)
#define METEORA_TILES(MB, NB, D)                          \
    METEORA_BOTH(MB, NB, D, kEpiStore);                   \
    METEORA_RING(MB, NB, D, kEpiStore, kBehindExt);       \
    METEORA_RING(MB, NB, D, kEpiStore, kBehindExtLook);   \
    METEORA_RING(MB, NB, D, kEpiStore, kBehindAnyLook);   \
    METEORA_RING(MB, NB, D, kEpiAccumulate, kBehindExtLook)
    METEORA_TILES(8, 8, 2);
    METEORA_TILES(8, 4, 3);
    METEORA_TILES(7, 4, 3);
    METEORA_TILES(6, 4, 3);
    METEORA_TILES(5, 4, 4);
    METEORA_TILES(4, 4, 3);
    METEORA_TILES(4, 4, 2);
    METEORA_BOTH(2, 2, 5, kEpiStore);
    METEORA_BOTH(3, 2, 5, kEpiStore);
    METEORA_BOTH(4, 2, 4, kEpiStore);
    METEORA_BOTH(4, 10, 2, kEpiPartialThrough);
    METEORA_BOTH(4, 5, 3, kEpiPartialThrough);
    METEORA_BOTH(4, 6, 3, kEpiPartialThrough);
    METEORA_BOTH(4, 7, 3, kEpiPartialThrough);
    METEORA_BOTH(4, 8, 2, kEpiPartialThrough);
    METEORA_BOTH(4, 9, 2, kEpiPartialThrough);
#define METEORA_PARTIAL(MB, NB, D)                          \
    METEORA_RING(MB, NB, D, kEpiPartial, kBehindNone);         \
    METEORA_RING(MB, NB, D, kEpiPartial, kBehindAny);          \
    METEORA_RING(MB, NB, D, kEpiPartialThrough, kBehindNone);  \
    METEORA_RING(MB, NB, D, kEpiPartialThrough, kBehindAny)
    METEORA_PARTIAL(4, 4, 2);
    METEORA_PARTIAL(3, 4, 2);
    METEORA_PARTIAL(3, 4, 5);
    METEORA_PARTIAL(4, 4, 4);
    METEORA_PARTIAL(5, 4, 4);
    METEORA_PARTIAL(6, 4, 3);
    METEORA_PARTIAL(7, 4, 3);
    METEORA_PARTIAL(8, 4, 3);
#undef METEORA_PARTIAL
#undef METEORA_TILES
#undef METEORA_BOTH
#undef METEORA_RING
    return e;
}

hipError_t launch_gemm(const void* x, const void* W, int T, int d_in, int d_out, bool bf16,
                       const void* hdense, int ext_stride, const void* Bt, int ext_k,
                       void* out, int accumulate, float* splitk_ws, hipStream_t stream,
                       const int32_t* topk_idx, int k, int r) {
    if (bf16) {
        if (hdense && (ext_stride % kGemmBK != 0 || ext_stride < ext_k || !Bt)) return hipErrorInvalidValue;
        GemmArgs a{};
        a.x = (const bf16_t*)x; a.W = (const bf16_t*)W; a.hd = (const bf16_t*)hdense; a.Bt = (const bf16_t*)Bt;
        a.out = (bf16_t*)out; a.T = T; a.d_in = d_in; a.d_out = d_out;
        a.ext_k = hdense ? ext_k : 0; a.ext_stride = ext_stride; a.accumulate = accumulate;
        if (a.ext_k > 0 && r > 0 && a.ext_k <= 64 * kGemmBK) { a.topk_idx = topk_idx; a.topk = k; a.rank = r; }
        const int S = splitk_ws ? gemm_splitk_splits(T, d_in, d_out, true) : 0;
        if (S > 0 && d_in > 0) {
            a.partial = splitk_ws;
            a.splits = S;
            a.tiles_per_split = ceil_div(ceil_div(d_in, kGemmBK), S);
            return launch_skinny(a, stream);
        }
        // A base projection of few tokens (no extension, and no workspace to split K in): tiles of 64 columns, as low as one per CU
        // allows, 64 to 128 rows.  It is bound by how many CUs stream W and by the bytes they have in flight: against 64 x 64 tiles
        // with two slots up to 64 tokens and 128 x 128 above, W not in any cache, 1, 64, 96 and 300 tokens: 4096 -> 4096 45.0, 45.5,
        // 35.1, 30.2 and 15.5, 21.2, 17.7, 19.0 us; 14336 -> 4096 151, 152, 129, 104 and 48.1, 70.2, 57.2, 59.0; 4096 -> 1024 28.0, 28.3,
        // 24.2, 28.0 and 11.7, 12.6, 12.6, 12.6; 5120 -> 13824 58.3, 58.8, 59.9 and 25.5, 36.2, 45.0.  128-row tiles only: 200 x 5120 ->
        // 5120 38.0, and 24.8 with 96 rows; rings as deep as LDS allows (9, 7, 6): 1 us slower at most sizes.  Short contractions and W in
        // cache gain too or are level (280 sizes of 64 to 4096 inputs, GPU alone): 200 x 128 -> 1024 4.1 and 3.2 cold, 4.1 and 3.1 warm,
        // 96 x 512 -> 4096 7.9 and 5.1, 6.0 and 4.4, 1 x 256 -> 1024 3.4 and 3.5 warm.
        const int row_tiles_64 = 256 / ceil_div(d_out, 64);
        if (a.ext_k == 0 && !accumulate && row_tiles_64 > 0 && dma_ok(a, 128, 64)) {
            const int blocks = ceil_div(ceil_div(T, row_tiles_64), 32);
            if (blocks <= 2) return launch_small_tiles<2, 2, 5>(a, stream);
            if (blocks == 3) return launch_small_tiles<3, 2, 5>(a, stream);
            if (blocks == 4) return launch_small_tiles<4, 2, 4>(a, stream);
        }
        const int64_t big_tiles = (int64_t)ceil_div(T, 256) * ceil_div(d_out, 256);
        // 256 x 256 tiles once they fill most of the 256 CUs; below that 128 x 128 tiles keep more CUs busy
        // (T = 2048, 4096 -> 4096: 128 tiles of 256 x 256 take 109 us, 512 tiles of 128 x 128 take 98 us)
        // ... except a little more than one tile per CU (257 to 328 tiles), where the second, nearly empty round of
        // 256 x 256 tiles costs more than the smaller tiles' lower efficiency (4096 -> 4096: T = 4608, 288 tiles, 174
        // us against 155 with 128 x 128 tiles; T = 5120 176 against 163; 336 tiles and more: the big tiles win again,
        // and with two rounds or more they always do: 544 tiles 275 against 279)
        if (T > 128 && big_tiles >= 160 && !(big_tiles > 256 && big_tiles <= 328))
            return dma_ok(a, 256, 256) ? launch_tiles<8, 8, 2>(a, stream) : launch_plain<4>(a, stream);
        if (T > 64 && !dma_ok(a, 256, 128)) return launch_plain<2>(a, stream);
        // otherwise tiles of 128 columns, one per CU, as low as that allows, with a ring that is as deep as helps: more CUs
        // busy and less padding than at 256 rows (a wavefront's 128 x 64 piece has 0.75 fragment reads per MFMA, a 64 x
        // 64 piece 1.0, so not lower than needed).  The GEMM inside the layer against 256-row
        // tiles (or two 128-row tiles per CU) with shallower rings: 4096 -> 4096 T = 1000 44.8 -> 41.3 us, 1280 59.1 ->
        // 47.3, 1531 61.0 -> 52.8, 1700 63.1 -> 59.6; 4096 -> 14336 T = 300 57.7 -> 50.5; 5120 -> 5120 T = 1000 79.7 ->
        // 64.1; 14336 -> 4096 T = 1280 177 -> 149.
        const int row_tiles = 256 / ceil_div(d_out, 128);
        if (T > 64 && row_tiles > 0) {
            switch (ceil_div(ceil_div(T, row_tiles), 32)) {
                case 1: case 2: case 3: case 4:
                    // three tiles ahead cover a load from HBM (four cost the start of the kernel more than they save); up
                    // to 8 K tiles that start is most of it, and two are enough.  Two, three and four tiles, W in cache and
                    // out of it: 65 x 512 -> 1024 6.8, 6.4, 6.8 and 6.5, 6.5, 7.0 us; 65 x 1024 -> 1024 8.6, 9.0, 9.3 and
                    // 9.2, 9.0, 9.5; 65 x 4096 -> 1024 23.8, 24.2, 24.5 and 35.2, 30.9, 31.3
                    return (a.d_in + (a.ext_k > 0 ? a.ext_stride : 0)) / kGemmBK <= 8 ? launch_tiles<4, 4, 2>(a, stream)
                                                                                      : launch_tiles<4, 4, 3>(a, stream);
                case 5: return launch_tiles<5, 4, 4>(a, stream);
                case 6: return launch_tiles<6, 4, 3>(a, stream);
                case 7: return launch_tiles<7, 4, 3>(a, stream);
                case 8: return launch_tiles<8, 4, 3>(a, stream);
            }
        }
        if (T > 64) return launch_tiles<4, 4, 2>(a, stream);   // more than one tile per CU: two share it
        return launch_skinny(a, stream);
    }
    if (accumulate) return hipErrorInvalidValue;   // the expand adds to the output by itself
    return launch_gemm_f32((const float*)x, (const float*)W, T, d_in, d_out, (float*)out, stream);
}

}  // namespace meteora
