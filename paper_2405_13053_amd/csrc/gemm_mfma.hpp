// bf16 MFMA kernel for the base projection out = x * W^T (first term of Eq. 1 / Eq. 2), with the
// LoRA expand optionally fused as an extension of the contraction:
//
//     out[t, c] = sum_{i < d_in} x[t,i] * W[c,i]  +  sum_{j < ext_k} hd[t,j] * Bst[j,c]
//
// where hd[t, a*r+q] = scale * w * h[t,slot,q] for the adapters a the token selected (zero
// elsewhere) and Bst is the stacked B[N, r, d_out] viewed as [N*r, d_out]; the kernels read it
// transposed (Bt[c, j], rows of ext_stride elements, columns j >= ext_k zero), which makes the
// extension one more stretch of K tiles with the same operand layout as x and W.  The second sum is
// exactly scale * sum_{i in I(x)} w_i (x A_i) B_i of Eq. 2, accumulated in the same fp32
// registers as the base term, so the output is rounded once.
//
// Three kernels share the operand layout (a workgroup of 4 wavefronts, 2 x 2, owns an output tile; K advances in steps of
// 64 through LDS tiles whose rows are 128 B, their 16-B chunks XOR-swizzled with the row index (see swz) so that a
// ds_read_b128 pass touches every bank once; W is the MFMA's first operand, so a lane ends up with 4 consecutive output
// columns of one token row):
//   gemm_mfma_ring_kernel  more than 64 tokens, base projections of up to 16384 outputs, and every fp32-tile launch of more than
//                          64: v_mfma_f32_16x16x32_bf16 on a ring of LDS slots that global->LDS loads fill two to five K
//                          tiles ahead;
//   gemm_mfma_dma_kernel   otherwise up to 64 tokens: 64 x 64 tiles, v_mfma_f32_32x32x16_bf16, two slots;
//   gemm_mfma_kernel       sizes whose byte offsets pass 32 bits: v_mfma_f32_32x32x16_bf16, tiles through registers into
//                          two LDS buffers.
#pragma once
#include <type_traits>
#include <utility>

#include "common.hpp"
#include "topk_key.hpp"

namespace meteora {

constexpr int kGemmBK = 64;          // K elements per LDS tile
constexpr int kGemmChunks = 8;       // 16-byte chunks per LDS row

// LDS staging of the output tile in the two-slot kernel: a wavefront's (MI*32) x (NI*32) bf16 block,
// rows padded by 16 bytes; the dynamic LDS size is the larger of the operand ring and this stage.
template <int NI>
__host__ __device__ constexpr int gemm_epilogue_stride() { return NI * 64 + 16; }
// fp32 partial tiles (split K) are staged one block row (32 tile rows) per wavefront at a time
template <int NI>
__host__ __device__ constexpr int gemm_partial_stride() { return NI * 128 + 16; }
template <int MI, int NI>
__host__ __device__ constexpr int gemm_lds_bytes() {
    constexpr int ring = 2 * (MI * 64 + NI * 64) * kGemmBK * 2;
    constexpr int stage = 4 * (MI * 32) * gemm_epilogue_stride<NI>();
    constexpr int pstage = 4 * 32 * gemm_partial_stride<NI>();
    constexpr int m = ring > stage ? ring : stage;
    return m > pstage ? m : pstage;
}

struct GemmArgs {
    const bf16_t* x;      // [T, d_in]
    const bf16_t* W;      // [d_out, d_in]
    const bf16_t* hd;     // [T, ext_stride] or nullptr
    const bf16_t* Bt;     // [d_out, ext_stride] (stacked B transposed, zero-padded columns) or nullptr
    bf16_t* out;          // [T, d_out]
    int T, d_in, d_out;
    int ext_k;            // N*r; 0 = no extension
    int ext_stride;       // row stride of hd and Bt: ext_k rounded up to a multiple of 64
    // The routing that hd was made from, or nullptr: topk_idx[T,k] adapters of rank r = ext_k / N.  hd is zero in the
    // columns of adapters a token did not select (the ring kernel skips K tiles that are zero for all its tokens)
    const int32_t* topk_idx;
    int topk, rank;
    int accumulate;       // 1: add previous contents of out
    int tiles_m, tiles_n;
    // split-K (skinny batches): blockIdx.y = split; split s < splits takes K tiles [s*tiles_per_split, ...), and the expand
    // extension (if ext_k > 0) is the last split's too in the ring kernel, split == splits in the two-slot one; fp32 tiles go
    // to partial[split][T][d_out]
    float* partial;       // nullptr: no split, the kernel writes `out` itself
    int splits, tiles_per_split;
    // few-tile batches (fp32 tiles of the ring kernel only): the column tiles of one launch may belong to
    // several row-major matrices that share x (the base weights of the layers of a group, and for each layer its
    // Wcat, so the routing products ride in the launch that reads W).  Segment e owns column tiles
    // [seg[e].tile0, seg[e+1].tile0) and writes fp32 tiles seg[e].partial[split][T][seg[e].rows].  nseg = 0: off.
    struct Segment {
        const bf16_t* W;   // [rows, d_in]
        float* partial;
        int rows, tile0;
    };
    static constexpr int kMaxSegments = 8;
    Segment seg[kMaxSegments];
    int nseg;
};

// LDS position of 16-byte chunk `chunk` of a 128-byte tile row.  A ds_read_b128 pass serves 16 lanes =
// 16 consecutive rows of one chunk; rows alternate between the two halves of the 64 banks, so rows 2m and
// 2m+1 may share a position and the 8 row pairs need 8 different ones: the pass then touches every bank
// once.  (chunk ^ (row & 7) puts rows m and m+8 on the same banks: a 2-way conflict on every read.)
__device__ __forceinline__ int swz(int row, int chunk) { return chunk ^ ((row >> 1) & 7); }

// Load a [ROWS x 64] bf16 tile (rows row0.., K columns k0..k0+64 of a row-major matrix with
// leading dimension ld) into registers: thread tid handles chunk (tid & 7) of rows (tid>>3) + 32*i.
template <int ROWS>
__device__ __forceinline__ void load_tile_regs(u32x4 (&regs)[ROWS / 32], const bf16_t* __restrict__ base, int ld,
                                               int row0, int nrows, int k0, int kmax, int tid) {
    const int chunk = tid & 7;
    const int kk = k0 + chunk * 8;
#pragma unroll
    for (int i = 0; i < ROWS / 32; ++i) {
        int row = row0 + (tid >> 3) + 32 * i;
        row = row < nrows ? row : nrows - 1;   // clamp: rows past the edge are computed but never stored
        if (kk < kmax)
            regs[i] = *reinterpret_cast<const u32x4*>(base + (size_t)row * ld + kk);
        else
            regs[i] = u32x4{0u, 0u, 0u, 0u};
    }
}

template <int ROWS>
__device__ __forceinline__ void store_tile_lds(const u32x4 (&regs)[ROWS / 32], bf16_t* lds_tile, int tid) {
    const int chunk = tid & 7;
#pragma unroll
    for (int i = 0; i < ROWS / 32; ++i) {
        const int row = (tid >> 3) + 32 * i;
        *reinterpret_cast<u32x4*>(lds_tile + row * kGemmBK + swz(row, chunk) * 8) = regs[i];
    }
}

template <int MI, int NI>
__device__ __forceinline__ void mma_tile(f32x16 (&acc)[MI][NI], const bf16_t* xs, const bf16_t* wsm, int wm, int wn,
                                         int lane) {
    const int lrow = lane & 31, khalf = lane >> 5;
#pragma unroll
    for (int ks = 0; ks < kGemmBK / 16; ++ks) {
        bf16x8 xf[MI], wf[NI];
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
            const int row = wm + mi * 32 + lrow;
            xf[mi] = *reinterpret_cast<const bf16x8*>(xs + row * kGemmBK + swz(row, ks * 2 + khalf) * 8);
        }
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
            const int row = wn + ni * 32 + lrow;
            wf[ni] = *reinterpret_cast<const bf16x8*>(wsm + row * kGemmBK + swz(row, ks * 2 + khalf) * 8);
        }
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
                acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[ni], xf[mi], acc[mi][ni], 0, 0, 0);
    }
}

template <int MI, int NI>
__global__ __launch_bounds__(256) void gemm_mfma_kernel(const GemmArgs a) {
    constexpr int BM = MI * 64, BN = NI * 64;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    bf16_t* smem = reinterpret_cast<bf16_t*>(smem_raw);
    // [2 buffers][x tile BM x 64 | w tile BN x 64]
    constexpr int kBufElems = (BM + BN) * kGemmBK;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = (wave >> 1) * (BM / 2), wn = (wave & 1) * (BN / 2);

    // XCD-aware tile order: consecutive workgroup ids go to different XCDs (8 of them), so give
    // each XCD a contiguous run of tiles, walked along n inside a band of tile rows.
    const int ntiles = a.tiles_m * a.tiles_n;
    int wg = blockIdx.x;
    {
        const int per_xcd = (ntiles + 7) / 8;
        const int xcd = wg % 8, local = wg / 8;
        const int remapped = xcd * per_xcd + local;
        wg = (local < per_xcd && remapped < ntiles && (ntiles % 8 == 0)) ? remapped : wg;
    }
    const int tile_m = wg / a.tiles_n, tile_n = wg % a.tiles_n;
    const int m0 = tile_m * BM, n0 = tile_n * BN;

    f32x16 acc[MI][NI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[mi][ni][i] = 0.f;

    const int nk_main = ceil_div(a.d_in, kGemmBK);
    const int nk_ext = a.ext_k > 0 ? a.ext_stride / kGemmBK : 0;
    const int nk = nk_main + nk_ext;

    u32x4 xr[BM / 32], wr[BN / 32];

    auto fetch = [&](int it) {   // global -> registers
        if (it < nk_main) {
            load_tile_regs<BM>(xr, a.x, a.d_in, m0, a.T, it * kGemmBK, a.d_in, tid);
            load_tile_regs<BN>(wr, a.W, a.d_in, n0, a.d_out, it * kGemmBK, a.d_in, tid);
        } else {
            load_tile_regs<BM>(xr, a.hd, a.ext_stride, m0, a.T, (it - nk_main) * kGemmBK, a.ext_stride, tid);
            load_tile_regs<BN>(wr, a.Bt, a.ext_stride, n0, a.d_out, (it - nk_main) * kGemmBK, a.ext_stride, tid);
        }
    };
    auto commit = [&](int, int buf) {   // registers -> LDS
        bf16_t* xs = smem + buf * kBufElems;
        store_tile_lds<BM>(xr, xs, tid);
        store_tile_lds<BN>(wr, xs + BM * kGemmBK, tid);
    };

    if (nk > 0) {
        fetch(0);
        commit(0, 0);
    }
    __syncthreads();
    for (int it = 0; it < nk; ++it) {
        const int buf = it & 1;
        if (it + 1 < nk) fetch(it + 1);
        const bf16_t* xs = smem + buf * kBufElems;
        mma_tile<MI, NI>(acc, xs, xs + BM * kGemmBK, wm, wn, lane);
        if (it + 1 < nk) commit(it + 1, buf ^ 1);
        __syncthreads();
    }

    // epilogue: lane holds, per block, 4 groups of 4 consecutive columns of token row (lane & 31)
    const int lrow = lane & 31, khalf = lane >> 5;
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
        const int row = m0 + wm + mi * 32 + lrow;
        if (row >= a.T) continue;
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int col = n0 + wn + ni * 32 + g * 8 + khalf * 4;
                if (col >= a.d_out) continue;   // d_out % 8 == 0, so a group of 4 is all in or all out
                uint2* dst = reinterpret_cast<uint2*>(a.out + (size_t)row * a.d_out + col);
                float v0 = acc[mi][ni][g * 4 + 0], v1 = acc[mi][ni][g * 4 + 1];
                float v2 = acc[mi][ni][g * 4 + 2], v3 = acc[mi][ni][g * 4 + 3];
                if (a.accumulate) {
                    const uint2 old = *dst;
                    v0 += bf16_bits_to_float(old.x & 0xffffu);
                    v1 += bf16_bits_to_float(old.x >> 16);
                    v2 += bf16_bits_to_float(old.y & 0xffffu);
                    v3 += bf16_bits_to_float(old.y >> 16);
                }
                uint2 pk;
                pk.x = pack_bf16x2(v0, v1);
                pk.y = pack_bf16x2(v2, v3);
                *dst = pk;
            }
        }
    }
}

// ------------------------------------------------------------------------------------------
// Two-slot version for few tokens: the tiles of both operands go from
// global memory straight into LDS with 16-byte buffer_load ... lds (no staging registers), the
// MFMA operand fragments are double-buffered in registers so the ds_reads of k-step s+1 are in
// flight while the MFMAs of k-step s run, and there is one barrier per 64-wide K tile, placed
// before the last k-step: behind it the next tile is visible, the tile after it is requested
// into the slot that has just been drained, and the first fragments of the next tile are read
// under the MFMAs of the last k-step.  The K tiles of the extension (hd x Bt) follow the main
// ones through the same pipeline; only the buffer resources and row strides change.
// ------------------------------------------------------------------------------------------
template <int MI, int NI>
struct Frags {
    bf16x8 x[MI];
    bf16x8 w[NI];
};

template <int MI, int NI>
__device__ __forceinline__ void load_frags(Frags<MI, NI>& f, const bf16_t* xs, const bf16_t* wsm, int wm, int wn,
                                           int lrow, int khalf, int ks) {
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
        const int row = wm + mi * 32 + lrow;
        f.x[mi] = *reinterpret_cast<const bf16x8*>(xs + row * kGemmBK + swz(row, ks * 2 + khalf) * 8);
    }
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
        const int row = wn + ni * 32 + lrow;
        f.w[ni] = *reinterpret_cast<const bf16x8*>(wsm + row * kGemmBK + swz(row, ks * 2 + khalf) * 8);
    }
}

// One MFMA operand fragment of k-step ks of an LDS tile pair: i < MI -> x block i, else W block i - MI.
template <int MI, int NI>
__device__ __forceinline__ void load_frag1(Frags<MI, NI>& f, const bf16_t* xs, const bf16_t* wsm, int wm, int wn,
                                           int lrow, int khalf, int ks, int i) {
    if (i < MI) {
        const int row = wm + i * 32 + lrow;
        f.x[i] = *reinterpret_cast<const bf16x8*>(xs + row * kGemmBK + swz(row, ks * 2 + khalf) * 8);
    } else {
        const int row = wn + (i - MI) * 32 + lrow;
        f.w[i - MI] = *reinterpret_cast<const bf16x8*>(wsm + row * kGemmBK + swz(row, ks * 2 + khalf) * 8);
    }
}

template <int MI, int NI>
__device__ __forceinline__ void mma_frags(f32x16 (&acc)[MI][NI], const Frags<MI, NI>& f) {
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
            acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.w[ni], f.x[mi], acc[mi][ni], 0, 0, 0);
}

// A [rows x 64-element-tiles] operand as the global->LDS loads see it.  An instruction moves 8 rows
// (8 lanes x 16 B per 128-byte tile row); lane (rsub, p) fetches the chunk whose swizzled position
// (see swz) is p, so the LDS image is the swizzled layout.  Wavefront `wave` moves rows (j*4 + wave)*8 .. +8 of the tile
// as piece j.  The address is rsrc base + voff (per lane: first row of piece 0, swizzled chunk)
// + a uniform offset (piece and K tile).  The resource covers exactly the matrix, so rows past
// its last one (ragged edge tiles) are out of range for the hardware and load zeros; they only
// feed output rows or columns that are never stored.
struct DmaOperand {
    __amdgpu_buffer_rsrc_t rsrc;
    uint32_t voff;        // per lane
    uint32_t piece_step;  // bytes between pieces: 32 rows
};

__device__ __forceinline__ DmaOperand dma_operand(const bf16_t* base, int nrows, int ld, int row0, int wave, int lane) {
    DmaOperand o;
    o.rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(base), 0, (uint32_t)nrows * (uint32_t)ld * 2u,
                                               0x00020000);
    // tile row of this lane in piece j: (j*4 + wave)*8 + rsub, so (row >> 1) & 7 = (wave & 1)*4 + (rsub >> 1)
    const int rsub = lane >> 3, p = lane & 7;
    o.voff = (uint32_t)(row0 + wave * 8 + rsub) * (uint32_t)ld * 2u +
             (uint32_t)((p ^ (((wave & 1) << 2) | (rsub >> 1))) << 4);
    o.piece_step = 32u * (uint32_t)ld * 2u;
    return o;
}

__device__ __forceinline__ void dma_piece(bf16_t* lds_tile, const DmaOperand& o, int ktile, int j, int wave) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        o.rsrc, (__attribute__((address_space(3))) void*)(lds_tile + (j * 4 + wave) * 8 * kGemmBK), 16, o.voff,
        (int)(o.piece_step * (uint32_t)j + (uint32_t)ktile * (kGemmBK * 2)), 0, 0);
}

// The K tiles behind the whole ones: first, where d_in is no multiple of 64, the rest of the main operands' columns (kt < 0),
// whose chunks past d_in load zeros, then those of the extension.  Both are requested by the same instructions, from
// the one resource or the other, so that no branch stands between loads and reads of LDS.  Base projections with tiles through registers for every such
// d_in, as it was, and so: 512 x 4104 -> 4096 68.5 and 38.1 us, 2000 97.8 and 69.1, 4096 173 and 97.7, 8192 x 4088 -> 4096 336
// and 195; with 4096 inputs 27.8, 55.0, 91.9 (rows of 8208 bytes straddle the lines of L2, which the lower tiles wait on).
struct PartTile {
    int columns;      // d_in % 64
    uint32_t offset;  // bytes from a row's start to the tile
    bool mine;        // this lane's chunk holds columns below d_in; if not it asks for what lies behind the matrix's last byte
};

__device__ __forceinline__ PartTile part_tile(int d_in, int wave, int lane) {
    PartTile t;
    t.columns = d_in % kGemmBK;
    t.offset = (uint32_t)(d_in / kGemmBK) * (kGemmBK * 2);
    t.mine = ((lane & 7) ^ (((wave & 1) << 2) | (lane >> 4))) * 8 < t.columns;
    return t;
}

// main_bytes: those of the main operand's matrix (with a piece's offset still below 2^32, see dma_ok).  PART, EXT: which there may be.
template <bool PART, bool EXT>
__device__ __forceinline__ void dma_piece_behind(bf16_t* lds_tile, const DmaOperand& main, uint32_t main_bytes, const DmaOperand& ext,
                                                 const PartTile& t, int kt, int j, int wave) {
    if constexpr (!PART) {
        dma_piece(lds_tile, ext, kt, j, wave);
    } else {
        const bool of_main = !EXT || kt < 0;
        const uint32_t voff = of_main ? (t.mine ? main.voff : main_bytes) : ext.voff;
        const uint32_t soff = of_main ? main.piece_step * (uint32_t)j + t.offset
                                      : ext.piece_step * (uint32_t)j + (uint32_t)kt * (kGemmBK * 2);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            of_main ? main.rsrc : ext.rsrc, (__attribute__((address_space(3))) void*)(lds_tile + (j * 4 + wave) * 8 * kGemmBK), 16,
            voff, (int)soff, 0, 0);
    }
}

// Map a workgroup id to an output tile: ids are dealt round-robin to the 8 XCDs, so each XCD
// gets a contiguous run of the tile order, and the order walks groups of 4 tile rows column by
// column: the 32 tiles an XCD works on at a time share few rows of x and W in its L2.
__device__ __forceinline__ void tile_of_workgroup(int wg, int tiles_m, int tiles_n, int& tile_m, int& tile_n) {
    const int ntiles = tiles_m * tiles_n;
    int id = wg;
    if (ntiles % 8 == 0) id = (wg % 8) * (ntiles / 8) + wg / 8;
    constexpr int GM = 4;
    const int group = id / (GM * tiles_n);
    const int first_m = group * GM;
    const int gm = min(GM, tiles_m - first_m);
    const int in_group = id - group * GM * tiles_n;
    tile_m = first_m + in_group % gm;
    tile_n = in_group / gm;
}

// Epilogue of the two-slot kernel: store a workgroup's 32 x 32 accumulators.
template <int MI, int NI>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& a, f32x16 (&acc)[MI][NI], unsigned char* smem_raw, int m0,
                                              int n0, int wm, int wn, int wave, int lane) {
    const int lrow = lane & 31, khalf = lane >> 5;
    // Epilogue.  A lane holds 4 consecutive columns per block row, so direct stores are 8-byte pieces
    // of 32 different rows per instruction; when the output is simply written (no split-K partials,
    // no accumulate) the bf16 tile is staged in this wavefront's own LDS region and stored as
    // 16-byte pieces that cover whole 128-byte lines.
    if (a.partial == nullptr && !a.accumulate) {
        constexpr int EST = gemm_epilogue_stride<NI>();   // bytes per staged row
        __syncthreads();                                   // every wavefront is done with the operand tiles
        unsigned char* ep = smem_raw + wave * (MI * 32) * EST;
        constexpr int LPR = NI * 4, RPI = 64 / LPR;        // lanes per staged row, rows per store instruction
        const int r_in = lane / LPR, c = (lane % LPR) * 8;
        const int col = n0 + wn + c;
        // one block row (32 tile rows) at a time, so the stores of a block row are under way while the next
        // one is converted; the region is this wavefront's own, and a wavefront's LDS accesses stay in order
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    uint2 pk;
                    pk.x = pack_bf16x2(acc[mi][ni][g * 4 + 0], acc[mi][ni][g * 4 + 1]);
                    pk.y = pack_bf16x2(acc[mi][ni][g * 4 + 2], acc[mi][ni][g * 4 + 3]);
                    *reinterpret_cast<uint2*>(ep + (mi * 32 + lrow) * EST + (ni * 32 + g * 8 + khalf * 4) * 2) = pk;
                }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int i = 0; i < 32 / RPI; ++i) {
                const int r = mi * 32 + i * RPI + r_in;
                const int row = m0 + wm + r;
                const u32x4 v = *reinterpret_cast<const u32x4*>(ep + r * EST + c * 2);
                if (row < a.T && col < a.d_out) *reinterpret_cast<u32x4*>(a.out + (size_t)row * a.d_out + col) = v;
            }
        }
        return;
    }

    if (a.partial != nullptr) {
        // fp32 split-K tile: same staging, one block row at a time, so the stores are 16-byte pieces of whole rows
        constexpr int PST = gemm_partial_stride<NI>();
        __syncthreads();
        unsigned char* ep = smem_raw + wave * 32 * PST;
        constexpr int PPR = NI * 8;                        // 16-byte pieces per staged row
        float* dst = a.partial + (size_t)blockIdx.y * a.T * a.d_out;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const f32x4 v = {acc[mi][ni][g * 4 + 0], acc[mi][ni][g * 4 + 1], acc[mi][ni][g * 4 + 2],
                                     acc[mi][ni][g * 4 + 3]};
                    *reinterpret_cast<f32x4*>(ep + lrow * PST + (ni * 32 + g * 8 + khalf * 4) * 4) = v;
                }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int i = 0; i < 32 * PPR / 64; ++i) {
                const int p = i * 64 + lane;
                const int r = p / PPR, c = (p % PPR) * 4;
                const int row = m0 + wm + mi * 32 + r, col = n0 + wn + c;
                const f32x4 v = *reinterpret_cast<const f32x4*>(ep + r * PST + c * 4);
                if (row < a.T && col < a.d_out) *reinterpret_cast<f32x4*>(dst + (size_t)row * a.d_out + col) = v;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        return;
    }

#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
        const int row = m0 + wm + mi * 32 + lrow;
        if (row >= a.T) continue;
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int col = n0 + wn + ni * 32 + g * 8 + khalf * 4;
                if (col >= a.d_out) continue;
                float v0 = acc[mi][ni][g * 4 + 0], v1 = acc[mi][ni][g * 4 + 1];
                float v2 = acc[mi][ni][g * 4 + 2], v3 = acc[mi][ni][g * 4 + 3];
                uint2* dst = reinterpret_cast<uint2*>(a.out + (size_t)row * a.d_out + col);
                if (a.accumulate) {
                    const uint2 old = *dst;
                    v0 += bf16_bits_to_float(old.x & 0xffffu);
                    v1 += bf16_bits_to_float(old.x >> 16);
                    v2 += bf16_bits_to_float(old.y & 0xffffu);
                    v3 += bf16_bits_to_float(old.y >> 16);
                }
                uint2 pk;
                pk.x = pack_bf16x2(v0, v1);
                pk.y = pack_bf16x2(v2, v3);
                *dst = pk;
            }
        }
    }
}

// PART: the inputs may end in a partial K tile
template <int MI, int NI, bool PART>
__global__ __launch_bounds__(256) void gemm_mfma_dma_kernel(const GemmArgs a) {
    constexpr int BM = MI * 64, BN = NI * 64;
    constexpr int PX = BM / 32, PW = BN / 32;   // pieces per wavefront per tile
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    bf16_t* smem = reinterpret_cast<bf16_t*>(smem_raw);
    constexpr int kBufElems = (BM + BN) * kGemmBK;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: keeps LDS bases in SGPRs
    const int wm = (wave >> 1) * (BM / 2), wn = (wave & 1) * (BN / 2);
    const int lrow = lane & 31, khalf = lane >> 5;
    int tile_m, tile_n;
    tile_of_workgroup(blockIdx.x, a.tiles_m, a.tiles_n, tile_m, tile_n);
    const int m0 = tile_m * BM, n0 = tile_n * BN;

    f32x16 acc[MI][NI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[mi][ni][i] = 0.f;

    // this workgroup's share of the contraction: whole K tiles [kt0, kt0 + nk_main), the partial one, and/or the extension
    int kt0 = 0, nk_main = a.d_in / kGemmBK, nk_part = PART && a.d_in % kGemmBK != 0 ? 1 : 0;
    int nk_ext = a.ext_k > 0 ? a.ext_stride / kGemmBK : 0;
    if (a.partial != nullptr) {
        const int split = blockIdx.y;
        if (split < a.splits) {
            kt0 = split * a.tiles_per_split;
            if (nk_main < kt0 || nk_main >= kt0 + a.tiles_per_split) nk_part = 0;
            nk_main = max(0, min(a.tiles_per_split, nk_main - kt0));
            nk_ext = 0;
        } else {
            nk_main = nk_part = 0;
        }
    }
    const int nk = nk_main + nk_part + nk_ext;

    // (x, W) feed local tiles [0, nk_main + nk_part), (hd, Bt) the tiles after them
    const DmaOperand ox = dma_operand(a.x, a.T, a.d_in, m0, wave, lane);
    const DmaOperand ow = dma_operand(a.W, a.d_out, a.d_in, n0, wave, lane);
    const DmaOperand oh = dma_operand(a.hd, nk_ext > 0 ? a.T : 0, a.ext_stride, m0, wave, lane);
    const DmaOperand ob = dma_operand(a.Bt, nk_ext > 0 ? a.d_out : 0, a.ext_stride, n0, wave, lane);
    const PartTile part = part_tile(a.d_in, wave, lane);
    const uint32_t x_bytes = (uint32_t)a.T * (uint32_t)a.d_in * 2u, w_bytes = (uint32_t)a.d_out * (uint32_t)a.d_in * 2u;

    // piece i of local tile `it` (x-like pieces first) into LDS slot `slot`
    auto request_piece = [&](int it, int slot, int i, auto is_ext) {
        bf16_t* xs = smem + slot * kBufElems;
        if constexpr (decltype(is_ext)::value) {
            const int kt = it - nk_main - nk_part;
            if (i < PX) dma_piece_behind<PART, true>(xs, ox, x_bytes, oh, part, kt, i, wave);
            else dma_piece_behind<PART, true>(xs + BM * kGemmBK, ow, w_bytes, ob, part, kt, i - PX, wave);
        } else {
            if (i < PX) dma_piece(xs, ox, kt0 + it, i, wave);
            else dma_piece(xs + BM * kGemmBK, ow, kt0 + it, i - PX, wave);
        }
    };
    auto request_tile = [&](int it, int slot) {
#pragma unroll
        for (int i = 0; i < PX + PW; ++i) {
            if (it < nk_main) request_piece(it, slot, i, std::false_type{});
            else request_piece(it, slot, i, std::true_type{});
        }
    };

    Frags<MI, NI> f0, f1;
    if (nk > 1) {
        // both slots are free: request the first two tiles together, wait for the older one only
        request_tile(0, 0);
        request_tile(1, 1);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PX + PW) : "memory");
        __syncthreads();
        load_frags<MI, NI>(f0, smem, smem + BM * kGemmBK, wm, wn, lrow, khalf, 0);
    } else if (nk > 0) {
        request_tile(0, 0);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        load_frags<MI, NI>(f0, smem, smem + BM * kGemmBK, wm, wn, lrow, khalf, 0);
    }
    // One K tile = 4 phases of (MI*NI MFMA + the fragment reads of the next k-step); sched_barrier keeps
    // each phase's reads from sinking into the next phase, where they would be waited on at once.
    auto phase = [&](Frags<MI, NI>& fnext, const Frags<MI, NI>& fcur, const bf16_t* xs, int ks) {
        load_frags<MI, NI>(fnext, xs, xs + BM * kGemmBK, wm, wn, lrow, khalf, ks);
        mma_frags<MI, NI>(acc, fcur);
        __builtin_amdgcn_sched_barrier(0);
    };
    // REQ: 0 = tile it+2 is a whole main tile, 1 = it is one behind those, 2 = there is none (last two tiles)
    auto tile_step = [&](int it, auto req) {
        constexpr int REQ = decltype(req)::value;
        const bf16_t* xs = smem + (it & 1) * kBufElems;
        phase(f1, f0, xs, 1);
        phase(f0, f1, xs, 2);
        phase(f1, f0, xs, 3);
        // tile it+1 (requested one tile ago) must have landed; every wavefront has read tile it
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        const bf16_t* xn = smem + ((it + 1) & 1) * kBufElems;
        if constexpr (REQ < 2) {
            // Program order = the order the LDS accesses must keep (the compiler does not move an LDS
            // read across a global->LDS load): the first fragments of tile it+1 with pieces of tile
            // it+2 between them, then the remaining pieces; tile it+2 goes into the slot just drained.
            constexpr int NR = MI + NI, NPC = PX + PW;
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                load_frag1<MI, NI>(f0, xn, xn + BM * kGemmBK, wm, wn, lrow, khalf, 0, i);
                request_piece(it + 2, it & 1, i, std::integral_constant<bool, REQ == 1>{});
            }
#pragma unroll
            for (int i = NR; i < NPC; ++i) request_piece(it + 2, it & 1, i, std::integral_constant<bool, REQ == 1>{});
            mma_frags<MI, NI>(acc, f1);
        } else {
            if (it + 1 < nk) load_frags<MI, NI>(f0, xn, xn + BM * kGemmBK, wm, wn, lrow, khalf, 0);
            mma_frags<MI, NI>(acc, f1);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    int it = 0;
    for (; it + 2 < nk_main; ++it) tile_step(it, std::integral_constant<int, 0>{});
    for (; it + 2 < nk; ++it) tile_step(it, std::integral_constant<int, 1>{});
    for (; it < nk; ++it) tile_step(it, std::integral_constant<int, 2>{});

    gemm_epilogue<MI, NI>(a, acc, smem_raw, m0, n0, wm, wn, wave, lane);
}

// ------------------------------------------------------------------------------------------
// The same pipeline with a ring of D x-slots and D+1 W-slots: the loads of D K tiles are in flight.  D = 2 fills the
// whole 160 KB of LDS for the 256 x 256 tile; smaller tiles of one workgroup per CU take as many slots as fit, since
// with two their K tile is shorter than a load's latency (300 x 4096 -> 4096 as K-split 160 x 128 tiles, 22 K tiles
// each: 21 us with D = 4, 28.9 us with 256 x 128 tiles and D = 2; 512 rows, 256 x 128 tiles: 26.8 against 29.7 us).
// A global->LDS load occupies the CU's address unit for ~16 cycles, so the
// four wavefronts can sustain one load per two 32-cycle MFMAs each; issued in one burst (all pieces of a tile in
// the last phase, the only time a slot of x is free) they stall the MFMAs queued behind them.
// So tile it+D's W pieces go out during the first k-step of tile it, into the W-slot that no
// wavefront has read since the previous barrier, and only its x pieces wait for the barrier, spread over
// the MFMAs of the second.  Loads complete in order, so the barrier of tile it waits for everything
// but the newest tiles and W pieces (vmcnt).
//
// The contraction runs on v_mfma_f32_16x16x32_bf16: on the layer's data the chip is power-limited, and per multiply
// this shape reads and writes half as many accumulator registers as 32x32x16.  Measured against the same kernel with
// 32x32x16 (256 x 256 tiles, extension of 256, back to back): 95.1 against 104-106 us at 4096 x 4096 x 4096, 666
// against 725 us at 8192 x 4096 x 14336; inside the layer 101.2 against 111.2 us.  The instruction is written in assembly with the accumulator tied in an AGPR: from the builtin
// the compiler lets the result land in other registers than the accumulator and moves about 100 of them per K tile.
// The compiler does not know that the statement is an MFMA, so (1) the source states the order of MFMAs, LDS reads
// and loads itself, group by group between scheduling barriers; (2) nothing but MFMAs touches an accumulator inside
// the K loop, and mfma_drain() stands between the last MFMA and the first read of a result; (3) the accumulators' first
// values are written ahead of mfma_start(), two wait states or more before the first MFMA.  What the source cannot state
// (that the compiler writes no copy of a fragment right in front of an MFMA) tests/test_mfma_waits_host.py checks in the
// assembly of every instance.
// ------------------------------------------------------------------------------------------
template <int MB, int NB, int D>
__host__ __device__ constexpr int gemm_ring_lds_bytes() {
    constexpr int ring = (D * MB * 32 + (D + 1) * NB * 32) * kGemmBK * 2;
    constexpr int stage = 4 * 32 * (NB * 64 + 16);   // the widest epilogue: 32 fp32 rows per wavefront
    return ring > stage ? ring : stage;
}

// how many of NPC pieces go out right after the i-th of NR fragment reads (evenly spread, the last read included)
__host__ __device__ constexpr int pieces_after_read(int i, int NPC, int NR) {
    return (i + 1) * NPC / NR - i * NPC / NR;
}

constexpr int kEpiStore = 0, kEpiAccumulate = 1, kEpiPartial = 2, kEpiPartialThrough = 3;
// Cache policy of the output's stores ("sc1"): written through the L2.  Where all workgroups of a launch end together,
// lines left in the L2 are only written back when the launch is over, and the next one waits for that.  Whole calls,
// ordinary stores, "nt", "sc1": the fp32 tiles of 300 x 4096 -> 4096 26.35, 25.6, 25.2 us, of 1531 x 4096 -> 1024 of rank
// 16 38.1, 37.75, 36.7; bf16 outputs: a training step of 4096 tokens 273.1 and 271.0 ("sc1"), 3000 x 5120 -> 5120 from its
// parts 174.5 and 172.8.  The routing products on 128 x 128 tiles (kEpiPartial, two workgroups per CU at different stages) gain
// nothing: 4096 tokens 120.9 and 121.7.  bf16 outputs beside weights that come from HBM, 96 to 4096 tokens, base projections and
// whole layers of 4096 -> 4096 and 14336, 14336 -> 4096, 5120 -> 5120 and 13824, ordinary and "sc1": 3% faster to 0.7% slower.
// The ends: 2000 x 4096 -> 4096 54.0 and 52.2, 700 x 4096 -> 14336 with adapters 92.3 and 90.1; 3000 x 4096 -> 14336 256.5
// and 258.4 (two runs 1.2% apart), 160 x 5120 -> 13824 53.3 and 53.6.
constexpr int kWriteThrough = 16;
// Epilogue of the ring kernel.  EPI fixes at compile time which form a kernel carries: with one form the
// accumulators leave their registers as they are converted (with all three behind run-time branches the compiler
// copies every accumulator out, and spills, before it branches).  A lane holds 4 consecutive output columns of token
// row l & 15 per block; the tile is staged in this wavefront's own LDS region, RS rows at a time, and leaves as
// 16-byte pieces that cover whole rows (the direct 8-byte stores touch 16 rows per instruction; with accumulate the
// old output comes in by the same pieces: 24.6 against 36.4 us for 3000 x 5120 outputs and K = 224).
template <int MB, int NB, int EPI>
__device__ __forceinline__ void gemm_epilogue16(const GemmArgs& a, f32x4 (&acc)[MB][NB], unsigned char* smem_raw, int m0,
                                                int n0, int wm, int wn, int wave, int lane) {
    constexpr bool F32 = EPI == kEpiPartial || EPI == kEpiPartialThrough;
    constexpr int POLICY = EPI == kEpiPartial ? 0 : kWriteThrough;
    constexpr int RS = MB % 2 == 0 ? 32 : 16;                  // staged rows
    constexpr int EB = F32 ? 4 : 2;                            // bytes per staged value
    constexpr int EST = NB * 16 * EB + 16;                     // bytes per staged row
    constexpr int PPR = NB * 16 * EB / 16;                     // 16-byte pieces per staged row
    constexpr int NP = RS * PPR / 64;                          // pieces per lane
    static_assert(RS * PPR % 64 == 0, "whole wavefronts of pieces");
    const int l15 = lane & 15, kq = lane >> 4;
    __syncthreads();                                           // every wavefront is done with the operand tiles
    unsigned char* ep = smem_raw + wave * RS * EST;            // this wavefront's own; its LDS accesses stay in order
    // The workgroup's rows of the output as a buffer: pieces past its last row or column are dropped by the hardware.
    // The whole offset of a piece is in the per-lane operand, which the bounds check covers.
    constexpr int BM = MB * 32;
    void* base = F32 ? (void*)(a.partial + ((size_t)blockIdx.y * a.T + m0) * a.d_out) : (void*)(a.out + (size_t)m0 * a.d_out);
    const uint32_t row_bytes = (uint32_t)a.d_out * EB;
    const __amdgpu_buffer_rsrc_t out =
        __builtin_amdgcn_make_buffer_rsrc(base, 0, (uint32_t)min(a.T - m0, BM) * row_bytes, 0x00020000);
    const uint32_t kOutside = 0xffffffffu;
    uint32_t voff[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        const int p = i * 64 + lane, col = n0 + wn + (p % PPR) * (16 / EB);   // d_out % 8 == 0: all in or all out
        voff[i] = col < a.d_out ? (uint32_t)(wm + p / PPR) * row_bytes + (uint32_t)col * EB : kOutside;
    }
    auto offset = [&](int i, int mb) {
        return voff[i] == kOutside ? kOutside : voff[i] + (uint32_t)(mb * 16) * row_bytes;
    };
    auto sync = [] {   // orders this wavefront's own LDS accesses
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
#pragma unroll
    for (int mb = 0; mb < MB; mb += RS / 16) {
        if constexpr (EPI == kEpiAccumulate) {   // the old output comes in the way the new one leaves
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const int p = i * 64 + lane;
                *reinterpret_cast<u32x4*>(ep + (p / PPR) * EST + (p % PPR) * 16) =
                    __builtin_amdgcn_raw_buffer_load_b128(out, offset(i, mb), 0, 0);
            }
            sync();
        }
#pragma unroll
        for (int h = 0; h < RS / 16; ++h)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                f32x4 v = acc[mb + h][nb];
                unsigned char* dst = ep + (h * 16 + l15) * EST + (nb * 16 + kq * 4) * EB;
                if constexpr (F32) {
                    *reinterpret_cast<f32x4*>(dst) = v;
                } else {
                    if constexpr (EPI == kEpiAccumulate) {
                        const uint2 old = *reinterpret_cast<const uint2*>(dst);
                        v[0] += bf16_bits_to_float(old.x & 0xffffu);
                        v[1] += bf16_bits_to_float(old.x >> 16);
                        v[2] += bf16_bits_to_float(old.y & 0xffffu);
                        v[3] += bf16_bits_to_float(old.y >> 16);
                    }
                    uint2 pk;
                    pk.x = pack_bf16x2(v[0], v[1]);
                    pk.y = pack_bf16x2(v[2], v[3]);
                    *reinterpret_cast<uint2*>(dst) = pk;
                }
            }
        sync();
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int p = i * 64 + lane;
            const u32x4 v = *reinterpret_cast<const u32x4*>(ep + (p / PPR) * EST + (p % PPR) * 16);
            __builtin_amdgcn_raw_buffer_store_b128(v, out, offset(i, mb), 0, POLICY);
        }
        sync();
        __builtin_amdgcn_sched_barrier(0);   // accumulators leave their registers 32 rows at a time
    }
}

// Which K tiles of the extension hold anything for tokens row0 .. row0 + ROWS - 1: with a skewed load most adapters are in
// no token's choice.  Where every tile holds something the look at the routing must cost nothing, so the ids, which lie
// next to each other, are read 16 bytes a lane, all at once and ahead of the first operand tiles, on whose arrival the
// workgroup waits anyway.  Layers of 4096 -> 4096 without a look, with one id after the other read up front, and so:
// 4096 tokens, 64 adapters of rank 32, top-4, every tile in use 206.3, 210.4, 206.0 us, logits falling off as -2 log(j)
// 198.1, 176.3, 172.7; 28 adapters of rank 8, top-8 (four tiles) 123.5, 129.1, 123.9.
template <int ROWS>
struct ExtIds {
    static constexpr int P = ROWS * kMaxTopK / 256;   // pieces of 4 ids per lane
    u32x4 v[P];
    int n;
    __device__ __forceinline__ void load(const GemmArgs& a, int row0, int lane) {
        n = min(ROWS, a.T - row0) * a.topk;
        const __amdgpu_buffer_rsrc_t ids = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<int32_t*>(a.topk_idx) + (size_t)row0 * a.topk, 0, (uint32_t)n * 4, 0x00020000);
#pragma unroll
        for (int i = 0; i < P; ++i)   // the last piece again past the end (fewer than 4 ids: zeros)
            v[i] = __builtin_amdgcn_raw_buffer_load_b128(ids, max(min((i * 64 + lane) * 16, n * 4 - 16), 0), 0, 0);
    }
    // Bit e = one of the tokens selected an adapter with columns in tile e (or an id outside [0, N) that shares its low
    // bits with such a one: that tile is multiplied for nothing).  Uniform over the wavefront.
    __device__ __forceinline__ uint64_t used(const GemmArgs& a, int lane) const {
        uint64_t mine = 0;   // adapters
#pragma unroll
        for (int i = 0; i < P; ++i) {
            if (i * 256 >= n) break;
#pragma unroll
            for (int j = 0; j < 4; ++j) mine |= 1ull << (v[i][j] & (kMaxAdapters - 1));
        }
        const uint64_t all = (uint64_t)wave_or((uint32_t)(mine >> 32)) << 32 | wave_or((uint32_t)mine);
        // lane = tile: its columns belong to adapters lo to hi (the halves keep the quotients clear of whole numbers)
        const float inv = 1.f / (float)a.rank;
        const int lo = min((int)((lane * kGemmBK + 0.5f) * inv), 63), hi = min((int)((lane * kGemmBK + 63.5f) * inv), 63);
        return __ballot(lane * kGemmBK < a.ext_k && (all >> lo << lo & ~0ull >> (63 - hi)) != 0);
    }
};

// Fragments of one k-step of 32 for a wavefront's MB x NB blocks of 16 x 16: lane l holds row (l & 15), k chunk l >> 4.
template <int MB, int NB>
struct Frags16 {
    bf16x8 x[MB];
    bf16x8 w[NB];
};

__device__ __forceinline__ void mfma16(f32x4& acc, const bf16x8& w, const bf16x8& x) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(w), "v"(x));
}
// The accumulators' first values, in place here: an MFMA may read a register two wait states after another vector
// instruction has written it (the compiler sees to that for the builtin only).
template <int MB, int NB>
__device__ __forceinline__ void mfma_start(f32x4 (&acc)[MB][NB]) {
#pragma unroll
    for (int mi = 0; mi < MB; ++mi)
#pragma unroll
        for (int ni = 0; ni < NB; ++ni) {
            acc[mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};
            asm volatile("" : "+a"(acc[mi][ni]));
        }
    asm volatile("s_nop 1" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}
// The wait states between an MFMA and another instruction's read of its result (the compiler inserts them for the
// builtin only; 16x16x32 is 8 passes: at most 12 are required).
__device__ __forceinline__ void mfma_drain() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}
// The same for what the compiler may read: behind this statement, and not before it, the accumulators have values.  (The
// wait alone does not say so: where the K loop's exits meet, reads of a result have been moved in front of it.)
template <int MB, int NB>
__device__ __forceinline__ void mfma_results(f32x4 (&acc)[MB][NB]) {
    mfma_drain();
#pragma unroll
    for (int mi = 0; mi < MB; ++mi)
#pragma unroll
        for (int ni = 0; ni < NB; ++ni) asm volatile("" : "+a"(acc[mi][ni]));
    __builtin_amdgcn_sched_barrier(0);
}

// Order of the MB x NB products of a k-step: 2 x 2 micro-blocks, each a cycle, walked as a snake, so that one operand
// register changes from one MFMA to the next (0.5% less time than sweeping whole rows).  An odd last row is swept; with an odd
// number of columns rows and columns change places.
template <int R, int C>
__host__ __device__ constexpr int snake_row(int k) {
    return k >= R / 2 * 2 * C ? R - 1 : (k / (2 * C)) * 2 + ((k >> 1) & 1);
}
template <int R, int C>
__host__ __device__ constexpr int snake_col(int k) {
    if (k >= R / 2 * 2 * C) return k - R / 2 * 2 * C;
    const int col = (k >> 2) % (C / 2), in = k & 3;
    return (((k / (2 * C)) & 1) ? C / 2 - 1 - col : col) * 2 + ((in == 1 || in == 2) ? 1 : 0);
}
template <int MB, int NB>
__host__ __device__ constexpr int order_mi(int k) {
    if constexpr (NB % 2 == 0) return snake_row<MB, NB>(k);
    else return snake_col<NB, MB>(k);
}
template <int MB, int NB>
__host__ __device__ constexpr int order_ni(int k) {
    if constexpr (NB % 2 == 0) return snake_col<MB, NB>(k);
    else return snake_row<NB, MB>(k);
}

// Fragment number i in the order the MFMAs need them: two of the operand that is walked in pairs (x; W with an odd NB), every
// one of the other, the rest of the first.
template <int MB, int NB>
__device__ __forceinline__ void load_frag16(Frags16<MB, NB>& f, const bf16_t* xs, const bf16_t* wsm, int wm, int wn, int l15,
                                            int kq, int ks, int i) {
    constexpr bool XPAIRS = NB % 2 == 0;
    constexpr int OTHER = XPAIRS ? NB : MB;
    const bool other = i >= 2 && i < 2 + OTHER;
    const int n = other ? i - 2 : i < 2 ? i : i - OTHER;
    if (other == XPAIRS) {
        const int row = wn + n * 16 + l15;
        f.w[n] = *reinterpret_cast<const bf16x8*>(wsm + row * kGemmBK + swz(row, ks * 4 + kq) * 8);
    } else {
        const int row = wm + n * 16 + l15;
        f.x[n] = *reinterpret_cast<const bf16x8*>(xs + row * kGemmBK + swz(row, ks * 4 + kq) * 8);
    }
}

template <int... PH, typename F>
__device__ __forceinline__ void for_each_phase(std::integer_sequence<int, PH...>, F f) {
    (f(std::integral_constant<int, PH>{}), ...);
}

// BEHIND: which K tiles there may be behind the whole ones of the main operands: the partial one (see PartTile), those of the
// extension, and whether the kernel looks for empty ones among these.  Code that is not run costs a short call with cold weights 0.8 us
// (65 x 1024 -> 4096 11.5 with the look against 10.6), and two more buffer resources and the tests of what there is cost the others 0.3 to
// 0.5% and more: whole calls, any and none, 300 x 4096 -> 4096 25.1 and 24.7 us, 1531 x 4096 -> 1024 of rank 16 37.2 and 36.4, 3000 x
// 5120 -> 5120 from its parts 170.4 and 169.1, a training step of 4096 x 4096 -> 4096 263.9 and 261.7.  Calls that are mostly extension
// feel the choice between its operands and the partial tile's in every request, with it and without: 1846 x 512 -> 856, 64 adapters of rank
// 32 (8 K tiles and 32 of the extension) 53.9 and 51.2, 137 x 256 -> 4096 40.7 and 40.1, lora_forward of 40 x 624 -> 5120 20.8 and 20.6.
constexpr int kBehindNone = 0, kBehindPart = 1, kBehindExt = 2, kBehindAny = 3, kBehindExtLook = 6, kBehindAnyLook = 7;

template <int MB, int NB, int D, int EPI, int BEHIND>
__global__ __launch_bounds__(256) void gemm_mfma_ring_kernel(const GemmArgs a_in) {
    GemmArgs a = a_in;
    constexpr bool PART = (BEHIND & 1) != 0, EXT = (BEHIND & 2) != 0, LOOK = (BEHIND & 4) != 0, ANY = BEHIND != kBehindNone;
    constexpr int BM = MB * 32, BN = NB * 32;   // 2 x 2 wavefronts of MB x NB blocks of 16 x 16
    constexpr int PX = BM / 32, PW = BN / 32;   // pieces per wavefront per tile
    static_assert((NB % 2 == 0 || MB % 2 == 0) && D >= 2 && (D - 1) * (PX + PW) < 64, "whole 2 x 2 micro-blocks; vmcnt holds 6 bits");
    constexpr int NR = MB + NB, NM = MB * NB;   // fragment reads and MFMAs per k-step
    // MFMAs per fragment read: k-step 0's reads (of k-step 1) end early, since the barrier waits for them; k-step 1's
    // (of the next tile) are spread over all of it
    constexpr int RA = NM * 3 / 4 / NR > 0 ? NM * 3 / 4 / NR : 1, RB = NM / NR;
    static_assert(RB >= 1, "a k-step needs one MFMA per fragment read");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    bf16_t* smem = reinterpret_cast<bf16_t*>(smem_raw);
    constexpr int kXElems = BM * kGemmBK, kWElems = BN * kGemmBK;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = (wave >> 1) * (BM / 2), wn = (wave & 1) * (BN / 2);
    const int l15 = lane & 15, kq = lane >> 4;
    int tile_m, tile_n;
    tile_of_workgroup(blockIdx.x, a.tiles_m, a.tiles_n, tile_m, tile_n);
    const int m0 = tile_m * BM;
    int n0 = tile_n * BN;
    if (a.nseg > 0) {   // uniform: the tile is an ordinary tile of its segment's matrix (split-K launches only)
        int e = 0;
        for (int i = 1; i < a.nseg; ++i)
            if (tile_n >= a_in.seg[i].tile0) e = i;
        n0 = (tile_n - a_in.seg[e].tile0) * BN;
        a.W = a_in.seg[e].W;
        a.d_out = a_in.seg[e].rows;
        a.partial = a_in.seg[e].partial;
    }

    // this workgroup's share of the contraction: whole K tiles [kt0, kt0 + nk_main), the partial one, and/or the extension
    int kt0 = 0, nk_main = a.d_in / kGemmBK, nk_part = PART && a.d_in % kGemmBK != 0 ? 1 : 0;
    int nk_ext = EXT && a.ext_k > 0 ? a.ext_stride / kGemmBK : 0;
    if (a.partial != nullptr) {
        kt0 = (int)blockIdx.y * a.tiles_per_split;
        if (nk_main < kt0 || nk_main >= kt0 + a.tiles_per_split) nk_part = 0;
        nk_main = max(0, min(a.tiles_per_split, nk_main - kt0));
        if ((int)blockIdx.y != a.splits - 1) nk_ext = 0;
    }
    const bool look = LOOK && nk_ext > 0 && a.topk_idx != nullptr;   // uniform
    ExtIds<BM> ids;
    if (look) ids.load(a, m0, lane);

    const DmaOperand ox = dma_operand(a.x, a.T, a.d_in, m0, wave, lane);
    const DmaOperand ow = dma_operand(a.W, a.d_out, a.d_in, n0, wave, lane);
    const DmaOperand oh = dma_operand(a.hd, nk_ext > 0 ? a.T : 0, a.ext_stride, m0, wave, lane);
    const DmaOperand ob = dma_operand(a.Bt, nk_ext > 0 ? a.d_out : 0, a.ext_stride, n0, wave, lane);
    const PartTile part = part_tile(a.d_in, wave, lane);
    const uint32_t x_bytes = (uint32_t)a.T * (uint32_t)a.d_in * 2u, w_bytes = (uint32_t)a.d_out * (uint32_t)a.d_in * 2u;

    auto xslot = [&](int it) { return smem + (it % D) * kXElems; };
    auto wslot = [&](int it) { return smem + D * kXElems + (it % (D + 1)) * kWElems; };
    // piece i of the x-like / W-like operand of whole K tile kt, or of tile kt of those behind the whole ones
    auto request_x = [&](bf16_t* slot, int kt, int i, auto is_ext) {
        if constexpr (decltype(is_ext)::value) dma_piece_behind<PART, EXT>(slot, ox, x_bytes, oh, part, kt, i, wave);
        else dma_piece(slot, ox, kt, i, wave);
    };
    auto request_w = [&](bf16_t* slot, int kt, int i, auto is_ext) {
        if constexpr (decltype(is_ext)::value) dma_piece_behind<PART, EXT>(slot, ow, w_bytes, ob, part, kt, i, wave);
        else dma_piece(slot, ow, kt, i, wave);
    };
    auto request_tile = [&](int it, int kt, auto is_ext) {
#pragma unroll
        for (int i = 0; i < PX; ++i) request_x(xslot(it), kt, i, is_ext);
#pragma unroll
        for (int i = 0; i < PW; ++i) request_w(wslot(it), kt, i, is_ext);
    };
    // the extension's K tiles: all of them, or those that hold anything for this workgroup's tokens
    uint64_t ext_left = nk_ext >= 64 ? ~0ull : (1ull << nk_ext) - 1;
    f32x4 acc[MB][NB];
    if (!LOOK || nk_main >= D) {
#pragma unroll
        for (int t = 0; t < D; ++t)
            if (LOOK || t < nk_main) request_tile(t, kt0 + t, std::false_type{});
        mfma_start<MB, NB>(acc);   // while the first tile is on its way
        if (look) ext_left &= ids.used(a, lane);
    } else {   // looks by itself: behind a join of the two branches the compiler would wait for every load
#pragma unroll
        for (int t = 0; t < D - 1; ++t)
            if (t < nk_main) request_tile(t, kt0 + t, std::false_type{});
        mfma_start<MB, NB>(acc);
        if (look) ext_left &= ids.used(a, lane);
    }
    // the last tile may hold data in its first k-step only (28 adapters of rank 8: 224 of 256 columns; the rest is zero
    // padding): that k-step is all it gets
    bool half_last = nk_ext > 0 && ((a.ext_k - 1) % kGemmBK) < kGemmBK / 2 && (ext_left >> (nk_ext - 1) & 1) != 0;
    nk_ext = __popcll(ext_left);
    if (PART && nk_ext == 0) half_last = nk_part > 0 && part.columns <= kGemmBK / 2;
    const int nk = nk_main + nk_part + nk_ext;
    // tiles are requested in order: the one that comes next behind the whole ones, see PartTile
    auto next_ext = [&]() {
        if (PART && nk_part > 0) {
            nk_part = 0;
            return -1;
        }
        const int e = __ffsll((unsigned long long)ext_left) - 1;
        ext_left &= ext_left - 1;
        return e;
    };
#pragma unroll
    for (int t = 0; t < D; ++t)
        if (ANY && t >= nk_main && t < nk) request_tile(t, next_ext(), std::true_type{});

    Frags16<MB, NB> f0, f1;
    // tile t is needed next: the loads of at most `left` tiles, requested after it, may still be in flight
    auto wait_tiles = [&](int left) {
        if (D > 4 && left >= 4) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(D > 4 ? 4 * (PX + PW) : 0) : "memory");
        else if (D > 3 && left == 3) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(D > 3 ? 3 * (PX + PW) : 0) : "memory");
        else if (D > 2 && left == 2) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(D > 2 ? 2 * (PX + PW) : 0) : "memory");
        else if (left == 1) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(PX + PW) : "memory");
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    };
    static_assert(D <= 5, "wait_tiles");
    if (nk > 0) {
        wait_tiles(min(nk, D) - 1);
#pragma unroll
        for (int i = 0; i < NR; ++i) load_frag16<MB, NB>(f0, xslot(0), wslot(0), wm, wn, l15, kq, 0, i);
    }

    // MFMAs [K0, K1) of a k-step
    auto mfmas = [&](const Frags16<MB, NB>& f, int k0, int k1) {
#pragma unroll
        for (int k = k0; k < k1; ++k)
            mfma16(acc[order_mi<MB, NB>(k)][order_ni<MB, NB>(k)], f.w[order_ni<MB, NB>(k)], f.x[order_mi<MB, NB>(k)]);
    };
    // Where tile `it` lies, outside the unrolled main loop: carried along, since the remainders by D and D + 1 sit between
    // two tiles (64 K tiles of 128 x 128, one workgroup per CU, D = 4: 27.2 us with them, 24.5 without)
    int slot_x = 0, slot_w = D * kXElems;
    // REQ: 0 = tile it+D is a whole main tile, 1 = it is one behind those, 2 = there is none (last D tiles)
    // PH: `it` in its trip when it is known at compile time (the unrolled main loop: every slot address is then a
    // constant and no address arithmetic sits between two tiles), -1 otherwise
    auto tile_step = [&](int it, auto req, auto ph) __attribute__((always_inline)) {
        constexpr int REQ = decltype(req)::value, PH = decltype(ph)::value;
        using IsExt = std::integral_constant<bool, REQ == 1>;
        auto xsl = [&](int d) {   // x-slot / W-slot of tile it + d, d = 0, 1 or D
            if constexpr (PH >= 0) return smem + ((PH + d) % D) * kXElems;
            else return smem + (d != 1 ? slot_x : slot_x == (D - 1) * kXElems ? 0 : slot_x + kXElems);
        };
        auto wsl = [&](int d) {
            constexpr int first = D * kXElems, last = first + D * kWElems;
            if constexpr (PH >= 0) return smem + first + ((PH + d) % (D + 1)) * kWElems;
            else if (d == 0) return smem + slot_w;
            else if (d == 1) return smem + (slot_w == last ? first : slot_w + kWElems);
            else return smem + (slot_w == first ? last : slot_w - kWElems);
        };
        const bf16_t* xs = xsl(0);
        const bf16_t* ws = wsl(0);
        bf16_t* const xreq = xsl(D);
        bf16_t* const wreq = wsl(D);
        // k-step 0: its MFMAs, the fragment reads of k-step 1 and the W pieces of tile it+D
        int issued = 0;
        const int kt = REQ == 1 ? next_ext() : kt0 + it + D;
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            mfmas(f0, i * RA, (i + 1) * RA);
            load_frag16<MB, NB>(f1, xs, ws, wm, wn, l15, kq, 1, i);
            if constexpr (REQ < 2) {
#pragma unroll
                for (int c = 0; c < pieces_after_read(i, PW, NR); ++c) request_w(wreq, kt, issued++, IsExt{});
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        mfmas(f0, NR * RA, NM);
        __builtin_amdgcn_sched_barrier(0);
        // tile it+1 (requested D-1 tiles ago) must have landed, and every wavefront's reads of tile it must be complete;
        // the tiles after it and the W pieces of tile it+D just issued may still be in flight
        // (a plain s_barrier: __syncthreads() carries a fence, for which the compiler waits for every load)
        if constexpr (REQ < 2)
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(PW + (D - 2) * (PX + PW)) : "memory");
        else
            wait_tiles(nk - 2 - it);
        // k-step 1: its MFMAs, the first fragments of tile it+1 and the x pieces of tile it+D into the x-slot just
        // drained
        const bf16_t* xn = xsl(1);
        const bf16_t* wnx = wsl(1);
        if constexpr (REQ < 2) {
            issued = 0;
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                mfmas(f1, i * RB, (i + 1) * RB);
                load_frag16<MB, NB>(f0, xn, wnx, wm, wn, l15, kq, 0, i);
#pragma unroll
                for (int c = 0; c < pieces_after_read(i, PX, NR); ++c) request_x(xreq, kt, issued++, IsExt{});
                __builtin_amdgcn_sched_barrier(0);
            }
            mfmas(f1, NR * RB, NM);
        } else {
            if (it + 1 < nk) {   // reads only: MFMAs in both arms of a branch make the compiler copy accumulators
#pragma unroll
                for (int i = 0; i < NR; ++i) load_frag16<MB, NB>(f0, xn, wnx, wm, wn, l15, kq, 0, i);
            }
            __builtin_amdgcn_sched_barrier(0);
            mfmas(f1, 0, NM);
        }
        if constexpr (PH < 0) {
            slot_x = (int)(xn - smem);
            slot_w = (int)(wnx - smem);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    using Req0 = std::integral_constant<int, 0>;
    using Rt = std::integral_constant<int, -1>;
    // A wavefront whose whole piece of the tile lies past the matrix (ragged last tile row or column: of few tokens the third
    // 128-column tile of 320 routing products is half empty) moves its share of the operand tiles and keeps the
    // barriers, one per K tile like the others, and skips the fragment reads and the MFMAs.
    const bool idle = n0 + wn >= a.d_out || m0 + wm >= a.T;   // uniform per wavefront
    int it = 0;
    if (idle) {
        for (; it < nk - (half_last ? 1 : 0); ++it) {
            if (it + D < nk) {
                const bool ext = ANY && it + D >= nk_main;
                const int kt = ext ? next_ext() : kt0 + it + D;
#pragma unroll
                for (int i = 0; i < PW; ++i) {
                    if (ext) request_w(wslot(it + D), kt, i, std::true_type{});
                    else request_w(wslot(it + D), kt, i, std::false_type{});
                }
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(PW + (D - 2) * (PX + PW)) : "memory");
#pragma unroll
                for (int i = 0; i < PX; ++i) {
                    if (ext) request_x(xslot(it + D), kt, i, std::true_type{});
                    else request_x(xslot(it + D), kt, i, std::false_type{});
                }
            } else {
                wait_tiles(nk - 2 - it);
            }
        }
        it = nk;
    }
    // The main loop of the large tiles, a whole period of both rings (6 or 12 tiles) per trip: no slot arithmetic between two
    // tiles.  12 tiles against one, 256 x 128 tiles: 2000 x 4096 -> 4096 54.4 and 51.6 us, with 64 adapters of rank 32 103.3
    // and 100.8; 192 and 224 x 128: 850 28.7 and 27.2, 1531 41.5 and 40.1.  6 tiles, 128 x 320: layers
    // of 16384 x 14336 -> 1024 with 544 rows of Wcat 585 and 575.  128 x 128 tiles wait on memory: no difference.
    constexpr int TRIP = D * (D + 1);
    if constexpr ((MB >= 6 || NB > 8) && D <= 3) {
        for (; it + TRIP - 1 + D < nk_main; it += TRIP)
            for_each_phase(std::make_integer_sequence<int, TRIP>{}, [&](auto ph) __attribute__((always_inline)) {
                tile_step(it + decltype(ph)::value, Req0{}, ph);
            });
        slot_x = (int)(xslot(it) - smem);
        slot_w = (int)(wslot(it) - smem);
    }
    for (; it + D < nk_main; ++it) tile_step(it, Req0{}, Rt{});
    if constexpr (ANY)
        for (; it + D < nk; ++it) tile_step(it, std::integral_constant<int, 1>{}, Rt{});
    for (; it < nk - (half_last ? 1 : 0); ++it) tile_step(it, std::integral_constant<int, 2>{}, Rt{});
    if (half_last && !idle) {   // read, behind the barrier, in the previous step's last phase
        mfmas(f0, 0, NM);
        mfma_drain();
    }
    mfma_results<MB, NB>(acc);

    gemm_epilogue16<MB, NB, EPI>(a, acc, smem_raw, m0, n0, wm, wn, wave, lane);
}

}  // namespace meteora
