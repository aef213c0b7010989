// Grouped LoRA expand (second product and weighted sum of Eq. 2 / Eq. 5):
//   out[t,:] (+)= scale * sum_slot w[t,slot] * h[t,slot,:] * B_a,   a = I(t)_slot.
//
// A workgroup owns whole output rows, so every output element has exactly one writer:
// no atomics, and the k contributions of a token are added in slot order (deterministic).
#include "common.hpp"
#include "kernels.hpp"

namespace meteora {

// Plain-FMA version: one workgroup per token, threads stride over d_out.
template <typename TX>
__global__ __launch_bounds__(256) void expand_fma_kernel(const float* __restrict__ h32, const TX* __restrict__ B,
                                                         const int32_t* __restrict__ topk_idx,
                                                         const float* __restrict__ topk_w, int d_out, int N,
                                                         int r, int k, float scale, TX* __restrict__ out,
                                                         int accumulate) {
    __shared__ float hs[kMaxTopK * kMaxRank];   // scale * w * h for the k slots
    __shared__ int as[kMaxTopK];
    const int t = blockIdx.x;
    for (int i = threadIdx.x; i < k * r; i += 256) {
        const int slot = i / r;
        hs[i] = scale * topk_w[(size_t)t * k + slot] * h32[(size_t)t * k * r + i];
    }
    if (threadIdx.x < k) {
        const int a = topk_idx[(size_t)t * k + threadIdx.x];
        as[threadIdx.x] = (a >= 0 && a < N) ? a : -1;
    }
    __syncthreads();
    for (int c = threadIdx.x; c < d_out; c += 256) {
        float acc = accumulate ? to_float(out[(size_t)t * d_out + c]) : 0.f;
        for (int slot = 0; slot < k; ++slot) {
            const int a = as[slot];
            if (a < 0) continue;
            const TX* Ba = B + (size_t)a * r * d_out + c;
            float d = 0.f;
            for (int q = 0; q < r; ++q) d = fmaf(hs[slot * r + q], to_float(Ba[(size_t)q * d_out]), d);
            acc += d;
        }
        out[(size_t)t * d_out + c] = from_float<TX>(acc);
    }
}

hipError_t launch_expand(const float* h32, const void* B, const int32_t* topk_idx, const float* topk_w,
                         int T, int d_out, int N, int r, int k, float scale, bool bf16, void* out,
                         int accumulate, hipStream_t stream) {
    if (bf16)
        expand_fma_kernel<bf16_t><<<T, 256, 0, stream>>>(h32, (const bf16_t*)B, topk_idx, topk_w, d_out, N, r, k,
                                                         scale, (bf16_t*)out, accumulate);
    else
        expand_fma_kernel<float><<<T, 256, 0, stream>>>(h32, (const float*)B, topk_idx, topk_w, d_out, N, r, k,
                                                        scale, (float*)out, accumulate);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// The expand alone, from the dense operand (bf16, up to 256 columns of it): out (+)= hd * B, B viewed as [N*r, d_out] and read
// as the caller stores it.
//
// Bound by the output's way in and out.  A workgroup owns 256 columns and a run of rows, one per CU: its slab of B goes to LDS
// once, transposed in registers (8 x 8 values a lane), so nothing packs B in front; then eight independent wavefronts
// take 32 rows x 128 columns each at a time, hd from memory as MFMA fragments.  A lane's rows of an MFMA pair are chosen so that
// its results are 8 consecutive columns of one token: the old output comes in and the new one leaves in 16-byte pieces
// without a stage in LDS.  K steps of 32 columns that are zero for a wavefront's tokens are left out.
// Whole lora_forward calls that accumulate, 28 adapters of rank 8, 4096 inputs, the GEMM on packed rows of B and this: 100 tokens,
// 14336 outputs 24.9 and 21.3 us, 3000, 14336 71.9 and 61.2, 8000, 4096 63.9 and 60.6; 3000 x 5120 -> 5120 41.5 and 40.0 (ordinary
// stores 41.0); output written only 3000 x 4096 -> 14336 59.5 and 52.7, 16000 x 1024 -> 4096 47.5 and 41.5.
// ------------------------------------------------------------------------------------------
constexpr int kExpCols = 256, kExpThreads = 512, kExpMaxK = 256;
constexpr int kExpRow = kExpMaxK * 2;                       // bytes per column of the slab
constexpr int kExpLds = kExpCols * kExpRow;
constexpr int kThrough = 16;                                // "sc1": written through the L2, as in the GEMM's epilogue

template <bool ACC>
__global__ __launch_bounds__(kExpThreads) void expand_dense_kernel(const bf16_t* __restrict__ hd, const bf16_t* __restrict__ B,
                                                                   bf16_t* __restrict__ out, int T, int d_out, int ext_k,
                                                                   int ext_stride, int slabs, int rows_per_wg) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l15 = lane & 15, kq = lane >> 4;
    const int c0 = (blockIdx.x % slabs) * kExpCols, row0 = blockIdx.x / slabs * rows_per_wg;
    const int nrows = min(rows_per_wg, T - row0), nks = ceil_div(ext_k, 32);
    const uint32_t b_bytes = (uint32_t)ext_k * (uint32_t)d_out * 2u, out_bytes = (uint32_t)T * (uint32_t)d_out * 2u;
    auto resource = [](const void* p, uint32_t bytes) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
    };
    const __amdgpu_buffer_rsrc_t rb = resource(B, b_bytes), ro = resource(out, out_bytes),
                                 rh = resource(hd, (uint32_t)T * (uint32_t)ext_stride * 2u);

    // the slab: a lane's piece is 8 rows of B (8 columns of hd) x 8 outputs; what lies past B's rows or columns is zero
    const int tasks = ceil_div(ext_k, 128) * 8;              // 128 rows x 32 outputs a wavefront
    u32x4 v[2][8];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int task = wave + 8 * u, k8 = (task >> 3) * 16 + (lane >> 2), c = c0 + (task & 7) * 32 + (lane & 3) * 8;
        if (task < tasks) {                                  // uniform
#pragma unroll
            for (int j = 0; j < 8; ++j)
                v[u][j] = __builtin_amdgcn_raw_buffer_load_b128(
                    rb, c < d_out ? (uint32_t)(k8 * 8 + j) * (uint32_t)d_out * 2u + (uint32_t)c * 2u : b_bytes, 0, 0);
        }
    }

    // this wavefront's items: (32 rows, 128 columns)
    const int items = 2 * ceil_div(nrows, 32), each = ceil_div(items, kExpThreads / 64);
    const int first = wave * each, last = min(items, first + each);
    bf16x8 x[2][kExpMaxK / 32];
    u32x4 old[2][4];
    auto load_hd = [&](int item) {
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
#pragma unroll
            for (int ks = 0; ks < kExpMaxK / 32; ++ks)
                if (ks < nks)                                // uniform
                    x[tb][ks] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(
                        rh, (uint32_t)(row0 + (item >> 1) * 32 + tb * 16 + l15) * (uint32_t)ext_stride * 2u + (uint32_t)(ks * 64 + kq * 16), 0, 0));
    };
    auto out_offset = [&](int item, int tb, int p) {
        const int c = c0 + (item & 1) * 128 + p * 32 + kq * 8, row = row0 + (item >> 1) * 32 + tb * 16 + l15;
        return c < d_out && row < T ? (uint32_t)row * (uint32_t)d_out * 2u + (uint32_t)c * 2u : out_bytes;
    };
    auto load_old = [&](int item) {
        if constexpr (ACC) {
#pragma unroll
            for (int tb = 0; tb < 2; ++tb)
#pragma unroll
                for (int p = 0; p < 4; ++p) old[tb][p] = __builtin_amdgcn_raw_buffer_load_b128(ro, out_offset(item, tb, p), 0, 0);
        }
    };
    if (first < last) {
        load_hd(first);
        load_old(first);
    }
    // column c of the slab: chunk k8 at k8 ^ key(c), so that neither these writes nor the fragment reads meet in a bank
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int task = wave + 8 * u, k8 = (task >> 3) * 16 + (lane >> 2), c = (task & 7) * 32 + (lane & 3) * 8;
        if (task < tasks) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                u32x4 w;
#pragma unroll
                for (int d = 0; d < 4; ++d)
                    w[d] = __builtin_amdgcn_perm(v[u][2 * d + 1][j / 2], v[u][2 * d][j / 2], j % 2 == 0 ? 0x05040100u : 0x07060302u);
                *reinterpret_cast<u32x4*>(smem + (c + j) * kExpRow + ((k8 ^ ((lane & 3) * 4 + (j & 3))) << 4)) = w;
            }
        }
    }
    __syncthreads();
    const unsigned char* slab = smem + ((l15 >> 2) * 8 + (l15 & 3)) * kExpRow;   // of the first MFMA's rows; its key is l15
    for (int item = first; item < last; ++item) {
        f32x4 acc[2][8];
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
#pragma unroll
            for (int nb = 0; nb < 8; ++nb) acc[tb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < kExpMaxK / 32; ++ks) {
            if (ks >= nks) break;
            const u32x4 a = __builtin_bit_cast(u32x4, x[0][ks]), b = __builtin_bit_cast(u32x4, x[1][ks]);
            if (__ballot(((a[0] | a[1]) | (a[2] | a[3]) | (b[0] | b[1]) | (b[2] | b[3])) != 0u) == 0ull) continue;
            const unsigned char* at = slab + (item & 1) * 128 * kExpRow + (((ks * 4 + kq) ^ l15) << 4);
#pragma unroll
            for (int nb = 0; nb < 8; ++nb) {
                const bf16x8 w = *reinterpret_cast<const bf16x8*>(at + ((nb >> 1) * 32 + (nb & 1) * 4) * kExpRow);
                acc[0][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, x[0][ks], acc[0][nb], 0, 0, 0);
                acc[1][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, x[1][ks], acc[1][nb], 0, 0, 0);
            }
        }
        u32x4 done[2][4];
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                f32x4 lo = acc[tb][2 * p], hi = acc[tb][2 * p + 1];
                if constexpr (ACC) {
                    const u32x4 o = old[tb][p];
                    lo += f32x4{bf16_bits_to_float(o[0] & 0xffffu), bf16_bits_to_float(o[0] >> 16), bf16_bits_to_float(o[1] & 0xffffu),
                                bf16_bits_to_float(o[1] >> 16)};
                    hi += f32x4{bf16_bits_to_float(o[2] & 0xffffu), bf16_bits_to_float(o[2] >> 16), bf16_bits_to_float(o[3] & 0xffffu),
                                bf16_bits_to_float(o[3] >> 16)};
                }
                done[tb][p] = u32x4{pack_bf16x2(lo[0], lo[1]), pack_bf16x2(lo[2], lo[3]), pack_bf16x2(hi[0], hi[1]), pack_bf16x2(hi[2], hi[3])};
            }
        if (item + 1 < last) {                               // the next item's loads go out ahead of the stores
            if (((item + 1) & 1) == 0) load_hd(item + 1);
            load_old(item + 1);
        }
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
#pragma unroll
            for (int p = 0; p < 4; ++p) __builtin_amdgcn_raw_buffer_store_b128(done[tb][p], ro, out_offset(item, tb, p), 0, kThrough);
    }
}

// Narrow outputs leave a workgroup few rows for its 128 KB of B (3000 x 4096 -> 1024 27.7 by the GEMM, 29.6 by this), up to 64
// tokens the split GEMM is ahead (64 x 4096 -> 4096 27.3 and 28.1); from 500 to 2000 tokens of 4096 outputs they are level.
bool expand_dense_applies(int T, int d_out, int ext_k, int ext_stride) {
    const uint64_t most = 1ull << 32;
    return T > 64 && d_out >= 4096 && ext_k <= kExpMaxK && d_out % 8 == 0 && ((uint64_t)T + 32) * d_out * 2 < most && ((uint64_t)T + 32) * ext_stride * 2 < most &&
           (uint64_t)(kExpMaxK + 8) * d_out * 2 < most;
}

hipError_t launch_expand_dense(const void* hdense, int ext_stride, const void* B, int ext_k, int T, int d_out, void* out,
                               int accumulate, hipStream_t stream) {
    if (!expand_dense_applies(T, d_out, ext_k, ext_stride) || ext_stride % 8 != 0 || ext_stride < ext_k) return hipErrorInvalidValue;
    const int slabs = ceil_div(d_out, kExpCols), most = slabs < 256 ? 256 / slabs : 1;
    const int rows = (int)align_up(ceil_div(T, most), 32), chunks = ceil_div(T, rows);
    auto go = [&](auto kern) -> hipError_t {
        const hipError_t e = ensure_lds_limit(reinterpret_cast<const void*>(kern), kExpLds);
        if (e != hipSuccess) return e;
        kern<<<slabs * chunks, kExpThreads, kExpLds, stream>>>((const bf16_t*)hdense, (const bf16_t*)B, (bf16_t*)out, T, d_out, ext_k,
                                                              ext_stride, slabs, rows);
        return hipGetLastError();
    };
    return accumulate ? go(&expand_dense_kernel<true>) : go(&expand_dense_kernel<false>);
}

hipError_t expand_init_kernels() {
    const hipError_t e = ensure_lds_limit(reinterpret_cast<const void*>(&expand_dense_kernel<true>), kExpLds);
    return e != hipSuccess ? e : ensure_lds_limit(reinterpret_cast<const void*>(&expand_dense_kernel<false>), kExpLds);
}

}  // namespace meteora
