// fp32 gate logits of one token by a workgroup of four wavefronts (Sec. 3.1: G(x) = x * W_gate), for fp32 storage.
//
// The four wavefronts share d_in, and inside a wavefront the columns of W_gate take as many lanes as they need (the
// next power of two), the rest of the lanes other rows: with 4 adapters a wavefront reads 16 rows of W_gate at once
// and 256 inputs are two steps of loads.
#pragma once
#include "common.hpp"

namespace meteora {

constexpr int kRowThreads = 256;

// Sum over i of x[i] * M[i * ld + offset of this thread's column], the rows dealt to `parts` threads per column.  Eight
// rows' loads are in flight at a time, from clamped addresses.
__device__ __forceinline__ float row_dot(const float* __restrict__ x, const float* __restrict__ M, int ld, int d_in,
                                         int part, int parts) {
    float acc[4] = {0.f, 0.f, 0.f, 0.f};   // four chains: less latency and a smaller rounding error than one
    for (int i0 = part; i0 < d_in; i0 += 8 * parts) {
        float xv[8], mv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i0 + u * parts, ic = i < d_in ? i : d_in - 1;
            xv[u] = x[ic];
            mv[u] = M[(size_t)ic * ld];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (i0 + u * parts < d_in) acc[u & 3] = fmaf(xv[u], mv[u], acc[u & 3]);
    }
    return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

// Sum over the lanes of a wavefront that hold the same column (lane % cols, cols a power of two).
__device__ __forceinline__ float sum_columns(float v, int cols) {
    for (int off = cols; off < kWave; off <<= 1) v += __shfl_xor(v, off);
    return v;
}

// cols: N rounded up to a power of two.  On return, behind a barrier, red[w][j] holds wavefront w's sum of column j.
__device__ __forceinline__ void gate_row(const float* __restrict__ x, const float* __restrict__ W_gate, int d_in, int N,
                                         int cols, float (&red)[4][kMaxAdapters]) {
    const int col = threadIdx.x & (cols - 1);
    float v = 0.f;
    if (col < N) v = row_dot(x, W_gate + col, N, d_in, threadIdx.x / cols, kRowThreads / cols);
    v = sum_columns(v, cols);
    if ((threadIdx.x & 63) < cols) red[threadIdx.x >> 6][col] = v;
    __syncthreads();
}

inline int pow2_at_least(int n) {
    int p = 1;
    while (p < n) p <<= 1;
    return p;
}

}  // namespace meteora
