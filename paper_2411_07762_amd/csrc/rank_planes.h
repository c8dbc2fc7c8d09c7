// The factors of the rank-r branch as bf16 planes (aser_rank_down, aser_internal.h), for the launches that make them.
#pragma once
#include "aser_internal.h"
#include "bf16_pair.h"

__host__ __device__ static inline int64_t split_factors_lb_blocks(int64_t n, int r_pad) { return (n + 255) / 256 * (r_pad / 8); }
static inline int64_t split_factors_blocks(int64_t m, int64_t n, int r_pad) {
    const int64_t la = ceil_div64(m * r_pad, 256 * 4);
    return split_factors_lb_blocks(n, r_pad) + (la < 2048 ? la : 2048);
}

// Both factors as NP bf16 planes, each what the ones before it leave of the value, rounded.  L_A (m x r) as [m][r_pad] with zeros behind r; L_B (r x n) in the
// order in which rank_down_kernel feeds it to the MFMA: [32 channels][plane][32 rows][8-channel slice][lane][8 channels], lane 32 h + i holding
// channels 16 h + 8 slice .. + 7 of row i, zeros past r and n; three planes: one block of 32 rows after the other.  PLAIN: as planes [r_pad][n] (n % 32 == 0).
// By `blocks` workgroups of 256 threads, split_factors_blocks of them; this is number `block`.
template <int NP, bool PLAIN>
__device__ __forceinline__ void split_factors(int64_t block, int64_t blocks, const float* __restrict__ L_A, const float* __restrict__ L_B, int64_t m, int64_t n,
                                              int r, int r_pad, const AserRankPlanes& out) {
    const int64_t lb_blocks = split_factors_lb_blocks(n, r_pad);
    if (block < lb_blocks) {                                 // eight rows, 256 channels
        const int64_t k = (block % ((n + 255) / 256)) * 256 + 8 * (threadIdx.x & 31);
        const int row = (int)(block / ((n + 255) / 256)) * 8 + (threadIdx.x >> 5);
        if (k >= (n + 31) / 32 * 32) return;
        float f[8];
        const float* src = L_B + (int64_t)(row < r ? row : 0) * n;
        if (((uintptr_t)src & 15) == 0 && k + 8 <= n) {
            const float4 x = *(const float4*)(src + k), y = *(const float4*)(src + k + 4);
            f[0] = x.x; f[1] = x.y; f[2] = x.z; f[3] = x.w; f[4] = y.x; f[5] = y.y; f[6] = y.z; f[7] = y.w;
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) f[e] = k + e < n ? src[k + e] : 0.f;
        }
        const int c8 = (int)(k & 31) >> 3, h = c8 >> 1, sl = c8 & 1, tall = r_pad / 32;
        const int together = NP == 3 ? 1 : tall;             // blocks of rows that a workgroup takes
        const int64_t step = NP == 3 ? row / 32 * ((n + 31) / 32) + k / 32 : k / 32;
        uint4* lb = (uint4*)out.lb + (PLAIN ? (row * n + k) / 8 : ((step * NP * together + (NP == 3 ? 0 : row / 32)) * 2 + sl) * 64 + 32 * h + (row & 31));
#pragma unroll
        for (int p = 0; p < NP; ++p, lb += PLAIN ? r_pad * n / 8 : (int64_t)together * 128) {
            uint32_t pair[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float &f0 = f[2 * q], &f1 = f[2 * q + 1];
                pair[q] = row < r ? bf16_pair(f0, f1) : 0u;
                f0 -= __uint_as_float(pair[q] << 16);
                f1 -= __uint_as_float(pair[q] & 0xFFFF0000u);
            }
            *lb = make_uint4(pair[0], pair[1], pair[2], pair[3]);
        }
        return;
    }
    const int64_t total = m * r_pad;
    for (int64_t t = (block - lb_blocks) * 256 + threadIdx.x; t < total; t += (blocks - lb_blocks) * 256) {
        const int64_t i = t / r_pad;
        const int j = (int)(t % r_pad);
        float x = j < r ? L_A[i * r + j] : 0.f;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const uint32_t part = bf16_rne(x);
            out.la[p][t] = (uint16_t)part;
            x -= __uint_as_float(part << 16);
        }
    }
}
