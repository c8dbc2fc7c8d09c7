// Rules on sizes that pick a kernel, in a file without HIP so that a host test can hold them against the measured figures.
#pragma once
#include <stdint.h>

// True where the kernels for a few tokens (forward_few.hip) are faster than the tiles of the prefill kernels.
// Up to 64 tokens they are.  Up to one workgroup per two compute units of their widest tile (128 tokens x 64 outputs) too, but for
// many tokens with a wide rank-r branch: its first product reads L_B once per 16 tokens.  Up to one workgroup per compute unit they
// re-use less per load than the 256 x 256 tiles, so there the contraction has to be long against the fixed part and against the
// rank-r branch, less so where the prefill kernels split the factors into two planes.  At most 2048 tokens, so that the partial sums
// fit the workspace (see aser_compensated_forward).
// Measured (us, prefill kernels -> few tokens; channels, outputs, tokens; int4).  r = 0: 4096, 4096, 300: 49 -> 32; 4096, 1024, 2048:
// 45 -> 35; 1024, 4096, 512: 20.3 -> 19.5; 512, 3072, 512: 15.8 -> 17.3 (prefill); 256, 4096, 384: 20.9 -> 15.2; 4096, 14336, 256: 47 -> 68 (prefill).
// r = 64, plain: 4096, 4096, 512: 86 -> 73; 2048, 8192, 256: 55 -> 52; 1024, 1024, 2048: 40 -> 48 and 4096, 1024, 2048: 86 -> 94 (prefill);
// split: 1024, 4096, 512: 48 -> 45; 4096, 1024, 2048: 101 -> 93; 512, 768, 1536: 38 -> 44 (prefill).  r = 128, plain: 8192, 256, 2048: 168 -> 166;
// 8192, 512, 2048: 168 -> 184 (prefill); split: 1024, 8192, 256: 68 -> 61; 4096, 1024, 2048: 136 -> 149 (prefill).
static inline bool aser_forward_few_pays(int64_t rows, int64_t n, int64_t m, int r, bool split) {
    const int64_t tiles = ((rows + 127) / 128) * ((m + 63) / 64), rank_work = (int64_t)((r + 15) / 16 * 16) * rows;
    if (rows > 2048 || tiles > 256) return false;
    if (rows <= 64) return true;
    if (tiles <= 128) return split || tiles <= 64 || rank_work <= 128 * 1536;
    if (r == 0) return n >= 1024 || (rows > 256 && rows < 1024 && ((rows - 1) & 255) < 128);   // or the last 256 tokens' tile would be half empty
    return split ? n >= 1024 && rank_work <= 64 * n && rank_work <= 128 * 1536 : n >= 2048 && rank_work <= 9 * n;
}

// True where f rounds of an arg-max in one workgroup select the outlier channels faster than the comparison of all pairs of
// channels: a round costs 1.6 to 3.3 us, the pairs n^2 / 5.4e6 us and one more launch, so the line is a constant plus n^2 (the rounds
// take 1024 threads instead of 512 above 16384 channels).
// Measured (us, rounds -> pairs): 4096 channels, f = 4: 17 -> 21, 8: 23 -> 22; 11008, 8: 33 -> 40; 14336, 16: 56 -> 59; 16384, 8: 36 -> 65, 16: 58 -> 66,
// 32: 102 -> 68; 32768, 8: 43 -> 201, 32: 121 -> 203, 64: 225 -> 206.
static inline bool aser_select_by_rounds(int64_t n, int f) { return f <= 4 + n * n / (n <= 16384 ? 17000000 : 20000000); }
