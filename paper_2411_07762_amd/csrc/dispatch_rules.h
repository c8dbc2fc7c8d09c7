// Rules on sizes that pick a kernel, in a file without HIP so that a host test can hold them against the measured figures.
#pragma once
#include <stdint.h>

// True where the kernels for a few tokens (forward_few.hip) are faster than the tiles of the prefill kernels, or, with split factors, as long as they are not
// much slower: P keeps all bits of the factors there (2e-7 of the rank-r branch instead of 5e-6).
// Up to 64 tokens they are faster.  Up to one workgroup per two compute units of their widest tile (128 tokens x 64 outputs) too, but for
// many tokens with a wide rank-r branch: its first product reads L_B once per 16 tokens.  Up to one workgroup per compute unit they
// re-use less per load than the 256 x 256 tiles, so there the contraction has to be long against the fixed part and, the more so the larger
// the rank, against the rank-r branch.  At most 2048 tokens, so that the partial sums fit the workspace (see aser_compensated_forward).
// Measured (us, prefill kernels -> few tokens; channels, outputs, tokens; int4).  r = 0: 4096, 4096, 300: 49 -> 33; 4096, 1024, 2048:
// 44 -> 35; 1024, 4096, 512: 19.7 -> 18.9; 512, 3072, 512: 15.5 -> 17.3 (prefill); 256, 4096, 384: 20.6 -> 15.2; 4096, 14336, 256: 47 -> 68 (prefill).
// Plain, r = 64: 4096, 4096, 384: 72 -> 66; 8192, 4096, 512: 109 -> 97; 11008, 1024, 1536: 140 -> 152 and 2048, 8192, 256: 44 -> 48 (prefill);
// 4096, 512, 2048: 65 -> 58.
// r = 128: 4096, 14336, 128: 90 -> 91; 8192, 4096, 512: 123 -> 138 (prefill); 8192, 1024, 1024: 122 -> 112; 8192, 512, 1536: 123 -> 133 (prefill);
// 4096, 256, 2048: 75 -> 76; 8192, 256, 2048: 121 -> 136 (prefill).  r = 16: 2048, 4096, 512: 40 -> 46 (prefill), 2048, 14336, 65: 42 -> 35, 4096, 1024, 2048: 61 -> 64 (prefill).
// Split, the furthest on the wrong side: r = 64: 4096, 1024, 2048: 75 -> 85; r = 128: 4096, 1024, 1536: 94 -> 120; r = 16: 1024, 1024, 2048: 32 -> 40.
// Over 540 plain calls (65 to 2048 tokens, 512 to 11008 channels, 256 to 14336 outputs, r 16 to 128) the rule loses at
// most 3 %, but 12 to 16 % at 65 tokens of 1024 channels and 6 % at 384 tokens of 2048.
static inline bool aser_forward_few_pays(int64_t rows, int64_t n, int64_t m, int r, bool split) {
    const int64_t tiles = ((rows + 127) / 128) * ((m + 63) / 64), rank = (r + 15) / 16 * 16, rank_work = rank * rows;
    if (rows > 2048 || tiles > 256) return false;
    if (rows <= 64) return true;
    if (tiles <= 128) {
        if (split || rank_work <= 128 * 1280) return true;
        return tiles <= 64 ? rank_work <= 128 * 1536 || n <= 6144 : rank_work <= 128 * 1536 && n <= 1024;
    }
    if (r == 0) return n >= 1024 || (rows > 256 && rows < 1024 && ((rows - 1) & 255) < 128);   // or the last 256 tokens' tile would be half empty
    if (split) return n >= 1024 && rank_work <= 64 * n && rank_work <= 128 * 1536;
    return rows <= 96 ? n >= 2048 : n >= (rows <= 512 ? 3072 : 5120) && rank * rank_work <= 512 * n;    // so few leave a quarter of the prefill kernels' tiles of 128 and more empty
}

// First product of the prefill kernels' rank-r branch, r_pad columns: true where 128 tokens per workgroup with both operands through LDS are faster than 32
// tokens with L_B read straight (forward.hip).  Beyond two rounds of 32 x 256 tokens always; in the second round (a few workgroups of it run
// beside the first) where the contraction is so short that a workgroup's start and end count: there are a quarter as many of them.
// Measured (us of the call, 32 tokens -> 128; channels, outputs, tokens): r = 40: 256, 107, 16384: 26.1 -> 24.2; 512, 107, 16384: 31.8 -> 28.3; 768, 1024, 9000: 42.5
// -> 41.5; split, 512, 107, 16384: 38.5 -> 33.6; not 288, 107, 8193: 24.9 -> 25.8, nor 896, 1024, 8193: 40.1 -> 41.4.  Up to 32 columns, split, 512, 107, 12000:
// 29.6 -> 27.8, plain never (768, 1024, 14000: 41.7 -> 42.6); up to 128, split, 256, 107, 16384: 42.7 -> 38.6, plain 31.7 -> 29.8,
// 768, 1024, 9000: 50.0 -> 50.7; 96 never (768, 1024, 9000, split: 54.0 -> 56.5).
// The rule loses at most 3 % (split, up to 32 columns: 288, 1024, 9000: 35.1 -> 36.2).
static inline bool aser_down_staged(int64_t rows, int64_t n, int r_pad, bool split) {
    if (rows <= 8448 || rows > 16384) return rows > 16384;
    return r_pad != 96 && n <= (split || r_pad == 64 ? 768 : (r_pad == 128 ? 320 : 0));
}

// True where f rounds of an arg-max in one workgroup select the outlier channels faster than the comparison of all pairs of
// channels: a round costs 1.6 to 3.3 us, the pairs n^2 / 5.4e6 us and one more launch, so the line is a constant plus n^2 (the rounds
// take 1024 threads instead of 512 above 16384 channels).
// Measured (us, rounds -> pairs): 4096 channels, f = 4: 17 -> 21, 8: 23 -> 22; 11008, 8: 33 -> 40; 14336, 16: 56 -> 59; 16384, 8: 36 -> 65, 16: 58 -> 66,
// 32: 102 -> 68; 32768, 8: 43 -> 201, 32: 121 -> 203, 64: 225 -> 206.
static inline bool aser_select_by_rounds(int64_t n, int f) { return f <= 4 + n * n / (n <= 16384 ? 17000000 : 20000000); }

// Gram update of a chunk of tokens that the LDS-direct schedule does not fill its rounds with by itself: the K chunks of that schedule
// and the split of its left-over tiles, or chunks = 0 where the plain grid of `parts` K parts and `steps64` 64-token steps each
// is faster.  T: 256 x 256 tiles of the lower triangle; steps: 32-token steps.
// EVERY tile, of the full rounds and left over, is summed in as many parts as the plain grid's, or up to a third more: fewer make the
// fp32 chains longer, more round G more often when a statistic comes in many calls.  Root mean square error of the diagonal against
// fp64, in 1e-8 (plain grid, then as many parts, then the left-over tiles alone in twice to eight times as many): 4096 channels, eight calls
// of 2000 tokens 9.05, 9.05, 9.01 to 9.54; four calls of 7503 10.2 (7 parts), 10.3 (8 parts), 10.4 to 10.6; one call of 7503 9.8, 9.1, 8.9 to 9.0.
// Costs in microseconds, fitted to 1040 .. 14336 channels and 256 .. 7503 tokens (nine tenths of the figures within 12 % for the
// LDS-direct schedule, 9 % for the plain grid, the medians within 2 %).  LDS-direct: 0.60 per step of the busiest workgroup and
// 0.186 per 256 x 256 tile flush of the launch (fp32 atomics that share the memory side).  Plain: per round of 256 workgroups 1.97
// a step and 4.3, 0.165 per flush.  Measured, plain -> LDS-direct: 1536 channels: 59 -> 42 us at 4000 tokens; 4096: 68 -> 61 at 1000, 137 -> 114 at
// 2000, 165 -> 133 at 3000, 240 -> 197 at 5000, 301 -> 305 at 7503, plain at 4000 (171 against 180); 8192: 409 -> 368 at 3000; 11008: 580 -> 467
// at 2000.  Left-over tiles in more parts: 104 instead of 114 us at 2000 tokens of 4096 channels, 117 instead of 133 at 3000.
struct AserGramSplit { int chunks, split; double cost; };
static inline AserGramSplit aser_gram_dma_split(int64_t T, int64_t steps, int64_t parts, int64_t steps64) {
    AserGramSplit best = {0, 1, 0.0};
    double best_cost = (double)((T * parts + 255) / 256) * (1.97 * (double)steps64 + 4.3) + 0.165 * (double)(T * parts) + 4.1;
    for (int c = 1; c <= 8; c *= 2) {
        const int64_t W = 256 / c, full = T / W, rem = T % W, steps_c = (steps + c - 1) / c;
        if (full > 0 && (c < parts || 3 * c > 4 * parts)) continue;
        for (int64_t sp = 1; sp <= (rem ? W / rem : 1); ++sp) {
            if (rem && (c * sp < parts || 3 * c * sp > 4 * parts)) continue;
            const int64_t last = rem ? (steps_c + sp - 1) / sp : 0;
            if (sp > 1 && last < 4) break;                  // the ring is filled once
            const double cost = 0.60 * (double)(full * steps_c + last) + 0.186 * (double)(c * (full * W + rem * sp)) + 8.9;
            if (cost <= best_cost) { best_cost = cost; best = AserGramSplit{c, (int)sp, 0.0}; }     // equal: more chunks, fewer XCDs on one slab
        }
    }
    best.cost = best_cost;
    return best;
}

// The same call on 256 x 128 tiles whose sums have two levels (gram_seg_kernel): the fp32 chains are half as long as those of `parts` K parts
// whatever the split, and G is rounded once per chunk (left-over tiles: per chunk and part, at most a third more often than by the plain grid).
// T: 256 x 128 tiles of the lower triangle.  Root mean square error of the diagonal over four seeds, without -> with, in 1e-8: 4096 channels, four
// calls of 7503 tokens 10.3 -> 6.9, of 3000 10.9 -> 7.9; 2048, four of 6000 10.6 -> 7.4; 1536, eight of 2000 9.0 -> 7.2; 8192, two of 3000 12.8 -> 8.6.
// Costs fitted to the same range (half of 200 figures within 3 %): 0.47 us per step of the busiest workgroup, 0.084 per tile flush.  It is taken
// where it promises 3 %, because the other models are that good.  Measured, without -> with: 1536 channels: 39 -> 31 us at 1000 tokens, 62 -> 53
// at 6000; 4096: 146 -> 106 at 3000, 203 -> 130 at 4300, 317 -> 179 at 7500, not at 1800 (85 against 93); 6144: 307 -> 230 at 4300; 8192: 367 -> 316
// at 3000, not at 7500 (605 against 609); 14336: never (728 against 836 at 3000).
// No range is shorter than the loads that are in flight at its start (aser_gram_shortest); the costs alone keep to 8 steps and more.
constexpr int kAserGramSegAhead = 5;
// The shortest range of `steps` in c chunks, each of them in sp parts (rounded up to whole steps; the last chunk and part get what is left).
static inline int64_t aser_gram_shortest(int64_t steps, int64_t c, int64_t sp) {
    const int64_t chunk = (steps + c - 1) / c;
    const int64_t chunks[2] = {chunk, steps - (steps - 1) / chunk * chunk};
    int64_t least = steps;
    for (int64_t k : chunks) {
        const int64_t part = (k + sp - 1) / sp, left = k - (k - 1) / part * part;
        least = left < least ? left : least;
    }
    return least;
}
static inline AserGramSplit aser_gram_seg_split(int64_t T, int64_t steps, int64_t parts) {
    AserGramSplit best = {0, 1, 1e30};
    for (int c = 1; c <= 8; c *= 2) {
        if (c > 1 && 3 * c > 4 * parts) break;
        const int64_t W = 256 / c, full = T / W, rem = T % W, steps_c = (steps + c - 1) / c;
        for (int64_t sp = 1; sp <= (rem ? W / rem : 1); ++sp) {
            if (c * sp > 1 && rem && 3 * c * sp > 4 * parts) break;
            if (aser_gram_shortest(steps, c, sp) < kAserGramSegAhead) continue;
            const int64_t last = rem ? (steps_c + sp - 1) / sp : 0;
            const double cost = 0.47 * (double)(full * steps_c) + 0.458 * (double)last + 0.084 * (double)(c * (full * W + rem * sp)) + 8.5;
            if (cost < best.cost) best = AserGramSplit{c, (int)sp, cost};
        }
    }
    return best;
}

// How many finished block rows a whitening step applies at a time to the block rows that are not due yet (whiten.hip).  Fewer keep a step's
// launch as short as the factorisation of the diagonal block beside it; more read and write the trailing matrix less often, which counts
// once there are several tiles per compute unit.  The slower tiles (six products, or operands fetched word by word) take one.
// Measured (us, lag 1, 2, 3, 4): 1536 columns 304, 302, 320, 352; 4096: 801, 793, 860, 973; 6000: 1440, 1324, 1460, 1620; 8192: 2393, 2065, 2101, 2175;
// 9000: 3221, 2764, 2741, 2857; 11008: 4928, 4016, 3868, 3899; 14336: 9658, 7427, 6882, 6770; (3, 4, 6, 8): 16384: 9578, 9170, 9644, 9981; 20480: 17124,
// 16288, 16216, 16516; 28672: 41349, 38928, 37149, 36671.  Six products, 1000 columns: 233, 247, 281, 300; word by word, 6001: 2354, 2811, 3660, 4552.
static inline int aser_whiten_lag(int64_t n, bool slow_tiles) {
    if (slow_tiles) return 1;
    return n <= 8192 ? 2 : (n <= 12288 ? 3 : (n <= 18432 ? 4 : (n <= 24576 ? 6 : 8)));
}
