// MFMA contraction kernel of the ASER calibration path for gfx950 (CDNA4).
//
// One kernel form serves the dense contractions of the path:  C (op)= alpha * A^T B  with
// both operands stored K-major (A: K x M, B: K x N, row-major).  The Gram matrix of Eq. 5
// (G = X^T X with X tokens x channels) has exactly this form, and the whitened error T S, the
// subspace-iteration products and the small Gram matrices of the orthogonalisation are arranged
// by their callers to have it too.  (The updates and panels of the whitening have it as well and
// share the tile of gemm_tile.h, in the launches of whiten.hip.)
//
// Data path.  Each workgroup (256 threads = 4 waves in a 2 x 2 grid; 512 threads and 8 waves for 256 x 128) owns a BM x BN
// tile of C.
// Per K step a thread fetches an 8(k) x 8(bf16) or 8(k) x 4(fp32) block of each operand with
// 16-byte loads that are contiguous along the channel dimension, turns it in registers into
// k-contiguous 8 x bf16 chunks (a byte-permute transpose for bf16; for fp32 the hi/lo split
// packs pairs along k directly), and stores the chunks to LDS in the order the MFMA operands
// are read: chunk (k-block, row) at [kb][swizzle(row)].  v_mfma_f32_32x32x16_bf16 reads one
// chunk per lane (row = lane % 32, k-block = lane / 32).  Global loads run one step (256 x 256
// tile) or two steps (smaller tiles, two register sets) ahead of the MFMAs; LDS is double
// buffered with one barrier per step.  fp32 operands are split as x = hi + lo (bf16 each) and
// contribute hi*hi + hi*lo + lo*hi, accumulated in fp32.
#include <type_traits>

#include "aser_internal.h"
#include "dispatch_rules.h"
#include "gemm_tile.h"

namespace {

// Tile and K-part of a workgroup for the plain schedules.
template <int IN, int BM, int BN, bool FAST, bool WIDE>
__device__ __forceinline__ void gemm_tn_workgroup(const GemmArgs& g, uint4* smem) {
    constexpr int BK = InTraits<IN>::BK;
    if (g.gate && *g.gate == 0) return;
    const int64_t tm = (g.M + BM - 1) / BM, tn = (g.N + BN - 1) / BN;
    int64_t ti, tj;
    const int64_t t = blockIdx.x;
    if (g.long_first) {                                   // column by column: with K_GE_COL the tiles with the longest K start first
        ti = t % tm;
        tj = t / tm;
    } else if (g.tiles == GEMM_TILES_ALL) {
        ti = t / tn;
        tj = t % tn;
    } else {
        // t enumerates pairs (p, q) with p >= q: p (p + 1) / 2 + q
        int64_t p = (int64_t)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
        while (p * (p + 1) / 2 > t) --p;
        while ((p + 1) * (p + 2) / 2 <= t) ++p;
        const int64_t q = t - p * (p + 1) / 2;
        if (g.tiles == GEMM_TILES_LOWER) { ti = p; tj = q; } else { ti = q; tj = p; }
    }
    const int64_t I0 = ti * BM, J0 = tj * BN;
    int64_t k0 = 0;
    if (g.krange == GEMM_K_GE_COL) k0 = (J0 / BK) * BK;
    const int64_t ksteps = (g.K - k0 + BK - 1) / BK;
    const int64_t per = (ksteps + g.k_parts - 1) / g.k_parts;
    const int64_t kBeg = k0 + (int64_t)blockIdx.y * per * BK;
    int64_t kEnd = kBeg + per * BK;
    if (kEnd > g.K) kEnd = g.K;
    if (kBeg >= kEnd && g.epi != GEMM_EPI_STORE) return;
    if constexpr (WIDE) tile_body_wide<IN, 256, 128, FAST>(g, I0, J0, kBeg, kEnd, smem);
    else tile_body<IN, BM, BN, FAST>(g, I0, J0, kBeg, kEnd, smem);
}

template <int IN, int BM, int BN, bool FAST>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_tn_kernel(GemmArgs g) {
    extern __shared__ uint4 smem[];
    gemm_tn_workgroup<IN, BM, BN, FAST, false>(g, smem);
}

template <int IN, bool FAST>
__global__ __launch_bounds__(kWideThreads) void gemm_tn_wide_kernel(GemmArgs g) {
    extern __shared__ uint4 smem[];
    gemm_tn_workgroup<IN, 256, 128, FAST, true>(g, smem);
}

// True when both operands allow the branch-free 16-byte fetch path.
template <int IN>
bool operands_fast(const GemmArgs& g) {
    constexpr int VEC = InTraits<IN>::VEC;
    return (((uintptr_t)g.A & 15) == 0) && (((uintptr_t)g.B & 15) == 0) && (g.lda % VEC == 0) && (g.ldb % VEC == 0) &&
           (g.M % VEC == 0) && (g.N % VEC == 0) && g.K > 0;
}

template <int IN, int BM, int BN, bool FAST>
int launch_plain(aser_ctx* ctx, const GemmArgs& g) {
    using Cfg = TileCfg<IN, BM, BN>;
    static bool attr_set[16] = {false};
    constexpr bool WIDE = BM == 256 && BN == 128;          // see tile_body_wide
    void (*kern)(GemmArgs);
    if constexpr (WIDE) kern = gemm_tn_wide_kernel<IN, FAST>;
    else kern = gemm_tn_kernel<IN, BM, BN, FAST>;
    if (ctx->device >= 0 && ctx->device < 16 && !attr_set[ctx->device]) {
        ASER_HIP(ctx, hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)Cfg::LDS_BYTES));
        attr_set[ctx->device] = true;
    }
    const int64_t tm = ceil_div64(g.M, BM), tn = ceil_div64(g.N, BN);
    int64_t tiles = (g.tiles == GEMM_TILES_ALL) ? tm * tn : tm * (tm + 1) / 2;
    dim3 grid((unsigned)tiles, (unsigned)g.k_parts, 1);
    hipLaunchKernelGGL(kern, grid, dim3(WIDE ? kWideThreads : kThreads), Cfg::LDS_BYTES, ctx->stream, g);
    return aser_check_launch(ctx, "gemm_tn");
}

template <int IN, bool FAST>
int dispatch_tile2(aser_ctx* ctx, const GemmArgs& g) {
    if (g.bm == 256 && g.bn == 256) {
        if constexpr (IN == GEMM_IN_F32X6) {
            ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "gemm_tn: the six-product form has no 256 x 256 tile (LDS)");
        } else {
            return launch_plain<IN, 256, 256, FAST>(ctx, g);
        }
    }
    if constexpr (IN != GEMM_IN_BF16) {
        if (g.bm == 256 && g.bn == 128) return launch_plain<IN, 256, 128, FAST>(ctx, g);
    }
    if (g.bm == 128 && g.bn == 128) return launch_plain<IN, 128, 128, FAST>(ctx, g);
    ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "gemm_tn: unsupported tile %dx%d", g.bm, g.bn);
}

template <int IN>
int dispatch_tile(aser_ctx* ctx, const GemmArgs& g) {
    if (operands_fast<IN>(g)) return dispatch_tile2<IN, true>(ctx, g);
    return dispatch_tile2<IN, false>(ctx, g);
}

// ---------------------------------------------------------------------------------------------
// Gram update with an XCD-aware persistent schedule.
//
// One workgroup per compute unit (256 of them; the tile's LDS footprint allows no more).  Work-
// groups are dealt to the 8 XCDs round-robin, so workgroup w runs on XCD w % 8 as slot w / 8.
// The token range is cut into C chunks (C = 1, 2, 4 or 8, chosen on the host); 8 / C XCDs share
// a chunk and split the lower-triangle tiles among them, each XCD taking 32 consecutive tiles of
// the tile order per round.  The tile order (strips of 8 tile columns, row-major inside a strip)
// makes 32 consecutive tiles a 4 x 8 patch that needs only 12 distinct 256-channel slabs of X
// per K step, and the 32 workgroups of an XCD sweep their chunk in lock step, so a slab is
// fetched from HBM about once per XCD and served to the other workgroups from that XCD's L2.
// Tiles left over after the full rounds are split along K so that every workgroup stays busy.
// Partial tiles are added to G with fp32 atomics (C chunks contribute to every tile).
__device__ __forceinline__ void tri_strip_tile(int64_t t, int nt, int* p_out, int* q_out) {
    for (int q0 = 0; q0 < nt; q0 += 8) {
        for (int p = q0; p < nt; ++p) {
            const int cnt = (p - q0 + 1 < 8) ? (p - q0 + 1) : 8;
            if (t < cnt) { *p_out = p; *q_out = q0 + (int)t; return; }
            t -= cnt;
        }
    }
    *p_out = 0; *q_out = 0;
}

template <int IN, int BM, bool FAST>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1))) void gram_persistent_kernel(GemmArgs g) {
    extern __shared__ uint4 smem[];
    constexpr int BK = InTraits<IN>::BK;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int slots = gridDim.x >> 3;                                 // workgroups per XCD
    const int C = g.k_parts;                                          // K chunks: 1, 2, 4 or 8
    const int gsz = 8 / C;                                            // XCDs that share one K chunk
    const int chunk = xcd / gsz, xi = xcd % gsz;
    const int64_t W = (int64_t)gsz * slots;                           // workgroups per K chunk
    const int64_t widx = (int64_t)xi * slots + slot;                  // an XCD takes `slots` consecutive tiles
    const int nt = (int)((g.N + BM - 1) / BM);
    const int64_t T = (int64_t)nt * (nt + 1) / 2;
    const int64_t ksteps = (g.K + BK - 1) / BK;
    const int64_t per = (ksteps + C - 1) / C;
    const int64_t kx0 = (int64_t)chunk * per * BK;
    int64_t kx1 = kx0 + per * BK;
    if (kx1 > g.K) kx1 = g.K;
    if (kx0 >= kx1) return;
    const int64_t full = T / W, rem = T % W;
    const int64_t split = g.split;                                    // K split of the left-over tiles
    const int64_t rounds = full + ((rem > 0 && widx < rem * split) ? 1 : 0);
    for (int64_t round = 0; round < rounds; ++round) {
        int64_t t = round * W + widx, k0 = kx0, k1 = kx1;
        if (round == full) {                                          // left-over tile, one K part of it
            t = full * W + widx % rem;
            const int64_t xsteps = (kx1 - kx0 + BK - 1) / BK;
            const int64_t pp = (xsteps + split - 1) / split;
            k0 = kx0 + (widx / rem) * pp * BK;
            k1 = k0 + pp * BK;
            if (k1 > kx1) k1 = kx1;
            if (k0 >= k1) break;
        }
        int p, q;
        tri_strip_tile(t, nt, &p, &q);
        tile_body<IN, BM, BM, FAST>(g, (int64_t)p * BM, (int64_t)q * BM, k0, k1, smem);
    }
}

template <int IN, bool FAST>
int launch_gram_persistent2(aser_ctx* ctx, const GemmArgs& g) {
    using Cfg = TileCfg<IN, 256, 256>;
    static bool attr_set[16] = {false};
    auto kern = gram_persistent_kernel<IN, 256, FAST>;
    if (ctx->device >= 0 && ctx->device < 16 && !attr_set[ctx->device]) {
        ASER_HIP(ctx, hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)Cfg::LDS_BYTES));
        attr_set[ctx->device] = true;
    }
    hipLaunchKernelGGL(kern, dim3(256), dim3(kThreads), Cfg::LDS_BYTES, ctx->stream, g);
    return aser_check_launch(ctx, "gram_persistent");
}

// ---------------------------------------------------------------------------------------------
// Gram tiles for bf16 X without a register stage (the main path of the Gram update).
//
// X is tokens x channels, so a slab of 32 tokens x 256 channels is 32 rows of 512 contiguous
// bytes.  global_load_lds_dwordx4 copies it straight into LDS: a wavefront instruction moves
// 64 x 16 bytes to 1 KB of consecutive LDS (two slab rows), and each lane chooses which 16-byte
// chunk of the row it fetches, which is how the layout gets its XOR swizzle: chunk c of slab row
// k sits at chunk slot c ^ 4 (k & 3).  The MFMA operands (8 consecutive tokens of one channel
// per lane) come out of that token-major layout through ds_read_b64_tr_b16: 16 lanes read a
// 4 token x 16 channel block (4 lanes per row, 8 bytes each) and each lane receives the 4 tokens
// of its channel; with the swizzle the 4 rows of a block lie 64 bytes apart in the bank map, which is
// what this read needs to run without bank conflicts (the conflict counter reads zero; with rows 32
// bytes apart every read took twice as long).  So
// there is no transpose in registers, no LDS store instruction and no staging VGPRs; a ring of
// four 32 KB stages keeps three steps of loads in flight.  Rows past the token range and
// channels past n are fetched from a block of zeros.
__device__ uint4 g_zero_chunk[4];

typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x8_t __attribute__((ext_vector_type(8)));

constexpr int kDmaBK = 32;
constexpr int kDmaStages = 4;
constexpr int kDmaSlabBytes = kDmaBK * 512;
constexpr int kDmaStageBytes = 2 * kDmaSlabBytes;
constexpr size_t kDmaLdsBytes = (size_t)kDmaStages * kDmaStageBytes;

__device__ __forceinline__ bf16x8_t lds_tr_frag(const char* p, int off_lo, int off_hi) {
    typedef s16x4_t __attribute__((address_space(3))) * lds_s4p;
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4p)(p + off_lo));
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4p)(p + off_hi));
    const s16x8_t v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8_t, v);
}

// One 256 x 256 tile of G over tokens [kBeg, kEnd): G[I0.., J0..] += X[:, I0..]^T X[:, J0..].
//
// Step s multiplies stage s % 4 in two 16-token slices of 16 MFMAs each.  One wave per SIMD means
// nothing but instruction order hides latencies, so the order is pinned by hand: the operand reads
// of slice 1 are interleaved with the MFMAs of slice 0; the wait for the next stage, the barrier,
// the loads of stage s + 3 and the operand reads of the next step's slice 0 are interleaved with
// the MFMAs of slice 1.
__device__ __forceinline__ void gram_tile_dma(const GemmArgs& g, int64_t I0, int64_t J0, int64_t kBeg, int64_t kEnd,
                                              char* smem) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm0 = (wave >> 1) * 128, wn0 = (wave & 1) * 128;

    // ---- fetch roles: this wave issues instructions 4 wave .. 4 wave + 3 of each slab; instruction i
    // covers slab rows 2 i and 2 i + 1, lane l is chunk slot l % 32 of row 2 i + l / 32
    const int drow = lane >> 5, slot = lane & 31;
    const char* zero = (const char*)g_zero_chunk;
    const int64_t ld_bytes = g.lda * 2;
    const int row0 = 8 * wave + drow;                    // slab row of this lane in its wave's first instruction
    const char* gp[2][4];                                // next source address per (operand, instruction)
    int64_t gstep[2][2];                                 // its advance per step (0 for chunks past n: they stay on the zeros)
    int64_t tok_next = kBeg + row0;                      // token of gp[.][0]
#pragma unroll
    for (int par = 0; par < 2; ++par) {
        const int chunk = slot ^ (4 * ((2 * par + drow) & 3));
        const int64_t ca = I0 + 8 * chunk, cb = J0 + 8 * chunk;
        gstep[0][par] = (ca < g.M) ? kDmaBK * ld_bytes : 0;
        gstep[1][par] = (cb < g.N) ? kDmaBK * ld_bytes : 0;
#pragma unroll
        for (int t = par; t < 4; t += 2) {
            gp[0][t] = (ca < g.M) ? (const char*)g.A + ca * 2 + (tok_next + 2 * t) * ld_bytes : zero;
            gp[1][t] = (cb < g.N) ? (const char*)g.B + cb * 2 + (tok_next + 2 * t) * ld_bytes : zero;
        }
    }
    // LDS byte address of the ring (what M0 must hold for the LDS-direct loads)
    const uint32_t ring = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem + wave * 4096;
    // One load of stage `step` (op, t fixed at compile time by the callers' unrolling).  Written as
    // inline assembly on purpose: the compiler makes every LDS read wait for all LDS-direct loads it
    // knows of (it cannot tell the ring stages apart), which would undo the prefetch.  The stages are
    // kept apart by the explicit vmcnt waits and barriers below instead.
    auto issue_one = [&](int64_t step, int op, int t, bool tail) {
        const char* src = gp[op][t];
        if (tail && tok_next + 2 * t >= kEnd) src = zero;
        const uint32_t dst = ring + (uint32_t)(step & (kDmaStages - 1)) * kDmaStageBytes + op * kDmaSlabBytes + t * 1024;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(dst), "v"(src) : "memory", "m0");
        gp[op][t] += gstep[op][t & 1];
    };
    auto issue_all = [&](int64_t step) {
        const bool tail = kBeg + (step + 1) * kDmaBK > kEnd;
#pragma unroll
        for (int op = 0; op < 2; ++op)
#pragma unroll
            for (int t = 0; t < 4; ++t) issue_one(step, op, t, tail);
        tok_next += kDmaBK;
    };

    // ---- operand read offsets inside a stage (bytes), first of the four (k16 slice, half) reads
    int offa[4], offb[4];
    {
        const int krow = 8 * (lane >> 5) + ((lane & 15) >> 2);
        const int xr = 4 * ((lane & 15) >> 2);
        const int msub = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int ma = wm0 + 32 * i + msub, mb = wn0 + 32 * i + msub;
            offa[i] = krow * 512 + (((ma >> 3) ^ xr) * 16) + (ma & 7) * 2;
            offb[i] = kDmaSlabBytes + krow * 512 + (((mb >> 3) ^ xr) * 16) + (mb & 7) * 2;
        }
    }

    f32x16_t acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    const int64_t nsteps = (kEnd - kBeg + kDmaBK - 1) / kDmaBK;
    __syncthreads();                                     // the previous tile's readers are done with the ring
    for (int64_t s = 0; s < kDmaStages - 1 && s < nsteps; ++s) issue_all(s);
    if (nsteps >= 3) __builtin_amdgcn_s_waitcnt(0x4F70);             // vmcnt(16): stage 0 landed
    else if (nsteps == 2) __builtin_amdgcn_s_waitcnt(0x0F78);        // vmcnt(8)
    else __builtin_amdgcn_s_waitcnt(0x0F70);                         // vmcnt(0)
    __syncthreads();
    bf16x8_t a0[4], b0[4], a1[4], b1[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        a0[i] = lds_tr_frag(smem + offa[i], 0, 4 * 512);
        b0[i] = lds_tr_frag(smem + offb[i], 0, 4 * 512);
    }
    // STEADY steps have a successor, a stage to fetch and no ragged rows in it: no branch in the body.
    auto step = [&](int64_t s, auto steady_tag) {
        constexpr bool STEADY = decltype(steady_tag)::value;
        const char* st = smem + (int)(s & (kDmaStages - 1)) * kDmaStageBytes;
        const char* sn = smem + (int)((s + 1) & (kDmaStages - 1)) * kDmaStageBytes;
        const bool more = STEADY || s + 1 < nsteps;
        const bool fetch = STEADY || s + kDmaStages - 1 < nsteps;
        const bool tail = !STEADY && fetch && (kBeg + (s + kDmaStages) * kDmaBK > kEnd);
        // slice 0: 16 MFMAs, one operand fragment of slice 1 read after every second one
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0[i], b0[j], acc[i][j], 0, 0, 0);
                if (j == 1) a1[i] = lds_tr_frag(st + offa[i], 16 * 512, 20 * 512);
                if (j == 3) b1[i] = lds_tr_frag(st + offb[i], 16 * 512, 20 * 512);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // slice 1: row 0 of MFMAs covers the wait and the barrier, rows 1 and 2 the eight loads of
        // stage s + 3, rows 2 and 3 the reads of the next step's slice 0
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[i], b1[j], acc[i][j], 0, 0, 0);
                if (i == 0 && j == 1 && more) {
                    // stage s + 1 has landed when at most the loads of stage s + 2 are in flight
                    if (STEADY || s + 2 < nsteps) __builtin_amdgcn_s_waitcnt(0x0F78);    // vmcnt(8)
                    else __builtin_amdgcn_s_waitcnt(0x0F70);                             // vmcnt(0)
                    __syncthreads();                      // everyone's share landed; stage s - 1 is free
                }
                if (fetch && i == 1) { issue_one(s + kDmaStages - 1, 0, j, tail); }
                if (fetch && i == 2 && j < 2) { issue_one(s + kDmaStages - 1, 1, 2 * j, tail); issue_one(s + kDmaStages - 1, 1, 2 * j + 1, tail); }
                if (more && i == 2 && j >= 2) {
                    a0[2 * (j - 2)] = lds_tr_frag(sn + offa[2 * (j - 2)], 0, 4 * 512);
                    a0[2 * (j - 2) + 1] = lds_tr_frag(sn + offa[2 * (j - 2) + 1], 0, 4 * 512);
                }
                if (more && i == 3) b0[j] = lds_tr_frag(sn + offb[j], 0, 4 * 512);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (fetch) tok_next += kDmaBK;
    };
    const int64_t full_steps = (kEnd - kBeg) / kDmaBK;               // stages without ragged rows
    int64_t s = 0;
    for (; s + kDmaStages - 1 < full_steps; ++s) step(s, std::true_type{});
    for (; s < nsteps; ++s) step(s, std::false_type{});

    // acc[i][j][e] is G(row, col) with row = 32 i + 8 (e / 4) + 4 (lane / 32) + e % 4, col = 32 j + lane % 32
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t col = J0 + wn0 + 32 * j + (lane & 31);
            const int64_t rbase = I0 + wm0 + 32 * i + 4 * (lane >> 5);
            if (col >= g.N) continue;
            float* cbase = g.C + rbase * g.ldc + col;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int dr = 8 * (e >> 2) + (e & 3);
                if (rbase + dr < g.M) unsafeAtomicAdd(cbase + (int64_t)dr * g.ldc, g.alpha * acc[i][j][e]);
            }
        }
}

// The persistent XCD-aware schedule of gram_persistent_kernel with the LDS-direct tile body.
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1))) void gram_dma_kernel(GemmArgs g) {
    extern __shared__ uint4 smem[];
    constexpr int BK = kDmaBK, BM = 256;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int slots = gridDim.x >> 3;
    const int C = g.k_parts;
    const int gsz = 8 / C;
    const int chunk = xcd / gsz, xi = xcd % gsz;
    const int64_t W = (int64_t)gsz * slots;
    const int64_t widx = (int64_t)xi * slots + slot;
    const int nt = (int)((g.N + BM - 1) / BM);
    const int64_t T = (int64_t)nt * (nt + 1) / 2;
    const int64_t ksteps = (g.K + BK - 1) / BK;
    const int64_t per = (ksteps + C - 1) / C;
    const int64_t kx0 = (int64_t)chunk * per * BK;
    int64_t kx1 = kx0 + per * BK;
    if (kx1 > g.K) kx1 = g.K;
    if (kx0 >= kx1) return;
    const int64_t full = T / W, rem = T % W;
    const int64_t split = g.split;
    const int64_t rounds = full + ((rem > 0 && widx < rem * split) ? 1 : 0);
    for (int64_t round = 0; round < rounds; ++round) {
        int64_t t = round * W + widx, k0 = kx0, k1 = kx1;
        if (round == full) {
            t = full * W + widx % rem;
            const int64_t xsteps = (kx1 - kx0 + BK - 1) / BK;
            const int64_t pp = (xsteps + split - 1) / split;
            k0 = kx0 + (widx / rem) * pp * BK;
            k1 = k0 + pp * BK;
            if (k1 > kx1) k1 = kx1;
            if (k0 >= k1) break;
        }
        int p, q;
        tri_strip_tile(t, nt, &p, &q);
        gram_tile_dma(g, (int64_t)p * BM, (int64_t)q * BM, k0, k1, (char*)smem);
    }
}

int launch_gram_dma(aser_ctx* ctx, const GemmArgs& g) {
    static bool attr_set[16] = {false};
    if (ctx->device >= 0 && ctx->device < 16 && !attr_set[ctx->device]) {
        ASER_HIP(ctx, hipFuncSetAttribute((const void*)gram_dma_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kDmaLdsBytes));
        attr_set[ctx->device] = true;
    }
    hipLaunchKernelGGL(gram_dma_kernel, dim3(256), dim3(kThreads), kDmaLdsBytes, ctx->stream, g);
    return aser_check_launch(ctx, "gram_dma");
}

// One 256 x 128 tile of G over tokens [kBeg, kEnd), with sums in two levels (bound by the operand stream, 24 KB per 0.47 us and compute unit, and by the
// flush, 0.084 us per tile of the launch; both figures from fits over 70 sizes): every `seg` steps of 32 tokens the accumulators of the MFMAs are
// added to a second set and start anew, so the fp32 chains are as short as with a flush to G every `seg` steps and G is
// touched once.  (The 256 x 256 tile has no registers for a second set.)  Data path as in gram_tile_dma, for slabs of 256 and 128 channels in a
// ring of six stages of 24 KB; four wavefronts of 128 x 64.
constexpr int kSegStages = 6;
static_assert(kSegStages - 1 == kAserGramSegAhead, "the rule keeps ranges that fill the ring");
constexpr int kSegStageBytes = kDmaBK * (512 + 256);
constexpr size_t kSegLdsBytes = (size_t)kSegStages * kSegStageBytes;

__device__ __forceinline__ void gram_tile_seg(const GemmArgs& g, int64_t I0, int64_t J0, int64_t kBeg, int64_t kEnd, int seg, char* smem) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm0 = (wave >> 1) * 128, wn0 = (wave & 1) * 64;

    // ---- fetch roles: rows 8 wave .. 8 wave + 7 of both slabs; of A two rows of 32 chunks per load (0 .. 3), of B four rows of 16 (4, 5).  Chunk c of
    // row k stands in slot c ^ 4 (k & 3).
    const char* zero = (const char*)g_zero_chunk;
    const int64_t ld_bytes = g.lda * 2;
    const char* gp[6];
    int64_t gstep[6];
    int krow[6];                                          // slab row of this lane in each load
#pragma unroll
    for (int t = 0; t < 6; ++t) {
        krow[t] = 8 * wave + (t < 4 ? 2 * t + (lane >> 5) : 4 * (t - 4) + (lane >> 4));
        const int chunk = (t < 4 ? (lane & 31) : (lane & 15)) ^ (4 * (krow[t] & 3));
        const int64_t c = (t < 4 ? I0 : J0) + 8 * chunk;
        const bool in = c < g.M;                          // M == N
        gp[t] = in ? (const char*)g.A + c * 2 + (kBeg + krow[t]) * ld_bytes : zero;
        gstep[t] = in ? kDmaBK * ld_bytes : 0;
    }
    const uint32_t ring = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
    const uint32_t dst_a = ring + wave * 4096, dst_b = ring + kDmaBK * 512 + wave * 2048;
    auto issue_one = [&](int stage, int t, int64_t first, bool tail) {      // first: token of the stage's first row
        const char* src = gp[t];
        if (tail && first + krow[t] >= kEnd) src = zero;
        const uint32_t dst = (uint32_t)(stage * kSegStageBytes) + (t < 4 ? dst_a + t * 1024 : dst_b + (t - 4) * 1024);
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(dst), "v"(src) : "memory", "m0");
        gp[t] += gstep[t];
    };

    // ---- operand read offsets inside a stage, first of the four (k16 slice, half) reads
    int offa[4], offb[2];
    {
        const int kr = 8 * (lane >> 5) + ((lane & 15) >> 2);
        const int xr = 4 * ((lane & 15) >> 2);
        const int msub = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int ma = wm0 + 32 * i + msub;
            offa[i] = kr * 512 + (((ma >> 3) ^ xr) * 16) + (ma & 7) * 2;
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int mb = wn0 + 32 * j + msub;
            offb[j] = kDmaBK * 512 + kr * 256 + (((mb >> 3) ^ xr) * 16) + (mb & 7) * 2;
        }
    }

    f32x16_t acc[4][2], sum[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = sum[i][j][e] = 0.f;

    const int nsteps = (int)((kEnd - kBeg + kDmaBK - 1) / kDmaBK);
    const int full_steps = (int)((kEnd - kBeg) / kDmaBK);            // stages without ragged rows
    __syncthreads();                                     // the previous tile's readers are done with the ring
    for (int s = 0; s < kSegStages - 1; ++s) {           // a range has at least as many steps
        const int64_t first = kBeg + (int64_t)s * kDmaBK;
#pragma unroll
        for (int t = 0; t < 6; ++t) issue_one(s, t, first, s >= full_steps);
    }
    __builtin_amdgcn_s_waitcnt(0x4F78);                              // vmcnt(24): stage 0 landed
    __syncthreads();
    bf16x8_t a0[4], b0[2], a1[4], b1[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) a0[i] = lds_tr_frag(smem + offa[i], 0, 4 * 512);
#pragma unroll
    for (int j = 0; j < 2; ++j) b0[j] = lds_tr_frag(smem + offb[j], 0, 4 * 256);

    int stage = 0, left = seg;
    // STEADY steps have a successor, a stage to fetch and no ragged rows in it
    auto step = [&](int s, auto steady_tag) {
        constexpr bool STEADY = decltype(steady_tag)::value;
        const int nstage = stage == kSegStages - 1 ? 0 : stage + 1, fstage = stage == 0 ? kSegStages - 1 : stage - 1;
        const char* st = smem + stage * kSegStageBytes;
        const char* sn = smem + nstage * kSegStageBytes;
        const bool more = STEADY || s + 1 < nsteps;
        const bool fetch = STEADY || s + kSegStages - 1 < nsteps;
        const int64_t first = kBeg + (int64_t)(s + kSegStages - 1) * kDmaBK;
        const bool tail = !STEADY && s + kSegStages - 1 >= full_steps;
        // slice 0: the operands of slice 1 are read between its products
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            acc[m >> 1][m & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0[m >> 1], b0[m & 1], acc[m >> 1][m & 1], 0, 0, 0);
            if (m < 2) b1[m] = lds_tr_frag(st + offb[m], 16 * 256, 20 * 256);
            else if (m < 6) a1[m - 2] = lds_tr_frag(st + offa[m - 2], 16 * 512, 20 * 512);
            __builtin_amdgcn_sched_barrier(0);
        }
        // slice 1: the wait and the barrier, the loads of stage s + 5, the operands of the next step's slice 0
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            acc[m >> 1][m & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[m >> 1], b1[m & 1], acc[m >> 1][m & 1], 0, 0, 0);
            if (m == 1 && more) {
                if (STEADY) __builtin_amdgcn_s_waitcnt(0x4F72);      // vmcnt(18): stage s + 1 has landed, three more may be in flight
                else __builtin_amdgcn_s_waitcnt(0x0F70);             // vmcnt(0)
                __syncthreads();                                     // everyone's share landed; stage s - 1 is free
            }
            if (m >= 2 && fetch) issue_one(fstage, m - 2, first, tail);
            if (m >= 2 && more) {
                if (m < 4) b0[m - 2] = lds_tr_frag(sn + offb[m - 2], 0, 4 * 256);
                else a0[m - 4] = lds_tr_frag(sn + offa[m - 4], 0, 4 * 512);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        stage = nstage;
        if (--left == 0 || (!STEADY && s + 1 == nsteps)) {
            left = seg;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        sum[i][j][e] += acc[i][j][e];
                        acc[i][j][e] = 0.f;
                    }
        }
    };
    int s = 0;
    for (; s + kSegStages - 1 < full_steps; ++s) step(s, std::true_type{});
    for (; s < nsteps; ++s) step(s, std::false_type{});

#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int64_t col = J0 + wn0 + 32 * j + (lane & 31);
            const int64_t rbase = I0 + wm0 + 32 * i + 4 * (lane >> 5);
            if (col >= g.N) continue;
            float* cbase = g.C + rbase * g.ldc + col;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int dr = 8 * (e >> 2) + (e & 3);
                if (rbase + dr < g.M) unsafeAtomicAdd(cbase + (int64_t)dr * g.ldc, sum[i][j][e]);
            }
        }
}

// Tile t of the lower triangle in 256 x 128 tiles: strips of 8 tile columns, row by row, so that 32 consecutive ones are about a 4 x 8 patch.
__device__ __forceinline__ void tri_strip_half_tile(int64_t t, int nt, int* p_out, int* q_out) {
    for (int q0 = 0; q0 < 2 * nt; q0 += 8)
        for (int p = q0 / 2; p < nt; ++p) {
            const int cnt = (2 * p + 2 - q0 < 8) ? (2 * p + 2 - q0) : 8;
            if (t < cnt) { *p_out = p; *q_out = q0 + (int)t; return; }
            t -= cnt;
        }
    *p_out = 0; *q_out = 0;
}

// The schedule of gram_dma_kernel on 256 x 128 tiles with two-level sums.
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1))) void gram_seg_kernel(GemmArgs g, int seg) {
    extern __shared__ uint4 smem[];
    constexpr int BK = kDmaBK;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int slots = gridDim.x >> 3;
    const int C = g.k_parts;
    const int gsz = 8 / C;
    const int chunk = xcd / gsz, xi = xcd % gsz;
    const int64_t W = (int64_t)gsz * slots;
    const int64_t widx = (int64_t)xi * slots + slot;
    const int nt = (int)((g.N + 255) / 256);
    const int64_t T = (int64_t)nt * (nt + 1);
    const int64_t ksteps = (g.K + BK - 1) / BK;
    const int64_t per = (ksteps + C - 1) / C;
    const int64_t kx0 = (int64_t)chunk * per * BK;
    int64_t kx1 = kx0 + per * BK;
    if (kx1 > g.K) kx1 = g.K;
    if (kx0 >= kx1) return;
    const int64_t full = T / W, rem = T % W;
    const int64_t split = g.split;
    const int64_t rounds = full + ((rem > 0 && widx < rem * split) ? 1 : 0);
    for (int64_t round = 0; round < rounds; ++round) {
        int64_t t = round * W + widx, k0 = kx0, k1 = kx1;
        if (round == full) {
            t = full * W + widx % rem;
            const int64_t xsteps = (kx1 - kx0 + BK - 1) / BK;
            const int64_t pp = (xsteps + split - 1) / split;
            k0 = kx0 + (widx / rem) * pp * BK;
            k1 = k0 + pp * BK;
            if (k1 > kx1) k1 = kx1;
            if (k0 >= k1) break;
        }
        int p, q;
        tri_strip_half_tile(t, nt, &p, &q);
        if ((int64_t)q * 128 >= g.N) continue;           // the second half of a ragged last tile
        gram_tile_seg(g, (int64_t)p * 256, (int64_t)q * 128, k0, k1, seg, (char*)smem);
    }
}

int launch_gram_seg(aser_ctx* ctx, const GemmArgs& g, int seg) {
    static bool attr_set[16] = {false};
    if (ctx->device >= 0 && ctx->device < 16 && !attr_set[ctx->device]) {
        ASER_HIP(ctx, hipFuncSetAttribute((const void*)gram_seg_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSegLdsBytes));
        attr_set[ctx->device] = true;
    }
    hipLaunchKernelGGL(gram_seg_kernel, dim3(256), dim3(kThreads), kSegLdsBytes, ctx->stream, g, seg);
    return aser_check_launch(ctx, "gram_seg");
}

template <int IN>
int launch_gram_persistent(aser_ctx* ctx, const GemmArgs& g) {
    if (operands_fast<IN>(g)) return launch_gram_persistent2<IN, true>(ctx, g);
    return launch_gram_persistent2<IN, false>(ctx, g);
}

}  // namespace

int aser_gemm_tn(aser_ctx* ctx, const GemmArgs& g) {
    if (g.M <= 0 || g.N <= 0 || g.K < 0) ASER_FAIL(ctx, ASER_ERR_SHAPE, "gemm_tn: bad sizes");
    if (g.k_parts < 1 || (g.k_parts > 1 && g.epi != GEMM_EPI_ATOMIC))
        ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "gemm_tn: split K needs the atomic epilogue");
    if (g.tiles != GEMM_TILES_ALL && (g.M != g.N || g.bm != g.bn))
        ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "gemm_tn: triangular tiling needs a square problem and tile");
    if (g.Ct && g.epi != GEMM_EPI_STORE) ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "gemm_tn: Ct needs the store epilogue");
    if (g.long_first && g.tiles != GEMM_TILES_ALL) ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "gemm_tn: this tile order needs all tiles");
    if (g.epi == GEMM_EPI_RESID && (!g.sumsq || g.k_parts != 1 || g.bm != 128 || g.bn != 128))
        ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "gemm_tn: the residual epilogue needs sumsq, k_parts == 1 and 128 x 128 tiles");
    if (g.in_type == GEMM_IN_BF16) return dispatch_tile<GEMM_IN_BF16>(ctx, g);
    if (g.in_type == GEMM_IN_F32X3) return dispatch_tile<GEMM_IN_F32X3>(ctx, g);
    if (g.in_type == GEMM_IN_F32X6) return dispatch_tile<GEMM_IN_F32X6>(ctx, g);
    ASER_FAIL(ctx, ASER_ERR_DTYPE, "gemm_tn: unknown input type");
}

// Gram update: lower-triangle tiles of G += X^T X.  Aligned bf16 activations take the LDS-direct persistent schedule
// wherever it is faster; fp32 or unaligned ones the register-staged persistent schedule from 8192 tokens (bf16; 4096
// fp32) on; the rest splits K over a plain grid.  Partial tiles are added with fp32 atomics.
int aser_syrk_gram(aser_ctx* ctx, const void* X, int x_dtype, int64_t rows, int64_t n, int64_t ldx,
                   float* G, int64_t ldg) {
    GemmArgs g{};
    g.A = X; g.lda = ldx; g.B = X; g.ldb = ldx;
    g.C = G; g.ldc = ldg; g.Ct = nullptr; g.ldct = 0;
    g.M = n; g.N = n; g.K = rows; g.alpha = 1.f;
    g.in_type = (x_dtype == ASER_DTYPE_BF16) ? GEMM_IN_BF16 : aser_f32_form(ctx, n * n);
    g.epi = GEMM_EPI_ATOMIC; g.tiles = GEMM_TILES_LOWER; g.krange = GEMM_K_FULL;
    const bool six = g.in_type == GEMM_IN_F32X6;         // no 256 x 256 tile: the plain grid with 128 x 128 tiles
    const int bk = (g.in_type == GEMM_IN_BF16) ? 64 : 32;
    const int64_t ksteps = ceil_div64(rows, bk);
    const int64_t t256 = ceil_div64(n, 256);
    const int64_t T256 = t256 * (t256 + 1) / 2;
    if (T256 >= 32 && ksteps >= 8 * 16 && !six) {
        // Number of K chunks: fewest steps on the busiest workgroup, each tile visit charged with
        // the cost of flushing a tile through atomics (about a dozen K steps).
        int best_c = 8;
        int64_t best_cost = -1;
        for (int c = 1; c <= 8; c *= 2) {
            const int64_t W = 256 / c, full = T256 / W, rem = T256 % W;
            const int64_t steps_c = ceil_div64(ksteps, c);
            const int64_t split = rem ? W / rem : 1;
            const int64_t cost = full * (steps_c + 12) + (rem ? ceil_div64(steps_c, split) + 12 : 0);
            if (best_cost < 0 || cost < best_cost) { best_cost = cost; best_c = c; }
        }
        const int64_t W = 256 / best_c, rem = T256 % W;
        g.bm = g.bn = 256; g.k_parts = best_c; g.split = rem ? (int)(W / rem) : 1;
        if (g.in_type == GEMM_IN_BF16 && operands_fast<GEMM_IN_BF16>(g)) return launch_gram_dma(ctx, g);
        return (g.in_type == GEMM_IN_BF16) ? launch_gram_persistent<GEMM_IN_BF16>(ctx, g)
                                           : launch_gram_persistent<GEMM_IN_F32X3>(ctx, g);
    }
    g.bm = g.bn = (n <= 1024 || six) ? 128 : 256;
    const int64_t t = ceil_div64(n, g.bm), tiles = t * (t + 1) / 2;
    int64_t parts = ceil_div64(1024, tiles);              // aim at >= 4 workgroups per CU
    const int64_t max_parts = ksteps / 16 > 0 ? ksteps / 16 : 1;   // keep >= 16 steps per part
    if (parts > max_parts) parts = max_parts;
    if (parts < 1) parts = 1;
    // up to 1024 channels the plain grid's 128 x 128 tiles split K further (4096 tokens: 24 us against 40), and a few tokens of
    // wide channels are all flushes (256 of 3584: 31.5 us against 32.2, of 8192: 148 against 160)
    if (n > 1024 && rows >= (n > 5120 ? 512 : (n > 2560 ? 384 : 256)) && g.in_type == GEMM_IN_BF16 && operands_fast<GEMM_IN_BF16>(g)) {
        const AserGramSplit sp = aser_gram_dma_split(T256, ceil_div64(rows, kDmaBK), parts, ceil_div64(ksteps, parts));
        const AserGramSplit sg = aser_gram_seg_split(2 * T256, ceil_div64(rows, kDmaBK), parts);
        if (sg.cost < 0.97 * sp.cost) {
            g.k_parts = sg.chunks; g.split = sg.split;
            return launch_gram_seg(ctx, g, (int)ceil_div64(ceil_div64(rows, kDmaBK), 2 * parts));
        }
        if (sp.chunks > 0) {
            g.k_parts = sp.chunks; g.split = sp.split;
            return launch_gram_dma(ctx, g);
        }
    }
    g.k_parts = (int)parts;
    return aser_gemm_tn(ctx, g);
}
