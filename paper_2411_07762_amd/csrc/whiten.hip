// Whitening factor of Eq. 5 / Algorithm 1: S = chol(M^-1 G M^-1), blocked, one block row of 128 at a time.
//
// The factorisation runs on the upper triangle (G' = R^T R, R = S^T) so that every contraction
// has the K-major "A^T B" form of the MFMA kernel.  For block row k (rows k .. k+b):
//   update           G'[k:k+b, k:] -= R[:k, k:k+b]^T R[:k, k:]   (A, B = the finished rows above)
//   diagonal block   R11 = chol(D), R11^-1                       (one workgroup, LDS)
//   row panel        R12 = (R11^-1)^T * G'[k, k+b:]              (A = R11^-1, B = the panel, in place)
// The chain of diagonal blocks and panels bounds it up to about 8192 columns; the updates run beside the diagonal blocks, and the
// products of the update from there on.  Measured (ms; update, block and panel one after the other -> this): 1024 columns 0.40 -> 0.23,
// 2048 0.75 -> 0.40, 4096 1.69 -> 0.79, 6000 2.63 -> 1.32, 8192 3.97 -> 2.07, 11008 6.33 -> 3.87, 16384 -> 9.17, 28672 -> 36.7.
// A final pass moves R to the lower triangle (S = R^T) and clears the strict upper triangle; writing
// R12^T from the panel kernel instead cost 4 us per panel in scattered 16-byte stores.
#include <limits.h>

#include "chol_block.h"
#include "dispatch_rules.h"
#include "gemm_tile.h"

namespace {

constexpr int kNb = 128;

// S[i][j] = S[j][i] = G[i][j] / (m_i m_j) for i >= j, plus the damping term on the diagonal.
__global__ __launch_bounds__(256) void whiten_prep_kernel(const float* G, int64_t ldg, int64_t n, const float* mdiag,
                                                          float* S, int64_t lds, const double* diag_sum, float damp) {
    __shared__ float tile[64][65];
    // blockIdx.x enumerates tile pairs (bi >= bj)
    const int64_t t = blockIdx.x;
    int64_t bi = (int64_t)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
    while (bi * (bi + 1) / 2 > t) --bi;
    while ((bi + 1) * (bi + 2) / 2 <= t) ++bi;
    const int64_t bj = t - bi * (bi + 1) / 2;
    const int64_t r0 = bi * 64, c0 = bj * 64;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const float add = (damp > 0.f && diag_sum) ? (float)((double)damp * (*diag_sum) / (double)n) : 0.f;
    for (int i = ty; i < 64; i += 4) {
        const int64_t r = r0 + i, c = c0 + tx;
        float v = 0.f;
        if (r < n && c < n) {
            const float g = (r >= c) ? G[r * ldg + c] : G[c * ldg + r];
            const float mi = mdiag ? mdiag[r] : 1.f, mj = mdiag ? mdiag[c] : 1.f;
            v = g / (mi * mj);
            if (r == c) v += add;
        }
        tile[i][tx] = v;
    }
    __syncthreads();
    if (bi == bj) {                                      // only the upper triangle is worked on from here
        for (int i = ty; i < 64; i += 4) {
            const int64_t r = r0 + i, c = c0 + tx;
            if (r < n && c < n) S[r * lds + c] = tile[i][tx];
        }
    } else {
        for (int i = ty; i < 64; i += 4) {
            const int64_t r = c0 + i, c = r0 + tx;      // transposed tile
            if (r < n && c < n) S[r * lds + c] = tile[tx][i];
        }
    }
}

__global__ __launch_bounds__(256) void diag_scaled_sum_kernel(const float* G, int64_t ldg, int64_t n, const float* mdiag,
                                                              double* out) {
    __shared__ double red[4];
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) {
        const double mi = mdiag ? (double)mdiag[i] : 1.0;
        acc += (double)G[i * ldg + i] / (mi * mi);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) *out = red[0] + red[1] + red[2] + red[3];
}

// The factor was built as R = S^T in the upper triangle.  One pass over pairs of 64 x 64 tiles moves it
// to the lower triangle (through LDS, both sides coalesced) and clears the strict upper triangle.
__global__ __launch_bounds__(256) void upper_to_lower_kernel(float* S, int64_t n, int64_t lds) {
    __shared__ float tile[64][65];
    const int64_t t = blockIdx.x;
    int64_t bi = (int64_t)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
    while (bi * (bi + 1) / 2 > t) --bi;
    while ((bi + 1) * (bi + 2) / 2 <= t) ++bi;
    const int64_t bj = t - bi * (bi + 1) / 2;          // bi >= bj: upper tile (bj, bi) -> lower tile (bi, bj)
    const int64_t u0 = bj * 64, v0 = bi * 64;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    for (int i = ty; i < 64; i += 4) {
        const int64_t r = u0 + i, c = v0 + tx;
        float v = 0.f;
        if (r < n && c < n) {
            v = S[r * lds + c];
            if (c > r) S[r * lds + c] = 0.f;
        }
        tile[i][tx] = v;
    }
    __syncthreads();
    for (int i = ty; i < 64; i += 4) {
        const int64_t r = v0 + i, c = u0 + tx;          // lower entry (r, c) = upper entry (c, r)
        if (r < n && c < n && r > c) S[r * lds + c] = tile[tx][i];
    }
}

// One step of the factorisation in one launch (R = S^T in the upper triangle, block rows of 128; j is the current one):
//   workgroup 0           D = S[j, j] -= R[j - 1, j]^T R[j - 1, j], then its factor and the inverse of that
//   the next `now` ones   the rest of block row j -= R[j - 1, j]^T R[j - 1, right] (K = 128), 256 columns each
//   all others            block rows i = j + 1, j + 1 + lag, ... -= R[j - lag .. j - 1, i]^T R[j - lag .. j - 1, right], 256 columns each
// so a block row has received all finished rows but the last when its turn comes (at j = i - 1, and every `lag` steps before that, `lag` block
// rows at a time).  The factorisation keeps one compute unit busy for 17 us, and nothing else here is needed before the panel that
// follows.  Every entry has one writer per launch: with the whole contribution to block row j + 1 formed in one step, split
// over workgroups that meet in fp32 atomics, the flushes (1.4 TB/s) took 18 of 50 us in the middle of 11008 columns.  A 128 x 256 tile
// takes 5 us and 1.15 per K step of 32 on eight wavefronts; with operands split into bf16 pairs once, by the panel, and copied straight to LDS
// a step takes 0.87, which changed the whole by 2 to 5 % and needs rows of whole cache lines, so that was left out.
struct WhitenStep {
    float* S;
    int64_t lds, n, k0;
    float* Rinv;
    int32_t* info;
    int now, lag;
};

// acc += A^T B over the first `slices` (even) 16-deep slices of a K = 128 product whose operands stand in LDS as four K steps of 32 in the layout of
// tile_body (chunks [term][k / 8][column]); pa, pb: this lane's chunk of the first step.  Four slices' operands are read at a time.
template <int IN, int BMA, int BMB>
__device__ __forceinline__ void mfma_k128(f32x16_t& acc, const uint4* pa, const uint4* pb, int slices) {
    constexpr int NP = InTraits<IN>::NP, KB = 4;
    for (int s0 = 0; s0 < slices; s0 += 4) {
        bf16x8_t a[4][NP], b[4][NP];
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                a[s][p] = __builtin_bit_cast(bf16x8_t, pa[((s >> 1) * NP * KB + p * KB + 2 * (s & 1)) * BMA]);
                b[s][p] = __builtin_bit_cast(bf16x8_t, pb[((s >> 1) * NP * KB + p * KB + 2 * (s & 1)) * BMB]);
            }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (s == 2 && s0 + 2 >= slices) break;
#pragma unroll
            for (int q = NP - 1; q >= 0; --q)             // terms whose orders add up to q, the smallest products first
#pragma unroll
                for (int p = 0; p <= q; ++p) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s][q - p], b[s][p], acc, 0, 0, 0);
        }
        pa += 2 * NP * KB * BMA;
        pb += 2 * NP * KB * BMB;
    }
}

// D -= P^T P for the 128 x b block P (the operand form IN), D on its way to As.  Two and three terms of P take 64 and 96 KB; the former fit beside As, so
// only the corner is finished before the pivot chain starts.
template <int IN, bool FAST>
struct UpdatedBlock {
    static constexpr int NP = InTraits<IN>::NP, kStage = NP * 4 * kNb;      // chunks of one K step of 32
    static constexpr bool kBeside = (size_t)4 * kStage * 16 <= (size_t)kN * kP * 4;
    const float* D;
    const float* P;                                       // null: nothing to subtract
    int64_t ld;
    int b;

    // tile t of the ten 32 x 32 tiles of the upper triangle: (0,0) (0,1) (0,2) (0,3) (1,1) (1,2) (1,3) (2,2) (2,3) (3,3)
    static __device__ __forceinline__ void place(int t, int* ti, int* tj) {
        *ti = t < 4 ? 0 : (t < 7 ? 1 : (t < 9 ? 2 : 3));
        *tj = t < 4 ? t : (t < 7 ? t - 3 : (t < 9 ? t - 5 : 3));
    }
    static __device__ __forceinline__ void product(const float* stage, int t, f32x16_t& c) {
        const int lane = threadIdx.x & 63;
        int ti, tj;
        place(t, &ti, &tj);
#pragma unroll
        for (int e = 0; e < 16; ++e) c[e] = 0.f;
        const uint4* st = (const uint4*)stage + (lane >> 5) * kNb;
        mfma_k128<IN, kNb, kNb>(c, st + swz(32 * ti + (lane & 31)), st + swz(32 * tj + (lane & 31)), 8);
    }
    __device__ __forceinline__ void subtract(float* As, int t, const f32x16_t& c) const {
        const int lane = threadIdx.x & 63;
        int ti, tj;
        place(t, &ti, &tj);
        const int col = 32 * tj + (lane & 31), row = 32 * ti + 4 * (lane >> 5);
        float* out = As + row * kP + col;
        if (col >= b) return;                             // rows beyond b lie below the diagonal there
        float old[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) old[e] = out[(8 * (e >> 2) + (e & 3)) * kP];
#pragma unroll
        for (int e = 0; e < 16; ++e) out[(8 * (e >> 2) + (e & 3)) * kP] = old[e] - c[e];
    }

    __device__ __forceinline__ void load(float* As, float* Xs, bool vec) const {
        const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        BlockLoad d;
        if (!P) {
            d.load(D, ld, b, vec);
            d.store(As);
            return;
        }
        float* stage = kBeside ? Xs : As;
        Fetch<IN, kNb, FAST> f;
        Staged r;
        const int step = tid >> 7;
        f.init(P, ld, 0, b, 32 * step, kNb, tid & 127);
        f.load(r, kNb);
        d.load(D, ld, b, vec);
        f.store(r, (uint4*)stage + step * kStage);
        if (kBeside) {
            d.store(As);
            return;
        }
        __syncthreads();
        f32x16_t acc[2];
        product(stage, wave, acc[0]);
        if (wave < 2) product(stage, 8 + wave, acc[1]);
        __syncthreads();
        d.store(As);
        __syncthreads();
        subtract(As, wave, acc[0]);
        if (wave < 2) subtract(As, 8 + wave, acc[1]);
    }
    __device__ __forceinline__ void first(float* As, const float* Xs) const {
        if (!kBeside || !P) return;
        f32x16_t c;
        product(Xs, 0, c);
        subtract(As, 0, c);
    }
    __device__ __forceinline__ void rest(float* As, const float* Xs, int wave) const {
        if (!kBeside || !P) return;
        for (int t = wave; t < 10; t += 7) {              // wavefronts 1 .. 7; the ones with two tiles are not on the chain's SIMD
            f32x16_t c;
            product(Xs, t, c);
            subtract(As, t, c);
        }
    }
};

template <int IN, bool FAST>
__global__ __launch_bounds__(kCholThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void whiten_step_kernel(WhitenStep w) {
    extern __shared__ __align__(16) uint4 smem[];
    const int64_t rem = w.n - w.k0;
    if (blockIdx.x == 0) {
        const int b = (int)(rem < kNb ? rem : kNb);
        float* D = w.S + w.k0 * w.lds + w.k0;
        const UpdatedBlock<IN, FAST> source{D, w.k0 ? D - kNb * w.lds : nullptr, w.lds, b};
        chol_block_body(source, (float*)smem, D, w.lds, b, w.Rinv, w.info, (int32_t)w.k0, 0, nullptr);
        return;
    }
    int t = (int)blockIdx.x - 1;
    int64_t kBeg = w.k0 - kNb;
    int64_t row = w.k0, col = w.k0 + kNb;                 // first row and column of the block row's part
    if (t >= w.now) {
        t -= w.now;
        kBeg = w.k0 > w.lag * kNb ? w.k0 - w.lag * kNb : 0;
        row = col;
        for (;;) {
            const int tiles = (int)((w.n - row + 255) / 256);
            if (t < tiles) break;
            t -= tiles;
            row += w.lag * kNb;
        }
        col = row;
    }
    GemmArgs g{};
    g.lda = g.ldb = g.ldc = w.lds;
    g.alpha = -1.f;
    g.A = w.S + row;
    g.B = w.S + col;
    g.C = w.S + row * w.lds + col;
    g.M = w.n - row < kNb ? w.n - row : kNb;
    g.N = w.n - col;
    g.K = w.k0;
    tile_body_wide<IN, 128, 256, FAST, true>(g, 0, (int64_t)t * 256, kBeg, w.k0, smem);
}

template <int IN, bool FAST>
int launch_step(aser_ctx* ctx, const WhitenStep& w) {
    static bool attr_set[16] = {false};
    constexpr size_t lds = kCholLdsBytes > TileCfg<IN, 128, 256>::LDS_BYTES ? kCholLdsBytes : TileCfg<IN, 128, 256>::LDS_BYTES;
    auto kern = whiten_step_kernel<IN, FAST>;
    if (ctx->device >= 0 && ctx->device < 16 && !attr_set[ctx->device]) {
        ASER_HIP(ctx, hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        attr_set[ctx->device] = true;
    }
    int64_t groups = 1 + w.now;
    if (w.now)
        for (int64_t row = w.k0 + kNb; row < w.n; row += w.lag * kNb) groups += ceil_div64(w.n - row, 256);
    hipLaunchKernelGGL(kern, dim3((unsigned)groups), dim3(kCholThreads), lds, ctx->stream, w);
    return aser_check_launch(ctx, "whiten_step");
}

// Row panel: the 128 rows from k0 on, right of the diagonal block, become (R11^-1)^T times themselves, 64 columns per workgroup.  K is 128 only, so
// all operands are fetched at once and there is one wait and one barrier: 4.7 us a launch at 4096 columns (9.4 with four K steps
// through the tiles of the other products).
template <int IN, bool FAST>
__global__ __launch_bounds__(kCholThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void whiten_panel_kernel(WhitenStep w) {
    extern __shared__ __align__(16) uint4 smem[];
    constexpr int NP = InTraits<IN>::NP, KB = 4, BN = 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float* C = w.S + w.k0 * w.lds + w.k0 + kNb;
    const int64_t N = w.n - w.k0 - kNb, J0 = (int64_t)blockIdx.x * BN;
    uint4* sb = smem + 4 * NP * KB * kNb;
    const int step = tid >> 7, unit = tid & 127;
    {
        Fetch<IN, kNb, true> fa;
        FetchRows<IN, BN, 4, FAST> fb;
        Staged ra;
        uint4 rb[4];
        fa.init(w.Rinv, kNb, 0, kNb, 32 * step, kNb, unit);
        fb.init(C, w.lds, J0, N, 32 * step, kNb, unit);
        fa.load(ra, kNb);
        fb.load(rb, kNb);
        __builtin_amdgcn_sched_barrier(0);
        fa.store(ra, smem + step * NP * KB * kNb);
        fb.store(rb, sb + step * NP * KB * BN);
    }
    __syncthreads();
    // row tile i needs k < 32 (i + 1): the two wavefronts of a SIMD take a long and a short one
    const int ti = wave < 4 ? wave : 7 - wave, tj = (wave >> 2) ^ (ti & 1);
    f32x16_t acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    mfma_k128<IN, kNb, BN>(acc, smem + (lane >> 5) * kNb + swz(32 * ti + (lane & 31)), sb + (lane >> 5) * BN + swz(32 * tj + (lane & 31)), 2 * (ti + 1));
    const int64_t col = J0 + 32 * tj + (lane & 31);
    float* out = C + (int64_t)(32 * ti + 4 * (lane >> 5)) * w.lds + col;
    if (col >= N) return;
#pragma unroll
    for (int e = 0; e < 16; ++e) out[(int64_t)(8 * (e >> 2) + (e & 3)) * w.lds] = acc[e];
}

template <int IN, bool FAST>
int launch_panel(aser_ctx* ctx, const WhitenStep& w) {
    static bool attr_set[16] = {false};
    constexpr size_t lds = (size_t)4 * InTraits<IN>::NP * 4 * (kNb + 64) * 16;
    auto kern = whiten_panel_kernel<IN, FAST>;
    if (ctx->device >= 0 && ctx->device < 16 && !attr_set[ctx->device]) {
        ASER_HIP(ctx, hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        attr_set[ctx->device] = true;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)ceil_div64(w.n - w.k0 - kNb, 64)), dim3(kCholThreads), lds, ctx->stream, w);
    return aser_check_launch(ctx, "whiten_panel");
}

}  // namespace

extern "C" int aser_whiten(aser_ctx* ctx, const float* G, int64_t ldg, int64_t n, const float* mdiag, float damp,
                           float* S, int64_t lds, int32_t* info) {
    if (!ctx) return ASER_ERR_INVALID_ARG;
    if (!G || !S) ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "whiten: null pointer");
    if (n <= 0 || ldg < n || lds < n) ASER_FAIL(ctx, ASER_ERR_SHAPE, "whiten: bad shape");
    if (!(damp >= 0.f)) ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "whiten: damp must be >= 0");
    if (((uintptr_t)G & 3) || ((uintptr_t)S & 3)) ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "whiten: misaligned pointer");
    const size_t need = (size_t)kNb * kNb * 4 + 512 + kAserWsTail;
    if (!ctx->ws || ctx->ws_bytes < need) ASER_FAIL(ctx, ASER_ERR_WORKSPACE, "whiten: workspace too small");
    ASER_TRY(aser_prepare_device(ctx));

    float* Rinv = (float*)ctx->ws;
    int32_t* info_dev = (int32_t*)((char*)ctx->ws + ctx->ws_bytes - kAserWsTail);
    double* diag_sum = (double*)((char*)ctx->ws + (size_t)kNb * kNb * 4 + 256);

    // A flag still pending from an earlier asynchronous call is kept (the factorisation lowers it with
    // atomicMin): that call's failed pivot is then still reported, by whichever call synchronises next.
    if (ctx->pending_info_dev != info_dev) ASER_TRY(aser_set_i32(ctx, info_dev, (int32_t)INT_MAX));
    if (damp > 0.f) {
        hipLaunchKernelGGL(diag_scaled_sum_kernel, dim3(1), dim3(256), 0, ctx->stream, G, ldg, n, mdiag, diag_sum);
        ASER_TRY(aser_check_launch(ctx, "diag_sum"));
    }
    const int64_t t64 = ceil_div64(n, 64);
    hipLaunchKernelGGL(whiten_prep_kernel, dim3((unsigned)(t64 * (t64 + 1) / 2)), dim3(256), 0, ctx->stream, G, ldg, n,
                       mdiag, S, lds, (const double*)diag_sum, damp);
    ASER_TRY(aser_check_launch(ctx, "whiten_prep"));

    // Blocked Cholesky on the upper triangle (R = S^T), a block row at a time: two launches per block row, the step (see WhitenStep) and the row panel.
    const bool six = aser_f32_form(ctx, n * n) == GEMM_IN_F32X6;     // three or six bf16 products per fp32 product
    const bool fast = ((uintptr_t)S & 15) == 0 && (lds & 3) == 0 && (n & 3) == 0;
    const int lag = aser_whiten_lag(n, six || !fast);
    for (int64_t k0 = 0; k0 < n; k0 += kNb) {
        const int64_t right = n - k0 - kNb;              // columns to the right of the block
        const WhitenStep w{S, lds, n, k0, Rinv, info_dev, (k0 > 0 && right > 0) ? (int)ceil_div64(right, 256) : 0, lag};
        ASER_TRY(six ? (fast ? launch_step<GEMM_IN_F32X6, true>(ctx, w) : launch_step<GEMM_IN_F32X6, false>(ctx, w))
                     : (fast ? launch_step<GEMM_IN_F32X3, true>(ctx, w) : launch_step<GEMM_IN_F32X3, false>(ctx, w)));
        if (right > 0)
            ASER_TRY(six ? (fast ? launch_panel<GEMM_IN_F32X6, true>(ctx, w) : launch_panel<GEMM_IN_F32X6, false>(ctx, w))
                         : (fast ? launch_panel<GEMM_IN_F32X3, true>(ctx, w) : launch_panel<GEMM_IN_F32X3, false>(ctx, w)));
    }
    hipLaunchKernelGGL(upper_to_lower_kernel, dim3((unsigned)(t64 * (t64 + 1) / 2)), dim3(256), 0, ctx->stream, S, n, lds);
    ASER_TRY(aser_check_launch(ctx, "upper_to_lower"));

    if (!info) {                                         // asynchronous: the flag is read by the next synchronising call
        ctx->pending_info_dev = info_dev;
        return ASER_OK;
    }
    ctx->pending_info_dev = info_dev;
    AserPending pend;
    ASER_TRY(aser_sync_status(ctx, &pend));
    *info = (pend.pivot == INT_MAX) ? 0 : pend.pivot;
    return aser_report_pending(ctx, pend, "whiten");
}
