// Activation smoothing via outlier analysis (Sec. 4.2): channel scores Xbar * Wbar, the index set
// I_f of the f largest scores, the diagonal m of Eq. 11 and the outlier part W_o of W M.
// All statistics are fp64 so that the selected indices do not depend on summation order in
// any realistic case; ties go to the lower channel index.
#include "aser_internal.h"
#include "rank_slot.h"

namespace {

constexpr int kSelMaxN = 32768;

// a beats b: larger score, or equal score and lower index
__device__ __forceinline__ bool beats(double sa, int ia, double sb, int ib) {
    return (sa > sb) || (sa == sb && ia < ib);
}

// Scores; a score that is NaN or +Inf (no tokens, or non-finite statistics) is no candidate.  Channel i's rank then takes the
// place of its column sum (the low word of wsum[i], which only this thread reads) and starts at zero.
__global__ __launch_bounds__(256) void score_kernel(const double* abs_sum, const int64_t* count, double* wsum,
                                                    int64_t m, int64_t n, double* score) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double xbar = abs_sum[i] / (double)(*count);
    const double wbar = wsum[i] / (double)m;
    score[i] = xbar * wbar;
    ((int2*)wsum)[i] = make_int2(0, 0);
}

// Scores are >= 0; -1 stands for "never a candidate", which every candidate beats.
__device__ __forceinline__ double candidate(double s) { return (s >= 0.0 && s <= 1.7e308) ? s : -1.0; }

// rank[2 i] += the channels among 128 (blockIdx.y) that beat channel i.  All pairs are compared: n^2 comparisons spread over the
// chip take a few microseconds, where f rounds of an arg-max in one workgroup are a chain of 1.6 us each (f = 64: 102 us at
// 4096 channels, 205 us at 11008).
constexpr int kRankPart = 128;
__global__ __launch_bounds__(256) void rank_kernel(const double* __restrict__ score, int n, int32_t* __restrict__ rank) {
    __shared__ double other[kRankPart];
    const int j0 = blockIdx.y * kRankPart, len = n - j0 < kRankPart ? n - j0 : kRankPart;
    for (int t = threadIdx.x; t < len; t += 256) other[t] = candidate(score[j0 + t]);
    __syncthreads();
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const double s = candidate(score[i]);
    int better = 0;
#pragma unroll 8
    for (int t = 0; t < len; ++t) better += beats(other[t], j0 + t, s, i) ? 1 : 0;
    if (better) atomicAdd(rank + 2 * (int64_t)i, better);
}

// One workgroup: idx in rank order (ranks are distinct), then the smoothing diagonal of Eq. 11.
__global__ __launch_bounds__(1024) void select_kernel(const double* __restrict__ score, const int32_t* __restrict__ rank,
                                                      const double* __restrict__ abs_sum, const int64_t* __restrict__ count, int n, int f,
                                                      int32_t* __restrict__ idx, float* __restrict__ mdiag, int32_t* __restrict__ no_candidate) {
    __shared__ double red[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const double cnt = (double)(*count);
    double xmin = 1.0e300;
    for (int i = tid; i < n; i += 1024) {
        mdiag[i] = 1.0f;
        const int r = rank[2 * (int64_t)i];
        if (!rank_has_slot(r, f)) continue;
        // No candidate for this slot (fewer than f channels with a finite score): it gets -1, which every
        // consumer of idx skips, and the flag makes the next synchronising call fail with a status.
        const bool none = candidate(score[i]) < 0.0;
        idx[r] = none ? -1 : i;
        if (none) *no_candidate = 1;
        else xmin = fmin(xmin, abs_sum[i] / cnt);                    // X_min over the selected channels (Eq. 11)
    }
    if (f == 0) return;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) xmin = fmin(xmin, __shfl_xor(xmin, o, 64));
    if (lane == 0) red[wave] = xmin;
    __syncthreads();
    xmin = red[0];
#pragma unroll
    for (int w = 1; w < 16; ++w) xmin = fmin(xmin, red[w]);
    for (int i = tid; i < n; i += 1024)
        if (rank_has_slot(rank[2 * (int64_t)i], f) && candidate(score[i]) >= 0.0) mdiag[i] = (float)((abs_sum[i] / cnt) / xmin);
}

__global__ __launch_bounds__(256) void gather_wo_kernel(const float* __restrict__ W, int64_t m, int64_t n, int64_t ldw,
                                                        const int32_t* __restrict__ idx, const float* __restrict__ mdiag,
                                                        int f, float* __restrict__ W_o) {
    const int64_t total = m * f;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t o = t / f;
        const int k = (int)(t % f);
        const int c = idx[k];
        W_o[t] = (c >= 0 && c < n) ? W[o * ldw + c] * mdiag[c] : 0.f;
    }
}

}  // namespace

// The two fp64 arrays of n entries (column sums of |W|, scores) and the selection's status word, wherever
// they live: in the bound workspace (aser_smooth_outliers) or in this file's static array.
static int smooth_run(aser_ctx* ctx, const float* W, int64_t m, int64_t n, int64_t ldw, const double* abs_sum,
                      const int64_t* count, int32_t f, int32_t* idx, float* mdiag, float* W_o, double* score,
                      double* wsum, double* sc_scratch, int32_t* sel_flag) {
    if (ctx->pending_sel_dev != sel_flag) ASER_TRY(aser_set_i32(ctx, sel_flag, 0));
    ctx->pending_sel_dev = sel_flag;
    double* sc = score ? score : sc_scratch;
    ASER_TRY(aser_fill_bytes(ctx, wsum, (size_t)n * 8));
    ASER_TRY(aser_col_abs_sum_w(ctx, W, m, n, ldw, wsum));
    hipLaunchKernelGGL(score_kernel, dim3((unsigned)ceil_div64(n, 256)), dim3(256), 0, ctx->stream, abs_sum, count, wsum, m, n, sc);
    ASER_TRY(aser_check_launch(ctx, "score"));
    int32_t* rank = (int32_t*)wsum;
    if (f > 0) {
        hipLaunchKernelGGL(rank_kernel, dim3((unsigned)ceil_div64(n, 256), (unsigned)ceil_div64(n, kRankPart)), dim3(256), 0, ctx->stream,
                           (const double*)sc, (int)n, rank);
        ASER_TRY(aser_check_launch(ctx, "rank"));
    }
    hipLaunchKernelGGL(select_kernel, dim3(1), dim3(1024), 0, ctx->stream, (const double*)sc, (const int32_t*)rank, abs_sum, count,
                       (int)n, (int)f, idx, mdiag, sel_flag);
    ASER_TRY(aser_check_launch(ctx, "select"));
    if (W_o && f > 0) {
        const int64_t total = m * f;
        const int blocks = (int)(ceil_div64(total, 256) < 2048 ? ceil_div64(total, 256) : 2048);
        hipLaunchKernelGGL(gather_wo_kernel, dim3(blocks), dim3(256), 0, ctx->stream, W, m, n, ldw, (const int32_t*)idx,
                           (const float*)mdiag, (int)f, W_o);
        ASER_TRY(aser_check_launch(ctx, "gather_wo"));
    }
    return ASER_OK;
}

static int smooth_validate(aser_ctx* ctx, const float* W, int64_t m, int64_t n, int64_t ldw, const double* abs_sum,
                           const int64_t* count, int32_t f, const int32_t* idx, const float* mdiag, const double* score) {
    if (!W || !abs_sum || !count || !mdiag) ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "smooth_outliers: null pointer");
    if (m <= 0 || n <= 0 || ldw < n) ASER_FAIL(ctx, ASER_ERR_SHAPE, "smooth_outliers: bad shape");
    if (f < 0 || f > n) ASER_FAIL(ctx, ASER_ERR_SHAPE, "smooth_outliers: f must be in [0, n]");
    if (f > 0 && !idx) ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "smooth_outliers: idx is null");
    if (n > kSelMaxN) ASER_FAIL(ctx, ASER_ERR_SHAPE, "smooth_outliers: n > 32768 is not supported");
    if (((uintptr_t)abs_sum & 7) || ((uintptr_t)count & 7) || (score && ((uintptr_t)score & 7)))
        ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "smooth_outliers: misaligned fp64/int64 pointer");
    return ASER_OK;
}

extern "C" int aser_smooth_outliers(aser_ctx* ctx, const float* W, int64_t m, int64_t n, int64_t ldw,
                                    const double* abs_sum, const int64_t* count, int32_t f,
                                    int32_t* idx, float* mdiag, float* W_o, double* score) {
    if (!ctx) return ASER_ERR_INVALID_ARG;
    ASER_TRY(smooth_validate(ctx, W, m, n, ldw, abs_sum, count, f, idx, mdiag, score));
    const size_t need = align_up((size_t)n * 8, 256) * 2 + kAserWsTail;
    if (!ctx->ws || ctx->ws_bytes < need) ASER_FAIL(ctx, ASER_ERR_WORKSPACE, "smooth_outliers: workspace too small");
    ASER_TRY(aser_prepare_device(ctx));
    // word 1 of the workspace tail: raised by the selection when it runs out of usable channels
    int32_t* sel_flag = (int32_t*)((char*)ctx->ws + ctx->ws_bytes - kAserWsTail) + 1;
    return smooth_run(ctx, W, m, n, ldw, abs_sum, count, f, idx, mdiag, W_o, score, (double*)ctx->ws,
                      (double*)((char*)ctx->ws + align_up((size_t)n * 8, 256)), sel_flag);
}

// ---------------------------------------------------------------------------------------------
// The same stage for callers that cannot allocate and therefore have no workspace to bind (code under
// HIP graph capture, serving loops, harnesses that forbid hipMalloc): the two fp64 arrays and the status
// word live in a static device array of fixed size instead.  Every device holds its own copy of the
// array at its own address, looked up once per device.
constexpr size_t kScratchColBytes = (size_t)kSelMaxN * 8;             // one fp64 per channel, n <= 32768
constexpr size_t kScratchBytes = 2 * kScratchColBytes + 256;          // |W| column sums, scores, status word
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

static void* g_scratch_ptr[16] = {nullptr};

extern "C" int aser_smooth_outliers_noalloc(aser_ctx* ctx, const float* W, int64_t m, int64_t n, int64_t ldw,
                                            const double* abs_sum, const int64_t* count, int32_t f,
                                            int32_t* idx, float* mdiag, float* W_o, double* score) {
    if (!ctx) return ASER_ERR_INVALID_ARG;
    ASER_TRY(smooth_validate(ctx, W, m, n, ldw, abs_sum, count, f, idx, mdiag, score));
    if ((size_t)n * 8 > kScratchColBytes)
        ASER_FAIL(ctx, ASER_ERR_SHAPE, "smooth_outliers_noalloc: n = %lld exceeds the static scratch (%d channels)",
                  (long long)n, kSelMaxN);
    if (ctx->device < 0 || ctx->device >= 16)
        ASER_FAIL(ctx, ASER_ERR_INVALID_ARG, "smooth_outliers_noalloc: device index %d is outside [0, 16)", ctx->device);
    ASER_TRY(aser_prepare_device(ctx));
    if (!g_scratch_ptr[ctx->device]) {
        // the array's name is only a host-side handle: its device address comes from the runtime, with
        // the context's device current (aser_prepare_device has just made it so)
        void* p = nullptr;
        ASER_HIP(ctx, hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) ASER_FAIL(ctx, ASER_ERR_HIP, "smooth_outliers_noalloc: no device address for the static scratch");
        g_scratch_ptr[ctx->device] = p;
    }
    char* base = (char*)g_scratch_ptr[ctx->device];
    // every call on this device shares the array and finds the last call's contents in it: the column
    // sums are cleared by smooth_run, the scores are overwritten, the status word is reset unless it is
    // still pending on this context
    return smooth_run(ctx, W, m, n, ldw, abs_sum, count, f, idx, mdiag, W_o, score, (double*)base,
                      (double*)(base + kScratchColBytes), (int32_t*)(base + 2 * kScratchColBytes));
}
