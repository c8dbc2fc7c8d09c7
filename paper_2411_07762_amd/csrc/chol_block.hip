// Launch of the 128-block Cholesky kernel (see chol_block.h).
#include "chol_block.h"

namespace {

__global__ __launch_bounds__(kCholThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void chol_block_kernel(float* D, int64_t ld, int b, float* Rinv, int32_t* info,
                                                                  int32_t pivot_base, int clear_d, float* beta_out, const int* gate) {
    extern __shared__ __align__(16) float sm[];
    if (gate && *gate == 0) return;
    chol_block_body(PlainBlock{D, ld, b}, sm, D, ld, b, Rinv, info, pivot_base, clear_d, beta_out);
}

}  // namespace

int aser_chol_block(aser_ctx* ctx, float* D, int64_t ld, int b, float* Rinv, int32_t* info, int32_t pivot_base, bool clear_d,
                    float* beta_out, const int* gate) {
    if (b <= 0 || b > kN) ASER_FAIL(ctx, ASER_ERR_SHAPE, "chol_block: block size out of range");
    static bool attr_set[16] = {false};
    if (ctx->device >= 0 && ctx->device < 16 && !attr_set[ctx->device]) {
        ASER_HIP(ctx, hipFuncSetAttribute((const void*)chol_block_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kCholLdsBytes));
        attr_set[ctx->device] = true;
    }
    hipLaunchKernelGGL(chol_block_kernel, dim3(1), dim3(kCholThreads), kCholLdsBytes, ctx->stream, D, ld, b, Rinv, info, pivot_base,
                       clear_d ? 1 : 0, beta_out, gate);
    return aser_check_launch(ctx, "chol_block");
}
