// Two fp32 values as two bf16 values in one word, the first in the lower half.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {            // rounded to nearest even, two at a time by one instruction
    typedef float pair_t __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16_pair_t __attribute__((ext_vector_type(2)));
    const pair_t v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16_pair_t));
}
// Their upper halves: truncated, exact for values that are bf16 already.
__device__ __forceinline__ uint32_t upper_halves(float a, float b) { return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u); }
__device__ __forceinline__ uint32_t bf16_rne(float x) {
    const uint32_t u = __float_as_uint(x);
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}
