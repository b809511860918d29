// Device code shared by the FFN kernels of ffn_kernels.hip and ffn_ring.hip.
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.h"

namespace fluxmoe {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

// What an LDS-direct load fetches for a 16-byte piece past the end of K.
static __device__ const uint4 g_zero_piece = {0, 0, 0, 0};

// SiLU(g) * u (Sec. 2.1's gated FFN) in FP32 with the hardware's exp2 and reciprocal, each within one
// ulp; the caller rounds the product to BF16.  g -> -inf gives exp2 = +inf, reciprocal 0, product -0.
__device__ __forceinline__ float swiglu(float g, float u) {
    const float e = __builtin_amdgcn_exp2f(-1.4426950408889634f * g);
    return g * __builtin_amdgcn_rcpf(1.0f + e) * u;
}

// Two FP32 values rounded to BF16 (nearest even) and packed, lo in bits 0..15: one v_cvt_pk_bf16_f32.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16_rne(float lo, float hi) {
    const f32x2_t v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

}  // namespace fluxmoe
