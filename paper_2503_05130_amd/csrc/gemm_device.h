// What the full-size product (gemm.hip) and the decode-step product
// (decode.hip) share on the device: vector types, the kernels' parameters and
// the bf16 conversions.
#pragma once

#include "gelu.h"
#include "gemm.h"

namespace iefwd {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void *lds_ptr_t;

struct GemmParams {
    const bf16_t *a;
    const bf16_t *w;
    const bf16_t *bias;
    const float *resid;
    void *out;
    int M, N, K;
    int tiles_m, tiles_n;
    QkvDst qkv;
    LnResid ln;
    LnIn lnin;
    const bf16_t *aux;   // Epi::GeluBwdBf16: the GELU's input [M, N]
    bf16_t *out2;        // Epi::BiasGelu2Bf16: GELU(out) [M, N]
};

__device__ inline bf16_t f32_to_bf16(float f) {
    __bf16 b = (__bf16)f;   // round to nearest even
    return __builtin_bit_cast(bf16_t, b);
}

__device__ inline uint32_t pack2(float lo, float hi) {
    return (uint32_t)f32_to_bf16(lo) | ((uint32_t)f32_to_bf16(hi) << 16);
}

}  // namespace
}  // namespace iefwd
