// float32 operands as three bfloat16 parts each (what that is good for, and how far sums are from 64 bits: gemm_f32.hip).
#pragma once
#include "common.h"

namespace zo2 {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float v2f_t __attribute__((ext_vector_type(2)));
typedef float v4f_t __attribute__((ext_vector_type(4)));
typedef uint32_t v2u_t __attribute__((ext_vector_type(2)));
typedef uint32_t v4u_t __attribute__((ext_vector_type(4)));

// two neighbouring values: the nearest bfloat16 of each in one word, and what is left of them (5.5 instructions an element in
// all; cutting instead of rounding takes as many and is 2 % slower with many rows)
__device__ __forceinline__ uint32_t split_step(float& a, float& b) {
    const uint32_t h = __builtin_bit_cast(uint32_t, __builtin_convertvector(v2f_t{a, b}, bf16x2_t));
    a -= u2f(h << 16);
    b -= u2f(h & 0xffff0000u);
    return h;
}

__device__ __forceinline__ f32x16_t mfma_bf16(v4u_t w, v4u_t x, f32x16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, w), __builtin_bit_cast(bf16x8_t, x), c, 0, 0, 0);
}
template <int TM, int TN>
__device__ __forceinline__ void clear_acc(f32x16_t (&acc)[TM][TN]) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
}

// Two kinds of operands have no such parts.  An infinity (or a value that rounds to one in bfloat16): inf - inf is a NaN where
// float32 has inf.  A value below 2^-110: its later parts fall under bfloat16's range, to 2^-134 each in the worst case, which is nothing
// beside a sum of 2^-74 or more whose other factors are up to 2^20 (2^-40 of it, times K) and shows in one that is smaller.  A wavefront with
// a sum that is not finite, or below 2^-74 and not zero, computes its tile again with float32 products, straight from memory.  (To look
// at every operand as it is split takes 1.5 instructions an element more: 64 x 24576 x 1024 35 -> 40 us, 768 x 50272 x 2048 822 -> 868.)
struct OddSums {
    float odd = 0.f;                       // 0 x finite sums to 0; anything else to a NaN
    uint32_t least = 0xffffffffu;          // (bits << 1) - 1 has the magnitudes in order, zero last
    __device__ __forceinline__ void look(float x) {
        odd = __builtin_fmaf(x, 0.f, odd);
        least = min(least, (f2u(x) << 1) - 1u);
    }
    __device__ __forceinline__ bool any() const { return __any(odd != 0.f || least < ((uint32_t)(127 - 74) << 24) - 1u); }
};

}  // namespace zo2
