// What a lane of the projections for few tokens does with the weights (gemm_skinny_rows.hip, gemm_skinny_few.hip): read, update and write
// theta, draw the perturbation; and the 16-row matrix instructions that take the result.
#pragma once
#include "f32_parts.h"
#include "gemm_skinny.h"

namespace zo2 {

__device__ __forceinline__ v4f_t mfma16_bf16(v4u_t w, v4u_t x, v4f_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w), __builtin_bit_cast(bf16x8_t, x), c, 0, 0, 0);
}
// The matrix instruction's operands of 8 k: float32 as three bfloat16 parts, 16-bit formats as they are.
template <typename T> struct RowsMfma {
    static constexpr int kParts = 1;
    static __device__ __forceinline__ v4f_t run(v4u_t w, v4u_t x, v4f_t c);
};
template <> __device__ __forceinline__ v4f_t RowsMfma<f16_t>::run(v4u_t w, v4u_t x, v4f_t c) {
    typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, w), __builtin_bit_cast(f16x8_t, x), c, 0, 0, 0);
}
template <> __device__ __forceinline__ v4f_t RowsMfma<bf16_t>::run(v4u_t w, v4u_t x, v4f_t c) { return mfma16_bf16(w, x, c); }
template <> struct RowsMfma<float> { static constexpr int kParts = 3; };


// A lane's share of a slab of 64 k: two chunks of eight of one weight row, 32 apart.  The workgroup's rows are a buffer: rows past N are outside
// it, are read as zeros and not written.
template <typename T> struct WeightLane {
    static constexpr int Q = sizeof(T) == 4 ? 2 : 1;      // 16-byte pieces of eight elements
    struct Theta { v4u_t v[2][Q]; };
    __amdgpu_buffer_rsrc_t rows;
    int row_at;                  // of the first chunk at k 0, in bytes
    uint64_t we;                 // and in elements of the tensor (the random stream's counter)
    uint32_t tensor_id;

    // row `row` of the n_rows that start at row n0; k of the first chunk
    __device__ __forceinline__ WeightLane(const SkinnyArgs& a, const SkinnyProblem& p, int n0, int n_rows, int row, int k)
        : rows(__builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<T*>(p.theta) + (size_t)n0 * a.K, 0,
                                                 (int)((uint32_t)min(n_rows, a.N - n0) * a.K * (uint32_t)sizeof(T)), 0x00020000)),
          row_at((row * a.K + k) * (int)sizeof(T)), we((uint64_t)(n0 + row) * (uint64_t)a.K + (uint64_t)k), tensor_id(p.tensor_id) {}

    __device__ __forceinline__ void load(Theta& t, int k0) const {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < Q; ++e) t.v[h][e] = __builtin_amdgcn_raw_buffer_load_b128(rows, row_at + 32 * (int)sizeof(T) * h + 16 * e, k0 * (int)sizeof(T), 0);
    }
    __device__ __forceinline__ void draw(int k0, const PhiloxKeys& key, float (&z)[2][8]) const {
        uint32_t w[2][4];
        const uint64_t e = we + (uint64_t)k0;
        philox4x32_10_x2(e >> 3, (e >> 3) + 4, tensor_id, key, w);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < 4; ++i) box_muller(w[h][i], z[h][2 * i], z[h][2 * i + 1]);
    }
    __device__ __forceinline__ void values(const Theta& t, float (&th)[2][8]) const {
        Vec<T, 8> s[2];
        __builtin_memcpy(s, &t, sizeof(s));
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int j = 0; j < 8; ++j) th[h][j] = Fmt<T>::load(s[h].v[j]);
    }
    // th: theta on entry; theta' = theta - c z on return, and stored.  (k0 in the lanes' offsets: with a scalar offset in a register the
    // compiler lets the very next instruction write the store's data registers, here theta' - eps z over theta', and what arrives in
    // memory is now and then the new value.)
    __device__ __forceinline__ void update(int k0, float c, const float (&z)[2][8], float (&th)[2][8]) const {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            Vec<T, 8> s;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                s.v[j] = Fmt<T>::store(__builtin_fmaf(-c, z[h][j], th[h][j]));
                th[h][j] = Fmt<T>::load(s.v[j]);
            }
            v4u_t u[Q];
            __builtin_memcpy(u, &s, sizeof(u));
#pragma unroll
            for (int q = 0; q < Q; ++q) __builtin_amdgcn_raw_buffer_store_b128(u[q], rows, row_at + 32 * (int)sizeof(T) * h + 16 * q + k0 * (int)sizeof(T), 0, 0);
        }
    }
};

}  // namespace zo2
