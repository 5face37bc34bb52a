// Row-wise and elementwise kernels around the GEMMs: random-stream test hooks, format
// conversion (Sec. 5.5 pack / unpack), LayerNorm, embedding gather with on-the-fly
// update + perturb, cross-entropy, and the scalar epilogue that forms g (Eq. 2).
#include "rowops.h"

#include <algorithm>

#include "philox.h"

namespace zo2 {

// ------------------------------------------------------------------ wave / block reductions
template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}
// all threads of a 256-thread block receive the sum
template <typename T>
__device__ __forceinline__ T block_sum(T v, T* sh) {
    v = wave_sum(v);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[w] = v;
    __syncthreads();
    T r = sh[0];
    for (int i = 1; i < (int)(blockDim.x >> 6); ++i) r += sh[i];
    return r;
}
__device__ __forceinline__ float block_max(float v, float* sh) {
    v = wave_max(v);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[w] = v;
    __syncthreads();
    float r = sh[0];
    for (int i = 1; i < (int)(blockDim.x >> 6); ++i) r = fmaxf(r, sh[i]);
    return r;
}

// ------------------------------------------------------------------ random-stream hooks
__global__ void philox_words_kernel(PhiloxKeys k, uint32_t tensor_id, uint64_t e0, uint64_t n, uint32_t* out) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint64_t e = e0 + i, q = e >> 2;
    uint32_t w[4];
    philox4x32_10((uint32_t)q, (uint32_t)(q >> 32), tensor_id, 0u, k, w);
    const uint32_t r = (uint32_t)(e & 3);
    out[i] = r == 0 ? w[0] : r == 1 ? w[1] : r == 2 ? w[2] : w[3];
}

__global__ void gaussian_kernel(PhiloxKeys k, uint32_t tensor_id, uint64_t e0, uint64_t n, float* out) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint64_t e = e0 + i;
    float z[4];
    gaussian4(k, tensor_id, e & ~(uint64_t)3, z);
    const uint32_t r = (uint32_t)(e & 3);
    out[i] = r == 0 ? z[0] : r == 1 ? z[1] : r == 2 ? z[2] : z[3];
}

zo2_status philox_words(uint64_t seed, uint32_t tid, uint64_t e0, uint64_t n, uint32_t* out, hipStream_t st) {
    if (n == 0) return ZO2_OK;
    ZO2_OP_CHECK(out != nullptr, ZO2_EINVAL, "philox_words: out is NULL");
    ZO2_OP_CHECK(n < (1ull << 39), ZO2_EINVAL, "philox_words: n too large");
    hipLaunchKernelGGL(philox_words_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, philox_keys(seed), tid, e0, n, out);
    ZO2_HIP_LAUNCH_CHECK();
    return ZO2_OK;
}
zo2_status gaussian(uint64_t seed, uint32_t tid, uint64_t e0, uint64_t n, float* out, hipStream_t st) {
    if (n == 0) return ZO2_OK;
    ZO2_OP_CHECK(out != nullptr, ZO2_EINVAL, "gaussian: out is NULL");
    ZO2_OP_CHECK(n < (1ull << 39), ZO2_EINVAL, "gaussian: n too large");
    hipLaunchKernelGGL(gaussian_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, philox_keys(seed), tid, e0, n, out);
    ZO2_HIP_LAUNCH_CHECK();
    return ZO2_OK;
}

// ------------------------------------------------------------------ pack / unpack
template <typename S, typename D>
__global__ __launch_bounds__(256) void convert_kernel(const S* __restrict__ src, D* __restrict__ dst, uint64_t n,
                                                      float mul, int vec_ok) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    if (vec_ok) {
        const uint64_t groups = n / 8;
        for (uint64_t gi = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; gi < groups; gi += stride) {
            const Vec<S, 8> s = load_vec<S, 8>(src + gi * 8);
            Vec<D, 8> d;
#pragma unroll
            for (int j = 0; j < 8; ++j) d.v[j] = Fmt<D>::store(Fmt<S>::load(s.v[j]) * mul);
            store_vec<D, 8>(dst + gi * 8, d);
        }
        for (uint64_t i = groups * 8 + (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
            dst[i] = Fmt<D>::store(Fmt<S>::load(src[i]) * mul);
    } else {
        for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
            dst[i] = Fmt<D>::store(Fmt<S>::load(src[i]) * mul);
    }
}

zo2_status convert(const void* src, int sdt, float sscale, void* dst, int ddt, float dscale, uint64_t n, hipStream_t st) {
    if (n == 0) return ZO2_OK;
    ZO2_OP_CHECK(src && dst, ZO2_EINVAL, "convert: NULL buffer");
    ZO2_OP_CHECK(sscale > 0.f && dscale > 0.f, ZO2_EINVAL, "convert: scales must be positive");
    const float mul = dscale / sscale;
    const uint64_t want = (n / 8 + 255) / 256 + 1;
    const unsigned grid = (unsigned)(want > 65536 ? 65536 : want);
    ZO2_DISPATCH_WIRE(sdt, S, {
        ZO2_DISPATCH_WIRE(ddt, D, {
            const int vec_ok = ((uintptr_t)src % (sizeof(S) * 8) == 0) && ((uintptr_t)dst % (sizeof(D) * 8) == 0);
            hipLaunchKernelGGL((convert_kernel<S, D>), dim3(grid), dim3(256), 0, st, (const S*)src, (D*)dst, n, mul, vec_ok);
        });
    });
    ZO2_HIP_LAUNCH_CHECK();
    return ZO2_OK;
}

// ------------------------------------------------------------------ LayerNorm
// One 256-thread workgroup per row.  Rows of up to 12288 elements are read once and held in
// registers for the mean, the centred variance and the output; longer rows are re-read from cache.
template <typename C, bool CACHED>
__global__ __launch_bounds__(256) void layernorm_kernel(const float* __restrict__ x, const C* __restrict__ w, const C* __restrict__ b,
                                                        const C* __restrict__ w2, const C* __restrict__ b2, C* __restrict__ y,
                                                        int rows_first, int d, float eps) {
    constexpr int kMaxVec = 12;                     // float4 per lane held in registers
    __shared__ float sh[4];
    const int r = blockIdx.x;
    const float4* xr = reinterpret_cast<const float4*>(x + (size_t)r * d);
    const C* ww = r < rows_first ? w : w2;
    const C* bb = r < rows_first ? b : b2;
    const int nv = d >> 2;
    float4 v[kMaxVec];
    float s = 0.f;
    if (CACHED) {
#pragma unroll
        for (int k = 0; k < kMaxVec; ++k) {
            const int i = threadIdx.x + 256 * k;
            v[k] = i < nv ? xr[i] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int k = 0; k < kMaxVec; ++k) s += (v[k].x + v[k].y) + (v[k].z + v[k].w);
    } else {
        for (int i = threadIdx.x; i < nv; i += 256) {
            const float4 t = xr[i];
            s += (t.x + t.y) + (t.z + t.w);
        }
    }
    const float mean = block_sum(s, sh) / (float)d;
    float q = 0.f;
    if (CACHED) {
#pragma unroll
        for (int k = 0; k < kMaxVec; ++k) {
            if (threadIdx.x + 256 * k < nv) {
                const float a0 = v[k].x - mean, a1 = v[k].y - mean, a2 = v[k].z - mean, a3 = v[k].w - mean;
                q += (a0 * a0 + a1 * a1) + (a2 * a2 + a3 * a3);
            }
        }
    } else {
        for (int i = threadIdx.x; i < nv; i += 256) {
            const float4 t = xr[i];
            const float a0 = t.x - mean, a1 = t.y - mean, a2 = t.z - mean, a3 = t.w - mean;
            q += (a0 * a0 + a1 * a1) + (a2 * a2 + a3 * a3);
        }
    }
    const float var = block_sum(q, sh) / (float)d;
    const float rstd = 1.0f / sqrtf(var + eps);
    C* yr = y + (size_t)r * d;
    auto emit = [&](int i, const float4& t) {
        const Vec<C, 4> wv = load_vec<C, 4>(ww + 4 * i), bv = load_vec<C, 4>(bb + 4 * i);
        Vec<C, 4> o;
        o.v[0] = Fmt<C>::store((t.x - mean) * rstd * Fmt<C>::load(wv.v[0]) + Fmt<C>::load(bv.v[0]));
        o.v[1] = Fmt<C>::store((t.y - mean) * rstd * Fmt<C>::load(wv.v[1]) + Fmt<C>::load(bv.v[1]));
        o.v[2] = Fmt<C>::store((t.z - mean) * rstd * Fmt<C>::load(wv.v[2]) + Fmt<C>::load(bv.v[2]));
        o.v[3] = Fmt<C>::store((t.w - mean) * rstd * Fmt<C>::load(wv.v[3]) + Fmt<C>::load(bv.v[3]));
        store_vec<C, 4>(yr + 4 * i, o);
    };
    if (CACHED) {
#pragma unroll
        for (int k = 0; k < kMaxVec; ++k) {
            const int i = threadIdx.x + 256 * k;
            if (i < nv) emit(i, v[k]);
        }
    } else {
        for (int i = threadIdx.x; i < nv; i += 256) emit(i, xr[i]);
    }
}

// One wavefront per row (rows of up to 4 * 64 * KV elements): the row lives in the wave's registers and
// both reductions are cross-lane only, so the four waves of a workgroup never wait for each other.
template <typename C, int KV>
__global__ __launch_bounds__(256) void layernorm_wave_kernel(const float* __restrict__ x, const C* __restrict__ w, const C* __restrict__ b,
                                                             const C* __restrict__ w2, const C* __restrict__ b2, C* __restrict__ y,
                                                             int rows, int rows_first, int d, float eps) {
    const int lane = threadIdx.x & 63;
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= rows) return;
    const float4* xr = reinterpret_cast<const float4*>(x + (size_t)r * d);
    const C* ww = r < rows_first ? w : w2;
    const C* bb = r < rows_first ? b : b2;
    const int nv = d >> 2;
    float4 v[KV];
#pragma unroll
    for (int k = 0; k < KV; ++k) {
        const int i = lane + 64 * k;
        v[k] = i < nv ? xr[i] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < KV; ++k) s += (v[k].x + v[k].y) + (v[k].z + v[k].w);
    const float mean = wave_sum(s) / (float)d;
    float q = 0.f;
#pragma unroll
    for (int k = 0; k < KV; ++k) {
        if (lane + 64 * k < nv) {
            const float a0 = v[k].x - mean, a1 = v[k].y - mean, a2 = v[k].z - mean, a3 = v[k].w - mean;
            q += (a0 * a0 + a1 * a1) + (a2 * a2 + a3 * a3);
        }
    }
    const float var = wave_sum(q) / (float)d;
    const float rstd = 1.0f / sqrtf(var + eps);
    C* yr = y + (size_t)r * d;
#pragma unroll
    for (int k = 0; k < KV; ++k) {
        const int i = lane + 64 * k;
        if (i < nv) {
            const Vec<C, 4> wv = load_vec<C, 4>(ww + 4 * i), bv = load_vec<C, 4>(bb + 4 * i);
            Vec<C, 4> o;
            o.v[0] = Fmt<C>::store((v[k].x - mean) * rstd * Fmt<C>::load(wv.v[0]) + Fmt<C>::load(bv.v[0]));
            o.v[1] = Fmt<C>::store((v[k].y - mean) * rstd * Fmt<C>::load(wv.v[1]) + Fmt<C>::load(bv.v[1]));
            o.v[2] = Fmt<C>::store((v[k].z - mean) * rstd * Fmt<C>::load(wv.v[2]) + Fmt<C>::load(bv.v[2]));
            o.v[3] = Fmt<C>::store((v[k].w - mean) * rstd * Fmt<C>::load(wv.v[3]) + Fmt<C>::load(bv.v[3]));
            store_vec<C, 4>(yr + 4 * i, o);
        }
    }
}

// The same with 8 consecutive elements per lane and piece (two adjacent 16-byte loads, one 16-byte store of 16-bit
// results): for rows whose length is a multiple of 8.  WAVES rows per workgroup.  Rows come in runs of rows_first, each with gain
// and offset of its own (a stream of a direction), w_step and b_step elements on from the run's before; the last run has the rest.
template <typename C, int KP, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void layernorm_wave8_kernel(const float* __restrict__ x, const C* __restrict__ w, const C* __restrict__ b,
                                                                     int64_t w_step, int64_t b_step, int last_run, C* __restrict__ y,
                                                                     int rows, int rows_first, int d, float eps) {
    const int lane = threadIdx.x & 63;
    const int r = blockIdx.x * WAVES + (threadIdx.x >> 6);
    if (r >= rows) return;
    const float4* xr = reinterpret_cast<const float4*>(x + (size_t)r * d);
    const int run = min(r / rows_first, last_run);
    const C* ww = w + run * w_step;
    const C* bb = b + run * b_step;
    const int n8 = d >> 3;
    float4 v[KP][2];
#pragma unroll
    for (int k = 0; k < KP; ++k) {
        const int i = lane + 64 * k;
        if (i < n8) { v[k][0] = xr[2 * i]; v[k][1] = xr[2 * i + 1]; }
        else v[k][0] = v[k][1] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < KP; ++k)
#pragma unroll
        for (int h = 0; h < 2; ++h) s += (v[k][h].x + v[k][h].y) + (v[k][h].z + v[k][h].w);
    const float mean = wave_sum(s) / (float)d;
    float q = 0.f;
#pragma unroll
    for (int k = 0; k < KP; ++k) {
        if (lane + 64 * k < n8) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float a0 = v[k][h].x - mean, a1 = v[k][h].y - mean, a2 = v[k][h].z - mean, a3 = v[k][h].w - mean;
                q += (a0 * a0 + a1 * a1) + (a2 * a2 + a3 * a3);
            }
        }
    }
    const float var = wave_sum(q) / (float)d;
    const float rstd = 1.0f / sqrtf(var + eps);
    C* yr = y + (size_t)r * d;
#pragma unroll
    for (int k = 0; k < KP; ++k) {
        const int i = lane + 64 * k;
        if (i < n8) {
            const Vec<C, 8> wv = load_vec<C, 8>(ww + 8 * i), bv = load_vec<C, 8>(bb + 8 * i);
            Vec<C, 8> o;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                o.v[4 * h + 0] = Fmt<C>::store((v[k][h].x - mean) * rstd * Fmt<C>::load(wv.v[4 * h + 0]) + Fmt<C>::load(bv.v[4 * h + 0]));
                o.v[4 * h + 1] = Fmt<C>::store((v[k][h].y - mean) * rstd * Fmt<C>::load(wv.v[4 * h + 1]) + Fmt<C>::load(bv.v[4 * h + 1]));
                o.v[4 * h + 2] = Fmt<C>::store((v[k][h].z - mean) * rstd * Fmt<C>::load(wv.v[4 * h + 2]) + Fmt<C>::load(bv.v[4 * h + 2]));
                o.v[4 * h + 3] = Fmt<C>::store((v[k][h].w - mean) * rstd * Fmt<C>::load(wv.v[4 * h + 3]) + Fmt<C>::load(bv.v[4 * h + 3]));
            }
            store_vec<C, 8>(yr + 8 * i, o);
        }
    }
}

static constexpr int kLnWaves = 1;      // rows per workgroup of the kernel above (1, 2, 4, 8 measured inside the step: within 2 %, 1 ahead)

static constexpr int kLnWaveMax = 5120; // longest row of the wavefront-per-row kernels
// does a row go to the kernel that moves 8 elements at a time?
static bool layernorm_by8(int dtype, int d, const void* y, const void* w, const void* b, const void* w2, const void* b2) {
    return zo2_dtype_size(dtype) == 2 && d % 8 == 0 && d <= kLnWaveMax &&
           (((uintptr_t)y | (uintptr_t)w | (uintptr_t)b | (uintptr_t)w2 | (uintptr_t)b2) % 16) == 0;
}

template <typename C>
static void launch_ln8(const float* x, const void* w, const void* b, int64_t w_bytes, int64_t b_bytes, int last_run, void* y, int rows, int rows_first, int d, float eps, hipStream_t st) {
    // pieces of 512 elements per row: instances for rows of up to 2048 and 5120 elements
    const dim3 grid((rows + kLnWaves - 1) / kLnWaves), block(64 * kLnWaves);
    const int64_t ws = w_bytes / (int64_t)sizeof(C), bs = b_bytes / (int64_t)sizeof(C);
    if (d <= 4 * 512) hipLaunchKernelGGL((layernorm_wave8_kernel<C, 4, kLnWaves>), grid, block, 0, st, x, (const C*)w, (const C*)b, ws, bs, last_run, (C*)y, rows, rows_first, d, eps);
    else hipLaunchKernelGGL((layernorm_wave8_kernel<C, 10, kLnWaves>), grid, block, 0, st, x, (const C*)w, (const C*)b, ws, bs, last_run, (C*)y, rows, rows_first, d, eps);
}

bool layernorm_sets_applicable(int dtype, int d, const void* y, const void* w, const void* b, int64_t step_bytes) {
    return layernorm_by8(dtype, d, y, w, b, (const void*)(uintptr_t)step_bytes, nullptr);
}
zo2_status layernorm_sets(int dtype, const float* x, const void* w, const void* b, int64_t step_bytes, void* y, int rows, int rows_per_set, int d, float eps,
                          hipStream_t st) {
    ZO2_OP_CHECK(rows > 0 && rows_per_set > 0 && x && w && b && y && ((uintptr_t)x % 16) == 0 && layernorm_sets_applicable(dtype, d, y, w, b, step_bytes), ZO2_EINVAL,
                 "layernorm: rows %d, d %d, or buffers not aligned to 8 elements", rows, d);
    if (dtype == ZO2_BF16) launch_ln8<bf16_t>(x, w, b, step_bytes, step_bytes, (rows - 1) / rows_per_set, y, rows, rows_per_set, d, eps, st);
    else launch_ln8<f16_t>(x, w, b, step_bytes, step_bytes, (rows - 1) / rows_per_set, y, rows, rows_per_set, d, eps, st);
    ZO2_HIP_LAUNCH_CHECK();
    return ZO2_OK;
}

zo2_status layernorm(int dtype, const float* x, const void* w, const void* b, const void* w2, const void* b2, void* y,
                     int rows, int rows_first, int d, float eps, hipStream_t st) {
    if (rows == 0) return ZO2_OK;
    ZO2_OP_CHECK(rows > 0 && d > 0 && d % 4 == 0, ZO2_EINVAL, "layernorm: rows %d, d %d (d must be a multiple of 4)", rows, d);
    ZO2_OP_CHECK(x && w && b && y, ZO2_EINVAL, "layernorm: NULL buffer");
    ZO2_OP_CHECK(rows_first >= rows || (w2 && b2), ZO2_EINVAL, "layernorm: second gain / bias missing");
    {   // rows are moved in groups of 4 elements
        const uintptr_t ca = 4 * (uintptr_t)zo2_dtype_size(dtype);
        ZO2_OP_CHECK(ca != 0 && ((uintptr_t)x % 16) == 0 && ((uintptr_t)y % ca) == 0 && ((uintptr_t)w % ca) == 0 && ((uintptr_t)b % ca) == 0 &&
                     ((uintptr_t)w2 % ca) == 0 && ((uintptr_t)b2 % ca) == 0, ZO2_EINVAL, "layernorm: unknown dtype, or buffers not aligned to 4 elements");
    }
    const bool by8 = layernorm_by8(dtype, d, y, w, b, w2, b2);
    ZO2_DISPATCH_COMPUTE(dtype, C, {
        // rows of up to 5120 elements by one wavefront each; longer rows take too many
        // registers for one wavefront (measured at 8192 rows: 5120 46 us against 55 with the kernels below, 7168 76
        // against 69, 12288 145 against 115) and stay with the workgroup-per-row kernel
        if (by8) {
            const bool first = rows_first > 0, one = !first || rows_first >= rows;      // (without rows of the first stream all are the second's)
            const void *w0 = first ? w : w2, *b0 = first ? b : b2;
            launch_ln8<C>(x, w0, b0, one ? 0 : (intptr_t)w2 - (intptr_t)w0, one ? 0 : (intptr_t)b2 - (intptr_t)b0, one ? 0 : 1, y, rows, one ? rows : rows_first, d, eps, st);
        } else if (d <= 8 * 64 * 4)
            hipLaunchKernelGGL((layernorm_wave_kernel<C, 8>), dim3((rows + 3) / 4), dim3(256), 0, st, x, (const C*)w, (const C*)b,
                               (const C*)w2, (const C*)b2, (C*)y, rows, rows_first, d, eps);
        else if (d <= kLnWaveMax)
            hipLaunchKernelGGL((layernorm_wave_kernel<C, 20>), dim3((rows + 3) / 4), dim3(256), 0, st, x, (const C*)w, (const C*)b,
                               (const C*)w2, (const C*)b2, (C*)y, rows, rows_first, d, eps);
        else if (d <= 12 * 256 * 4)
            hipLaunchKernelGGL((layernorm_kernel<C, true>), dim3(rows), dim3(256), 0, st, x, (const C*)w, (const C*)b,
                               (const C*)w2, (const C*)b2, (C*)y, rows_first, d, eps);
        else
            hipLaunchKernelGGL((layernorm_kernel<C, false>), dim3(rows), dim3(256), 0, st, x, (const C*)w, (const C*)b,
                               (const C*)w2, (const C*)b2, (C*)y, rows_first, d, eps);
    });
    ZO2_HIP_LAUNCH_CHECK();
    return ZO2_OK;
}

// One workgroup per row, a thread for every four columns (up to 1024 threads, two pieces each beyond 4096 columns), the row in
// registers.  Steps of few tokens are a chain of launches of 4 - 5 us each, most of it start and end; what is left here is the
// latency of the pieces' loads, sixteen in flight per thread.  2 x 16 rows, d 2048, 32 slices: 6.6 us instead of 5.3 for the sum
// and 4.5 for the LayerNorm; 2 x 64 rows, d 768, float32, 6 pieces: 3.9 instead of 4.0 and 4.5.
// Whether a projection is cut along k, and whether a sweep sits between its sum and this LayerNorm, must not show in the results:
// mean and variance are added up as layernorm() does for the same row.  Every thread leaves the sum of its four columns in LDS, and
// every wavefront adds those in the order of that kernel's lanes.
enum { kLnWave = 0, kLnWave8 = 1, kLnBlock = 2 };      // layernorm_wave_kernel, layernorm_wave8_kernel, layernorm_kernel
template <int ORDER>
__device__ __forceinline__ float layernorm_total(const float* part, int nv) {
    constexpr int kGroups = ORDER == kLnBlock ? 4 : 1;
    float tot = 0.f;
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
        float s = 0.f;
        if (ORDER == kLnWave8) {
#pragma unroll 4
            for (int i = 2 * (threadIdx.x & 63); i < nv; i += 128) {
                s += part[i];
                s += part[i + 1];
            }
        } else {
#pragma unroll 4
            for (int i = (threadIdx.x & 63) + 64 * g; i < nv; i += 64 * kGroups) s += part[i];
        }
        s = wave_sum(s);
        tot = g == 0 ? s : tot + s;
    }
    return tot;
}

template <typename C, int V, int ORDER>      // V: 16-byte pieces per thread
__global__ __launch_bounds__(1024) void reduce_layernorm_kernel(RowSum a, float* __restrict__ h, const C* __restrict__ w, const C* __restrict__ b,
                                                               const C* __restrict__ w2, const C* __restrict__ b2, C* __restrict__ y,
                                                               int rows_first, int d, float eps) {
    __shared__ float sh_s[1024 * V], sh_q[1024 * V];
    const int r = blockIdx.x, nv = d >> 2, nt = blockDim.x;
    const bool second = r >= rows_first;
    const float* src = a.part + (second ? a.stream_stride + (size_t)(r - rows_first) * d : (size_t)r * d);
    const C* bias = reinterpret_cast<const C*>(second ? a.bias2 : a.bias);
    const C* ww = second ? w2 : w;
    const C* bb = second ? b2 : b;
    float4* hr = reinterpret_cast<float4*>(h + (size_t)r * d);
    float4 v[V];
#pragma unroll
    for (int k = 0; k < V; ++k) {
        const int i = threadIdx.x + nt * k;
        v[k] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (i < nv) {
            const float4 res = hr[i];
            const Vec<C, 4> bv = load_vec<C, 4>(bias + 4 * i);
            for (int p0 = 0; p0 < a.pieces; p0 += 16) {
                float4 t[16];
#pragma unroll
                for (int p = 0; p < 16; ++p)
                    if (p0 + p < a.pieces) t[p] = *reinterpret_cast<const float4*>(src + (size_t)(p0 + p) * a.piece_stride + 4 * i);
#pragma unroll
                for (int p = 0; p < 16; ++p)
                    if (p0 + p < a.pieces) { v[k].x += t[p].x; v[k].y += t[p].y; v[k].z += t[p].z; v[k].w += t[p].w; }
            }
            v[k].x = (v[k].x + Fmt<C>::load(bv.v[0])) + res.x;
            v[k].y = (v[k].y + Fmt<C>::load(bv.v[1])) + res.y;
            v[k].z = (v[k].z + Fmt<C>::load(bv.v[2])) + res.z;
            v[k].w = (v[k].w + Fmt<C>::load(bv.v[3])) + res.w;
            hr[i] = v[k];
            sh_s[i] = (v[k].x + v[k].y) + (v[k].z + v[k].w);
        }
    }
    __syncthreads();
    const float mean = layernorm_total<ORDER>(sh_s, nv) / (float)d;
#pragma unroll
    for (int k = 0; k < V; ++k) {
        const int i = threadIdx.x + nt * k;
        if (i < nv) {
            const float a0 = v[k].x - mean, a1 = v[k].y - mean, a2 = v[k].z - mean, a3 = v[k].w - mean;
            sh_q[i] = (a0 * a0 + a1 * a1) + (a2 * a2 + a3 * a3);
        }
    }
    __syncthreads();
    const float rstd = 1.0f / sqrtf(layernorm_total<ORDER>(sh_q, nv) / (float)d + eps);
    C* yr = y + (size_t)r * d;
#pragma unroll
    for (int k = 0; k < V; ++k) {
        const int i = threadIdx.x + nt * k;
        if (i >= nv) continue;
        const Vec<C, 4> wv = load_vec<C, 4>(ww + 4 * i), bv = load_vec<C, 4>(bb + 4 * i);
        Vec<C, 4> o;
        o.v[0] = Fmt<C>::store((v[k].x - mean) * rstd * Fmt<C>::load(wv.v[0]) + Fmt<C>::load(bv.v[0]));
        o.v[1] = Fmt<C>::store((v[k].y - mean) * rstd * Fmt<C>::load(wv.v[1]) + Fmt<C>::load(bv.v[1]));
        o.v[2] = Fmt<C>::store((v[k].z - mean) * rstd * Fmt<C>::load(wv.v[2]) + Fmt<C>::load(bv.v[2]));
        o.v[3] = Fmt<C>::store((v[k].w - mean) * rstd * Fmt<C>::load(wv.v[3]) + Fmt<C>::load(bv.v[3]));
        store_vec<C, 4>(yr + 4 * i, o);
    }
}

bool reduce_layernorm_applicable(int d) { return d > 0 && d % 4 == 0 && d <= 8192; }

zo2_status reduce_layernorm(int dtype, const RowSum& a, float* h, const void* w, const void* b, const void* w2, const void* b2, void* y, int rows,
                            int rows_first, int d, float eps, hipStream_t st) {
    if (rows == 0) return ZO2_OK;
    ZO2_OP_CHECK(rows > 0 && reduce_layernorm_applicable(d) && a.pieces >= 1, ZO2_EINVAL, "reduce_layernorm: rows %d, d %d, %d pieces", rows, d, a.pieces);
    ZO2_OP_CHECK(a.part && a.bias && h && w && b && y && (rows_first >= rows || (a.bias2 && w2 && b2)), ZO2_EINVAL, "reduce_layernorm: NULL buffer");
    const uintptr_t ca = 4 * (uintptr_t)zo2_dtype_size(dtype);
    ZO2_OP_CHECK(ca != 0 && (((uintptr_t)a.part | (uintptr_t)h) & 15) == 0 && a.piece_stride % 4 == 0 && a.stream_stride % 4 == 0 &&
                 (((uintptr_t)w | (uintptr_t)b | (uintptr_t)w2 | (uintptr_t)b2 | (uintptr_t)y | (uintptr_t)a.bias | (uintptr_t)a.bias2) & (ca - 1)) == 0,
                 ZO2_EINVAL, "reduce_layernorm: unknown dtype, or buffers not aligned to 4 elements");
    const bool by8 = layernorm_by8(dtype, d, y, w, b, w2, b2);
#define ZO2_RLN(V, ORDER)                                                                                                           \
    hipLaunchKernelGGL((reduce_layernorm_kernel<C, V, ORDER>), dim3(rows), dim3(std::min(1024, (d / 4 + 63) / 64 * 64)), 0, st, a, h, (const C*)w, (const C*)b, (const C*)w2, \
                       (const C*)b2, (C*)y, rows_first, d, eps)
    ZO2_DISPATCH_COMPUTE(dtype, C, {
        constexpr int kBy8 = sizeof(C) == 2 ? kLnWave8 : kLnWave;
        if (by8 && d <= 4096) ZO2_RLN(1, kBy8);
        else if (by8) ZO2_RLN(2, kBy8);
        else if (d <= 4096) ZO2_RLN(1, kLnWave);
        else if (d <= kLnWaveMax) ZO2_RLN(2, kLnWave);
        else ZO2_RLN(2, kLnBlock);
    });
#undef ZO2_RLN
    ZO2_HIP_LAUNCH_CHECK();
    return ZO2_OK;
}

// ------------------------------------------------------------------ embedding gather (Alg. 2, DualForward(Embedding))
// h+[t] = W+tok[id_t] + W+pos[t + off], h-[t] likewise, with the pending update and the
// perturbation evaluated only for the rows the batch touches.  The tables themselves are
// brought up to date by K1 afterwards; both evaluate the same per-element expression.
// UPDATES: 0, 1, or 2 for any number of them.  (One alone is not a loop: where float16 results are made, whether the compiler folds a rounding
// into the multiply-add in front of it depends on such things, and a run is to keep its bits.)
template <typename W, typename C, int UPDATES>
__global__ __launch_bounds__(256) void embed_kernel(EmbedArgs a) {
    const int dv = a.d >> 2;
    const int64_t gi = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gi >= (int64_t)a.T * dv) return;
    const int t = (int)(gi / dv), j = (int)(gi % dv) * 4;
    const int id = a.tokens[t];
    const int pos = t % a.seq + a.pos_offset;
    constexpr bool kScaled = (Fmt<W>::kBytes == 1);
    float hp[4] = {0.f, 0.f, 0.f, 0.f}, hm[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int which = 0; which < 2; ++which) {
        const W* table = reinterpret_cast<const W*>(which == 0 ? a.tok_emb : a.pos_emb);
        const uint64_t e = (uint64_t)(which == 0 ? id : pos) * a.d + j;
        const float scale = which == 0 ? a.scale_tok : a.scale_pos, inv_scale = 1.0f / scale;
        const Vec<W, 4> tv = load_vec<W, 4>(table + e);
        float th[4], z[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            th[i] = Fmt<W>::load(tv.v[i]);
            if (kScaled) th[i] *= inv_scale;
        }
        auto update = [&](int n) {
            const float c = a.c_ptr[n];
            gaussian4(a.k_upd[n], (uint32_t)which, e, z);
            uint32_t rw[4] = {0u, 0u, 0u, 0u};
            const bool sr = Fmt<W>::kBytes < 4 && a.stochastic != 0;
            if (sr) rounding_words(a.k_upd[n], (uint32_t)which, e >> 3, rw);
            // this group of 4 is the lower or the upper half of its Philox call: rounding words 0, 1 or 2, 3
            const uint32_t r2[2] = {(e & 4) ? rw[2] : rw[0], (e & 4) ? rw[3] : rw[1]};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float u = __builtin_fmaf(-c, z[i], th[i]);
                const float us = kScaled ? u * scale : u;
                const uint32_t r16 = (r2[i >> 1] >> (16 * (i & 1))) & 0xffffu;
                th[i] = Fmt<W>::load(sr ? store_stochastic<W>(us, r16) : Fmt<W>::store(us));
                if (kScaled) th[i] *= inv_scale;
            }
        };
        if constexpr (UPDATES == 1) update(0);
        if constexpr (UPDATES == 2) {
#pragma unroll 1
            for (int n = 0; n < a.n_upd; ++n) update(n);
        }
        if (a.single) {
#pragma unroll
            for (int i = 0; i < 4; ++i) hp[i] += Fmt<C>::load(Fmt<C>::store(th[i]));
            continue;
        }
        gaussian4(a.k_cur, (uint32_t)which, e, z);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            hp[i] += Fmt<C>::load(Fmt<C>::store(__builtin_fmaf(a.eps, z[i], th[i])));
            hm[i] += Fmt<C>::load(Fmt<C>::store(__builtin_fmaf(-a.eps, z[i], th[i])));
        }
    }
    float* op = a.h + (size_t)t * a.d + j;
    *reinterpret_cast<float4*>(op) = make_float4(hp[0], hp[1], hp[2], hp[3]);
    if (a.single) return;
    float* om = a.h + ((size_t)a.T + t) * a.d + j;
    *reinterpret_cast<float4*>(om) = make_float4(hm[0], hm[1], hm[2], hm[3]);
}

zo2_status embed_gather(const EmbedArgs& a, int wire_dtype, int compute_dtype, hipStream_t st) {
    if (a.T == 0) return ZO2_OK;
    ZO2_OP_CHECK(a.n_upd >= 0 && a.n_upd <= EmbedArgs::kMaxUpdates, ZO2_EINVAL, "embed: %d updates", a.n_upd);
    ZO2_OP_CHECK(a.d % 4 == 0, ZO2_EINVAL, "embed: d %d not a multiple of 4", a.d);
    const int64_t n = (int64_t)a.T * (a.d / 4);
    const dim3 grid((unsigned)((n + 255) / 256)), block(256);
    ZO2_DISPATCH_WIRE(wire_dtype, W, {
        ZO2_DISPATCH_COMPUTE(compute_dtype, C, {
            if constexpr (__is_same(C, bf16_t) && !__is_same(W, f16_t)) {      // the formats of a round in one sweep (k1_round_applicable)
                if (a.n_upd > 1) {
                    hipLaunchKernelGGL((embed_kernel<W, C, 2>), grid, block, 0, st, a);
                    ZO2_HIP_LAUNCH_CHECK();
                    return ZO2_OK;
                }
            }
            ZO2_OP_CHECK(a.n_upd <= 1, ZO2_EINVAL, "embed: %d updates in these formats", a.n_upd);
            if (a.n_upd) hipLaunchKernelGGL((embed_kernel<W, C, 1>), grid, block, 0, st, a);
            else hipLaunchKernelGGL((embed_kernel<W, C, 0>), grid, block, 0, st, a);
        });
    });
    ZO2_HIP_LAUNCH_CHECK();
    return ZO2_OK;
}

// ------------------------------------------------------------------ cross-entropy per row
// NT threads per row: 1024 (a row of 50272 logits is a dozen 16-byte loads each: a launch of 64 rows takes 12.7 us against 25 with 256
// threads), 256 where the order of the sums is kept
template <int NT>
__global__ __launch_bounds__(NT) void ce_rows_kernel(const float* __restrict__ logits, int64_t ld, const int32_t* __restrict__ labels,
                                                      int row0, int label_period, int vocab, float* __restrict__ row_loss) {
    __shared__ float shf[NT / 64];
    __shared__ double shd[NT / 64];
    // logits row blockIdx.x is row (row0 + blockIdx.x) of the stacked [+ rows; - rows] batch
    const int r = row0 + blockIdx.x;
    const int lab = labels[r % label_period];
    if (lab < 0) {                       // ignored position (uniform per workgroup)
        if (threadIdx.x == 0) row_loss[r] = 0.f;
        return;
    }
    const float* lr = logits + (size_t)blockIdx.x * ld;
    // one pass: running maximum m and sum s of exp(x - m) per lane, rescaled when m grows; while m is -inf (logits of -inf, which
    // add nothing, or NaN, which is to stay) the exponents are taken against 0
    float m = -INFINITY, s = 0.f;
    auto base = [&]() { return m == -INFINITY ? 0.f : m; };
    const bool vec = ((ld & 3) == 0) && (((uintptr_t)logits & 15) == 0);
    const int nv = vec ? (vocab >> 2) : 0;
    for (int i = threadIdx.x; i < nv; i += NT) {
        const float4 x = reinterpret_cast<const float4*>(lr)[i];
        const float mx = fmaxf(fmaxf(x.x, x.y), fmaxf(x.z, x.w));
        if (mx > m) { s *= expf(m - mx); m = mx; }
        s += (expf(x.x - base()) + expf(x.y - base())) + (expf(x.z - base()) + expf(x.w - base()));
    }
    for (int i = nv * 4 + threadIdx.x; i < vocab; i += NT) {
        const float x = lr[i];
        if (x > m) { s *= expf(m - x); m = x; }
        s += expf(x - base());
    }
    const float mall = block_max(m, shf);
    const double tot = block_sum((double)(m == -INFINITY ? s : s * expf(m - mall)), shd);
    if (threadIdx.x == 0) row_loss[r] = (float)(log(tot) + (double)mall - (double)lr[lab]);
}

zo2_status cross_entropy_rows(const float* logits, int64_t ld, const int32_t* labels, int rows, int row0, int label_period,
                              int vocab, float* row_loss, hipStream_t st, bool keep_order) {
    if (rows == 0) return ZO2_OK;
    ZO2_OP_CHECK(logits && labels && row_loss, ZO2_EINVAL, "cross_entropy: NULL buffer");
    ZO2_OP_CHECK(vocab > 0 && ld >= vocab && label_period > 0 && row0 >= 0, ZO2_EINVAL, "cross_entropy: bad shape");
    if (keep_order) hipLaunchKernelGGL(ce_rows_kernel<256>, dim3(rows), dim3(256), 0, st, logits, ld, labels, row0, label_period, vocab, row_loss);
    else hipLaunchKernelGGL(ce_rows_kernel<1024>, dim3(rows), dim3(1024), 0, st, logits, ld, labels, row0, label_period, vocab, row_loss);
    ZO2_HIP_LAUNCH_CHECK();
    return ZO2_OK;
}

// ------------------------------------------------------------------ combine the LM-head kernel's cross-entropy partials
// Row r has n_parts pairs (m_i, s_i), span-major ([i * part_ld + r]), with s_i = sum over a 64-column span of
// exp(y - m_i); then logsumexp = M + log(sum_i s_i exp(m_i - M)), M = max_i m_i.
// The maximum of spans whose logits are all NaN is -inf (fmaxf passes them over), like that of spans that add nothing: exponents are taken against 0
// then, so that what is added is the spans' sums times exp(-inf) = 0, which is 0, or the NaN that is to reach the row's loss.
__device__ __forceinline__ float ce_base(float m) { return m == -INFINITY ? 0.f : m; }
// Eight rows per workgroup and 128 lanes to a row, so that a row's 788 spans of a 50272-word vocabulary are seven loads a lane, all under way
// at once, and few rows still are several workgroups: bound by the latency of one such load and of the launch.  (32 rows per workgroup walked
// 25 spans a lane, twice: 15, 17, 22 and 23 us at 32, 370, 1026 and 8192 rows; this 7, 8, 9.5 and 24.6.)  The four workgroups that share a 128-byte line of
// partials have indexes 8 apart, which the hardware deals to one XCD and so to one L2.
__global__ __launch_bounds__(1024) void ce_combine_kernel(const float* __restrict__ part_max, const float* __restrict__ part_sum,
                                                          const float* __restrict__ label_logit, const int32_t* __restrict__ labels,
                                                          int rows, int n_parts, int64_t part_ld, int row0, int label_period,
                                                          float* __restrict__ row_loss) {
    constexpr int kRows = 8, kLanes = 128, kLoads = 8;
    __shared__ float sh_m[16][kRows];
    __shared__ double sh_s[16][kRows];
    const int lr = threadIdx.x & (kRows - 1), grp = threadIdx.x / kRows, wave = threadIdx.x >> 6;
    const int line = (blockIdx.x >> 5) * 8 + (blockIdx.x & 7);
    const int first = (line * 4 + ((blockIdx.x >> 3) & 3)) * kRows, r = first + lr;
    if (first >= rows) return;
    const int rc = r < rows ? r : rows - 1;
    const float* pm = part_max + rc;
    const float* ps = part_sum + rc;
    float m = -INFINITY;
    double s = 0.0;
    for (int i0 = grp; i0 < n_parts; i0 += kLanes * kLoads) {
        float mi[kLoads], si[kLoads];
#pragma unroll
        for (int j = 0; j < kLoads; ++j) {
            const int i = i0 + kLanes * j;
            mi[j] = i < n_parts ? pm[(size_t)i * part_ld] : -INFINITY;
            si[j] = i < n_parts ? ps[(size_t)i * part_ld] : 0.f;
        }
        float mx = m;
#pragma unroll
        for (int j = 0; j < kLoads; ++j) mx = fmaxf(mx, mi[j]);
        if (mx > m) {
            s *= (double)expf(m - mx);
            m = mx;
        }
        const float base = ce_base(m);
#pragma unroll
        for (int j = 0; j < kLoads; ++j) s += (double)(si[j] * expf(mi[j] - base));       // a span past the last column has sum 0 and exp(-inf) = 0
    }
    // the row's lanes of this wavefront (8 apart), then the wavefronts
    auto merge = [](float& m0, double& s0, float m1, double s1) {
        const float mm = fmaxf(m0, m1);
        const double a = m0 == -INFINITY ? s0 : s0 * (double)expf(m0 - mm), b = m1 == -INFINITY ? s1 : s1 * (double)expf(m1 - mm);
        m0 = mm;
        s0 = a + b;
    };
#pragma unroll
    for (int d = kRows; d < 64; d <<= 1) merge(m, s, __shfl_xor(m, d, 64), __shfl_xor(s, d, 64));
    if ((threadIdx.x & 63) < kRows) {
        sh_m[wave][lr] = m;
        sh_s[wave][lr] = s;
    }
    __syncthreads();
    if (threadIdx.x >= kRows || r >= rows) return;
    const int lab = labels[(row0 + r) % label_period];
    if (lab < 0) {
        row_loss[row0 + r] = 0.f;
        return;
    }
    float mm = -INFINITY;
#pragma unroll
    for (int k = 0; k < 16; ++k) mm = fmaxf(mm, sh_m[k][lr]);
    double ss = 0.0;
    const float base = ce_base(mm);
#pragma unroll
    for (int k = 0; k < 16; ++k) ss += sh_s[k][lr] * (double)expf(sh_m[k][lr] - base);
    row_loss[row0 + r] = (float)(log(ss) + (double)mm - (double)label_logit[r]);
}

// 32 rows per block; kGroups groups of lanes split the spans, so every load is 32 consecutive floats.  Two sweeps (max, then sum) keep the loads
// independent of each other.  Eight groups, a thread walking 99 of the 788 spans of a 50272-word vocabulary, for contexts that keep the order of their
// sums (with eight loads under way: 55 us at 4096 rows instead of 32).  32 groups for more than 8192 rows, where whole 128-byte lines are
// worth more than short walks (beside loss_epilogue_kernel, eight rows a workgroup -> this, us: 8192 rows 33 and 34, 16384 55 -> 50, 32768 110 -> 91).
template <int kGroups>
__global__ __launch_bounds__(32 * kGroups) void ce_combine_rows_kernel(const float* __restrict__ part_max, const float* __restrict__ part_sum,
                                                         const float* __restrict__ label_logit, const int32_t* __restrict__ labels,
                                                         int rows, int n_parts, int64_t part_ld, int row0, int label_period,
                                                         float* __restrict__ row_loss) {
    constexpr int kRows = 32, kUnroll = kGroups == 8 ? 4 : 8;
    __shared__ float sh_m[kGroups][kRows];
    __shared__ double sh_s[kGroups][kRows];
    const int lr = threadIdx.x & (kRows - 1), grp = threadIdx.x / kRows;
    const int r = blockIdx.x * kRows + lr;
    const int rc = r < rows ? r : rows - 1;
    const float* pm = part_max + rc;
    const float* ps = part_sum + rc;
    float m = -INFINITY;
#pragma unroll kUnroll
    for (int i = grp; i < n_parts; i += kGroups) m = fmaxf(m, pm[(size_t)i * part_ld]);
    double s = 0.0;
    const float base = ce_base(m);
#pragma unroll kUnroll
    for (int i = grp; i < n_parts; i += kGroups) {
        const float mi = pm[(size_t)i * part_ld];
        s += (double)(ps[(size_t)i * part_ld] * expf(mi - base));     // a span past the last column has sum 0 and exp(-inf) = 0
    }
    sh_m[grp][lr] = m;
    sh_s[grp][lr] = s;
    __syncthreads();
    if (grp != 0 || r >= rows) return;
    const int lab = labels[(row0 + r) % label_period];
    if (lab < 0) {
        row_loss[row0 + r] = 0.f;
        return;
    }
    float mm = -INFINITY;
#pragma unroll
    for (int k = 0; k < kGroups; ++k) mm = fmaxf(mm, sh_m[k][lr]);
    double ss = 0.0;
    const float base_all = ce_base(mm);
#pragma unroll
    for (int k = 0; k < kGroups; ++k) ss += sh_s[k][lr] * (double)expf(sh_m[k][lr] - base_all);
    row_loss[row0 + r] = (float)(log(ss) + (double)mm - (double)label_logit[r]);
}

zo2_status ce_combine(const float* part_max, const float* part_sum, const float* label_logit, const int32_t* labels, int rows,
                      int n_parts, int64_t part_ld, int row0, int label_period, float* row_loss, hipStream_t st, bool keep_order, int like_rows) {
    if (rows == 0) return ZO2_OK;
    ZO2_OP_CHECK(part_max && part_sum && label_logit && labels && row_loss && n_parts > 0 && label_period > 0 && part_ld >= rows,
                 ZO2_EINVAL, "ce_combine: bad argument");
    const dim3 by32((rows + 31) / 32);
    if (keep_order) hipLaunchKernelGGL(ce_combine_rows_kernel<8>, by32, dim3(256), 0, st, part_max, part_sum, label_logit, labels, rows, n_parts, part_ld, row0, label_period, row_loss);
    else if ((like_rows ? like_rows : rows) > 8192) hipLaunchKernelGGL(ce_combine_rows_kernel<32>, by32, dim3(1024), 0, st, part_max, part_sum, label_logit, labels, rows, n_parts, part_ld, row0, label_period, row_loss);
    else hipLaunchKernelGGL(ce_combine_kernel, dim3((rows + 255) / 256 * 32), dim3(1024), 0, st, part_max, part_sum, label_logit, labels, rows, n_parts, part_ld, row0, label_period, row_loss);
    ZO2_HIP_LAUNCH_CHECK();
    return ZO2_OK;
}

// ------------------------------------------------------------------ scalar epilogue (Eq. 2)
// l+ = mean of row_loss[0..T) over non-ignored labels, l- of row_loss[T..2T);
// g = (l+ - l-) / (2 eps); the pending step c = lr * g stays in device memory.
__global__ __launch_bounds__(256) void loss_epilogue_kernel(const float* __restrict__ row_loss, const int32_t* __restrict__ labels,
                                                            int T, float eps, float lr, int ns, float* __restrict__ result,
                                                            float* __restrict__ c_pending) {
    __shared__ double shd[4];
    double sp = 0.0, sm = 0.0, cnt = 0.0;
    for (int i = threadIdx.x; i < T; i += 256) {
        if (labels[i] >= 0) {
            sp += (double)row_loss[i];
            if (ns == 2) sm += (double)row_loss[T + i];
            cnt += 1.0;
        }
    }
    sp = block_sum(sp, shd);
    sm = block_sum(sm, shd);
    cnt = block_sum(cnt, shd);
    if (threadIdx.x == 0) {
        const float lp = (float)(sp / cnt), lm = ns == 2 ? (float)(sm / cnt) : lp;
        const float g = ns == 2 ? (lp - lm) / (2.0f * eps) : 0.f;
        result[0] = lp;
        result[1] = lm;
        result[2] = g;
        result[3] = (float)cnt;
        if (ns == 2) *c_pending = lr * g;
    }
}

zo2_status loss_epilogue(const float* row_loss, const int32_t* labels, int T, float eps, float lr, int ns, float* result,
                         float* c_pending, hipStream_t st) {
    hipLaunchKernelGGL(loss_epilogue_kernel, dim3(1), dim3(256), 0, st, row_loss, labels, T, eps, lr, ns, result, c_pending);
    ZO2_HIP_LAUNCH_CHECK();
    return ZO2_OK;
}

}  // namespace zo2
