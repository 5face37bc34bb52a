// The projections of few tokens in float32: gemm_skinny.hip's layout - a workgroup owns 128 output features and a slice of k, reads the
// stored weights once for both perturbation streams and forms W+- in registers - with the pending update in the same place: a lane
// reads its theta, writes theta' = theta - c z_prev back and multiplies with theta' +- eps z, each operand as three bfloat16 parts (f32_parts.h).
// The sweep's copies move 16 bytes a parameter and are read again, 8 more; here it is 8 in all.
//
// What bounds it: two draws and the parts of two copies are some 50 vector instructions an element; a slab of 64 rows, 1.5 us of them, 1.4 us of
// MFMAs and as much of LDS reads, takes 4 us on a compute unit.  At d 768 a launch is one or two slabs per workgroup and 9 us of first loads,
// last stores, start and end.  Steps, sweep and float32 GEMMs -> this, us: d 768, 12 blocks, 16 tokens 1162 -> 952, 64 1390 -> 1284, 96 1623 -> 1499;
// d 2048, 6 blocks, 16 2185 -> 1284, 64 2389 -> 1653, 96 2812 -> 2012; d 4096, 2 blocks, 30 3045 -> 1711; d 5120, 2 blocks, 60 4699 -> 3055.  128
// rows (one slab in LDS, its registers full) 1657 -> 1841, 2848 -> 2636, d 5120 5476 -> 5735: the line is drawn at 96.
// (Wavefronts of 32 features and half a slab's k, as in gemm_skinny.hip, read LDS half as often, but their halves have to meet and their
// lanes to store single floats: 1425 us where this takes 1284.)
#include <algorithm>

#include "f32_parts.h"
#include "gemm_skinny.h"

namespace zo2 {

static constexpr int kSfBN = 128, kSfBK = 64;      // weight rows per workgroup, k per slab

// v_mfma_f32_16x16x32_bf16: lane (r, g) = (l & 15, l >> 4) supplies k = 8 g .. + 7 of row r of either operand.  Wavefront w owns features 16 w ..
// + 15 of the workgroup's 128 over the whole slice, so nothing has to meet at the end; the lanes of a row read and write whole lines of theta.
// With the weights as the first operand a lane ends with row r of the activations and features 4 g .. + 3.
// MT: 32 rows of each stream.
__device__ __forceinline__ v4f_t mfma16_bf16(v4u_t w, v4u_t x, v4f_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w), __builtin_bit_cast(bf16x8_t, x), c, 0, 0, 0);
}
template <int MT, bool UPDATE>
__global__ __launch_bounds__(512, 2) void skinny_f32_kernel(const SkinnyArgs a) {
    constexpr int R = 64 * MT, NI = 4 * MT, PLANE = R * 8;     // activation rows of both streams, 16-row tiles, 16-byte chunks of one part of a slab
    extern __shared__ __attribute__((aligned(16))) char smem[];
    v4u_t* Xs = reinterpret_cast<v4u_t*>(smem);                // [2 slabs][3 parts][R rows][8 chunks], chunk kc of row m at kc ^ ((m >> 1) & 7)

    const SkinnyProblem p = a.p[blockIdx.z];
    const int n0 = blockIdx.x * kSfBN;
    const int k_begin = blockIdx.y * a.k_per_split, k_end = min(a.K, k_begin + a.k_per_split);
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float* __restrict__ Xp = reinterpret_cast<const float*>(p.Xp);
    const float* __restrict__ Xm = reinterpret_cast<const float*>(p.Xm);
    const float c = UPDATE ? *a.c_ptr : 0.f;

    // this lane's weight row; its chunks' place in the tensor (the random stream's counter) and in the workgroup's rows as a buffer: rows
    // past N are outside it, are read as zeros and not written
    const int row = wave * 16 + r;
    const uint64_t we = (uint64_t)(n0 + row) * (uint64_t)a.K + (uint64_t)(8 * g);
    const __amdgpu_buffer_rsrc_t rows =
        __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<float*>(p.theta) + (size_t)n0 * a.K, 0, (int)((uint32_t)min(kSfBN, a.N - n0) * a.K * 4u), 0x00020000);
    const int row_at = (row * a.K + 8 * g) * 4;

    struct Theta { v4u_t v[2][2]; };                           // two chunks of eight, 32 apart
    auto load_theta = [&](Theta& t, int k0) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 2; ++e) t.v[h][e] = __builtin_amdgcn_raw_buffer_load_b128(rows, row_at + 128 * h + 16 * e, k0 * 4, 0);
    };
    // theta' of both chunks, stored if this is where the update is applied.  (k0 in the lanes' offsets: with a scalar offset in a register the
    // compiler lets the very next instruction write the store's data registers, here theta' - eps z over theta', and what arrives in
    // memory is now and then the new value.)
    auto updated = [&](const Theta& t, int k0, bool apply, float (&th)[2][8]) {
        __builtin_memcpy(th, &t, sizeof(th));
        if (!apply) return;
        uint32_t w[2][4];
        const uint64_t e = we + (uint64_t)k0;
        philox4x32_10_x2(e >> 3, (e >> 3) + 4, p.tensor_id, a.key_prev, w);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            float z[8];
#pragma unroll
            for (int i = 0; i < 4; ++i) box_muller(w[h][i], z[2 * i], z[2 * i + 1]);
#pragma unroll
            for (int j = 0; j < 8; ++j) th[h][j] = __builtin_fmaf(-c, z[j], th[h][j]);
            v4u_t s[2];
            __builtin_memcpy(s, th[h], 32);
#pragma unroll
            for (int q = 0; q < 2; ++q) __builtin_amdgcn_raw_buffer_store_b128(s[q], rows, row_at + 128 * h + 16 * q + k0 * 4, 0, 0);
        }
    };
    auto draw = [&](int k0, float (&z)[2][8]) {
        uint32_t w[2][4];
        const uint64_t e = we + (uint64_t)k0;
        philox4x32_10_x2(e >> 3, (e >> 3) + 4, p.tensor_id, a.key, w);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < 4; ++i) box_muller(w[h][i], z[h][2 * i], z[h][2 * i + 1]);
    };
    // the parts of a chunk's W+ and W-: [stream][part]
    struct Parts { v4u_t w[2][3]; } part[2];
    auto perturb = [&](const Theta& t, int k0) {
        float th[2][8], z[2][8];
        updated(t, k0, UPDATE, th);
        draw(k0, z);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                float x[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) x[j] = __builtin_fmaf(s ? -a.eps : a.eps, z[h][j], th[h][j]);
#pragma unroll
                for (int q = 0; q < 3; ++q)
#pragma unroll
                    for (int j = 0; j < 4; ++j) part[h].w[s][q][j] = split_step(x[2 * j], x[2 * j + 1]);
            }
    };

    // activations: a thread's chunk i is (row (tid + 512 i) >> 3 of the 2 x 32 MT, chunk tid & 7); rows past M repeat row M - 1
    v4f_t xr[MT][2];
    const float* xsrc[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        const int m = (tid >> 3) + 64 * i, s = m >= 32 * MT;
        xsrc[i] = (s ? Xm : Xp) + (size_t)min(m - 32 * MT * s, a.M - 1) * a.ldx + (tid & 7) * 8;
    }
    auto load_x = [&](int k0) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int e = 0; e < 2; ++e) xr[i][e] = *reinterpret_cast<const v4f_t*>(xsrc[i] + k0 + 4 * e);
    };
    auto store_x = [&](int buf) {
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            const int m = (tid >> 3) + 64 * i, at = m * 8 + ((tid & 7) ^ ((m >> 1) & 7));
            float x[8];
            __builtin_memcpy(x, xr[i], 32);
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                v4u_t u;
#pragma unroll
                for (int j = 0; j < 4; ++j) u[j] = split_step(x[2 * j], x[2 * j + 1]);
                Xs[(buf * 3 + q) * PLANE + at] = u;
            }
        }
    };

    v4f_t hi[NI], low[NI];                 // tile i: rows 16 i .. + 15 of the 2 x 32 MT
#pragma unroll
    for (int i = 0; i < NI; ++i) hi[i] = low[i] = v4f_t{0.f, 0.f, 0.f, 0.f};
    // two tiles at a time: a product does not wait for the one before it
    auto multiply = [&](int buf) {
        const v4u_t* X = Xs + buf * 3 * PLANE;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const v4u_t* at = X + r * 8 + ((4 * h + g) ^ ((r >> 1) & 7));
#pragma unroll
            for (int i = 0; i < NI; i += 2) {
                const v4u_t(&w)[3] = part[h].w[i >= NI / 2];
                v4u_t x[2][3];
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int q = 0; q < 3; ++q) x[t][q] = at[q * PLANE + (i + t) * 128];
#pragma unroll
                for (int t = 0; t < 2; ++t) low[i + t] = mfma16_bf16(w[2], x[t][0], low[i + t]);
#pragma unroll
                for (int t = 0; t < 2; ++t) hi[i + t] = mfma16_bf16(w[0], x[t][0], hi[i + t]);
#pragma unroll
                for (int t = 0; t < 2; ++t) low[i + t] = mfma16_bf16(w[0], x[t][2], low[i + t]);
#pragma unroll
                for (int t = 0; t < 2; ++t) low[i + t] = mfma16_bf16(w[1], x[t][1], low[i + t]);
#pragma unroll
                for (int t = 0; t < 2; ++t) low[i + t] = mfma16_bf16(w[1], x[t][0], low[i + t]);
#pragma unroll
                for (int t = 0; t < 2; ++t) low[i + t] = mfma16_bf16(w[0], x[t][1], low[i + t]);
            }
        }
    };
    Theta t;
    load_theta(t, k_begin);
    load_x(k_begin);
    perturb(t, k_begin);
    store_x(0);
    int buf = 0;
    for (int k0 = k_begin;; k0 += kSfBK) {
        const bool more = k0 + kSfBK < k_end;
        if (more) {
            load_theta(t, k0 + kSfBK);
            load_x(k0 + kSfBK);
        }
        __syncthreads();                   // this slab's activations are there, and nobody reads those of the one before any more
        multiply(buf);
        if (!more) break;
        perturb(t, k0 + kSfBK);
        buf ^= 1;
        store_x(buf);
    }

    OddSums o;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            hi[i][e] += low[i][e];
            o.look(hi[i][e]);
        }
    if (o.any()) {                         // once more with float32 products: theta' from memory, which holds it by now, and the activations as they are
#pragma unroll
        for (int i = 0; i < NI; ++i) hi[i] = v4f_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int k0 = k_begin; k0 < k_end; k0 += kSfBK) {
            float th[2][8], z[2][8];
            load_theta(t, k0);
            updated(t, k0, false, th);
            draw(k0, z);
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const bool s = i >= NI / 2;
                const float* X = (s ? Xm : Xp) + (size_t)min((i - (s ? NI / 2 : 0)) * 16 + r, a.M - 1) * a.ldx + k0 + 8 * g;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    float x[8];
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const v4f_t f = *reinterpret_cast<const v4f_t*>(X + 32 * h + 4 * e);
                        __builtin_memcpy(x + 4 * e, &f, 16);
                    }
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        hi[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_fmaf(s ? -a.eps : a.eps, z[h][j], th[h][j]), x[j], hi[i], 0, 0, 0);
                }
            }
        }
    }
    const int n = n0 + wave * 16 + 4 * g;
    if (n >= a.N) return;                  // (N % 4 == 0)
    const size_t plane = (size_t)a.M * a.N;
    float* __restrict__ out = a.partial + ((size_t)blockIdx.z * a.splits + blockIdx.y) * 2 * plane + n;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int s = i >= NI / 2, m = (i - (s ? NI / 2 : 0)) * 16 + r;
        if (m < a.M) *reinterpret_cast<v4f_t*>(out + s * plane + (size_t)m * a.N) = hi[i];
    }
}

template <int MT, bool UPDATE>
static zo2_status launch_as(const SkinnyArgs& a, hipStream_t st) {
    const dim3 grid((a.N + kSfBN - 1) / kSfBN, a.splits, a.nprob);
    constexpr int lds = 2 * 3 * 64 * MT * 8 * 16;              // 48 KB a row tile
    static bool reserved_on[kMaxDevices] = {false};
    bool& reserved = reserved_on[current_device()];
    auto kern = skinny_f32_kernel<MT, UPDATE>;
    if (!reserved) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess) {
            set_op_error("skinny gemm: cannot reserve %d bytes of LDS", lds);
            return ZO2_EHIP;
        }
        reserved = true;
    }
    hipLaunchKernelGGL(kern, grid, dim3(512), lds, st, a);
    ZO2_HIP_LAUNCH_CHECK();
    return ZO2_OK;
}

bool skinny_f32_applicable(int M, int N, int K) { return M >= 1 && M <= 96 && N >= 1 && N % 4 == 0 && K >= 64 && K % 64 == 0 && K < 1 << 22; }

zo2_status skinny_f32_launch(const SkinnyArgs& a, hipStream_t st) {
    if (a.M <= 32) return a.c_ptr ? launch_as<1, true>(a, st) : launch_as<1, false>(a, st);
    if (a.M <= 64) return a.c_ptr ? launch_as<2, true>(a, st) : launch_as<2, false>(a, st);
    return a.c_ptr ? launch_as<3, true>(a, st) : launch_as<3, false>(a, st);
}

}  // namespace zo2
