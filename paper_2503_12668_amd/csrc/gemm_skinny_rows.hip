// The projections of up to 96 tokens (16 bits: those that gemm_skinny_few.hip does not take): gemm_skinny.hip's layout - a workgroup owns 128 output features and a slice of k, reads the stored
// weights once for both perturbation streams and forms W+- in registers - with wavefronts of 16 features over the whole slice on 16-row matrix
// instructions: nothing meets at the end, the four lanes of a row read (and write) its whole 128 bytes, and a lane ends with four
// neighbouring columns of a row.  The pending update can be applied in the same place: a lane writes theta' = theta - c z_prev back and multiplies with
// theta' +- eps z.
//
// 16 bits.  What bounds it is the generator, about 130 instructions per draw of eight elements; few registers (72 - 120) leave it four
// wavefronts per SIMD.  Per launch, wavefronts of 32 features and half a slab's k -> this, d 2048, 16 rows, us: QKV 14.8 -> 13.2, output 8.6 -> 7.3, FC1 16.0 -> 14.3,
// FC2 14.4 -> 13.3, LM head 84 -> 77.  Steps: 12 blocks, 16 tokens 1579 -> 1513, 96 2037 -> 1972; float16, d 2560, 6 blocks, 30 tokens 1236 -> 1134.  A matrix instruction
// reads its own kilobyte of activations from LDS, which beyond 96 rows takes longer than the generator (d 4096, 4 blocks, 128 tokens 2042 -> 2097).
//
// float32.  Each operand as three bfloat16 parts (f32_parts.h).  The sweep's copies move 16 bytes a parameter and are read again, 8 more; here it
// is 8 in all.
// What bounds it: two draws and the parts of two copies are some 50 vector instructions an element; a slab of 64 rows, 1.5 us of them, 1.4 us of
// MFMAs and as much of LDS reads, takes 4 us on a compute unit.  At d 768 a launch is one or two slabs per workgroup and 9 us of first loads,
// last stores, start and end.  Steps, sweep and float32 GEMMs -> this, us: d 768, 12 blocks, 16 tokens 1162 -> 952, 64 1390 -> 1284, 96 1623 -> 1499;
// d 2048, 6 blocks, 16 2185 -> 1284, 64 2389 -> 1653, 96 2812 -> 2012; d 4096, 2 blocks, 30 3045 -> 1711; d 5120, 2 blocks, 60 4699 -> 3055.  128
// rows (one slab in LDS, its registers full) 1657 -> 1841, 2848 -> 2636, d 5120 5476 -> 5735: the line is drawn at 96.
// (Wavefronts of 32 features and half a slab's k, as in gemm_skinny.hip, read LDS half as often, but their halves have to meet and their
// lanes to store single floats: 1425 us where this takes 1284.)
#include <algorithm>

#include "f32_parts.h"
#include "skinny_weights.h"

namespace zo2 {

static constexpr int kSfBN = 128, kSfBK = 64;      // weight rows per workgroup, k per slab

// v_mfma_f32_16x16x32_bf16: lane (r, g) = (l & 15, l >> 4) supplies k = 8 g .. + 7 of row r of either operand.  Wavefront w owns features 16 w ..
// + 15 of the workgroup's 128 over the whole slice, so nothing has to meet at the end; the lanes of a row read and write whole lines of theta.
// With the weights as the first operand a lane ends with row r of the activations and features 4 g .. + 3.
// MT: 32 rows of each stream.
template <typename T, int MT, bool UPDATE, bool CE>
__global__ __launch_bounds__(512, MT == 1 && sizeof(T) == 2 ? 4 : 2) void skinny_rows_kernel(const SkinnyArgs a) {
    constexpr bool F32 = sizeof(T) == 4;
    constexpr int R = 64 * MT, NI = 4 * MT, PLANE = R * 8;     // activation rows of both streams, 16-row tiles, 16-byte chunks of one part of a slab
    constexpr int P = RowsMfma<T>::kParts, Q = F32 ? 2 : 1;    // parts of an operand; 16-byte pieces of eight elements
    extern __shared__ __attribute__((aligned(16))) char smem[];
    v4u_t* Xs = reinterpret_cast<v4u_t*>(smem);                // [2 slabs][P parts][R rows][8 chunks], chunk kc of row m at kc ^ ((m >> 1) & 7)

    const SkinnyProblem p = a.p[blockIdx.z];
    const int n0 = blockIdx.x * kSfBN;
    const int k_begin = blockIdx.y * a.k_per_split, k_end = min(a.K, k_begin + a.k_per_split);
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const T* __restrict__ Xp = reinterpret_cast<const T*>(p.Xp);
    const T* __restrict__ Xm = reinterpret_cast<const T*>(p.Xm);
    const float c = UPDATE ? *a.c_ptr : 0.f;

    const WeightLane<T> lane_w(a, p, n0, kSfBN, wave * 16 + r, 8 * g);
    using Theta = typename WeightLane<T>::Theta;
    // the parts of a chunk's W+ and W-: [stream][part]
    struct Parts { v4u_t w[2][P]; } part[2];
    auto perturb = [&](const Theta& t, int k0) {
        float th[2][8], z[2][8];
        lane_w.values(t, th);
        if constexpr (UPDATE) {
            lane_w.draw(k0, a.key_prev, z);
            lane_w.update(k0, c, z, th);
        }
        lane_w.draw(k0, a.key, z);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                if constexpr (F32) {
                    float x[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) x[j] = __builtin_fmaf(s ? -a.eps : a.eps, z[h][j], th[h][j]);
#pragma unroll
                    for (int q = 0; q < P; ++q)
#pragma unroll
                        for (int j = 0; j < 4; ++j) part[h].w[s][q][j] = split_step(x[2 * j], x[2 * j + 1]);
                } else {
                    Vec<T, 8> x;
#pragma unroll
                    for (int j = 0; j < 8; ++j) x.v[j] = Fmt<T>::store(__builtin_fmaf(s ? -a.eps : a.eps, z[h][j], th[h][j]));
                    __builtin_memcpy(&part[h].w[s][0], &x, 16);
                }
            }
    };

    // activations: a thread's chunk i is (row (tid + 512 i) >> 3 of the 2 x 32 MT, chunk tid & 7); rows past M repeat row M - 1
    v4u_t xr[MT][Q];
    const T* xsrc[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        const int m = (tid >> 3) + 64 * i, s = m >= 32 * MT;
        xsrc[i] = (s ? Xm : Xp) + (size_t)min(m - 32 * MT * s, a.M - 1) * a.ldx + (tid & 7) * 8;
    }
    auto load_x = [&](int k0) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int e = 0; e < Q; ++e) xr[i][e] = *reinterpret_cast<const v4u_t*>(xsrc[i] + k0 + 4 * e);
    };
    auto store_x = [&](int buf) {
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            const int m = (tid >> 3) + 64 * i, at = m * 8 + ((tid & 7) ^ ((m >> 1) & 7));
            if constexpr (F32) {
                float x[8];
                __builtin_memcpy(x, xr[i], 32);
#pragma unroll
                for (int q = 0; q < P; ++q) {
                    v4u_t u;
#pragma unroll
                    for (int j = 0; j < 4; ++j) u[j] = split_step(x[2 * j], x[2 * j + 1]);
                    Xs[(buf * P + q) * PLANE + at] = u;
                }
            } else {
                Xs[buf * PLANE + at] = xr[i][0];
            }
        }
    };

    v4f_t hi[NI], low[F32 ? NI : 1];       // tile i: rows 16 i .. + 15 of the 2 x 32 MT
#pragma unroll
    for (int i = 0; i < NI; ++i) hi[i] = v4f_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; F32 && i < NI; ++i) low[i] = v4f_t{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](int buf) {
        const v4u_t* X = Xs + buf * P * PLANE;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const v4u_t* at = X + r * 8 + ((4 * h + g) ^ ((r >> 1) & 7));
            if constexpr (F32) {           // two tiles at a time: a product does not wait for the one before it
#pragma unroll
                for (int i = 0; i < NI; i += 2) {
                    const v4u_t(&w)[P] = part[h].w[i >= NI / 2];
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
            } else {
#pragma unroll
                for (int i = 0; i < NI; ++i) hi[i] = RowsMfma<T>::run(part[h].w[i >= NI / 2][0], at[i * 128], hi[i]);
            }
        }
    };
    Theta t;
    lane_w.load(t, k_begin);
    load_x(k_begin);
    perturb(t, k_begin);
    store_x(0);
    int buf = 0;
    for (int k0 = k_begin;; k0 += kSfBK) {
        const bool more = k0 + kSfBK < k_end;
        if (more) {
            lane_w.load(t, k0 + kSfBK);
            load_x(k0 + kSfBK);
        }
        __syncthreads();                   // this slab's activations are there, and nobody reads those of the one before any more
        multiply(buf);
        if (!more) break;
        perturb(t, k0 + kSfBK);
        buf ^= 1;
        store_x(buf);
    }

    if constexpr (F32) {
        OddSums o;
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                hi[i][e] += low[i][e];
                o.look(hi[i][e]);
            }
        if (o.any()) {                     // once more with float32 products: theta' from memory, which holds it by now, and the activations as they are
#pragma unroll
            for (int i = 0; i < NI; ++i) hi[i] = v4f_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
            for (int k0 = k_begin; k0 < k_end; k0 += kSfBK) {
                float th[2][8], z[2][8];
                lane_w.load(t, k0);
                lane_w.values(t, th);
                lane_w.draw(k0, a.key, z);
#pragma unroll
                for (int i = 0; i < NI; ++i) {
                    const bool s = i >= NI / 2;
                    const T* X = (s ? Xm : Xp) + (size_t)min((i - (s ? NI / 2 : 0)) * 16 + r, a.M - 1) * a.ldx + k0 + 8 * g;
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
    }
    if constexpr (CE) {
        // cross-entropy partials of this workgroup's 128 columns: a stream's logits are parked in LDS (16 KB x MT, the size of the
        // activations' buffers), then half a wavefront reduces a 64-column span of a row
        float* tile = reinterpret_cast<float*>(smem);
        const int span = lane >> 5, col = 64 * span + 2 * (lane & 31);
        constexpr float kL2e = 1.4426950408889634f;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NI / 2; ++i) *reinterpret_cast<v4f_t*>(tile + (i * 16 + r) * kSfBN + wave * 16 + 4 * g) = hi[s * (NI / 2) + i];
            __syncthreads();
            for (int m = wave; m < a.M; m += 8) {
                float2 y = *reinterpret_cast<const float2*>(tile + m * kSfBN + col);
                if (n0 + col >= a.N) y = make_float2(-INFINITY, -INFINITY);       // N % 4 == 0
                float mx = fmaxf(y.x, y.y);
#pragma unroll
                for (int d = 1; d < 32; d <<= 1) mx = fmaxf(mx, __shfl_xor(mx, d, 64));
                const float mb = mx == -INFINITY ? 0.f : mx;                      // a span past the last column sums to 0
                float sum = __builtin_amdgcn_exp2f((y.x - mb) * kL2e) + __builtin_amdgcn_exp2f((y.y - mb) * kL2e);
#pragma unroll
                for (int d = 1; d < 32; d <<= 1) sum += __shfl_xor(sum, d, 64);
                const size_t at = (size_t)(blockIdx.x * 2 + span) * (size_t)a.part_ld + (size_t)(s * a.M + m);
                if ((lane & 31) == 0) {
                    a.part_max[at] = mx;
                    a.part_sum[at] = sum;
                }
                const int dl = a.labels[m] - n0;
                if (lane == 0 && dl >= 0 && dl < kSfBN) a.label_logit[s * a.M + m] = tile[m * kSfBN + dl];
            }
        }
        return;
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

template <typename T, int MT, bool UPDATE, bool CE>
static zo2_status launch_as(const SkinnyArgs& a, hipStream_t st) {
    const dim3 grid((a.N + kSfBN - 1) / kSfBN, a.splits, a.nprob);
    constexpr int lds = 2 * RowsMfma<T>::kParts * 64 * MT * 8 * 16;              // 16 KB a row tile and part
    static bool reserved_on[kMaxDevices] = {false};
    bool& reserved = reserved_on[current_device()];
    auto kern = skinny_rows_kernel<T, MT, UPDATE, CE>;
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

template <bool UPDATE>
static zo2_status launch_f32(const SkinnyArgs& a, hipStream_t st) {
    return a.M <= 32 ? launch_as<float, 1, UPDATE, false>(a, st) : a.M <= 64 ? launch_as<float, 2, UPDATE, false>(a, st) : launch_as<float, 3, UPDATE, false>(a, st);
}
template <typename T, bool CE>
static zo2_status launch_16(const SkinnyArgs& a, hipStream_t st) {
    return a.M <= 32 ? launch_as<T, 1, false, CE>(a, st) : a.M <= 64 ? launch_as<T, 2, false, CE>(a, st) : launch_as<T, 3, false, CE>(a, st);
}

zo2_status skinny_rows_launch(const SkinnyArgs& a, int dtype, bool ce, hipStream_t st) {
    if (dtype == ZO2_F32) return a.c_ptr ? launch_f32<true>(a, st) : launch_f32<false>(a, st);
    if (dtype == ZO2_F16) return ce ? launch_16<f16_t, true>(a, st) : launch_16<f16_t, false>(a, st);
    if (!a.c_ptr) return ce ? launch_16<bf16_t, true>(a, st) : launch_16<bf16_t, false>(a, st);
    ZO2_OP_CHECK(a.M <= 32, ZO2_EINVAL, "skinny gemm: an update in the loader of bfloat16 takes at most 32 rows, not %d", a.M);
    return ce ? launch_as<bf16_t, 1, true, true>(a, st) : launch_as<bf16_t, 1, true, false>(a, st);
}

}  // namespace zo2
