// Projections of the dual forward when a step has few tokens (at most 256 per stream).
//
// With so few rows the projections are bound by reading the weights, not by the matrix cores, and the large-tile
// kernel has a handful of tiles for 256 compute units.  This kernel turns the layout around: a workgroup owns 128 output
// features and a slice of k, streams the stored weights theta through once for BOTH perturbation streams, and forms
// W+ = theta + eps z, W- = theta - eps z in its loader, chunk by chunk in registers (z regenerated from the counters,
// Alg. 2 "perturb"; the same arithmetic and rounding as the sweep kernel, so the same bits) - the two perturbed copies
// of a block are never written to memory nor read back.  The k range is cut into slices so that a launch has a few hundred
// workgroups; the slices' float32 partial sums go to a workspace and a second kernel adds them in slice order
// (deterministic, unlike atomics) and applies bias, scale, ReLU and residual.
#include "gemm_skinny.h"

#include <algorithm>

namespace zo2 {

typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t v4u_t __attribute__((ext_vector_type(4)));
typedef float v4f_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));

template <typename T> struct SkMfma;
template <> struct SkMfma<bf16_t> {
    static __device__ __forceinline__ f32x16_t run(v4u_t a, v4u_t b, f32x16_t c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
    }
};
template <> struct SkMfma<f16_t> {
    static __device__ __forceinline__ f32x16_t run(v4u_t a, v4u_t b, f32x16_t c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
    }
};

// Eight consecutive stored elements (one 16-byte chunk) and their Philox words -> the same chunk of W+ and of W-: one call, four Box-Muller pairs, one fused multiply-add and one rounding per element and sign.
template <typename T>
__device__ __forceinline__ void perturb_words(const uint32_t w[4], float eps, v4u_t th, v4u_t& wp, v4u_t& wm) {
    Vec<T, 8> t8, p8, m8;
    __builtin_memcpy(&t8, &th, 16);
    float z[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) box_muller(w[i], z[2 * i], z[2 * i + 1]);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const float t = Fmt<T>::load(t8.v[j]);
        p8.v[j] = Fmt<T>::store(__builtin_fmaf(eps, z[j], t));
        m8.v[j] = Fmt<T>::store(__builtin_fmaf(-eps, z[j], t));
    }
    __builtin_memcpy(&wp, &p8, 16);
    __builtin_memcpy(&wm, &m8, 16);
}
// one chunk, starting at element index e, a multiple of 8 (the test hook)
template <typename T>
__device__ __forceinline__ void perturb_chunk(const PhiloxKeys& key, uint32_t tensor_id, uint64_t e, float eps, v4u_t th, v4u_t& wp, v4u_t& wm) {
    uint32_t w[4];
    philox4x32_10((uint32_t)(e >> 3), (uint32_t)(e >> 35), tensor_id, 0u, key, w);
    perturb_words<T>(w, eps, th, wp, wm);
}
// two chunks, 16 elements apart, in step (the loader)
template <typename T>
__device__ __forceinline__ void perturb_pair(const PhiloxKeys& key, uint32_t tensor_id, uint64_t e, float eps, const v4u_t th[2], v4u_t wp[2], v4u_t wm[2]) {
    uint32_t w[2][4];
    philox4x32_10_x2(e >> 3, (e >> 3) + 2, tensor_id, key, w);
#pragma unroll
    for (int j = 0; j < 2; ++j) perturb_words<T>(w[j], eps, th[j], wp[j], wm[j]);
}

// The order asked of the scheduler for N MFMAs of one pair of chunks beside the generation of the next: the pair's vector
// instructions (about 190, and 32 transcendental ones) spread evenly behind the MFMAs, each of which occupies the matrix
// pipeline for 32 cycles, and the reads of activations four MFMAs ahead of their use.
template <int N, int J>
__device__ __forceinline__ void mix_from() {
    if constexpr (J == 0) __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    if constexpr ((J + 1) * 190 / N > J * 190 / N) __builtin_amdgcn_sched_group_barrier(0x002, (J + 1) * 190 / N - J * 190 / N, 0);
    if constexpr ((J + 1) * 32 / N > J * 32 / N) __builtin_amdgcn_sched_group_barrier(0x400, (J + 1) * 32 / N - J * 32 / N, 0);
    if constexpr (J + 4 < N) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    if constexpr (J + 1 < N) mix_from<N, J + 1>();
}

static constexpr int kSkRows = 96;          // rows of skinny_rows_kernel
static constexpr int kSkBN = 128, kSkBK = 64, kSkKC = 8;      // weight rows per workgroup, k per slab, 16-byte chunks per slab row

// MT: 32-row MFMA tiles per stream (the workgroup covers 32 MT rows of each stream, every wavefront all of them).
//
// A wavefront owns 32 of the workgroup's 128 output features.  The MFMA's weight operand wants, in lane (r, kh), the 8
// consecutive k of feature r starting at 16 ks + 8 kh: exactly one 16-byte chunk of the stored weight and one call of
// the generator, so a lane loads its chunk of theta, perturbs it in registers and feeds both MFMAs from there - the
// weights never pass through LDS and no wavefront waits for another's generation.  Only the activations are shared:
// their slab (2 streams x 32 MT rows x 64 k) is staged in LDS, double-buffered, one barrier per slab.
//
// What bounds it is the generator: about 130 instructions per chunk, 16 of them transcendental, which take twice an ordinary
// one's time.  One wavefront alone leaves a good part of that time unused on dependences, so a slab's
// two pairs of chunks go to two wavefronts (NW = 8; their sums meet in LDS at the end, a pair's MFMAs run under the
// generation of the wavefront's next) where two wavefronts per SIMD fit the registers: up to 128 rows per stream.  Beyond,
// one wavefront takes both pairs (NW = 4).
// Up to 96 rows skinny_rows_kernel (gemm_skinny_rows.hip) has taken its place, but for contexts that keep the order of their sums.
template <typename T, int MT, int NW, bool CE>
__global__ __launch_bounds__(64 * NW, (MT <= 4 ? 2 : 1)) void skinny_dual_kernel(const SkinnyArgs a) {
    constexpr int MP = 32 * MT, NT = 64 * NW, CX = (MP * kSkKC + NT - 1) / NT;      // rows per stream; X chunks each thread stages per stream and slab
    constexpr int PAIRS = 8 / NW;                             // pairs of chunks per wavefront and slab
    extern __shared__ __attribute__((aligned(16))) char smem[];
    v4u_t* Xs = reinterpret_cast<v4u_t*>(smem);               // [2 buffers][2 streams][MP rows][8 chunks], chunk index XOR-swizzled

    const SkinnyProblem p = a.p[blockIdx.z];
    const int n0 = blockIdx.x * kSkBN;
    const int k_begin = blockIdx.y * a.k_per_split, k_end = min(a.K, k_begin + a.k_per_split);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r = lane & 31, kh = lane >> 5;
    const int half = NW == 8 ? wave >> 2 : 0;                 // which pair of a slab this wavefront takes
    const T* __restrict__ Xp = reinterpret_cast<const T*>(p.Xp);
    const T* __restrict__ Xm = reinterpret_cast<const T*>(p.Xm);
    const T* __restrict__ Th = reinterpret_cast<const T*>(p.theta);

    // staging plan of the activations: chunk c = tid + NT i of a stream's slab is (row c >> 3, position c & 7); rows past
    // M re-read row M - 1.  Position kc of row m sits at chunk kc ^ ((m >> 1) & 7): sixteen lanes that read one position
    // of sixteen consecutive rows, and eight that write one row, each touch every bank once.
    // (96 rows over 512 threads: the second chunk is there for half of them only)
    auto staged = [&](int i) { return (i + 1) * NT <= MP * kSkKC || tid + NT * i < MP * kSkKC; };
    uint32_t xoff[CX];
    int xl[CX];
#pragma unroll
    for (int i = 0; i < CX; ++i) {
        const int c = tid + NT * i, row = c >> 3, kc = c & 7;
        xoff[i] = (uint32_t)((size_t)min(row, a.M - 1) * a.ldx + kc * 8);
        xl[i] = row * kSkKC + (kc ^ ((row >> 1) & 7));
    }
    // this lane's weight row (features past N re-read row N - 1; their sums are dropped) and, in elements from the
    // tensor's start, where its first chunk begins: the random stream's counter and the load address in one
    const int n = n0 + (wave & 3) * 32 + r;
    const uint64_t we = (uint64_t)min(n, a.N - 1) * (uint64_t)a.K + (uint64_t)(kh * 8);

    f32x16_t acc[2][MT];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[s][i][v] = 0.f;

    v4u_t xr[2][CX];
    auto load_x = [&](int k0) {
#pragma unroll
        for (int i = 0; i < CX; ++i) {
            if (!staged(i)) continue;
            xr[0][i] = *reinterpret_cast<const v4u_t*>(Xp + xoff[i] + k0);
            xr[1][i] = *reinterpret_cast<const v4u_t*>(Xm + xoff[i] + k0);
        }
    };
    auto store_x = [&](int buf) {
        v4u_t* Xb = Xs + buf * (2 * MP * kSkKC);
#pragma unroll
        for (int i = 0; i < CX; ++i) {
            if (!staged(i)) continue;
            Xb[xl[i]] = xr[0][i];
            Xb[MP * kSkKC + xl[i]] = xr[1][i];
        }
    };
    // A pair of chunks: 32 k.  While the MFMAs of one pair run, the wavefront's vector instructions generate the next; the
    // registers of a pair's theta are reloaded, a slab ahead, as soon as it is perturbed.
    struct Pair { v4u_t th[2], wp[2], wm[2]; } P[2];
    auto load_theta = [&](Pair& q, int k0) {
#pragma unroll
        for (int h = 0; h < 2; ++h) q.th[h] = *reinterpret_cast<const v4u_t*>(Th + we + min(k0, k_end - 32) + 16 * h);
    };
    auto perturb = [&](Pair& q, int k0) { perturb_pair<T>(a.key, p.tensor_id, we + (uint64_t)k0, a.eps, q.th, q.wp, q.wm); };
    auto mfma = [&](const Pair& q, const v4u_t* Xb, int ks) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int kc = (ks + h) * 2 + kh;
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                const int row = i * 32 + r, at = row * kSkKC + (kc ^ ((r >> 1) & 7));
                acc[0][i] = SkMfma<T>::run(Xb[at], q.wp[h], acc[0][i]);
                acc[1][i] = SkMfma<T>::run(Xb[MP * kSkKC + at], q.wm[h], acc[1][i]);
            }
        }
    };
    const v4u_t* Xb = Xs;
    int buf = 0, k0 = k_begin;
    auto next_slab = [&]() {
        buf ^= 1;
        store_x(buf);                      // last read before the barrier that ended the previous slab
        Xb = Xs + buf * (2 * MP * kSkKC);
        __syncthreads();
    };
    if constexpr (PAIRS == 1) {            // P[0]: this slab's pair, P[1]: the next one's
        const int ko = 32 * half;
        load_theta(P[0], k_begin + ko);
        load_x(k_begin);
        load_theta(P[1], k_begin + kSkBK + ko);
        perturb(P[0], k_begin + ko);
        store_x(0);
        __syncthreads();
        for (; k0 + kSkBK < k_end; k0 += kSkBK) {
            load_x(k0 + kSkBK);
            __builtin_amdgcn_sched_barrier(0);
            perturb(P[1], k0 + kSkBK + ko);
            mfma(P[0], Xb, 2 * half);
            mix_from<4 * MT, 0>();
            __builtin_amdgcn_sched_barrier(0);
            load_theta(P[1], k0 + 2 * kSkBK + ko);
            next_slab();
#pragma unroll
            for (int h = 0; h < 2; ++h) { P[0].wp[h] = P[1].wp[h]; P[0].wm[h] = P[1].wm[h]; }
        }
        mfma(P[0], Xb, 2 * half);
    } else {
        load_theta(P[0], k_begin);
        load_x(k_begin);
        load_theta(P[1], k_begin + 32);
        perturb(P[0], k_begin);
        load_theta(P[0], k_begin + kSkBK);
        store_x(0);
        __syncthreads();
        for (; k0 + kSkBK < k_end; k0 += kSkBK) {
            load_x(k0 + kSkBK);
            __builtin_amdgcn_sched_barrier(0);
            perturb(P[1], k0 + 32);
            mfma(P[0], Xb, 0);
            mix_from<4 * MT, 0>();
            __builtin_amdgcn_sched_barrier(0);
            load_theta(P[1], k0 + kSkBK + 32);
            perturb(P[0], k0 + kSkBK);
            mfma(P[1], Xb, 2);
            mix_from<4 * MT, 0>();
            __builtin_amdgcn_sched_barrier(0);
            load_theta(P[0], k0 + 2 * kSkBK);
            next_slab();
        }
        perturb(P[1], k0 + 32);
        mfma(P[0], Xb, 0);
        mfma(P[1], Xb, 2);
    }
    if constexpr (NW == 8) {               // the second half's sums join the first's, one stream at a time (16 KB x MT, the size of the X buffers)
        float* meet = reinterpret_cast<float*>(smem) + ((wave & 3) * 64 + lane) * 4;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            __syncthreads();
            if (half) {
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int v = 0; v < 16; v += 4)
                        *reinterpret_cast<v4f_t*>(meet + (i * 4 + v / 4) * 1024) = v4f_t{acc[s][i][v], acc[s][i][v + 1], acc[s][i][v + 2], acc[s][i][v + 3]};
            }
            __syncthreads();
            if (!half) {
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int v = 0; v < 16; v += 4) {
                        const v4f_t o = *reinterpret_cast<const v4f_t*>(meet + (i * 4 + v / 4) * 1024);
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[s][i][v + e] += o[e];
                    }
            }
        }
        if (!CE && half) return;
    }
    if constexpr (CE) {
        // cross-entropy partials of this workgroup's 128 columns: a stream's logits are parked in LDS (16 KB x MT, the size of the
        // X buffers), then half a wavefront reduces a 64-column span of a row
        float* tile = reinterpret_cast<float*>(smem);
        const int span = lane >> 5, col = 64 * span + 2 * (lane & 31);
        constexpr float kL2e = 1.4426950408889634f;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            __syncthreads();
            if (!half) {
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int v = 0; v < 16; ++v) tile[(i * 32 + 8 * (v >> 2) + 4 * kh + (v & 3)) * kSkBN + (wave & 3) * 32 + r] = acc[s][i][v];
            }
            __syncthreads();
            for (int m = wave; m < a.M; m += NW) {
                float2 y = *reinterpret_cast<const float2*>(tile + m * kSkBN + col);
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
                if (lane == 0 && dl >= 0 && dl < kSkBN) a.label_logit[s * a.M + m] = tile[m * kSkBN + dl];
            }
        }
        return;
    }

    // partial sums of this k slice: lane holds column n of each 32 x 32 tile and rows 8 (v / 4) + 4 kh + v % 4
    if (n >= a.N) return;
    const size_t plane = (size_t)a.M * a.N;
    float* __restrict__ part = a.partial + ((size_t)blockIdx.z * a.splits + blockIdx.y) * 2 * plane;
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int m = i * 32 + 8 * (v >> 2) + 4 * kh + (v & 3);
                if (m < a.M) part[s * plane + (size_t)m * a.N + n] = acc[s][i][v];
            }
}

// Sum of the k slices in slice order, then bias, scale, ReLU, residual; four consecutive columns per thread.
template <typename T, typename OutT>
__global__ __launch_bounds__(256) void skinny_reduce_kernel(const SkinnyArgs a) {
    const int n4 = a.N >> 2;
    const size_t per_stream = (size_t)a.M * n4;
    const size_t gi = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gi >= 2 * per_stream) return;
    const SkinnyProblem p = a.p[blockIdx.y];
    const int s = (int)(gi / per_stream);
    const size_t rem = gi - (size_t)s * per_stream;
    const int m = (int)(rem / n4), n = (int)(rem % n4) * 4;
    const size_t plane = (size_t)a.M * a.N;
    const float* part = a.partial + (size_t)blockIdx.y * a.splits * 2 * plane + (size_t)s * plane + (size_t)m * a.N + n;
    // slice order; the loads of sixteen slices are in flight together (one after the other, a thread would wait out the
    // memory latency once per slice, and so few threads run here that nothing else would hide it)
    v4f_t sum = {0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < a.splits; k0 += 16) {
        v4f_t t[16];
#pragma unroll
        for (int j = 0; j < 16; ++j)
            if (k0 + j < a.splits) t[j] = *reinterpret_cast<const v4f_t*>(part + (size_t)(k0 + j) * 2 * plane);
#pragma unroll
        for (int j = 0; j < 16; ++j)
            if (k0 + j < a.splits) sum += t[j];
    }
    const T* bias = reinterpret_cast<const T*>(s ? p.bias_m : p.bias_p);
    const float* res = s ? p.res_m : p.res_p;
    OutT* Y = reinterpret_cast<OutT*>(s ? p.Ym : p.Yp);
    const size_t o = (size_t)m * a.ldy + n;
    Vec<OutT, 4> out;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float y = (sum[e] + (bias ? Fmt<T>::load(bias[n + e]) : 0.f)) * p.out_scale;
        if (a.relu) y = fmaxf(y, 0.f);
        if (res) y += res[o + e];
        out.v[e] = Fmt<OutT>::store(y);
    }
    store_vec<OutT, 4>(Y + o, out);
}

template <typename T>
__global__ __launch_bounds__(256) void perturbed_rows_kernel(const T* theta, uint64_t e0, uint64_t chunks, uint32_t tensor_id, PhiloxKeys key,
                                                             float eps, T* w_plus, T* w_minus) {
    const uint64_t c = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= chunks) return;
    v4u_t wp, wm;
    perturb_chunk<T>(key, tensor_id, e0 + 8 * c, eps, *reinterpret_cast<const v4u_t*>(theta + 8 * c), wp, wm);
    *reinterpret_cast<v4u_t*>(w_plus + 8 * c) = wp;
    *reinterpret_cast<v4u_t*>(w_minus + 8 * c) = wm;
}

bool skinny_applicable(int M, int N, int K, int dtype) {
    if (dtype == ZO2_F32) return skinny_f32_applicable(M, N, K);
    return (dtype == ZO2_BF16 || dtype == ZO2_F16) && M >= 1 && M <= 256 && N >= 1 && N % 4 == 0 && K >= 64 && K % 64 == 0;
}

// How many pieces the k range is cut into: enough workgroups to occupy the chip (about two per compute unit for up to
// 32 rows, one above - measured on d_model 2048 shapes), but never more float32 partial sums than four times the bytes
// of the weights themselves (a piece writes 2 M x 128 sums for the 128 x k_per_split weights it reads).
static void pick_splits(int M, int N, int K, int nprob, int& splits, int& k_per_split) {
    const int n_tiles = (N + kSkBN - 1) / kSkBN, slabs = K / kSkBK;
    int want = (M <= 32 ? 512 : 256) / (n_tiles * nprob);
    const int cap = K / M > 1 ? K / M : 1;
    want = want > cap ? cap : want;
    want = want < 1 ? 1 : (want > slabs ? slabs : want);
    const int slabs_per = (slabs + want - 1) / want;
    k_per_split = slabs_per * kSkBK;
    splits = (slabs + slabs_per - 1) / slabs_per;
}

// float32: one workgroup per compute unit, of two slabs and more, as many pieces as the workspace holds
static void pick_splits_f32(int M, int N, int K, int nprob, size_t workspace_bytes, int& splits, int& k_per_split) {
    const int n_tiles = (N + kSkBN - 1) / kSkBN, slabs = K / kSkBK;
    const size_t room = workspace_bytes / ((size_t)nprob * 2 * M * N * sizeof(float));
    int want = std::min(std::max(1, 256 / (n_tiles * nprob)), slabs);
    want = (int)std::max<size_t>(1, std::min<size_t>(want, room));
    const int slabs_per = (slabs + want - 1) / want;
    k_per_split = slabs_per * kSkBK;
    splits = (slabs + slabs_per - 1) / slabs_per;
}

size_t skinny_workspace_bytes(int M, int N, int K, int nprob) {
    if (M <= 0 || N <= 0 || K < kSkBK || nprob <= 0) return 0;
    int splits, kps;
    pick_splits(M, N, K, nprob, splits, kps);
    return (size_t)nprob * splits * 2 * (size_t)M * N * sizeof(float);
}

template <typename T, int MT, bool CE, int NW>
static zo2_status skinny_launch_mt(const SkinnyArgs& a, hipStream_t st) {
    const dim3 grid((a.N + kSkBN - 1) / kSkBN, a.splits, a.nprob), block(64 * NW);
    constexpr int lds = 2 * 2 * 32 * MT * kSkKC * 16;
    static bool reserved_on[kMaxDevices] = {false};
    bool& reserved = reserved_on[current_device()];
    auto kern = skinny_dual_kernel<T, MT, NW, CE>;
    if (!reserved) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess) {
            set_op_error("skinny gemm: cannot reserve %d bytes of LDS", lds);
            return ZO2_EHIP;
        }
        reserved = true;
    }
    hipLaunchKernelGGL(kern, grid, block, lds, st, a);
    ZO2_HIP_LAUNCH_CHECK();
    return ZO2_OK;
}

template <typename T>
static zo2_status launch_reduce(const SkinnyArgs& a, hipStream_t st) {
    const size_t work = 2 * (size_t)a.M * (a.N / 4);
    const dim3 rgrid((unsigned)((work + 255) / 256), a.nprob), block(256);
    if (a.out_f32) hipLaunchKernelGGL((skinny_reduce_kernel<T, float>), rgrid, block, 0, st, a);
    else hipLaunchKernelGGL((skinny_reduce_kernel<T, T>), rgrid, block, 0, st, a);
    ZO2_HIP_LAUNCH_CHECK();
    return ZO2_OK;
}

template <typename T>
static zo2_status skinny_launch_t(const SkinnyArgs& a, hipStream_t st, bool sum) {
    const zo2_status s = !a.in_order && a.M <= kSkRows && a.K < 1 << 22 ? skinny_rows_launch(a, __is_same(T, bf16_t) ? ZO2_BF16 : ZO2_F16, false, st)
                       : a.M <= 32 ? skinny_launch_mt<T, 1, false, 4>(a, st) : a.M <= 64 ? skinny_launch_mt<T, 2, false, 4>(a, st)
                       : a.M <= 128 ? (a.in_order ? skinny_launch_mt<T, 4, false, 4>(a, st) : skinny_launch_mt<T, 4, false, 8>(a, st))
                       : a.M <= 192 ? skinny_launch_mt<T, 6, false, 4>(a, st) : skinny_launch_mt<T, 8, false, 4>(a, st);
    return s != ZO2_OK || !sum ? s : launch_reduce<T>(a, st);
}

// does an output lie where some workgroup still reads?  (The sums of all go to the workspace then, and the outputs are made from them.)
static bool writes_its_inputs(const SkinnyArgs& a, int dtype) {
    const size_t osz = a.out_f32 ? 4 : zo2_dtype_size(dtype), y_bytes = ((size_t)(a.M - 1) * a.ldy + a.N) * osz, x_bytes = ((size_t)(a.M - 1) * a.ldx + a.K) * zo2_dtype_size(dtype);
    auto meet = [](const void* y, size_t ny, const void* x, size_t nx) { return x && (uintptr_t)y < (uintptr_t)x + nx && (uintptr_t)x < (uintptr_t)y + ny; };
    for (int i = 0; i < a.nprob; ++i)
        for (const void* y : {(const void*)a.p[i].Yp, (const void*)a.p[i].Ym})
            for (int j = 0; j < a.nprob; ++j) {
                const SkinnyProblem& q = a.p[j];
                const size_t b = (size_t)a.N * zo2_dtype_size(dtype), r_bytes = ((size_t)(a.M - 1) * a.ldy + a.N) * 4;
                if (meet(y, y_bytes, q.Xp, x_bytes) || meet(y, y_bytes, q.Xm, x_bytes) || meet(y, y_bytes, q.bias_p, b) || meet(y, y_bytes, q.bias_m, b) ||
                    meet(y, y_bytes, q.theta, (size_t)a.N * a.K * zo2_dtype_size(dtype)))
                    return true;
                for (const void* res : {(const void*)q.res_p, (const void*)q.res_m})
                    if (res != y && meet(y, y_bytes, res, r_bytes)) return true;
            }
    return false;
}

// the launches whose kernels apply a pending update; the others would pass it by
static bool update_fits(const SkinnyArgs& a, int dtype) {
    return !a.c_ptr || dtype == ZO2_F32 || (dtype == ZO2_BF16 && a.M <= 32 && !a.in_order && a.K < 1 << 22);
}

zo2_status skinny_launch(SkinnyArgs& a, int dtype, void* workspace, size_t workspace_bytes, hipStream_t st, bool sum) {
    ZO2_OP_CHECK(skinny_applicable(a.M, a.N, a.K, dtype), ZO2_EINVAL,
                 "skinny gemm: needs 1 <= M <= 256 (float32: 96), N %% 4 == 0, K %% 64 == 0 (got %d x %d x %d)", a.M, a.N, a.K);
    ZO2_OP_CHECK(update_fits(a, dtype), ZO2_EINVAL, "skinny gemm: no update in the loader of this format, %d rows of %d (in order: %d)", a.M, a.K, a.in_order);
    ZO2_OP_CHECK(a.nprob >= 1 && a.nprob <= SkinnyArgs::kMaxProblems, ZO2_EINVAL, "skinny gemm: %d problems", a.nprob);
    ZO2_OP_CHECK(a.ldx >= a.K && a.ldx % 8 == 0 && a.ldy >= a.N && a.ldy % 4 == 0, ZO2_EINVAL, "skinny gemm: bad leading dimension");
    ZO2_OP_CHECK((size_t)a.M * (size_t)a.ldx < 0xffffffffull, ZO2_EINVAL, "skinny gemm: activation panel too large");
    const size_t osz = a.out_f32 || dtype == ZO2_F32 ? 4 : 2;
    for (int i = 0; i < a.nprob; ++i) {
        const SkinnyProblem& p = a.p[i];
        ZO2_OP_CHECK(p.Xp && p.Xm && p.theta && p.Yp && p.Ym, ZO2_EINVAL, "skinny gemm: NULL operand in problem %d", i);
        ZO2_OP_CHECK((((uintptr_t)p.Xp | (uintptr_t)p.Xm | (uintptr_t)p.theta) & 15) == 0, ZO2_EINVAL, "skinny gemm: operands must be 16-byte aligned");
        ZO2_OP_CHECK((((uintptr_t)p.Yp | (uintptr_t)p.Ym) & (4 * osz - 1)) == 0, ZO2_EINVAL, "skinny gemm: outputs must be aligned to 4 elements");
        ZO2_OP_CHECK((p.bias_p == nullptr) == (p.bias_m == nullptr) && (p.res_p == nullptr) == (p.res_m == nullptr), ZO2_EINVAL,
                     "skinny gemm: bias / residual must be given for both streams or neither");
        ZO2_OP_CHECK(!p.res_p || a.out_f32, ZO2_EINVAL, "skinny gemm: a residual needs float32 output");
    }
    if (dtype == ZO2_F32) pick_splits_f32(a.M, a.N, a.K, a.nprob, workspace_bytes, a.splits, a.k_per_split);
    else pick_splits(a.M, a.N, a.K, a.nprob, a.splits, a.k_per_split);
    const size_t need = (size_t)a.nprob * a.splits * 2 * (size_t)a.M * a.N * sizeof(float);
    ZO2_OP_CHECK(workspace && ((uintptr_t)workspace & 15) == 0 && workspace_bytes >= need, ZO2_EINVAL,
                 "skinny gemm: workspace of %zu bytes needed (16-byte aligned)", need);
    a.partial = reinterpret_cast<float*>(workspace);
    a.direct = 0;
    // (not by `sum`: who adds the pieces is a matter of the scratch's organisation and of how many directions a round has, and is not to show in a sum)
    if (dtype != ZO2_F32 && !a.in_order && skinny_few_pays(a, dtype)) {
        skinny_few_splits(a, a.splits, a.splits, a.k_per_split);
        a.direct = sum && a.splits == 1 && !writes_its_inputs(a, dtype);
        const zo2_status s = skinny_few_launch(a, dtype, st);
        return s != ZO2_OK || !sum || a.direct ? s : dtype == ZO2_BF16 ? launch_reduce<bf16_t>(a, st) : launch_reduce<f16_t>(a, st);
    }
    if (dtype == ZO2_F32) {
        const zo2_status s = skinny_rows_launch(a, ZO2_F32, false, st);
        return s != ZO2_OK || !sum ? s : launch_reduce<float>(a, st);
    }
    if (dtype == ZO2_BF16) return skinny_launch_t<bf16_t>(a, st, sum);
    return skinny_launch_t<f16_t>(a, st, sum);
}

zo2_status skinny_launch_sums(SkinnyArgs& a, float* out, hipStream_t st) {
    ZO2_OP_CHECK(skinny_f32_applicable(a.M, a.N, a.K) && a.nprob == 1 && a.ldx >= a.K && a.ldx % 4 == 0, ZO2_EINVAL,
                 "skinny gemm: %d x %d x %d in %d problems as sums", a.M, a.N, a.K, a.nprob);
    const SkinnyProblem& p = a.p[0];
    ZO2_OP_CHECK(p.Xp && p.Xm && p.theta && out && (((uintptr_t)p.Xp | (uintptr_t)p.Xm | (uintptr_t)p.theta | (uintptr_t)out) & 15) == 0, ZO2_EINVAL,
                 "skinny gemm: NULL operand, or operands not aligned to 16 bytes");
    a.splits = 1; a.k_per_split = a.K; a.partial = out;
    return skinny_rows_launch(a, ZO2_F32, false, st);
}

zo2_status skinny_launch_ce(SkinnyArgs& a, int dtype, hipStream_t st) {
    ZO2_OP_CHECK(dtype != ZO2_F32 && skinny_applicable(a.M, a.N, a.K, dtype) && a.M <= 128 && a.nprob == 1, ZO2_EINVAL,
                 "skinny head: needs 16-bit dtype, 1 <= M <= 128, N %% 4 == 0, K %% 64 == 0 (got %d x %d x %d)", a.M, a.N, a.K);
    ZO2_OP_CHECK(update_fits(a, dtype), ZO2_EINVAL, "skinny head: no update in the loader of this format, %d rows of %d (in order: %d)", a.M, a.K, a.in_order);
    ZO2_OP_CHECK(a.ldx >= a.K && a.ldx % 8 == 0 && (size_t)a.M * (size_t)a.ldx < 0xffffffffull, ZO2_EINVAL, "skinny head: bad leading dimension");
    const SkinnyProblem& p = a.p[0];
    ZO2_OP_CHECK(p.Xp && p.Xm && p.theta && a.labels && a.part_max && a.part_sum && a.label_logit && a.part_ld >= 2 * (int64_t)a.M, ZO2_EINVAL,
                 "skinny head: NULL operand or short partial arrays");
    ZO2_OP_CHECK((((uintptr_t)p.Xp | (uintptr_t)p.Xm | (uintptr_t)p.theta) & 15) == 0, ZO2_EINVAL, "skinny head: operands must be 16-byte aligned");
    a.splits = 1; a.k_per_split = a.K; a.partial = nullptr;      // a vocabulary has tiles for every compute unit
    if (a.M <= kSkRows && a.K < 1 << 22) return skinny_rows_launch(a, dtype, true, st);
    return dtype == ZO2_BF16 ? skinny_launch_mt<bf16_t, 4, true, 8>(a, st) : skinny_launch_mt<f16_t, 4, true, 8>(a, st);
}

zo2_status skinny_perturbed_rows(int dtype, const void* theta, int64_t K, int64_t n0, int64_t rows, uint32_t tensor_id, uint64_t seed,
                                 float eps, void* w_plus, void* w_minus, hipStream_t st) {
    ZO2_OP_CHECK(dtype == ZO2_BF16 || dtype == ZO2_F16, ZO2_EINVAL, "perturbed_rows: dtype must be BF16 or F16");
    ZO2_OP_CHECK(theta && w_plus && w_minus && K > 0 && K % 8 == 0 && n0 >= 0 && rows >= 0, ZO2_EINVAL, "perturbed_rows: bad argument");
    ZO2_OP_CHECK((((uintptr_t)theta | (uintptr_t)w_plus | (uintptr_t)w_minus) & 15) == 0, ZO2_EINVAL, "perturbed_rows: pointers must be 16-byte aligned");
    const uint64_t chunks = (uint64_t)rows * (uint64_t)K / 8;
    if (chunks == 0) return ZO2_OK;
    const PhiloxKeys key = philox_keys(seed);
    const dim3 grid((unsigned)((chunks + 255) / 256)), block(256);
    if (dtype == ZO2_BF16)
        hipLaunchKernelGGL(perturbed_rows_kernel<bf16_t>, grid, block, 0, st, reinterpret_cast<const bf16_t*>(theta), (uint64_t)n0 * (uint64_t)K, chunks,
                           tensor_id, key, eps, reinterpret_cast<bf16_t*>(w_plus), reinterpret_cast<bf16_t*>(w_minus));
    else
        hipLaunchKernelGGL(perturbed_rows_kernel<f16_t>, grid, block, 0, st, reinterpret_cast<const f16_t*>(theta), (uint64_t)n0 * (uint64_t)K, chunks,
                           tensor_id, key, eps, reinterpret_cast<f16_t*>(w_plus), reinterpret_cast<f16_t*>(w_minus));
    ZO2_HIP_LAUNCH_CHECK();
    return ZO2_OK;
}

}  // namespace zo2
