// Projection GEMMs of the dual forward (Alg. 2 "forward"): Y = act((X W^T + b) s) + R.
//
// Both operands are K-contiguous (activations [M, K], weights [N, K]), which is exactly
// the per-lane operand shape of the CDNA MFMA instructions: lane l of a wavefront supplies
// 8 consecutive k of row l % 32.  So tiles go global -> LDS -> registers as 16-byte chunks
// with no transposition; an XOR swizzle of the chunk index keeps the 128-bit LDS accesses
// conflict free.  bf16 / fp16 inputs use v_mfma_f32_32x32x16 (float32 accumulate); the
// float32 mode is in gemm_f32.hip.
//
// The +/- streams (and q, k, v) are independent problems of one shape: they share a launch
// through grid.z so that even the narrow projections fill 256 compute units.
#include <math.h>
#include <string.h>

#include <algorithm>

#include "gemm.h"

namespace zo2 {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
// (native vector types for everything staged in registers: arrays of HIP's struct-based float4 / uint4 are not always
// taken apart into registers by the compiler and then live in scratch memory)
typedef float v4f_t __attribute__((ext_vector_type(4)));
typedef uint32_t v4u_t __attribute__((ext_vector_type(4)));

template <typename T> struct Mfma;
template <> struct Mfma<bf16_t> {
    static __device__ __forceinline__ f32x16_t run(v4u_t a, v4u_t b, f32x16_t c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
    }
};
template <> struct Mfma<f16_t> {
    static __device__ __forceinline__ f32x16_t run(v4u_t a, v4u_t b, f32x16_t c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
    }
};

// ---------------------------------------------------------------------------------------
// MFMA kernel.  Block tile BM x BN x 64, four wavefronts in a 2 x 2 grid, each owning a
// (BM/2) x (BN/2) tile made of 32 x 32 MFMA tiles.  LDS holds two stages of 16-byte chunks:
// chunk (row, kc) of a tile lives at index row * 8 + (kc ^ (row & 7)).
// ---------------------------------------------------------------------------------------
template <typename T, int BM, int BN, typename OutT>
__global__ __launch_bounds__(256, 2) void gemm_mfma_kernel(const GemmArgs a) {
    constexpr int BK = 64, KC = BK / 8;            // 8 chunks of 8 elements per row
    constexpr int WM = BM / 2, WN = BN / 2, TM = WM / 32, TN = WN / 32;
    constexpr int CA = BM * KC / 256, CB = BN * KC / 256;   // chunks each thread stages per tile
    __shared__ v4u_t lds[2][(BM + BN) * KC];

    const GemmProblem p = a.p[blockIdx.z];
    const int tiles_n = (a.N + BN - 1) / BN;
    const int m0 = (blockIdx.x / tiles_n) * BM, n0 = (blockIdx.x % tiles_n) * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1, r = lane & 31, kh = lane >> 5;
    const T* __restrict__ X = reinterpret_cast<const T*>(p.X);
    const T* __restrict__ W = reinterpret_cast<const T*>(p.W);

    // per-thread staging plan
    const T* ga[CA];
    const T* gb[CB];
    int la[CA], lb[CB], kca[CA], kcb[CB];
#pragma unroll
    for (int i = 0; i < CA; ++i) {
        const int c = tid + 256 * i, row = c >> 3, kc = c & 7;
        const int m = min(m0 + row, a.M - 1);
        ga[i] = X + (size_t)m * a.ldx + kc * 8;
        la[i] = row * KC + (kc ^ (row & 7));
        kca[i] = kc * 8;
    }
#pragma unroll
    for (int i = 0; i < CB; ++i) {
        const int c = tid + 256 * i, row = c >> 3, kc = c & 7;
        const int n = min(n0 + row, a.N - 1);
        gb[i] = W + (size_t)n * a.ldw + kc * 8;
        lb[i] = BM * KC + row * KC + (kc ^ (row & 7));
        kcb[i] = kc * 8;
    }

    f32x16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    v4u_t ra[CA], rb[CB];
    const v4u_t zero4 = v4u_t{0u, 0u, 0u, 0u};
    auto load_tile = [&](int k0) {
#pragma unroll
        for (int i = 0; i < CA; ++i) ra[i] = (k0 + kca[i] < a.K) ? *reinterpret_cast<const v4u_t*>(ga[i] + k0) : zero4;
#pragma unroll
        for (int i = 0; i < CB; ++i) rb[i] = (k0 + kcb[i] < a.K) ? *reinterpret_cast<const v4u_t*>(gb[i] + k0) : zero4;
    };
    auto store_tile = [&](int buf) {
#pragma unroll
        for (int i = 0; i < CA; ++i) lds[buf][la[i]] = ra[i];
#pragma unroll
        for (int i = 0; i < CB; ++i) lds[buf][lb[i]] = rb[i];
    };

    const int nk = (a.K + BK - 1) / BK;
    load_tile(0);
    store_tile(0);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        const int cur = kt & 1;
        if (kt + 1 < nk) load_tile((kt + 1) * BK);
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            const int kc = ks * 2 + kh;
            v4u_t fa[TM], fb[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int row = wm * WM + i * 32 + r;
                fa[i] = lds[cur][row * KC + (kc ^ (row & 7))];
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int row = wn * WN + j * 32 + r;
                fb[j] = lds[cur][BM * KC + row * KC + (kc ^ (row & 7))];
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = Mfma<T>::run(fa[i], fb[j], acc[i][j]);
        }
        if (kt + 1 < nk) store_tile(cur ^ 1);
        __syncthreads();
    }

    // epilogue: lane holds column n = r of each 32 x 32 tile and rows 8 (v/4) + 4 kh + v%4
    const T* __restrict__ bias = reinterpret_cast<const T*>(p.bias);
    OutT* __restrict__ Y = reinterpret_cast<OutT*>(p.Y);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int n = n0 + wn * WN + j * 32 + r;
        if (n >= a.N) continue;
        const float bv = bias ? Fmt<T>::load(bias[n]) : 0.f;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int m = m0 + wm * WM + i * 32 + 8 * (v >> 2) + 4 * kh + (v & 3);
                if (m >= a.M) continue;
                float y = (acc[i][j][v] + bv) * p.out_scale;
                if (a.relu) y = fmaxf(y, 0.f);
                const size_t o = (size_t)m * a.ldy + n;
                if (p.residual) y += p.residual[o];
                Y[o] = Fmt<OutT>::store(y);
            }
        }
    }
}

template <typename T>
static zo2_status launch_mfma(const GemmArgs& a, hipStream_t st) {
    constexpr int BM = 128, BN = 128;
    const unsigned tiles = (unsigned)(((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN));
    const dim3 grid(tiles, 1, a.nprob), block(256);
    if (a.out_f32) hipLaunchKernelGGL((gemm_mfma_kernel<T, BM, BN, float>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((gemm_mfma_kernel<T, BM, BN, T>), grid, block, 0, st, a);
    ZO2_HIP_LAUNCH_CHECK();
    return ZO2_OK;
}

// Tile height and k pieces of a float32 launch, by a small cost model in ns: what the kernels of gemm_f32.hip were measured at.  All of
// them run two workgroups per compute unit, so per slab of 32 k a round of two tiles a unit costs 2860 (128 rows), 1800 (64) or 1050 (32),
// a launch or last round of one tile a unit 1120, 780 - 950 (nearly empty chip - full one) or 520 - 740, the launch itself 5300.  Pieces add
// the write and the re-read of their partial sums at 4 TB/s and a second launch (4 us).  With a k that ends inside a slab of 16, 128-row
// tiles were measured at 1130 - 1445 and, from one tile a unit to two, 2240 - 2800; the lower ones, whose last slab alone differs, as above
// (N 8192, K 2056, 128 | 64 | 32 rows, us: 64 rows 79 | 54 | 41, 256 81 | 63 | 75, 512 98 | 121 | 143, 768 155 | 182, 1024 185 | 242).
struct F32Pick { int rows, splits; };
static F32Pick f32_pick(int M, int N, int K, int nprob, int max_splits) {
    const double cu = (double)device_cu_count();
    const double tn = (double)((N + 127) / 128);
    const bool ragged = K % 16 != 0;
    F32Pick best = {128, 1};
    double best_ns = 1e30;
    for (int rows = 128; rows >= 32; rows /= 2) {
        for (int s = 1; s <= max_splits; ++s) {
            const int kp = ((K + s - 1) / s + 31) / 32 * 32;
            if (s > 1 && (kp < 64 || (K + kp - 1) / kp != s)) continue;
            const double tiles = nprob * s * tn * (double)((M + rows - 1) / rows);
            const double full = floor(tiles / (2.0 * cu)), rest = tiles - full * 2.0 * cu, fill = rest / cu;
            const double two = rows == 128 ? (ragged ? 2800.0 : 2860.0) : rows == 64 ? 1800.0 : 1050.0;
            const double one = rows == 128 ? (ragged ? 1070.0 + 375.0 * fill : 1120.0) : rows == 64 ? 780.0 + 170.0 * fill : 520.0 + 220.0 * fill;
            const double last = rows == 128 && ragged ? 2060.0 + 740.0 * (fill - 1.0) : two;
            const double slab = two * full + (fill > 1.0 ? last : fill > 0.0 ? one : 0.0);
            double ns = 5300.0 + kp / 32.0 * slab;
            if (s > 1) ns += 4000.0 + (double)nprob * s * (double)M * (double)N * 8.0 / 4.0e3;
            if (ns < 0.97 * best_ns) { best = {rows, s}; best_ns = ns; }
        }
    }
    return best;
}

int gemm_f32_tile_rows(int M, int N, int K, int nprob) { return f32_pick(M, N, K, nprob, 1).rows; }

// the large-tile kernel, or the general one for the shapes it does not take
static zo2_status launch_large(const GemmArgs& a, int dtype, hipStream_t st) {
    if (gemm256_applicable(a, dtype)) return gemm_launch_256(a, dtype, st);
    if (dtype == ZO2_BF16) return launch_mfma<bf16_t>(a, st);
    if (dtype == ZO2_F16) return launch_mfma<f16_t>(a, st);
    set_op_error("gemm: dtype %d is not a compute dtype", dtype);
    return ZO2_EINVAL;
}

// what every kernel takes for granted: 16-byte rows of operands that are there
static zo2_status check_operands(const GemmArgs& a) {
    ZO2_OP_CHECK(a.K % 8 == 0, ZO2_EINVAL, "gemm: K = %d is not a multiple of 8", a.K);
    ZO2_OP_CHECK(a.ldx >= a.K && a.ldw >= a.K && a.ldy >= a.N, ZO2_EINVAL, "gemm: leading dimension too small");
    ZO2_OP_CHECK(a.ldx % 8 == 0 && a.ldw % 8 == 0, ZO2_EINVAL, "gemm: ldx / ldw must be multiples of 8");
    ZO2_OP_CHECK(a.nprob >= 1 && a.nprob <= GemmArgs::kMaxProblems, ZO2_EINVAL, "gemm: %d problems", a.nprob);
    for (int i = 0; i < a.nprob; ++i) {
        ZO2_OP_CHECK(a.p[i].X && a.p[i].W && (a.p[i].Y || a.ce_mode), ZO2_EINVAL, "gemm: NULL operand in problem %d", i);
        ZO2_OP_CHECK(((uintptr_t)a.p[i].X & 15) == 0 && ((uintptr_t)a.p[i].W & 15) == 0, ZO2_EINVAL,
                     "gemm: operands must be 16-byte aligned");
    }
    return ZO2_OK;
}

zo2_status gemm_launch(const GemmArgs& a, int dtype, hipStream_t st, int of_rows) {
    ZO2_OP_CHECK(a.M >= 0 && a.N >= 0 && a.K > 0, ZO2_EINVAL, "gemm: bad shape %d x %d x %d", a.M, a.N, a.K);
    if (a.M == 0 || a.N == 0 || a.nprob == 0) return ZO2_OK;
    const int all_rows = std::max(a.M, of_rows);
    { const zo2_status s = check_operands(a); if (s != ZO2_OK) return s; }
    // cross-entropy mode has no output matrix (Y may be NULL): only the 256 x 256 kernel implements it, so every
    // other path must be refused before anything is launched
    ZO2_OP_CHECK(!a.ce_mode || (dtype != ZO2_F32 && gemm256_applicable(a, dtype)), ZO2_EINVAL,
                 "gemm: cross-entropy mode needs the large-tile kernel (16-bit inputs, K %% 128 == 0, N >= 256, N %% 4 == 0, 256 rows within 2 GiB)");
    if (dtype == ZO2_F32) {
        ZO2_OP_CHECK(a.out_f32, ZO2_EINVAL, "gemm: the float32 kernel writes float32 output");
        GemmArgs f = a;
        f.kpiece = a.K;
        return gemm_launch_f32(f, 1, f32_pick(all_rows, a.N, a.K, a.nprob, 1).rows, st);
    }
    GemmArgs m = a;
    m.M = all_rows;
    const GemmChoice k = gemm_choose(m, dtype, 0);
    if (!k.rows) return launch_large(a, dtype, st);
    m.M = a.M;
    m.kpiece = a.K;
    return gemm_launch_mid(m, dtype, k.rows, 1, st);
}


// ---------------------------------------------------------------------------------------- split-k
// With few rows per stream a projection has a handful of tiles for 256 compute units (attention output and FC2 of a
// d_model 2048 block at 512 tokens per stream: 64 tiles of 128 rows).  The k range is then cut into 2 or 4 pieces that
// run as problems of their own - the kernels take a list of problems of one shape - and a small second kernel sums a
// problem's pieces in piece order and finishes the values.
template <typename T, typename OutT>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const GemmArgs a, const float* __restrict__ part, int splits) {
    const int n4 = a.N >> 2;
    const size_t gi = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gi >= (size_t)a.M * n4) return;
    const GemmProblem p = a.p[blockIdx.y];
    const int m = (int)(gi / n4), n = (int)(gi % n4) * 4;
    const size_t plane = (size_t)a.M * a.N;
    const float* src = part + (size_t)blockIdx.y * splits * plane + (size_t)m * a.N + n;
    v4f_t sum = *reinterpret_cast<const v4f_t*>(src);
    for (int k0 = 1; k0 < splits; k0 += 8) {
        v4f_t t[8];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (k0 + k < splits) t[k] = *reinterpret_cast<const v4f_t*>(src + (size_t)(k0 + k) * plane);
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (k0 + k < splits) sum += t[k];
    }
    const T* bias = reinterpret_cast<const T*>(p.bias);
    OutT* Y = reinterpret_cast<OutT*>(p.Y);
    const size_t o = (size_t)m * a.ldy + n;
    Vec<OutT, 4> out;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float y = (sum[e] + (bias ? Fmt<T>::load(bias[n + e]) : 0.f)) * p.out_scale;
        if (a.relu) y = fmaxf(y, 0.f);
        if (p.residual) y += p.residual[o + e];
        out.v[e] = Fmt<OutT>::store(y);
    }
    store_vec<OutT, 4>(Y + o, out);
}

// Pieces per problem: a small cost model of the large kernel.  A launch of t tiles runs in ceil(t / CUs) rounds; a tile
// costs its k range plus a fixed part (prologue and epilogue, about 256 k), a 128-row tile two thirds of a 256-row one;
// split pieces add the write and the re-read of their float32 partial sums.  One k of a 256 x 256 tile is 26.75 ns at the
// rate the kernel reaches (1.25 PFLOP/s over 256 compute units), the partial sums move at about 4 TB/s.  A split, and a
// further doubling, must win 8 % to be taken (measured launches agree with the model to a few percent).  Splits are
// taken where tiles are few (128 - 1024 tokens per stream at d_model 2048) and where the tile count sits badly on the
// rounds with a long k (FC2 of the OPT-13B shape at 2048 tokens: 320 tiles, 1.25 rounds).
static double large_tile_ns(int M, int N, int K, int nprob, int s) {
    const double cu = (double)device_cu_count(), tn = (double)((N + 255) / 256), kk = (double)K / s + 256.0;
    const double t256 = nprob * s * (double)((M + 255) / 256) * tn, t128 = nprob * s * (double)((M + 127) / 128) * tn;
    double ns = ceil(t128 / cu) * kk * (2.0 / 3.0);
    if (M >= 256) ns = fmin(ns, ceil(t256 / cu) * kk);
    ns *= 26.75;
    if (s > 1) ns += (double)nprob * s * (double)M * (double)N * 8.0 / 4.0e3;      // bytes / (4e12 B/s) in ns
    return ns;
}
int gemm_pick_splits(int M, int N, int K, int nprob, int dtype) {
    if (!(dtype == ZO2_BF16 || dtype == ZO2_F16) || M <= 0 || N <= 0 || N % 4 != 0 || nprob <= 0) return 1;
    auto launch_ns = [&](int s) { return large_tile_ns(M, N, K, nprob, s); };
    int best = 1;
    double best_ns = launch_ns(1);
    for (int s = 2; s <= 4; s *= 2) {
        if (K % (s * 128) != 0 || K / s < 512 || nprob * s > GemmArgs::kMaxPieces) break;
        const double ns = launch_ns(s);
        if (ns < 0.92 * best_ns) { best = s; best_ns = ns; }
    }
    return best;
}

size_t gemm_splitk_workspace_bytes(int M, int N, int nprob, int splits) {
    return splits > 1 ? (size_t)nprob * splits * (size_t)M * N * sizeof(float) : 0;
}

template <typename T>
static void launch_splitk_reduce(const GemmArgs& a, const float* part, int splits, hipStream_t st) {
    const size_t work = (size_t)a.M * (a.N / 4);
    const dim3 grid((unsigned)((work + 255) / 256), a.nprob), block(256);
    if (a.out_f32) hipLaunchKernelGGL((splitk_reduce_kernel<T, float>), grid, block, 0, st, a, part, splits);
    else hipLaunchKernelGGL((splitk_reduce_kernel<T, T>), grid, block, 0, st, a, part, splits);
}

int gemm_f32_pick_splits(int M, int N, int K, int nprob, size_t workspace_bytes) {
    if (M <= 0 || N <= 0 || N % 4 != 0 || K < 128 || nprob <= 0) return 1;
    const size_t per_piece = (size_t)nprob * M * N * sizeof(float);
    return f32_pick(M, N, K, nprob, (int)std::min<size_t>(32, std::max<size_t>(1, workspace_bytes / per_piece))).splits;
}

// float32: the pieces are one more grid dimension of the kernel
zo2_status gemm_launch_f32_splitk(const GemmArgs& a, int splits, void* workspace, size_t workspace_bytes, hipStream_t st, bool sum) {
    if (splits <= 1) return gemm_launch(a, ZO2_F32, st);
    ZO2_OP_CHECK(a.out_f32 && !a.ce_mode && a.M > 0 && a.N > 0 && a.N % 4 == 0 && a.ldy % 4 == 0 && a.K % 8 == 0 && a.ldx % 4 == 0 && a.ldw % 4 == 0,
                 ZO2_EINVAL, "gemm split-k: bad shape %d x %d x %d", a.M, a.N, a.K);
    const size_t plane = (size_t)a.M * a.N, need = plane * a.nprob * splits * sizeof(float);
    ZO2_OP_CHECK(workspace && ((uintptr_t)workspace & 15) == 0 && workspace_bytes >= need, ZO2_EINVAL,
                 "gemm split-k: workspace of %zu bytes needed (16-byte aligned)", need);
    GemmArgs e = a;
    e.kpiece = ((a.K + splits - 1) / splits + 31) / 32 * 32;
    ZO2_OP_CHECK((a.K + e.kpiece - 1) / e.kpiece == splits, ZO2_EINVAL, "gemm split-k: %d pieces of K = %d", splits, a.K);
    e.ldy = a.N; e.relu = 0;
    float* part = reinterpret_cast<float*>(workspace);
    for (int i = 0; i < a.nprob; ++i) {
        ZO2_OP_CHECK(a.p[i].X && a.p[i].W && a.p[i].Y && (((uintptr_t)a.p[i].X | (uintptr_t)a.p[i].W | (uintptr_t)a.p[i].Y | (uintptr_t)a.p[i].residual) & 15) == 0,
                     ZO2_EINVAL, "gemm split-k: operands must be 16-byte aligned");
        e.p[i].bias = nullptr; e.p[i].residual = nullptr; e.p[i].out_scale = 1.0f;
        e.p[i].Y = part + (size_t)i * splits * plane;
    }
    zo2_status s = gemm_launch_f32(e, splits, f32_pick(a.M, a.N, e.kpiece, a.nprob * splits, 1).rows, st);
    if (s != ZO2_OK || !sum) return s;
    launch_splitk_reduce<float>(a, part, splits, st);
    ZO2_HIP_LAUNCH_CHECK();
    return ZO2_OK;
}

// Kernel, tile height and pieces of a block projection.  The 128 x 128 kernel's launch: 3.5 us, and per round of tiles and slab
// 0.44 us (128 rows) or 0.28 us (64) when the chip is nearly empty, two fifths or a third more when every compute unit has a tile;
// pieces add their partial sums at 4 TB/s and 4 us for the second launch.  The large kernel's launch: 3 us, and per round 4 us and
// 25.5 ns a k for 256-row tiles.  Measured inside steps, second launch included, large -> this kernel (us):
// d 2048, 185 rows: QKV 30.7 -> 20.5, output 20.9 -> 14.1 (64-row tiles), FC1 30.9 -> 22.2, FC2 38.6 -> 26.2 (2 pieces); 512 rows:
// output 27.4 -> 16.2, but FC1 37.2 against 44.5 (two rounds).
// Where the large kernel cannot run (K a multiple of 64 but not of 128) the other choice is the general one: two workgroups per compute
// unit, so twice the tiles per round, and 0.8 PFLOP/s once rounds are full (this kernel 0.7).  Its launch: 5.6 us and 0.9 us a slab with
// up to one tile per compute unit, beyond that 3 us and per round of 512 tiles 3.8 us and 1.25 a slab; several rounds of this kernel are
// told apart with 4.5 us a round (3 with 64 rows) and correspondingly less a slab.  General -> this kernel (us): K 832, N 832: 512 rows 16.6 ->
// 8.1, 4096 21.6 -> 15.2, 8192 25.9 against 27.8; K 704, N 2816: 1024 16.5 -> 11.8, 4096 36.6 against 38.0, 7504 57.9 against 70.7; K 1728, N
// 6080: 512 29.7 -> 20.5, 2048 66.9 -> 61.7, 8192 225 against 247.  The choice is the faster one or within 4 % of it in 90 launches.
// Tiles of 256 rows are for the launches of several directions at once (gemm_launch_groups), which have tiles for two rounds of 128 rows: the
// wavefronts of a compute unit then ask for three quarters of the bytes per product.  Eight problems of 512 rows, d 2048, in a step: FC2
// (K 8192) 161 -> 136 us, output 67 -> 54; a step of 4 x 128 tokens and four directions, 8 blocks, 7550 -> 7294.  Where k is no multiple of 128 a
// round has its fixed 4.5 us there too; rounds of four directions, tiles of up to 128 rows -> of up to 256, us: d 1728, 4 blocks, 2 x 128 tokens 3435 -> 3273, d 1088,
// 2 x 250 2976 -> 2805, d 832, 6 blocks, 200 1693 -> 1631; with up to 128 tokens they stay on the lower ones (d 1344, 64 tokens 1797, on 256 rows 1902).
static double general_ns(double tiles, double slabs) {
    const double cu = (double)device_cu_count();
    return tiles <= cu ? 5600.0 + 900.0 * slabs : 3000.0 + ceil(tiles / (2.0 * cu)) * (3800.0 + 1250.0 * slabs);
}
static double mid_ns(int rows, double tiles, int kp, bool large) {
    const double cu = (double)device_cu_count(), rounds = ceil(tiles / cu), fill = tiles / (rounds * cu);
    if (!large && rounds > 1.0)
        return 3000.0 + rounds * (rows == 256 ? 4500.0 + (kp / 64) * (780.0 + 260.0 * fill) : rows == 128 ? 4500.0 + (kp / 64) * (400.0 + 250.0 * fill) : 3000.0 + (kp / 64) * (240.0 + 120.0 * fill));
    if (rows == 256) return 3500.0 + rounds * (kp / 64) * (780.0 + 260.0 * fill);
    return 3500.0 + rounds * (kp / 64) * (rows == 128 ? 440.0 + 180.0 * fill : 280.0 + 90.0 * fill);
}
GemmChoice gemm_choose(const GemmArgs& a, int dtype, size_t workspace_bytes) {
    GemmChoice best = {0, gemm_pick_splits(a.M, a.N, a.K, a.nprob, dtype)};
    if (gemm_splitk_workspace_bytes(a.M, a.N, a.nprob, best.splits) > workspace_bytes) best.splits = 1;
    // Matrices of up to 2^19 elements (d 512 and less) stay with the older kernels, for the order of their sums and not for speed: in
    // models this small three updates at a learning rate of 1e-2 make percents of the loss of a late digit (evaluations after them lie
    // 0.1 - 9.7 % from the oracle over six draws of the weights, in the older order), and runs of that kind are held to 2 %.  What it
    // costs, large -> this kernel: launches of 100 - 1024 rows 8 - 19 -> 5 - 14 us; steps of d 256, ffn 2048, 8 blocks: 100 tokens 660 -> 530
    // us, 400 695 -> 622; d 512, ffn 1024, 12 blocks: 100 1063 -> 806, 1024 1395 -> 1202.
    if (a.large_only || gemm256_is_forced() || !gemm_mid_applicable(a, dtype) || (int64_t)a.N * a.K <= 1 << 19) return best;
    const double cu = (double)device_cu_count(), tn = (double)((a.N + 127) / 128);
    const bool large = gemm256_applicable(a, dtype);
    double best_ns = general_ns(a.nprob * tn * (double)((a.M + 127) / 128), (double)(a.K / 64));
    if (large) {
        best_ns = 1e30;
        for (int s = 1; s <= 4; s *= 2) {
            const size_t bytes = gemm_splitk_workspace_bytes(a.M, a.N, a.nprob, s);
            if (s > 1 && (a.K % (s * 128) != 0 || a.K / s < 512 || a.nprob * s > GemmArgs::kMaxPieces || bytes > workspace_bytes)) break;
            double ns = 1e30;
            for (int rows = 128; rows <= 256; rows += 64) {
                const double tiles = (double)a.nprob * s * (double)((a.N + 255) / 256) * (double)((a.M + rows - 1) / rows);
                ns = fmin(ns, 3000.0 + ceil(tiles / cu) * gemm256_tile_cost(rows) * (25.5 * a.K / s + 4000.0));
            }
            if (s > 1) ns += 4000.0 + 2.0 * (double)bytes / 4.0e3;
            if (ns < 0.97 * best_ns) { best = {0, s}; best_ns = ns; }
        }
    }
    for (int rows = 128; rows >= 64; rows -= 64)
        for (int s = 1; s <= 8; ++s) {
            const int kp = ((a.K + s - 1) / s + 63) / 64 * 64;
            const size_t bytes = (size_t)a.nprob * s * a.M * a.N * sizeof(float);
            if (s > 1 && (kp < 256 || (a.K + kp - 1) / kp != s || bytes > workspace_bytes)) continue;
            const double tiles = (double)a.nprob * s * tn * (double)((a.M + rows - 1) / rows);
            if (tiles >= (double)(1 << 22)) continue;              // the grid's limit
            double ns = mid_ns(rows, tiles, kp, large);
            if (s > 1) ns += 4000.0 + 2.0 * (double)bytes / 4.0e3;
            if (ns < 0.95 * best_ns) { best = {rows, s}; best_ns = ns; }
        }
    return best;
}

// The 128 x 128 kernel with its k range in pieces
zo2_status gemm_launch_mid_splitk(const GemmArgs& a, int dtype, int rows, int splits, void* workspace, size_t workspace_bytes, hipStream_t st, bool sum) {
    ZO2_OP_CHECK(a.M > 0 && a.N > 0 && a.K > 0, ZO2_EINVAL, "gemm: bad shape %d x %d x %d", a.M, a.N, a.K);
    { const zo2_status s = check_operands(a); if (s != ZO2_OK) return s; }
    GemmArgs e = a;
    e.kpiece = splits > 1 ? ((a.K + splits - 1) / splits + 63) / 64 * 64 : a.K;
    if (splits <= 1) return gemm_launch_mid(e, dtype, rows, 1, st);
    const size_t plane = (size_t)a.M * a.N, need = plane * a.nprob * splits * sizeof(float);
    ZO2_OP_CHECK(gemm_mid_applicable(a, dtype) && workspace && ((uintptr_t)workspace & 15) == 0 && workspace_bytes >= need, ZO2_EINVAL,
                 "gemm split-k: workspace of %zu bytes needed (16-byte aligned)", need);
    e.ldy = a.N; e.relu = 0; e.out_f32 = 1;
    float* part = reinterpret_cast<float*>(workspace);
    for (int i = 0; i < a.nprob; ++i) {
        e.p[i].bias = nullptr; e.p[i].residual = nullptr; e.p[i].out_scale = 1.0f;
        e.p[i].Y = part + (size_t)i * splits * plane;
    }
    zo2_status s = gemm_launch_mid(e, dtype, rows, splits, st);
    if (s != ZO2_OK) return s;
    if (!sum) return ZO2_OK;
    if (dtype == ZO2_BF16) launch_splitk_reduce<bf16_t>(a, part, splits, st);
    else launch_splitk_reduce<f16_t>(a, part, splits, st);
    ZO2_HIP_LAUNCH_CHECK();
    return ZO2_OK;
}

zo2_status gemm_launch_splitk(const GemmArgs& a, int dtype, int splits, void* workspace, size_t workspace_bytes, hipStream_t st, bool sum) {
    if (splits <= 1) return gemm_launch(a, dtype, st);
    ZO2_OP_CHECK(dtype == ZO2_BF16 || dtype == ZO2_F16, ZO2_EINVAL, "gemm split-k: 16-bit compute formats only");
    ZO2_OP_CHECK(!a.ce_mode, ZO2_EINVAL, "gemm split-k: not with the cross-entropy epilogue");
    ZO2_OP_CHECK(splits == 2 || splits == 4, ZO2_EINVAL, "gemm split-k: %d pieces (2 or 4)", splits);
    ZO2_OP_CHECK(a.M > 0 && a.N > 0 && a.N % 4 == 0 && a.ldy % 4 == 0 && a.K % (splits * 8) == 0, ZO2_EINVAL,
                 "gemm split-k: bad shape %d x %d x %d for %d pieces", a.M, a.N, a.K, splits);
    ZO2_OP_CHECK(a.nprob >= 1 && a.nprob * splits <= GemmArgs::kMaxProblems, ZO2_EINVAL, "gemm split-k: %d problems x %d pieces", a.nprob, splits);
    const size_t need = gemm_splitk_workspace_bytes(a.M, a.N, a.nprob, splits);
    ZO2_OP_CHECK(workspace && ((uintptr_t)workspace & 15) == 0 && workspace_bytes >= need, ZO2_EINVAL,
                 "gemm split-k: workspace of %zu bytes needed (16-byte aligned)", need);
    const size_t osz = a.out_f32 ? 4 : 2;
    for (int i = 0; i < a.nprob; ++i) {
        ZO2_OP_CHECK(a.p[i].X && a.p[i].W && a.p[i].Y, ZO2_EINVAL, "gemm split-k: NULL operand in problem %d", i);
        ZO2_OP_CHECK(((uintptr_t)a.p[i].Y & (4 * osz - 1)) == 0 && ((uintptr_t)a.p[i].residual & 15) == 0 && ((uintptr_t)a.p[i].bias & 7) == 0,
                     ZO2_EINVAL, "gemm split-k: output, residual and bias must be aligned to 4 elements");
        ZO2_OP_CHECK(!a.p[i].residual || a.out_f32, ZO2_EINVAL, "gemm split-k: a residual needs float32 output");
    }
    float* part = reinterpret_cast<float*>(workspace);
    const size_t plane = (size_t)a.M * a.N, esz = 2;
    const int kp = a.K / splits;
    GemmArgs e;
    memset(&e, 0, sizeof(e));
    e.M = a.M; e.N = a.N; e.K = kp; e.ldx = a.ldx; e.ldw = a.ldw; e.ldy = a.N; e.relu = 0; e.out_f32 = 1; e.nprob = a.nprob * splits;
    for (int i = 0; i < a.nprob; ++i)
        for (int k = 0; k < splits; ++k) {
            GemmProblem& q = e.p[i * splits + k];
            q.X = reinterpret_cast<const char*>(a.p[i].X) + (size_t)k * kp * esz;
            q.W = reinterpret_cast<const char*>(a.p[i].W) + (size_t)k * kp * esz;
            q.Y = part + ((size_t)i * splits + k) * plane;
            q.out_scale = 1.0f;
        }
    zo2_status s = check_operands(e);
    if (s == ZO2_OK) s = launch_large(e, dtype, st);
    if (s != ZO2_OK) return s;
    if (!sum) return ZO2_OK;
    if (dtype == ZO2_BF16) launch_splitk_reduce<bf16_t>(a, part, splits, st);
    else launch_splitk_reduce<f16_t>(a, part, splits, st);
    ZO2_HIP_LAUNCH_CHECK();
    return ZO2_OK;
}

int gemm_groups_rows(const GemmArgs& a, int dtype, GemmChoice k) {
    const int kp = k.splits > 1 ? ((a.K + k.splits - 1) / k.splits + 63) / 64 * 64 : a.K;
    const double n = (double)a.nprob * k.splits * (double)((a.N + 127) / 128);
    const bool large = gemm256_applicable(a, dtype);
    int rows = 64;
    for (int h = 128; h <= (dtype == ZO2_BF16 ? 256 : 128); h *= 2)      // (directions go together in bfloat16)
        if (mid_ns(h, n * ((a.M + h - 1) / h), kp, large) <= mid_ns(rows, n * ((a.M + rows - 1) / rows), kp, large)) rows = h;
    return rows;
}
zo2_status gemm_launch_groups(const GemmArgs& a, int dtype, GemmChoice k, int groups, void* workspace, size_t workspace_bytes, hipStream_t st) {
    ZO2_OP_CHECK(groups >= 1 && a.nprob >= groups && a.nprob % groups == 0 && a.nprob <= GemmArgs::kMaxProblems, ZO2_EINVAL, "gemm: %d problems in %d groups", a.nprob, groups);
    if (k.rows) return gemm_launch_mid_splitk(a, dtype, gemm_groups_rows(a, dtype, k), k.splits, workspace, workspace_bytes, st);
    if (k.splits <= 1) {
        { const zo2_status s = check_operands(a); if (s != ZO2_OK) return s; }
        return launch_large(a, dtype, st);
    }
    // as many groups at a time as the list of problems holds pieces of
    const int each = a.nprob / groups, at_once = std::max(1, std::min(groups, GemmArgs::kMaxProblems / (each * k.splits)));
    for (int g0 = 0; g0 < groups; g0 += at_once) {
        GemmArgs e = a;
        e.nprob = each * std::min(at_once, groups - g0);
        for (int i = 0; i < e.nprob; ++i) e.p[i] = a.p[g0 * each + i];
        const zo2_status s = gemm_launch_splitk(e, dtype, k.splits, workspace, workspace_bytes, st);
        if (s != ZO2_OK) return s;
    }
    return ZO2_OK;
}

}  // namespace zo2
