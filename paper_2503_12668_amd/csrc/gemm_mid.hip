// 16-bit projections with a few hundred rows per stream: 128 x 128 x 64 (64 x 128 x 64, 256 x 128 x 64) block tiles, eight
// wavefronts, a ring of LDS stages filled by direct-to-LDS loads.
//
// With so few rows a launch is a handful of k-slabs per compute unit, bound by the bytes a compute unit can have under way
// (about 64 KB, whatever the ring's depth: weights from HBM and activations from L2 alike, 46 - 50 GB/s a unit) and by its
// first and last microseconds, not by the matrix cores: the large tiles of gemm256.hip have too few tiles (or pieces of
// k whose partial sums are written and read back).  Here the tile is small enough that the launch fills the chip with little
// or no splitting, and a ring of four slabs keeps three of them under way (five and six are no faster, three cost 10 % on
// weights from HBM).  A wavefront owns
// 64 x 64 of the tile (32 x 64 of the lower one, 128 x 64 of the higher) for one half of each slab's k - two wavefronts per SIMD, no more LDS reads
// than four would make - and the two halves' sums meet in LDS at the end.
//
// Tiles of 256 rows (bfloat16, a ring of three slabs) are for launches with many of them: 1.04 us a slab with a tile on every compute unit where two
// tiles of 128 rows take 1.24, by 48 KB of loads in place of 64.  A sum has the same order at every height.
//
// Slab layout: rows of 8 chunks of 16 bytes, chunk kc of row m at position kc ^ ((m >> 1) & 7); a direct-to-LDS load lands
// lane i's 16 bytes at offset 16 i, so the permutation is applied to the address a lane fetches from.
#include <type_traits>

#include "gemm.h"

namespace zo2 {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float v4f_t __attribute__((ext_vector_type(4)));
typedef uint32_t v4u_t __attribute__((ext_vector_type(4)));

template <typename T> struct MidMfma;
template <> struct MidMfma<bf16_t> {
    static __device__ __forceinline__ f32x16_t run(v4u_t a, v4u_t b, f32x16_t c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
    }
};
template <> struct MidMfma<f16_t> {
    static __device__ __forceinline__ f32x16_t run(v4u_t a, v4u_t b, f32x16_t c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
    }
};

static constexpr int kMidBN = 128, kMidBK = 64;
template <int BM> struct MidTile {
    static constexpr int kStage = (BM + kMidBN) * kMidBK * 2;      // 48 KB / 32 KB / 24 KB
    static constexpr int kStages = BM == 256 ? 3 : 4;
    static constexpr int kLds = kStage * kStages;                  // 144 KB / 128 KB / 96 KB
};

// source address = wave-uniform base + per-lane 32-bit byte offset
__device__ __forceinline__ void mid_load_to_lds(const void* sbase, uint32_t voff, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds_base), "v"(voff), "s"(sbase) : "memory");
}
__device__ __forceinline__ void mid_load_to_lds(const void* sbase, int64_t off, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds_base), "v"((const char*)sbase + off) : "memory");
}
__device__ __forceinline__ const char* mid_uniform(const void* p) {      // a wave-uniform pointer into scalar registers
    const uint64_t v = (uint64_t)(uintptr_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (const char*)(uintptr_t)(((uint64_t)hi << 32) | lo);
}

// All loads of this wavefront but those of the `ahead` youngest slabs (LPW loads each) have landed.
template <int LPW, int AHEAD>
__device__ __forceinline__ void mid_wait(int ahead) {
    if constexpr (AHEAD == 0) {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    } else {
        if (ahead >= AHEAD) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"(AHEAD * LPW) : "memory");
        else mid_wait<LPW, AHEAD - 1>(ahead);
    }
}

template <typename T, typename OutT, int BM, bool FAR>          // FAR: rows lie too far apart for 32-bit offsets inside a tile
__global__ __launch_bounds__(512, 2) void gemm_mid_kernel(const GemmArgs a, int splits) {
    constexpr int KC = kMidBK / 8, TM = BM / 64, TN = 2;           // 32 x 32 MFMA tiles per wavefront: TM x 2
    constexpr int NST = MidTile<BM>::kStages, STAGE = MidTile<BM>::kStage;
    constexpr int XL = BM / 8 / 8, WL = kMidBN / 8 / 8, LPW = XL + WL;      // direct-to-LDS loads (8 rows each) per wavefront and slab
    extern __shared__ __attribute__((aligned(1024))) char smem[];

    // Workgroup ids go round robin over the 8 XCDs; each takes a contiguous run of the list (rows fastest, then columns,
    // pieces of k, problems), so that the row tiles of one panel of W are read through one L2.
    const int nblk = (int)gridDim.x, xcd = (int)(blockIdx.x & 7), in_xcd = (int)(blockIdx.x >> 3);
    int id = xcd * (nblk >> 3) + min(xcd, nblk & 7) + in_xcd;
    const int tiles_m = (a.M + BM - 1) / BM, tiles_n = (a.N + kMidBN - 1) / kMidBN;
    const int m0 = (id % tiles_m) * BM; id /= tiles_m;
    const int n0 = (id % tiles_n) * kMidBN; id /= tiles_n;
    const int piece = id % splits, prob = id / splits;
    const GemmProblem p = a.p[prob];
    const int k_first = piece * a.kpiece, nk = min(a.K - k_first, a.kpiece) / kMidBK;

    const int lane = threadIdx.x & 63, r = lane & 31, kh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int half = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;

    // this lane's sources: load t of the wavefront brings 8 rows (lane -> row lane / 8, position lane % 8); rows past the end of
    // a matrix repeat its last one, their products are never stored
    const char* base_x = mid_uniform(reinterpret_cast<const T*>(p.X) + (size_t)m0 * a.ldx + k_first);
    const char* base_w = mid_uniform(reinterpret_cast<const T*>(p.W) + (size_t)n0 * a.ldw + k_first);
    using Offset = std::conditional_t<FAR, int64_t, uint32_t>;
    Offset gx[XL], gw[WL];
    const int lrow = lane >> 3;
#pragma unroll
    for (int t = 0; t < XL; ++t) {
        const int row = (wave * XL + t) * 8 + lrow;
        gx[t] = (Offset)(min(row, a.M - 1 - m0) * a.ldx + ((lane & 7) ^ ((row >> 1) & 7)) * 8) * 2;
    }
#pragma unroll
    for (int t = 0; t < WL; ++t) {
        const int row = (wave * WL + t) * 8 + lrow;
        gw[t] = (Offset)(min(row, a.N - 1 - n0) * a.ldw + ((lane & 7) ^ ((row >> 1) & 7)) * 8) * 2;
    }
    auto issue_one = [&](int t, int kt, int stage) {               // load t of slab kt: weights first
        const uint32_t at = lds0 + (uint32_t)stage * STAGE;
        const size_t k = (size_t)kt * (kMidBK * 2);
        if (t < WL) mid_load_to_lds(base_w + k, gw[t < WL ? t : 0], at + BM * 128 + (wave * WL + t) * 1024);
        else mid_load_to_lds(base_x + k, gx[t < WL ? 0 : t - WL], at + (wave * XL + t - WL) * 1024);
    };
    auto issue = [&](int kt, int stage) {
#pragma unroll
        for (int t = 0; t < LPW; ++t) issue_one(t, kt, stage);
    };

    f32x16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    const int xrow = wm * (BM / 2) + r, wrow = wn * 64 + r;
    uint32_t off[2];                       // this lane's chunk of a row at the wavefront's two k-steps of a slab
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) off[ks] = (uint32_t)((((half * 2 + ks) * 2 + kh) ^ ((r >> 1) & 7)) * 16);
    // A wavefront holds its fragments of slab kt in registers when it reaches the barrier of iteration kt; behind it slab kt's
    // stage is refilled with slab kt + NST, and the fragments of slab kt + 1 are read under the MFMAs of slab kt (read only when
    // they were due, all wavefronts waited for LDS at the same moment: 2.5 times the MFMAs' own time per slab).
    struct Frag { v4u_t x[2][TM], w[2][TN]; } f0, f1;
    auto read = [&](Frag& f, int stage) {
        const char* xs = smem + stage * STAGE + xrow * 128;
        const char* ws = smem + stage * STAGE + BM * 128 + wrow * 128;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
            for (int j = 0; j < TN; ++j) f.w[ks][j] = *reinterpret_cast<const v4u_t*>(ws + j * 4096 + off[ks]);
#pragma unroll
            for (int i = 0; i < TM; ++i) f.x[ks][i] = *reinterpret_cast<const v4u_t*>(xs + i * 4096 + off[ks]);
        }
    };
    int stage = 0;
    // The wavefront's loads and LDS reads are dealt out between its MFMAs, which run on while it issues them.  (All loads ahead of the
    // MFMAs, the wavefronts queued for the one address unit behind the barrier with the matrix cores idle: a slab took the sum
    // of the time of its loads and of its MFMAs, 0.29 + 0.29 us, not the larger.  185 rows, weights in cache: N 2048, K 8192, two
    // problems 69.6 -> 49.3 us, N 2048, K 2048, six 25.2 -> 20.2, N 8192, K 2048, two 27.1 -> 22.5; from HBM 70.8 -> 58.4, 27.1 -> 24.9, 30.3 -> 27.9.)
    auto step = [&](int kt, const Frag& cur, Frag& next) {
        mid_wait<LPW, NST - 2>(max(0, min(NST - 2, nk - 2 - kt)));      // slab kt + 1 has landed
        __syncthreads();
        const int refill = stage;
        const bool more = kt + NST < nk;
        stage = stage == NST - 1 ? 0 : stage + 1;
        const char* xs = smem + stage * STAGE + xrow * 128;             // (past the last slab: bytes nobody uses)
        const char* ws = smem + stage * STAGE + BM * 128 + wrow * 128;
        // weights first: a lane ends with one row of the output and runs of four consecutive columns
#pragma unroll
        for (int u = 0; u < 2 * TM * TN; ++u) {
            const int ks = u / (TM * TN), i = u / TN % TM, j = u % TN;
            acc[i][j] = MidMfma<T>::run(cur.w[ks][j], cur.x[ks][i], acc[i][j]);
            __builtin_amdgcn_sched_barrier(0);
            // the next slab's fragments: TM + TN per k-step, under the first half of the MFMAs
            constexpr int FR = 2 * (TM + TN), RPM = (FR + TM * TN - 1) / (TM * TN);
#pragma unroll
            for (int q = u * RPM; q < (u + 1) * RPM; ++q)
                if (q < FR) {
                    const int kq = q / (TM + TN), e = q % (TM + TN);
                    if (e < TN) next.w[kq][e < TN ? e : 0] = *reinterpret_cast<const v4u_t*>(ws + e * 4096 + off[kq]);
                    else next.x[kq][e < TN ? 0 : e - TN] = *reinterpret_cast<const v4u_t*>(xs + (e - TN) * 4096 + off[kq]);
                }
            // the retired stage's refill: load t behind MFMA 2 t (128 rows: four loads, eight MFMAs); 64 rows: behind 0, 2 and 3 of four
            if (more && u * LPW % (2 * TM * TN) < LPW) issue_one(u * LPW / (2 * TM * TN), kt + NST, refill);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
#pragma unroll
    for (int s = 0; s < NST; ++s)
        if (s < nk) issue(s, s);
    mid_wait<LPW, NST - 1>(min(NST - 1, nk - 1));
    __syncthreads();
    read(f0, 0);
    for (int kt = 0; kt < nk; kt += 2) {
        step(kt, f0, f1);
        if (kt + 1 < nk) step(kt + 1, f1, f0);
    }

    // The two halves meet: of a pair of wavefronts, the first finishes the left 32 columns of their 64, the second the right.
    __syncthreads();
    {
        float* send = reinterpret_cast<float*>(smem) + (wave * TM * 4 * 64 + lane) * 4;
        const float* recv = reinterpret_cast<const float*>(smem) + ((wave ^ 4) * TM * 4 * 64 + lane) * 4;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int v = 0; v < 16; v += 4) {
                v4f_t x;
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = half ? acc[i][0][v + e] : acc[i][1][v + e];
                *reinterpret_cast<v4f_t*>(send + (i * 4 + v / 4) * 256) = x;
            }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int v = 0; v < 16; v += 4) {
                const v4f_t o = *reinterpret_cast<const v4f_t*>(recv + (i * 4 + v / 4) * 256);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[i][0][v + e] = half ? o[e] + acc[i][1][v + e] : acc[i][0][v + e] + o[e];
            }
    }
    const T* __restrict__ bias = reinterpret_cast<const T*>(p.bias);
    OutT* __restrict__ Y = reinterpret_cast<OutT*>(p.Y);
    const size_t ldy = splits > 1 ? (size_t)a.N : (size_t)a.ldy;
    if (splits > 1) Y += (size_t)piece * a.M * a.N;                // this piece's partial sums (no bias, residual or ReLU, scale 1)
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int m = m0 + wm * (BM / 2) + i * 32 + r;
        if (m >= a.M) continue;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int n = n0 + wn * 64 + half * 32 + 8 * q + 4 * kh;
            if (n >= a.N) continue;                                // N % 4 == 0: a run of four is inside the row or past its end
            float b4[4] = {0.f, 0.f, 0.f, 0.f};
            if (bias) {
                const Vec<T, 4> b = load_vec<T, 4>(bias + n);
#pragma unroll
                for (int e = 0; e < 4; ++e) b4[e] = Fmt<T>::load(b.v[e]) * p.out_scale;      // (acc + b) s = acc s + b s, as in the large kernel
            }
            float y[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) y[e] = __builtin_fmaf(acc[i][0][4 * q + e], p.out_scale, b4[e]);
            if (a.relu) {                                          // (no maximum with -inf in its place: that would lose a NaN)
#pragma unroll
                for (int e = 0; e < 4; ++e) y[e] = fmaxf(y[e], 0.f);
            }
            const size_t o = (size_t)m * ldy + n;
            if (p.residual) {
                const v4f_t rv = *reinterpret_cast<const v4f_t*>(p.residual + o);
#pragma unroll
                for (int e = 0; e < 4; ++e) y[e] += rv[e];
            }
            Vec<OutT, 4> out;
#pragma unroll
            for (int e = 0; e < 4; ++e) out.v[e] = Fmt<OutT>::store(y[e]);
            store_vec<OutT, 4>(Y + o, out);
        }
    }
}

template <typename T, typename OutT, int BM, bool FAR = false>
static zo2_status mid_launch_t(const GemmArgs& a, int splits, hipStream_t st) {
    auto kern = gemm_mid_kernel<T, OutT, BM, FAR>;
    static bool reserved_on[kMaxDevices] = {false};
    bool& reserved = reserved_on[current_device()];
    if (!reserved) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, MidTile<BM>::kLds);
        if (e != hipSuccess) {
            set_op_error("gemm: cannot reserve %d bytes of LDS: %s", MidTile<BM>::kLds, hipGetErrorString(e));
            return ZO2_EHIP;
        }
        reserved = true;
    }
    const int64_t blocks = (int64_t)((a.M + BM - 1) / BM) * ((a.N + kMidBN - 1) / kMidBN) * splits * a.nprob;
    ZO2_OP_CHECK(blocks < (int64_t)1 << 22, ZO2_EINVAL, "gemm: launch too large for the 128 x 128 kernel");
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(512), MidTile<BM>::kLds, st, a, splits);
    ZO2_HIP_LAUNCH_CHECK();
    return ZO2_OK;
}

bool gemm_mid_applicable(const GemmArgs& a, int dtype) {
    if ((dtype != ZO2_BF16 && dtype != ZO2_F16) || a.ce_mode || a.M < 1 || a.K % kMidBK != 0 || a.N % 4 != 0 || a.ldy % 4 != 0) return false;
    const size_t osz = a.out_f32 ? 4 : 2;
    for (int i = 0; i < a.nprob; ++i) {
        if (((uintptr_t)a.p[i].Y & (4 * osz - 1)) != 0 || ((uintptr_t)a.p[i].bias & 7) != 0 || ((uintptr_t)a.p[i].residual & 15) != 0) return false;
        if (a.p[i].residual && !a.out_f32) return false;
    }
    return true;
}

// splits > 1: a.kpiece k per piece (a multiple of 64), p[i].Y = the problem's float32 partial sums, one [M][N] plane per piece
zo2_status gemm_launch_mid(const GemmArgs& a, int dtype, int rows, int splits, hipStream_t st) {
    ZO2_OP_CHECK(gemm_mid_applicable(a, dtype) && (rows == 64 || rows == 128 || (rows == 256 && dtype == ZO2_BF16)) && splits >= 1 && a.kpiece > 0 && a.kpiece % kMidBK == 0 &&
                 (int64_t)a.kpiece * (splits - 1) < a.K && (int64_t)a.kpiece * splits >= a.K && (splits == 1 || a.out_f32),
                 ZO2_EINVAL, "gemm: shape or alignment not supported by the 128 x 128 kernel");
    // rows of 8 MB and more: 64-row tiles with 64-bit addresses (the height does not show in a sum)
    const bool far = a.ldx >= 1 << 22 || a.ldw >= 1 << 22;
#define ZO2_MID(T, OutT)                                                \
    if (far) return mid_launch_t<T, OutT, 64, true>(a, splits, st);     \
    if (rows == 64) return mid_launch_t<T, OutT, 64>(a, splits, st);    \
    if constexpr (std::is_same_v<T, bf16_t>)                            \
        if (rows == 256) return mid_launch_t<T, OutT, 256>(a, splits, st); \
    return mid_launch_t<T, OutT, 128>(a, splits, st)
    if (dtype == ZO2_BF16) {
        if (a.out_f32) { ZO2_MID(bf16_t, float); }
        ZO2_MID(bf16_t, bf16_t);
    }
    if (a.out_f32) { ZO2_MID(f16_t, float); }
    ZO2_MID(f16_t, f16_t);
#undef ZO2_MID
}

}  // namespace zo2
