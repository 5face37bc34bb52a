// float32 projections on the bfloat16 matrix cores: every operand as the sum of three bfloat16 numbers.
//
// A float32 significand has 24 bits, a bfloat16 one 8.  x = hi + mid + lo, each part the rest rounded to nearest, holds every
// bit of an x of 2^-110 or more (the rests are exact in float32; for smaller ones see OddSums), so x w is nine products of
// bfloat16 numbers, each exact in the matrix core's float32.  The six largest are taken.  mid is up to 2^-8 and lo up to 2^-17 of x, just
// above a power of two, so what is left out (mid lo, lo mid, lo lo) is up to 2^-24 of |x w|, as much as a float32 product's
// rounding; over random significands it is 2^-27.5 in the root mean square, a fifth of that rounding, and of random sign.  A
// product by itself is off by up to 2^-23 (2^-25.2 in the root mean square, as in float32), sums are nearer than float32's (below).
// v_mfma_f32_32x32x16_bf16 does 16 k in 32 cycles where v_mfma_f32_32x32x2_f32 needs 512, so six of them still are 2.7 times as fast.  hi hi goes to one accumulator and the five
// small products to another, added at the end: the large sums are rounded once per 16 k (every two k with float32 products).
//
// Measured, float32 products -> this, in us: 2 x 768 rows, d 2048 / ffn 8192: LM head 2468 -> 1633 (128 -> 194 TFLOP/s), FC1 410 ->
// 274, FC2 405 + 16 -> 321, QKV 342 -> 247, output 109 + 16 -> 92; 64 rows, N 24576, K 1024: 46 -> 34; 16 rows, N 8192, K 2048: 55 -> 42.
// Distance from the sums in 64 bits, of the result's norm: K 2048, normal operands 8.1e-7 -> 2.7e-7 (128-row tiles) and 1.9e-7; K 8192, X
// behind a ReLU 1.15e-6 -> 4.9e-7 and 3.3e-7; K 256 2.9e-7 -> 0.9e-7 and 0.7e-7.  (One accumulator for all six products: 7.0e-7, 1.35e-6.)
//
// Two kernels.  gemm_f32_split_kernel, many rows: operands are split once, on their way from registers into LDS, which holds
// three planes.  gemm_f32_ring_kernel, few rows: LDS is a ring of float32 slabs filled by direct-to-LDS loads, and a wavefront
// splits the fragments it reads.  What bounds the first is the matrix cores (and the clock they leave the chip), the second the vector
// ALU, which splits a slab in about the time its loads take.
#include <math.h>

#include <type_traits>

#include "gemm.h"
#include "f32_parts.h"
#include "gemm_f32_index.h"

namespace zo2 {

template <int TM, int TN>
__device__ __forceinline__ bool odd_sums(const f32x16_t (&acc)[TM][TN]) {
    OddSums o;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) o.look(acc[i][j][v]);
    return o.any();
}
// v_mfma_f32_32x32x2_f32: lanes 0..31 supply k = 0, lanes 32..63 k = 1 of a row.  A lane of half h reads k = 8 g + 4 h .. + 3 of its
// row with one load; issue t of group g contracts k = 8 g + t with k = 8 g + 4 + t.  (K is a multiple of 8.)
template <int TM, int TN>
__device__ __forceinline__ void float32_products(const GemmArgs& a, const float* X, const float* W, int m0, int n0, int K, f32x16_t (&acc)[TM][TN]) {
    const int lane = threadIdx.x & 63, r = lane & 31, kh = lane >> 5;
    clear_acc<TM, TN>(acc);
    const float* gx[TM];
    const float* gw[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) gx[i] = X + (size_t)min(m0 + i * 32 + r, a.M - 1) * a.ldx + 4 * kh;
#pragma unroll
    for (int j = 0; j < TN; ++j) gw[j] = W + (size_t)min(n0 + j * 32 + r, a.N - 1) * a.ldw + 4 * kh;
    for (int k = 0; k < K; k += 8) {
        v4f_t fx[TM], fw[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i) fx[i] = *reinterpret_cast<const v4f_t*>(gx[i] + k);
#pragma unroll
        for (int j = 0; j < TN; ++j) fw[j] = *reinterpret_cast<const v4f_t*>(gw[j] + k);
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fw[j][t], fx[i][t], acc[i][j], 0, 0, 0);
    }
}

// Four consecutive columns n .. n + 3 of output row m: in a 32 x 32 MFMA tile a lane holds row m = r (the second operand's row) and the
// columns 8 q + 4 kh + e (the first operand's rows), q = 0 .. 3.
__device__ __forceinline__ void store_run(const GemmArgs& a, const GemmProblem& p, int m, int n, const float acc[4]) {
    if (m >= a.M || n >= a.N) return;
    const float* __restrict__ bias = reinterpret_cast<const float*>(p.bias);
    float* __restrict__ Y = reinterpret_cast<float*>(p.Y);
    if (gridDim.y > 1) Y += (size_t)blockIdx.y * a.M * a.N;       // this piece's partial sums (no bias, scale 1: see gemm_launch_f32_splitk)
    const bool vec_ok = (a.N % 4 == 0) && (a.ldy % 4 == 0) && (((uintptr_t)Y & 15) == 0) &&
                        (!p.residual || ((uintptr_t)p.residual & 15) == 0) && (!bias || ((uintptr_t)bias & 15) == 0);
    const size_t o = (size_t)m * a.ldy + n;
    if (vec_ok) {                          // N % 4 == 0: the run of four is inside the row or entirely past its end
        const v4f_t b4 = bias ? *reinterpret_cast<const v4f_t*>(bias + n) : v4f_t{0.f, 0.f, 0.f, 0.f};
        v4f_t y;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            y[e] = (acc[e] + b4[e]) * p.out_scale;
            if (a.relu) y[e] = fmaxf(y[e], 0.f);
        }
        if (p.residual) y += *reinterpret_cast<const v4f_t*>(p.residual + o);
        *reinterpret_cast<v4f_t*>(Y + o) = y;
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (n + e >= a.N) continue;
            float v = (acc[e] + (bias ? bias[n + e] : 0.f)) * p.out_scale;
            if (a.relu) v = fmaxf(v, 0.f);
            if (p.residual) v += p.residual[o + e];
            Y[o + e] = v;
        }
    }
}

// ---------------------------------------------------------------------------------------
// Many rows: block tile 128 x 128 x 16, four wavefronts (2 x 2) of 64 x 64, two workgroups per compute unit.  LDS holds two
// stages of three planes, rows of 16 bfloat16; 16-byte chunk kc of row m sits at position kc ^ swz(m), so that eight and sixteen
// neighbouring rows at one kc lie in different columns of the banks.
//
// A slab's 24 MFMAs are six groups of four, and everything else is dealt out between the groups: the split of slab kt + 2 into the
// stage that slab kt has just left (its fragments are in registers when the barrier is reached), the fragments of slab kt + 1 - a
// part's registers are refilled as soon as its last product is issued, the high parts, needed throughout, have two sets -
// and the loads of slab kt + 4 into the registers that slab kt + 2 left: two slabs' time to come back.
// ---------------------------------------------------------------------------------------
struct F32Tile {
    static constexpr int BM = 128, BN = 128, BK = 16, kRow = BK * 2;
    static constexpr int kPlane = (BM + BN) * kRow, kStage = 3 * kPlane, kLds = 2 * kStage;      // 48 KB
};

template <bool KTAIL>                  // K is not a multiple of 16: zeros past the end of the rows
__global__ __launch_bounds__(256, 2) void gemm_f32_split_kernel(const GemmArgs a) {
    using Tile = F32Tile;
    constexpr int BM = Tile::BM, BN = Tile::BN, BK = Tile::BK, ROW = Tile::kRow, PLANE = Tile::kPlane, STAGE = Tile::kStage;
    extern __shared__ __attribute__((aligned(1024))) char smem[];

    const GemmProblem p = a.p[blockIdx.z];
    const int tiles_m = (a.M + BM - 1) / BM;
    // workgroup ids go round robin over the 8 XCDs; each takes a contiguous run of tiles, rows fastest, so that the row tiles of
    // one column panel of W are read through one L2
    const int nblk = (int)gridDim.x, xcd = (int)(blockIdx.x & 7), in_xcd = (int)(blockIdx.x >> 3);
    const int tile = xcd * (nblk >> 3) + min(xcd, nblk & 7) + in_xcd;
    const int m0 = (tile % tiles_m) * BM, n0 = (tile / tiles_m) * BN;
    const int k_first = (int)blockIdx.y * a.kpiece, K = min(a.K - k_first, a.kpiece);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1, r = lane & 31, kh = lane >> 5;
    const float* __restrict__ X = reinterpret_cast<const float*>(p.X) + k_first;
    const float* __restrict__ W = reinterpret_cast<const float*>(p.W) + k_first;

    auto swz = [](int m) { return ((m >> 2) ^ (m >> 3)) & 1; };
    // staging plan: chunks of four floats, four to a row of a slab; a thread takes rows tid / 4 and tid / 4 + 64 of either operand
    const int kc4 = (tid & 3) * 4;
    const float* g[4];                 // W, W, X, X
    int l[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int row = tid / 4 + 64 * (c & 1);
        g[c] = (c < 2 ? W + (size_t)min(n0 + row, a.N - 1) * a.ldw : X + (size_t)min(m0 + row, a.M - 1) * a.ldx) + (KTAIL ? 0 : kc4);
        l[c] = ((c < 2 ? BM : 0) + row) * ROW + (((tid & 3) >> 1) ^ swz(row)) * 16 + (tid & 1) * 8;
    }
    const int nk = (K + BK - 1) / BK;
    v4f_t rg[2][4];
    // (a chunk past the end of the row is fetched from the row's start, and zeros are parked: dropped where it is fetched, the
    // wavefront would wait for its loads there; 1024 x 3072 x 776: 58 -> 37 us)
    const int last_at = f32_chunk_at(nk - 1, nk, BK, kc4, K);
    const bool past = KTAIL && !f32_chunk_inside(nk - 1, nk, BK, kc4, K);
    auto load_slab = [&](v4f_t (&to)[4], int kt) {         // past the last slab: the last one again, which nobody reads
        const int slab = min(kt, nk - 1) * BK, at = !KTAIL ? slab : kt >= nk - 1 ? last_at : slab + kc4;
#pragma unroll
        for (int c = 0; c < 4; ++c) to[c] = *reinterpret_cast<const v4f_t*>(g[c] + at);
    };
    auto park = [&](v4f_t x, int kt, char* at) {           // a chunk of slab kt
        const bool drop = past && kt >= nk - 1;
        float e[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) e[t] = drop ? 0.f : x[t];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const uint32_t u0 = split_step(e[0], e[1]), u1 = split_step(e[2], e[3]);
            *reinterpret_cast<v2u_t*>(at + q * PLANE) = v2u_t{u0, u1};
        }
    };

    f32x16_t acc[2][2], low[2][2];
    clear_acc<2, 2>(acc);
    clear_acc<2, 2>(low);
    const int kc = (kh ^ swz(r)) * 16, xat = (wm * 64 + r) * ROW + kc, wat = (BM + wn * 64 + r) * ROW + kc;
    struct Part { v4u_t w[2], x[2]; } hi[2], mid, lo;
    auto read = [&](Part& f, const char* stage, int q) {
#pragma unroll
        for (int j = 0; j < 2; ++j) f.w[j] = *reinterpret_cast<const v4u_t*>(stage + q * PLANE + wat + j * 32 * ROW);
#pragma unroll
        for (int i = 0; i < 2; ++i) f.x[i] = *reinterpret_cast<const v4u_t*>(stage + q * PLANE + xat + i * 32 * ROW);
    };
    // weights are the instruction's first operand: a lane ends with one row of the output and runs of four consecutive columns
    auto products = [&](f32x16_t (&c)[2][2], const Part& w, const Part& x) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) c[i][j] = mfma_bf16(w.w[j], x.x[i], c[i][j]);
    };
    auto slab = [&](int kt, auto parity) {
        constexpr int P = decltype(parity)::value;         // kt & 1
        char* free_stage = smem + P * STAGE;
        const char* next = smem + (P ^ 1) * STAGE;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __syncthreads();
        products(low, lo, hi[P]);
        park(rg[P][0], kt + 2, free_stage + l[0]);
        __builtin_amdgcn_sched_barrier(0);
        products(low, hi[P], lo);
        park(rg[P][1], kt + 2, free_stage + l[1]);
        __builtin_amdgcn_sched_barrier(0);
        read(lo, next, 2);
        products(low, mid, mid);
        park(rg[P][2], kt + 2, free_stage + l[2]);
        __builtin_amdgcn_sched_barrier(0);
        read(hi[P ^ 1], next, 0);
        products(low, mid, hi[P]);
        park(rg[P][3], kt + 2, free_stage + l[3]);
        __builtin_amdgcn_sched_barrier(0);
        load_slab(rg[P], kt + 4);
        products(low, hi[P], mid);
        __builtin_amdgcn_sched_barrier(0);
        read(mid, next, 1);
        products(acc, hi[P], hi[P]);
        __builtin_amdgcn_sched_barrier(0);
    };
    load_slab(rg[0], 0);
    load_slab(rg[1], 1);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
#pragma unroll
        for (int c = 0; c < 4; ++c) park(rg[s][c], s, smem + s * STAGE + l[c]);
        load_slab(rg[s], s + 2);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __syncthreads();
    read(hi[0], smem, 0);
    read(mid, smem, 1);
    read(lo, smem, 2);
    int kt = 0;
    for (; kt + 1 < nk; kt += 2) {
        slab(kt, std::integral_constant<int, 0>{});
        slab(kt + 1, std::integral_constant<int, 1>{});
    }
    if (kt < nk) slab(kt, std::integral_constant<int, 0>{});

#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] += low[i][j];
    if (odd_sums<2, 2>(acc)) float32_products<2, 2>(a, X, W, m0 + wm * 64, n0 + wn * 64, K, acc);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float y[4] = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
                store_run(a, p, m0 + wm * 64 + i * 32 + r, n0 + wn * 64 + j * 32 + 8 * q + 4 * kh, y);
            }
}

// ---------------------------------------------------------------------------------------
// Few rows: a launch is bound by its weights' bytes and by the time its loads take to come back, so LDS is a ring of slabs of
// 32 k, as in gemm_mid.hip.  Block tile BM x 128 x 32, eight wavefronts: four side by side
// (32 rows: 32 x 32 each) or two by two (64 rows: 32 x 64 each), times the two halves of a slab's k, whose sums meet in LDS at
// the end.  Slab layout: rows of 8 chunks of 16 bytes, chunk kc of row m at position kc ^ ((m >> 1) & 7); the permutation is
// applied to the address a lane fetches from.
// ---------------------------------------------------------------------------------------
template <int BM> struct RingTile {
    static constexpr int BN = 128, BK = 32, kStage = (BM + BN) * BK * 4;      // 20 KB / 24 KB
    // (three stages leave room for a second workgroup: loads in flight are limited to about 64 KB a compute unit, so more
    // stages bring nothing; with seven a step of d 768, 64 tokens took 1473 us, with three 1422)
    static constexpr int kStages = 3, kLds = kStage * kStages;
};

// source address = wave-uniform base + per-lane 32-bit byte offset
__device__ __forceinline__ void ring_load_to_lds(const void* sbase, uint32_t voff, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds_base), "v"(voff), "s"(sbase) : "memory");
}
__device__ __forceinline__ const char* ring_uniform(const void* p) {     // a wave-uniform pointer into scalar registers
    const uint64_t v = (uint64_t)(uintptr_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (const char*)(uintptr_t)(((uint64_t)hi << 32) | lo);
}

// All loads of this wavefront but those of the `ahead` youngest slabs (three each) have landed.
template <int AHEAD>
__device__ __forceinline__ void ring_wait(int ahead) {
    if constexpr (AHEAD == 0) {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    } else {
        if (ahead >= AHEAD) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"(AHEAD * 3) : "memory");
        else ring_wait<AHEAD - 1>(ahead);
    }
}

template <int BM, bool KTAIL>          // K is not a multiple of 32: the last slab is used as far as the rows go
__global__ __launch_bounds__(512, 2) void gemm_f32_ring_kernel(const GemmArgs a) {
    using Tile = RingTile<BM>;
    constexpr int BN = Tile::BN, BK = Tile::BK, NST = Tile::kStages, STAGE = Tile::kStage;
    constexpr int WGN = BM == 32 ? 4 : 2, TN = BN / WGN / 32, QUADS = 4 * TN;      // a wavefront's 32 x 32 tiles are side by side
    extern __shared__ __attribute__((aligned(1024))) char smem[];

    const GemmProblem p = a.p[blockIdx.z];
    const int tiles_m = (a.M + BM - 1) / BM;
    const int nblk = (int)gridDim.x, xcd = (int)(blockIdx.x & 7), in_xcd = (int)(blockIdx.x >> 3);
    const int tile = xcd * (nblk >> 3) + min(xcd, nblk & 7) + in_xcd;
    const int m0 = (tile % tiles_m) * BM, n0 = (tile / tiles_m) * BN;
    const int k_first = (int)blockIdx.y * a.kpiece, K = min(a.K - k_first, a.kpiece), nk = KTAIL ? (K + BK - 1) / BK : K / BK;
    const int lane = threadIdx.x & 63, r = lane & 31, kh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int half = wave >> 2, wm = (wave & 3) / WGN, wn = (wave & 3) % WGN;
    const float* __restrict__ X = reinterpret_cast<const float*>(p.X) + k_first;
    const float* __restrict__ W = reinterpret_cast<const float*>(p.W) + k_first;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;

    // A load brings 8 rows (lane -> row lane / 8, position lane % 8); rows past the end of a matrix repeat its last one, their
    // products are never stored.  Per slab a wavefront loads 16 rows of W and 8 of X (32 rows: wavefronts 4 - 7 bring the same
    // rows as 0 - 3 to the same places, so that all of them count their loads alike).
    const int lrow = lane >> 3, xrow8 = BM == 32 ? (wave & 3) * 8 : wave * 8;
    const int xr = xrow8 + lrow;
    const char* base_x = ring_uniform(X + (size_t)m0 * a.ldx);
    const char* base_w = ring_uniform(W + (size_t)n0 * a.ldw);
    // offsets from a slab's first k; of the last slab from the rows' first (a chunk past the end of a row is then the row's first:
    // fill_tail() puts zeros in its place)
    const uint32_t gx = (uint32_t)(min(xr, a.M - 1 - m0) * a.ldx + ((lane & 7) ^ ((xr >> 1) & 7)) * 4) * 4u;
    uint32_t gw[2], last_w[2], last_x = 0;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int row = (wave * 2 + t) * 8 + lrow;
        gw[t] = (uint32_t)(min(row, a.N - 1 - n0) * a.ldw + ((lane & 7) ^ ((row >> 1) & 7)) * 4) * 4u;
        if (KTAIL) last_w[t] = (uint32_t)(min(row, a.N - 1 - n0) * a.ldw + f32_chunk_at(nk - 1, nk, BK, ((lane & 7) ^ ((row >> 1) & 7)) * 4, K)) * 4u;
    }
    if (KTAIL) last_x = (uint32_t)(min(xr, a.M - 1 - m0) * a.ldx + f32_chunk_at(nk - 1, nk, BK, ((lane & 7) ^ ((xr >> 1) & 7)) * 4, K)) * 4u;
    auto issue_one = [&](int t, int kt, int stage) {
        const uint32_t at = lds0 + (uint32_t)stage * STAGE;
        const bool last = KTAIL && kt == nk - 1;
        const size_t k = last ? 0 : (size_t)kt * (BK * 4);
        if (t < 2) ring_load_to_lds(base_w + k, last ? last_w[t & 1] : gw[t & 1], at + BM * 128 + (wave * 2 + t) * 1024);
        else ring_load_to_lds(base_x + k, last ? last_x : gx, at + xrow8 * 128);
    };
    auto issue = [&](int kt, int stage) {
#pragma unroll
        for (int t = 0; t < 3; ++t) issue_one(t, kt, stage);
    };

    f32x16_t acc[1][TN], low[1][TN];
    clear_acc<1, TN>(acc);
    clear_acc<1, TN>(low);

    // this lane's eight k of a row in this wavefront's half of a slab: chunks 4 half + 2 kh and the next
    const int xat = (wm * 32 + r) * 128, wat = BM * 128 + (wn * (32 * TN) + r) * 128, sw = (r >> 1) & 7;
    const int c0 = ((4 * half + 2 * kh) ^ sw) * 16, c1 = ((4 * half + 2 * kh + 1) ^ sw) * 16;
    struct Raw { v4f_t x[2], w[TN][2]; } raw;
    struct Parts { v4u_t x[3], w[TN][3]; } f0, f1;
    auto read = [&](int stage) {
        const char* at = smem + stage * STAGE;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            raw.w[j][0] = *reinterpret_cast<const v4f_t*>(at + wat + j * 4096 + c0);
            raw.w[j][1] = *reinterpret_cast<const v4f_t*>(at + wat + j * 4096 + c1);
        }
        raw.x[0] = *reinterpret_cast<const v4f_t*>(at + xat + c0);
        raw.x[1] = *reinterpret_cast<const v4f_t*>(at + xat + c1);
    };
    auto fill_tail = [&](int kt) {         // fragments of slab kt: a lane's eight k are inside the row or entirely past its end
        if (!KTAIL || kt + 1 < nk || kt * BK + 16 * half + 8 * kh < K) return;
        const v4f_t zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < TN; ++j) raw.w[j][0] = raw.w[j][1] = zero;
        raw.x[0] = raw.x[1] = zero;
    };
    auto split = [&](const v4f_t v[2], v4u_t part[3]) {
        float e[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) e[t] = v[t >> 2][t & 3];
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int t = 0; t < 4; ++t) part[q][t] = split_step(e[2 * t], e[2 * t + 1]);
    };
    auto split_all = [&](Parts& f) {
#pragma unroll
        for (int j = 0; j < TN; ++j) split(raw.w[j], f.w[j]);
        split(raw.x, f.x);
    };
    auto product = [&](int t, const Parts& f) {
        constexpr int order[6][2] = {{2, 0}, {0, 2}, {1, 1}, {1, 0}, {0, 1}, {0, 0}};
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            if (t < 5) low[0][j] = mfma_bf16(f.w[j][order[t][0]], f.x[order[t][1]], low[0][j]);
            else acc[0][j] = mfma_bf16(f.w[j][0], f.x[0], acc[0][j]);
        }
    };
    int stage = 0;
    // As in gemm_mid.hip: a wavefront holds its fragments of slab kt, split, when it reaches the barrier of iteration kt; behind it
    // that slab's stage is refilled and the fragments of slab kt + 1 are read under the first products, and split under the others
    // (split ahead of the products, all wavefronts kept the vector ALU busy at one time and the matrix cores at another).
    auto step = [&](int kt, const Parts& cur, Parts& next) {
        ring_wait<NST - 2>(max(0, min(NST - 2, nk - 2 - kt)));      // slab kt + 1 has landed
        __syncthreads();
        const int refill = stage;
        const bool more = kt + NST < nk;
        stage = stage == NST - 1 ? 0 : stage + 1;
        read(stage);                       // (past the last slab: bytes nobody uses)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            product(t, cur);
            __builtin_amdgcn_sched_barrier(0);
            if (more) issue_one(t, kt + NST, refill);
            __builtin_amdgcn_sched_barrier(0);
        }
        fill_tail(kt + 1);
        split_all(next);
#pragma unroll
        for (int t = 2; t < 6; ++t) product(t, cur);
#pragma unroll
        for (int t = 0; t < 4 * TN; ++t) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, (44 + 44 * TN) / (4 * TN), 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (more) issue_one(2, kt + NST, refill);
    };
#pragma unroll
    for (int s = 0; s < NST; ++s)
        if (s < nk) issue(s, s);
    ring_wait<NST - 1>(min(NST - 1, nk - 1));
    __syncthreads();
    read(0);
    fill_tail(0);
    split_all(f0);
    for (int kt = 0; kt < nk; kt += 2) {
        step(kt, f0, f1);
        if (kt + 1 < nk) step(kt + 1, f1, f0);
    }

    // The halves meet: of a pair of wavefronts, the first finishes the first half of their runs of four columns, the second the rest.
    __syncthreads();
    float y[QUADS / 2][4];
    {
        float* send = reinterpret_cast<float*>(smem) + (wave * (QUADS / 2) * 64 + lane) * 4;
        const float* recv = reinterpret_cast<const float*>(smem) + ((wave ^ 4) * (QUADS / 2) * 64 + lane) * 4;
        auto run = [&](int t) {            // run t of the wavefront's tiles
            v4f_t x;
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = acc[0][t >> 2][4 * (t & 3) + e] + low[0][t >> 2][4 * (t & 3) + e];
            return x;
        };
#pragma unroll
        for (int t = 0; t < QUADS / 2; ++t) {
            const v4f_t lo = run(t), hi = run(t + QUADS / 2);
            *reinterpret_cast<v4f_t*>(send + t * 256) = half ? lo : hi;
#pragma unroll
            for (int e = 0; e < 4; ++e) y[t][e] = half ? hi[e] : lo[e];
        }
        __syncthreads();
        OddSums odd;
#pragma unroll
        for (int t = 0; t < QUADS / 2; ++t) {
            const v4f_t o = *reinterpret_cast<const v4f_t*>(recv + t * 256);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                y[t][e] = half ? o[e] + y[t][e] : y[t][e] + o[e];
                odd.look(y[t][e]);
            }
        }
        if (odd.any()) {
            float32_products<1, TN>(a, X, W, m0 + wm * 32, n0 + wn * (32 * TN), K, acc);
#pragma unroll
            for (int t = 0; t < QUADS / 2; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) y[t][e] = half ? acc[0][(t + QUADS / 2) >> 2][4 * ((t + QUADS / 2) & 3) + e] : acc[0][t >> 2][4 * (t & 3) + e];
        }
    }
#pragma unroll
    for (int t = 0; t < QUADS / 2; ++t) {
        const int u = half ? t + QUADS / 2 : t;
        store_run(a, p, m0 + wm * 32 + r, n0 + wn * (32 * TN) + (u >> 2) * 32 + 8 * (u & 3) + 4 * kh, y[t]);
    }
}

template <typename K>
static zo2_status launch_f32_t(K kern, const GemmArgs& a, int bm, int threads, int lds, bool& reserved, int splits, hipStream_t st) {
    if (lds > 65536 && !reserved) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) {
            set_op_error("gemm: cannot reserve %d bytes of LDS: %s", lds, hipGetErrorString(e));
            return ZO2_EHIP;
        }
        reserved = true;
    }
    const unsigned tiles = (unsigned)(((a.M + bm - 1) / bm) * ((a.N + 127) / 128));
    hipLaunchKernelGGL(kern, dim3(tiles, splits, a.nprob), dim3(threads), lds, st, a);
    ZO2_HIP_LAUNCH_CHECK();
    return ZO2_OK;
}
template <bool KTAIL>
static zo2_status launch_split_t(const GemmArgs& a, int splits, hipStream_t st) {
    static bool reserved_on[kMaxDevices] = {false};
    return launch_f32_t(gemm_f32_split_kernel<KTAIL>, a, F32Tile::BM, 256, F32Tile::kLds, reserved_on[current_device()], splits, st);
}
template <int BM, bool KTAIL>
static zo2_status launch_ring_t(const GemmArgs& a, int splits, hipStream_t st) {
    static bool reserved_on[kMaxDevices] = {false};
    return launch_f32_t(gemm_f32_ring_kernel<BM, KTAIL>, a, BM, 512, RingTile<BM>::kLds, reserved_on[current_device()], splits, st);
}

zo2_status gemm_launch_f32(const GemmArgs& a, int splits, int rows, hipStream_t st) {
    const bool tail = a.K % 32 != 0;                                    // (pieces are multiples of 32: only the last one can end inside a slab)
    if (a.ldx >= 1 << 22 || a.ldw >= 1 << 22) rows = 128;               // the ring's offsets are 32 bits
    if (rows == 32) return tail ? launch_ring_t<32, true>(a, splits, st) : launch_ring_t<32, false>(a, splits, st);
    if (rows == 64) return tail ? launch_ring_t<64, true>(a, splits, st) : launch_ring_t<64, false>(a, splits, st);
    return a.K % 16 != 0 ? launch_split_t<true>(a, splits, st) : launch_split_t<false>(a, splits, st);
}

}  // namespace zo2
