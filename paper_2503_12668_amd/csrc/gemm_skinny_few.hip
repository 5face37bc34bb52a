// The projections of up to 32 tokens in 16 bits.  A workgroup owns 16 output features; its eight wavefronts take the slabs of its k in turn, each with
// its own activations straight from memory into the matrix instruction's registers, and meet once, at the end.  No barrier and no LDS until then,
// and k as long as a workgroup can make it: QKV and FC1 are finished here, with bias, ReLU and rounding, and the output projection and FC2 leave
// the LayerNorm behind them a few sums to add, not 32 (where skinny_few_pays takes them: FC2 of d 2048, ffn 8192 is beyond its line and leaves 32).
// (gemm_skinny_rows.hip's 128 features a workgroup need 8 - 32 pieces of k to fill the chip: a launch of 4.7 us for their sum behind QKV
// and FC1 each, and 8 MB of sums that a LayerNorm pass has to read.)  An activation is read once for 16 features instead of once for 128: from
// L2, 2 M bytes a weight, which is why the line is 32 rows.
// What bounds it is the generator, as there.  d 2048, 16 rows, update and perturbation, us: QKV 21.8 + 4.7 -> 21.7, FC1 22.5 + 4.9 -> 23.3, output 10.2 -> 8.4, the
// LayerNorm behind it 5.8 -> 4.8.  Steps, us: d 2048, 12 blocks, 16 tokens 1457 -> 1306, 32 1573 -> 1470, float16 16 1503 -> 1378; d 768, 12 blocks, 14
// 724 -> 537; d 512, 6 blocks, 24 391 -> 297.
#include <algorithm>

#include "skinny_weights.h"

namespace zo2 {

static constexpr int kFewBN = 16, kFewWaves = 8, kFewBK = 64;      // features per workgroup, wavefronts, k per slab

// NT: 16-row tiles of each stream
template <typename T, int NT, bool UPDATE>
__global__ __launch_bounds__(64 * kFewWaves, 4) void skinny_few_kernel(const SkinnyArgs a) {
    constexpr int NI = 2 * NT;
    __shared__ v4f_t sums[kFewWaves][NI][64];
    const SkinnyProblem p = a.p[blockIdx.z];
    const int n0 = blockIdx.x * kFewBN;
    const int k_begin = blockIdx.y * a.k_per_split, k_end = min(a.K, k_begin + a.k_per_split);
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float c = UPDATE ? *a.c_ptr : 0.f;

    const WeightLane<T> lane_w(a, p, n0, kFewBN, r, 8 * g);
    const T* xsrc[NI];                     // row r of tile i; rows past M repeat row M - 1
#pragma unroll
    for (int i = 0; i < NI; ++i)
        xsrc[i] = reinterpret_cast<const T*>(i >= NT ? p.Xm : p.Xp) + (size_t)min((i >= NT ? i - NT : i) * 16 + r, a.M - 1) * a.ldx + 8 * g;

    v4f_t acc[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) acc[i] = v4f_t{0.f, 0.f, 0.f, 0.f};
    typename WeightLane<T>::Theta t, next;
    v4u_t x[2][NI];
    auto load_x = [&](int k0) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < NI; ++i) x[h][i] = *reinterpret_cast<const v4u_t*>(xsrc[i] + k0 + 32 * h);
    };
    // theta is not touched before the slab's first draw: that covers the latency of the first load, and in the iterations behind it the
    // wait, which cannot tell them apart from the first, then finds the stores of the iteration before done
    auto wait_for = [](typename WeightLane<T>::Theta& t, const float (&z)[2][8]) {
        asm volatile("" : "+v"(t.v[0][0]), "+v"(t.v[1][0])
                     : "v"(z[0][0]), "v"(z[0][1]), "v"(z[0][2]), "v"(z[0][3]), "v"(z[0][4]), "v"(z[0][5]), "v"(z[0][6]), "v"(z[0][7]),
                       "v"(z[1][0]), "v"(z[1][1]), "v"(z[1][2]), "v"(z[1][3]), "v"(z[1][4]), "v"(z[1][5]), "v"(z[1][6]), "v"(z[1][7]));
    };
    int k0 = k_begin + wave * kFewBK;
    if (k0 < k_end) {
        lane_w.load(t, k0);
        load_x(k0);
        for (;;) {
            const int k1 = k0 + kFewWaves * kFewBK;
            if (k1 < k_end) lane_w.load(next, k1);
            float th[2][8], z[2][8];
            lane_w.draw(k0, UPDATE ? a.key_prev : a.key, z);
            wait_for(t, z);
            lane_w.values(t, th);
            if constexpr (UPDATE) {
                lane_w.update(k0, c, z, th);
                lane_w.draw(k0, a.key, z);
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                Vec<T, 8> w[2];
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int j = 0; j < 8; ++j) w[s].v[j] = Fmt<T>::store(__builtin_fmaf(s ? -a.eps : a.eps, z[h][j], th[h][j]));
#pragma unroll
                for (int i = 0; i < NI; ++i) {
                    v4u_t u;
                    __builtin_memcpy(&u, &w[i >= NT], 16);
                    acc[i] = RowsMfma<T>::run(u, x[h][i], acc[i]);
                }
            }
            if (k1 >= k_end) break;
            load_x(k1);
            t = next;
            k0 = k1;
        }
    }
    // a lane holds row r of a tile and features 4 g .. + 3; wavefront i finishes tile i.  Bias and residual are on their way while the others end.
    const int i = wave, s = i >= NT, m = (s ? i - NT : i) * 16 + r, n = n0 + 4 * g;
    const bool mine = i < NI && m < a.M && n < a.N;            // (N % 4 == 0)
    const size_t o = (size_t)m * a.ldy + n;
    const T* bias = reinterpret_cast<const T*>(s ? p.bias_m : p.bias_p);
    const float* res = s ? p.res_m : p.res_p;
    float b[4] = {0.f, 0.f, 0.f, 0.f}, q[4] = {0.f, 0.f, 0.f, 0.f};
    if (a.direct && mine && bias)
#pragma unroll
        for (int e = 0; e < 4; ++e) b[e] = Fmt<T>::load(bias[n + e]);
    if (a.direct && mine && res)
#pragma unroll
        for (int e = 0; e < 4; ++e) q[e] = res[o + e];
#pragma unroll
    for (int t = 0; t < NI; ++t) sums[wave][t][lane] = acc[t];
    __syncthreads();
    if (!mine) return;
    v4f_t y = sums[0][i][lane];            // the wavefronts' sums in order
#pragma unroll
    for (int w = 1; w < kFewWaves; ++w) y += sums[w][i][lane];
    if (!a.direct) {
        const size_t plane = (size_t)a.M * a.N;
        *reinterpret_cast<v4f_t*>(a.partial + (((size_t)blockIdx.z * a.splits + blockIdx.y) * 2 + s) * plane + (size_t)m * a.N + n) = y;
        return;
    }
    Vec<float, 4> f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        f.v[e] = (y[e] + b[e]) * p.out_scale;
        if (a.relu) f.v[e] = fmaxf(f.v[e], 0.f);
        if (res) f.v[e] += q[e];
    }
    if (a.out_f32) {
        store_vec<float, 4>(reinterpret_cast<float*>(s ? p.Ym : p.Yp) + o, f);
    } else {
        Vec<T, 4> v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v.v[e] = Fmt<T>::store(f.v[e]);
        store_vec<T, 4>(reinterpret_cast<T*>(s ? p.Ym : p.Yp) + o, v);
    }
}

// Up to 32 rows, while the activations that its workgroups read - once for 16 features, 16-row tiles of both streams - take less time than it saves: a
// launch where the sum is one of its own, a part of the LayerNorm behind it otherwise.  MB of them at which both sides meet, from the launches at d 2048
// and the steps at 2560 and 4096: what is left of them behind a generator that draws twice costs 0.03 us a MB (200 and 80 MB), behind one draw
// 0.07 (86 and 34).  float16 draws once here; bfloat16 once or twice, but an order of sums that depended on whether an update
// is pending would show in the losses of a step behind a flush: one line for both.  Nor does it ask who adds the pieces this time (a LayerNorm's pass does
// not in a round that goes through the blocks together, or under a smaller scratch set): a projection onto the residual stream has the second line always.
bool skinny_few_pays(const SkinnyArgs& a, int dtype) {
    if (a.M > 32 || a.K >= 1 << 22) return false;
    const double mb = 4e-6 * (a.M <= 16 ? 1 : 2) * a.N * (double)a.K * a.nprob;
    return mb <= (dtype == ZO2_BF16 ? (a.onto_residual ? 60. : 150.) : (a.onto_residual ? 34. : 86.));
}

// Pieces of k, at most max_splits of them.  The time is that of the slabs that one wavefront walks, while two workgroups a compute unit are resident (512 on
// the chip); a sum in a launch of its own costs as much as two slabs, one that a LayerNorm pass makes next to nothing a piece.
void skinny_few_splits(const SkinnyArgs& a, int max_splits, int& splits, int& k_per_split) {
    const int slabs = a.K / kFewBK, tiles = (a.N + kFewBN - 1) / kFewBN * a.nprob;
    float best = 0.f;
    splits = 0;
    for (int s = 1; s <= std::min(max_splits, slabs); ++s) {
        const int each = (slabs + s - 1) / s, n = (slabs + each - 1) / each;
        const float cost = (float)((each + kFewWaves - 1) / kFewWaves) * std::max(1.f, (float)tiles * (float)n / 512.f) + (a.onto_residual ? 0.05f * (float)n : n > 1 ? 2.f : 0.f);
        if (splits == 0 || cost < best) {
            best = cost;
            splits = n;
            k_per_split = each * kFewBK;
        }
    }
}

template <typename T, bool UPDATE>
static zo2_status launch_t(const SkinnyArgs& a, hipStream_t st) {
    const dim3 grid((a.N + kFewBN - 1) / kFewBN, a.splits, a.nprob), block(64 * kFewWaves);
    if (a.M <= 16) hipLaunchKernelGGL((skinny_few_kernel<T, 1, UPDATE>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((skinny_few_kernel<T, 2, UPDATE>), grid, block, 0, st, a);
    ZO2_HIP_LAUNCH_CHECK();
    return ZO2_OK;
}
zo2_status skinny_few_launch(const SkinnyArgs& a, int dtype, hipStream_t st) {
    if (dtype == ZO2_F16) return launch_t<f16_t, false>(a, st);
    return a.c_ptr ? launch_t<bf16_t, true>(a, st) : launch_t<bf16_t, false>(a, st);
}

}  // namespace zo2
