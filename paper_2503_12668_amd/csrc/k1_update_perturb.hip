// K1: fused regenerate + deferred update + perturb (Alg. 2 DualForward, Sec. 5.4).
//
// The paper sweeps a module's parameters four times per iteration (update, +eps, -2eps,
// +eps), drawing a fresh Gaussian vector each time.  Here one sweep reads theta once,
// regenerates z_prev (last iteration's direction) and z (this iteration's) from their
// counters, writes theta' = theta - c z_prev back in the transfer format, and writes the
// two perturbed copies W+ = theta' + eps z, W- = theta' - eps z in the compute format.
// theta itself is never perturbed, so "restore" costs nothing and is exact.
//
// HBM-streaming kernel: each lane moves groups of 8 consecutive elements with 128-bit
// accesses (bf16/fp16; two for fp32, one 64-bit for the 8-bit formats), a workgroup owns
// a contiguous chunk of one tensor, the grid covers up to 16 tensors of a bucket.
#include <math.h>

#include <algorithm>

#include "k1.h"
#include "philox.h"

namespace zo2 {

static constexpr int kThreads = 256;
static constexpr int kPerLane = 8;
// one group per lane and workgroup: measured inside the step, workgroups of 2048 elements sweep a block at 6.4 TB/s,
// of 8192 (four groups per lane, all loads up front) at 5.9 - many small workgroups keep the streams of consecutive
// addresses denser than few large ones
static constexpr int kIters = 1;
static constexpr int kChunk = kThreads * kPerLane * kIters;   // 2048 elements per workgroup

// The arithmetic of one group of 8 consecutive elements (one Philox call q per random stream): tv holds
// theta on entry and theta' on return.
template <typename W, typename C, bool UPDATE, bool PERTURB, bool SR, bool DRAW>
__device__ __forceinline__ void k1_group(const PhiloxKeys& k_prev, const PhiloxKeys& k_cur, uint32_t tensor_id, uint64_t q, float c, float eps, float scale,
                                         float inv_scale, Vec<W, kPerLane>& tv, Vec<C, kPerLane>& p, Vec<C, kPerLane>& m) {
    constexpr bool kScaled = (Fmt<W>::kBytes == 1);
    float th[kPerLane];
    if constexpr (kScaled) {        // 8-bit storage: the group's eight bytes are converted by the packed hardware instructions
        fp8_decode8<W>(tv, th);
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) th[j] *= inv_scale;
    } else {
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) th[j] = Fmt<W>::load(tv.v[j]);
    }
    if (UPDATE) {
        float zp[kPerLane];
        gaussian8(k_prev, tensor_id, q, zp);
        uint32_t rw[4] = {0u, 0u, 0u, 0u};
        constexpr bool sr = SR && Fmt<W>::kBytes < 4;
        if (sr) rounding_words(k_prev, tensor_id, q, rw);
        if constexpr (kScaled && !sr) {
            float ts[kPerLane];
#pragma unroll
            for (int j = 0; j < kPerLane; ++j) ts[j] = __builtin_fmaf(-c, zp[j], th[j]) * scale;
            fp8_encode8<W>(ts, tv);
            fp8_decode8<W>(tv, th);
#pragma unroll
            for (int j = 0; j < kPerLane; ++j) th[j] *= inv_scale;
        } else if constexpr (kScaled) {
            float ts[kPerLane];
#pragma unroll
            for (int j = 0; j < kPerLane; ++j) ts[j] = __builtin_fmaf(-c, zp[j], th[j]) * scale;
            fp8_encode8_stochastic<W>(ts, rw, tv, th);
#pragma unroll
            for (int j = 0; j < kPerLane; ++j) th[j] *= inv_scale;
        } else {
#pragma unroll
            for (int j = 0; j < kPerLane; ++j) {
                const float t = __builtin_fmaf(-c, zp[j], th[j]);
                tv.v[j] = sr ? store_stochastic<W>(t, rounding_bits_of(rw, j)) : Fmt<W>::store(t);
                th[j] = Fmt<W>::load(tv.v[j]);
            }
        }
    }
    if constexpr (PERTURB && DRAW) {
        float z[kPerLane];
        gaussian8(k_cur, tensor_id, q, z);
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) {
            p.v[j] = Fmt<C>::store(__builtin_fmaf(eps, z[j], th[j]));
            m.v[j] = Fmt<C>::store(__builtin_fmaf(-eps, z[j], th[j]));
        }
    } else if constexpr (PERTURB) {
        // eps = 0 (the single forward of an evaluation): W+ = theta' in the compute format, nothing to draw.  A kernel
        // instance of its own, chosen on the host: as a branch on eps inside one instance the two paths' 16-bit results
        // were merged through scratch memory.
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) p.v[j] = m.v[j] = Fmt<C>::store(th[j]);
    }
}

// MIXED: the block of a step whose projections perturb in their loader.  Its matrices are only updated, its vectors - a few
// workgroups of the sweep - perturbed as well (one launch of 36 us for 50 M elements; as a launch of
// their own the vectors took 4.7 us behind the 33 of the update).
template <typename W, typename C, bool UPDATE, bool PERTURB, bool SR, bool DRAW, bool MIXED = false>
__global__ __launch_bounds__(kThreads) void k1_kernel(const K1Args a) {
    // which tensor does this workgroup work on: first_chunk[] ascends (0xffffffff past the last segment),
    // so the segment index is the number of entries at or below this workgroup's index
    // Workgroups are dispatched in index order; chunks are taken in the opposite order, so that the sweep ends with
    // the first tensors of the list: the projections that run right after the sweep (q, k, v of a block) then find
    // their perturbed copies still in the memory-side cache, which a whole block's copies exceed.
    const uint32_t chunk = a.reverse ? a.total_chunks - 1u - blockIdx.x : blockIdx.x;
    int s = 0;
#pragma unroll
    for (int i = 1; i < K1Args::kMaxSeg; ++i) s += (chunk >= a.first_chunk[i]) ? 1 : 0;
    const K1Seg sg = a.seg[s];
    const uint64_t chunk0 = (uint64_t)(chunk - a.first_chunk[s]) * kChunk;
    W* __restrict__ theta = reinterpret_cast<W*>(a.theta) + sg.off;
    const int64_t wofs = a.packed_w ? sg.woff : sg.off - a.w_off0;
    C* __restrict__ wp = PERTURB ? reinterpret_cast<C*>(a.w_plus) + wofs : nullptr;
    const bool has_m = PERTURB && a.w_minus != nullptr;            // a single forward needs W+ only
    C* __restrict__ wm = has_m ? reinterpret_cast<C*>(a.w_minus) + wofs : nullptr;
    const float c = UPDATE ? (a.c_ptr ? *a.c_ptr : a.c_imm) : 0.f;
    const float eps = a.eps;
    const float scale = sg.scale, inv_scale = 1.0f / sg.scale;
    constexpr int kStride = kThreads * kPerLane;

    if constexpr (MIXED) {
        if (sg.woff < 0 && chunk0 + kChunk <= sg.n) {      // a matrix is whole chunks but for its last workgroup
            const uint64_t i = chunk0 + (uint64_t)threadIdx.x * kPerLane;
            Vec<W, kPerLane> tv = load_vec_stream<W, kPerLane>(theta + i);
            Vec<C, kPerLane> p, m;
            k1_group<W, C, true, false, SR, false>(a.k_prev, a.k_cur, sg.tensor_id, (sg.e0 + i) >> 3, c, eps, scale, inv_scale, tv, p, m);
            store_vec<W, kPerLane>(theta + i, tv);
            return;
        }
    }
    const bool copies = PERTURB && !(MIXED && sg.woff < 0);
    if (chunk0 + kChunk <= sg.n) {
        // whole chunk inside the tensor (all but the last workgroup of a segment): every load is in
        // flight before the first group is computed, and nothing is masked
        const uint64_t i0 = chunk0 + (uint64_t)threadIdx.x * kPerLane;
        Vec<W, kPerLane> tv[kIters];
#pragma unroll
        // (theta is read once per step: loaded with the streaming policy it leaves the caches to the perturbed copies,
        // which the projections read next - the sweep itself runs 5 % faster and the projections 1 %)
        for (int it = 0; it < kIters; ++it) tv[it] = load_vec_stream<W, kPerLane>(theta + i0 + (uint64_t)it * kStride);
#pragma unroll
        for (int it = 0; it < kIters; ++it) {
            const uint64_t i = i0 + (uint64_t)it * kStride;
            Vec<C, kPerLane> p, m;
            k1_group<W, C, UPDATE, PERTURB, SR, DRAW>(a.k_prev, a.k_cur, sg.tensor_id, (sg.e0 + i) >> 3, c, eps, scale, inv_scale, tv[it], p, m);
            // (theta' is not read again before the next step when the perturbed copies are written here: streamed past the
            // caches it leaves them to the copies; in an update-only sweep the projections read theta' next, so it stays)
            if (UPDATE && PERTURB) store_vec_stream<W, kPerLane>(theta + i, tv[it]);
            else if (UPDATE) store_vec<W, kPerLane>(theta + i, tv[it]);
            if (PERTURB) {
                store_vec<C, kPerLane>(wp + i, p);
                if (has_m) store_vec<C, kPerLane>(wm + i, m);
            }
        }
        return;
    }
    // last chunk of a segment: ragged end, element-wise masking
#pragma unroll 1
    for (int it = 0; it < kIters; ++it) {
        const uint64_t i0 = chunk0 + (uint64_t)it * kStride + (uint64_t)threadIdx.x * kPerLane;
        if (i0 >= sg.n) break;
        const int valid = (sg.n - i0 >= (uint64_t)kPerLane) ? kPerLane : (int)(sg.n - i0);
        Vec<W, kPerLane> tv;
        if (valid == kPerLane) {
            tv = load_vec<W, kPerLane>(theta + i0);
        } else {
#pragma unroll
            for (int j = 0; j < kPerLane; ++j) tv.v[j] = (j < valid) ? theta[i0 + j] : Fmt<W>::store(0.f);
        }
        Vec<C, kPerLane> p, m;
        k1_group<W, C, UPDATE, PERTURB, SR, DRAW>(a.k_prev, a.k_cur, sg.tensor_id, (sg.e0 + i0) >> 3, c, eps, scale, inv_scale, tv, p, m);
        if (valid == kPerLane) {
            if (UPDATE && PERTURB) store_vec_stream<W, kPerLane>(theta + i0, tv);
            else if (UPDATE) store_vec<W, kPerLane>(theta + i0, tv);
            if (copies) {
                store_vec<C, kPerLane>(wp + i0, p);
                if (has_m) store_vec<C, kPerLane>(wm + i0, m);
            }
        } else {
#pragma unroll
            for (int j = 0; j < kPerLane; ++j)
                if (j < valid) {
                    if (UPDATE) theta[i0 + j] = tv.v[j];
                    if (copies) { wp[i0 + j] = p.v[j]; if (has_m) wm[i0 + j] = m.v[j]; }
                }
        }
    }
}

// Where the loader applies the update, or there is none, the vectors are all that a step's blocks need swept: 13 workgroups a block at d 2048, a
// launch of 4.7 us that is start and end.  With resident blocks one launch does them for all, and for the final LayerNorm.
template <typename T, bool UPDATE>
__global__ __launch_bounds__(kThreads) void k1_vectors_kernel(const K1VectorsArgs a) {
    const bool last = blockIdx.y == (uint32_t)a.n_blocks;
    const K1VectorsArgs::List& li = last ? a.last : a.block;
    if (blockIdx.x >= li.total_chunks) return;
    int s = 0;
#pragma unroll
    for (int i = 1; i < K1Args::kMaxSeg; ++i) s += (blockIdx.x >= li.first_chunk[i]) ? 1 : 0;
    const K1Seg& sg = li.seg[s];
    const uint64_t i = (uint64_t)(blockIdx.x - li.first_chunk[s]) * kChunk + (uint64_t)threadIdx.x * kPerLane;
    if (i >= sg.n) return;
    const int64_t b = last ? 0 : (int64_t)blockIdx.y, w = sg.woff + b * a.w_stride + (int64_t)i;
    T* theta = reinterpret_cast<T*>(li.theta) + sg.off + b * a.theta_stride + (int64_t)i;
    const float c = UPDATE ? *a.c_ptr : 0.f;
    Vec<T, kPerLane> tv = load_vec<T, kPerLane>(theta), p, m;
    k1_group<T, T, UPDATE, true, false, true>(a.k_prev, a.k_cur, sg.tensor_id + (uint32_t)(b * a.tid_stride), i >> 3, c, a.eps, 1.f, 1.f, tv, p, m);
    if (UPDATE) store_vec<T, kPerLane>(theta, tv);
    store_vec<T, kPerLane>(reinterpret_cast<T*>(li.w_plus) + w, p);
    store_vec<T, kPerLane>(reinterpret_cast<T*>(li.w_minus) + w, m);
}

// A round of directions in one sweep (zo2_step_multi).  Bound by the vector ALU, which draws n_upd + n_dir Gaussians an element
// (busy 99 % of the cycles; at four and four the bytes alone would take about as long);
// sweep by sweep the same draws each wait for theta and its write: a block of 50 M bf16 elements, four updates and four directions
// 99 + 59 + 137 us in seven launches, 194 in one.  The group's arithmetic is k1_group's, update by update and direction by direction, so
// the stored bits are those of the single sweeps.
template <typename W, typename C, bool SR>
__global__ __launch_bounds__(kThreads) void k1_round_kernel(const K1RoundArgs a) {
    const uint32_t chunk = a.total_chunks - 1u - blockIdx.x;      // last to first, as in k1_kernel
    int s = 0;
#pragma unroll
    for (int i = 1; i < K1Args::kMaxSeg; ++i) s += (chunk >= a.first_chunk[i]) ? 1 : 0;
    const K1Seg sg = a.seg[s];
    const uint64_t i0 = (uint64_t)(chunk - a.first_chunk[s]) * kChunk + (uint64_t)threadIdx.x * kPerLane;
    if (i0 >= sg.n) return;
    W* __restrict__ theta = reinterpret_cast<W*>(a.theta) + sg.off + i0;
    const int64_t wofs = sg.off - a.w_off0 + (int64_t)i0;
    const int valid = (sg.n - i0 >= (uint64_t)kPerLane) ? kPerLane : (int)(sg.n - i0);
    const float scale = sg.scale, inv_scale = 1.0f / sg.scale;
    const uint64_t q = (sg.e0 + i0) >> 3;
    Vec<W, kPerLane> tv;
    Vec<C, kPerLane> p, m;
    if (valid == kPerLane) {
        tv = load_vec_stream<W, kPerLane>(theta);
    } else {
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) tv.v[j] = (j < valid) ? theta[j] : Fmt<W>::store(0.f);
    }
#pragma unroll 1
    for (int u = 0; u < a.n_upd; ++u)
        k1_group<W, C, true, false, SR, false>(a.k_upd[u], a.k_upd[u], sg.tensor_id, q, a.c_ptr[u], 0.f, scale, inv_scale, tv, p, m);
    if (a.n_upd > 0) {
        if (valid == kPerLane) {
            store_vec_stream<W, kPerLane>(theta, tv);
        } else {
#pragma unroll
            for (int j = 0; j < kPerLane; ++j)
                if (j < valid) theta[j] = tv.v[j];
        }
    }
#pragma unroll 1
    for (int d = 0; d < a.n_dir; ++d) {
        k1_group<W, C, false, true, false, true>(a.k_dir[d], a.k_dir[d], sg.tensor_id, q, 0.f, a.eps, scale, inv_scale, tv, p, m);
        C* __restrict__ wp = reinterpret_cast<C*>(a.w_plus[d]) + wofs;
        C* __restrict__ wm = reinterpret_cast<C*>(a.w_minus[d]) + wofs;
        if (valid == kPerLane) {
            store_vec<C, kPerLane>(wp, p);
            store_vec<C, kPerLane>(wm, m);
        } else {
#pragma unroll
            for (int j = 0; j < kPerLane; ++j)
                if (j < valid) { wp[j] = p.v[j]; wm[j] = m.v[j]; }
        }
    }
}

// (bfloat16 copies of anything but float16: where float16 is stored the compiler folds the rounding into the multiply-add in some
// instances and not in others, 34 of a million elements differ, and a round in one pass is to leave the bits of one in several)
bool k1_round_applicable(int wire_dtype, int compute_dtype) { return compute_dtype == ZO2_BF16 && wire_dtype != ZO2_F16; }
template <typename W, typename C>
static zo2_status launch_round(const K1RoundArgs& a, hipStream_t st) {
    if constexpr (__is_same(C, bf16_t) && !__is_same(W, f16_t)) {
        if (a.stochastic && sizeof(W) < 4) hipLaunchKernelGGL((k1_round_kernel<W, C, true>), dim3(a.total_chunks), dim3(kThreads), 0, st, a);
        else hipLaunchKernelGGL((k1_round_kernel<W, C, false>), dim3(a.total_chunks), dim3(kThreads), 0, st, a);
        ZO2_HIP_LAUNCH_CHECK();
        return ZO2_OK;
    }
    set_op_error("k1: no round in one sweep for these formats");
    return ZO2_EINVAL;
}

template <typename W, typename C>
static zo2_status launch_wc(const K1Args& a, bool update, bool perturb, hipStream_t st) {
    const dim3 grid(a.total_chunks), block(kThreads);
    const bool sr = update && a.stochastic != 0 && sizeof(W) < 4;      // stochastic rounding only concerns a low-bit theta'
    const bool draw = a.eps != 0.f;
    if constexpr (sizeof(W) == 2 && __is_same(W, C)) {
        if (a.mixed) {
            if (sr) hipLaunchKernelGGL((k1_kernel<W, C, true, true, true, true, true>), grid, block, 0, st, a);
            else hipLaunchKernelGGL((k1_kernel<W, C, true, true, false, true, true>), grid, block, 0, st, a);
            ZO2_HIP_LAUNCH_CHECK();
            return ZO2_OK;
        }
    }
#define ZO2_K1_LAUNCH(U, P, S, D) hipLaunchKernelGGL((k1_kernel<W, C, U, P, S, D>), grid, block, 0, st, a)
    if (update && perturb && sr) { if (draw) ZO2_K1_LAUNCH(true, true, true, true); else ZO2_K1_LAUNCH(true, true, true, false); }
    else if (update && perturb) { if (draw) ZO2_K1_LAUNCH(true, true, false, true); else ZO2_K1_LAUNCH(true, true, false, false); }
    else if (update && sr) ZO2_K1_LAUNCH(true, false, true, false);
    else if (update) ZO2_K1_LAUNCH(true, false, false, false);
    else if (perturb) { if (draw) ZO2_K1_LAUNCH(false, true, false, true); else ZO2_K1_LAUNCH(false, true, false, false); }
#undef ZO2_K1_LAUNCH
    ZO2_HIP_LAUNCH_CHECK();
    return ZO2_OK;
}

uint32_t k1_chunks(uint64_t n) { return (uint32_t)((n + kChunk - 1) / kChunk); }

// workgroups of the segments, and the checks that every sweep needs of them
static zo2_status plan_chunks(const K1Seg* seg, int nseg, uint32_t* first_chunk, uint32_t& total) {
    ZO2_OP_CHECK(nseg >= 1 && nseg <= K1Args::kMaxSeg, ZO2_EINVAL, "k1: %d segments", nseg);
    uint32_t chunks = 0;
    for (int i = 0; i < nseg; ++i) {
        ZO2_OP_CHECK((seg[i].e0 & 7) == 0 && (seg[i].off & 7) == 0, ZO2_EINVAL,
                     "k1: segment %d not aligned to 8 elements", i);
        int ex = 0;
        ZO2_OP_CHECK(seg[i].scale > 0.f && isfinite(seg[i].scale) && frexpf(seg[i].scale, &ex) == 0.5f, ZO2_EINVAL,
                     "k1: segment %d has scale %g (must be a power of two)", i, (double)seg[i].scale);
        first_chunk[i] = chunks;
        const uint64_t nc = (seg[i].n + kChunk - 1) / kChunk;
        ZO2_OP_CHECK(chunks + nc < 0x7fffffffull, ZO2_EINVAL, "k1: too many chunks");
        chunks += (uint32_t)nc;
    }
    for (int i = nseg; i < K1Args::kMaxSeg; ++i) first_chunk[i] = 0xffffffffu;
    total = chunks;
    return ZO2_OK;
}

zo2_status k1_launch(K1Args& a, int wire_dtype, int compute_dtype, bool update, bool perturb, hipStream_t st) {
    { const zo2_status s = plan_chunks(a.seg, a.nseg, a.first_chunk, a.total_chunks); if (s != ZO2_OK) return s; }
    if (a.total_chunks == 0 || (!update && !perturb)) return ZO2_OK;
    ZO2_OP_CHECK(a.theta != nullptr, ZO2_EINVAL, "k1: theta is NULL");
    ZO2_OP_CHECK(!perturb || a.w_plus, ZO2_EINVAL, "k1: W+ missing");
    ZO2_OP_CHECK(!a.mixed || (update && perturb && a.packed_w && a.w_minus && a.eps != 0.f && wire_dtype == compute_dtype && zo2_dtype_size(wire_dtype) == 2),
                 ZO2_EINVAL, "k1: a mixed sweep updates and perturbs 16-bit tensors into packed copies");
    ZO2_DISPATCH_WIRE(wire_dtype, W, {
        ZO2_DISPATCH_COMPUTE(compute_dtype, C, { return launch_wc<W, C>(a, update, perturb, st); });
    });
    return ZO2_OK;
}

zo2_status k1_vectors_launch(K1VectorsArgs& a, int dtype, bool update, hipStream_t st) {
    for (K1VectorsArgs::List* li : {&a.block, &a.last}) {
        const zo2_status s = plan_chunks(li->seg, li->nseg, li->first_chunk, li->total_chunks);
        if (s != ZO2_OK) return s;
        ZO2_OP_CHECK(li->theta && li->w_plus && li->w_minus, ZO2_EINVAL, "k1: NULL buffer");
        for (int i = 0; i < li->nseg; ++i)
            ZO2_OP_CHECK(li->seg[i].n % kPerLane == 0 && li->seg[i].woff >= 0 && li->seg[i].woff % kPerLane == 0 && li->seg[i].e0 == 0, ZO2_EINVAL, "k1: vectors in whole groups of eight");
    }
    ZO2_OP_CHECK(a.n_blocks >= 0 && a.n_blocks < 65535 && a.theta_stride % kPerLane == 0 && a.w_stride % kPerLane == 0 && (!update || a.c_ptr) &&
                 (dtype == ZO2_F32 || dtype == ZO2_BF16), ZO2_EINVAL, "k1: vectors of %d blocks", a.n_blocks);
    const dim3 grid(std::max(a.block.total_chunks, a.last.total_chunks), a.n_blocks + 1), block(kThreads);
    if (dtype == ZO2_F32) {
        if (update) hipLaunchKernelGGL((k1_vectors_kernel<float, true>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((k1_vectors_kernel<float, false>), grid, block, 0, st, a);
    } else {
        if (update) hipLaunchKernelGGL((k1_vectors_kernel<bf16_t, true>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((k1_vectors_kernel<bf16_t, false>), grid, block, 0, st, a);
    }
    ZO2_HIP_LAUNCH_CHECK();
    return ZO2_OK;
}

zo2_status k1_round_launch(K1RoundArgs& a, int wire_dtype, int compute_dtype, hipStream_t st) {
    { const zo2_status s = plan_chunks(a.seg, a.nseg, a.first_chunk, a.total_chunks); if (s != ZO2_OK) return s; }
    ZO2_OP_CHECK(a.n_upd >= 0 && a.n_upd <= K1RoundArgs::kMaxUpdates && a.n_dir >= 0 && a.n_dir <= K1RoundArgs::kMaxDirs && a.theta && (a.n_upd == 0 || a.c_ptr),
                 ZO2_EINVAL, "k1: a round of %d updates and %d directions", a.n_upd, a.n_dir);
    for (int j = 0; j < a.n_dir; ++j) ZO2_OP_CHECK(a.w_plus[j] && a.w_minus[j], ZO2_EINVAL, "k1: W+- of direction %d missing", j);
    if (a.total_chunks == 0 || a.n_upd + a.n_dir == 0) return ZO2_OK;
    ZO2_DISPATCH_WIRE(wire_dtype, W, {
        ZO2_DISPATCH_COMPUTE(compute_dtype, C, { return launch_round<W, C>(a, st); });
    });
    return ZO2_OK;
}

}  // namespace zo2
