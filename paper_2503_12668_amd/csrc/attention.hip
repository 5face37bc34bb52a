// Causal multi-head self-attention of the decoder block (Alg. 2 "forward"), flash style:
// keys / values are visited in tiles staged through LDS, the softmax is accumulated online,
// and the S x S score matrix is never written to memory.
//
// Three kernels: the matrix cores for 16-bit inputs (d_head 64, 80, 128) and for float32 (d_head 16, 32, 64, 80, 128), and
// a vector-ALU kernel with float32 arithmetic throughout as the general fallback: one wavefront per 64 queries of one
// (sequence, head); a lane owns one query row.
#include <algorithm>
#include <type_traits>

#include "attention.h"

namespace zo2 {

template <typename T, int DH>
__global__ __launch_bounds__(64) void attention_valu_kernel(const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
                                                            T* __restrict__ out, int seq, int64_t ld) {
    constexpr int KT = 16;                     // keys per tile
    __shared__ float Ks[KT][DH];
    __shared__ float Vs[KT][DH];
    const int lane = threadIdx.x;
    const int q0 = blockIdx.x * 64, head = blockIdx.y, sq = blockIdx.z;
    const size_t base = (size_t)sq * seq * ld + (size_t)head * DH;
    const int i = q0 + lane;                   // this lane's query position
    const bool live = i < seq;
    float qr[DH], o[DH];
#pragma unroll
    for (int d = 0; d < DH; d += 8) {
        Vec<T, 8> t;
        if (live) t = load_vec<T, 8>(q + base + (size_t)i * ld + d);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            qr[d + e] = live ? Fmt<T>::load(t.v[e]) : 0.f;
            o[d + e] = 0.f;
        }
    }
    float m = -INFINITY, l = 0.f;
    const int jend = min(seq, q0 + 64);
    for (int j0 = 0; j0 < jend; j0 += KT) {
        __syncthreads();
        // stage KT keys and values: KT * DH / 8 chunks of 8 elements over 64 lanes
        for (int c = lane; c < KT * DH / 8; c += 64) {
            const int jj = c / (DH / 8), d = (c % (DH / 8)) * 8;
            const int j = j0 + jj;
            if (j < seq) {
                const Vec<T, 8> kk = load_vec<T, 8>(k + base + (size_t)j * ld + d);
                const Vec<T, 8> vv = load_vec<T, 8>(v + base + (size_t)j * ld + d);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    Ks[jj][d + e] = Fmt<T>::load(kk.v[e]);
                    Vs[jj][d + e] = Fmt<T>::load(vv.v[e]);
                }
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) { Ks[jj][d + e] = 0.f; Vs[jj][d + e] = 0.f; }
            }
        }
        __syncthreads();
        float s[KT];
        float tmax = -INFINITY;
#pragma unroll
        for (int jj = 0; jj < KT; ++jj) {
            float acc = 0.f;
#pragma unroll
            for (int d = 0; d < DH; d += 4) {
                const float4 kv = *reinterpret_cast<const float4*>(&Ks[jj][d]);
                acc = __builtin_fmaf(qr[d], kv.x, acc);
                acc = __builtin_fmaf(qr[d + 1], kv.y, acc);
                acc = __builtin_fmaf(qr[d + 2], kv.z, acc);
                acc = __builtin_fmaf(qr[d + 3], kv.w, acc);
            }
            const bool ok = live && (j0 + jj <= i);
            s[jj] = ok ? acc : -INFINITY;
            tmax = fmaxf(tmax, s[jj]);
        }
        if (tmax == -INFINITY) continue;       // nothing visible for this lane in the tile (uniform barriers: none inside)
        const float mn = fmaxf(m, tmax);
        const float resc = expf(m - mn);       // exp(-inf) = 0 on the first visible tile
        l *= resc;
#pragma unroll
        for (int d = 0; d < DH; ++d) o[d] *= resc;
#pragma unroll
        for (int jj = 0; jj < KT; ++jj) {
            const float pj = expf(s[jj] - mn);  // 0 for masked keys
            l += pj;
#pragma unroll
            for (int d = 0; d < DH; d += 4) {
                const float4 vv = *reinterpret_cast<const float4*>(&Vs[jj][d]);
                o[d] = __builtin_fmaf(pj, vv.x, o[d]);
                o[d + 1] = __builtin_fmaf(pj, vv.y, o[d + 1]);
                o[d + 2] = __builtin_fmaf(pj, vv.z, o[d + 2]);
                o[d + 3] = __builtin_fmaf(pj, vv.w, o[d + 3]);
            }
        }
        m = mn;
    }
    if (live) {
        const float inv = 1.0f / l;
#pragma unroll
        for (int d = 0; d < DH; d += 8) {
            Vec<T, 8> t;
#pragma unroll
            for (int e = 0; e < 8; ++e) t.v[e] = Fmt<T>::store(o[d + e] * inv);
            store_vec<T, 8>(out + base + (size_t)i * ld + d, t);
        }
    }
}

// ---------------------------------------------------------------------------------------
// MFMA kernel (bf16 / fp16, d_head 64, 80 or 128).  One wavefront owns 32 queries and walks the
// keys in tiles of 32 staged through LDS.
//
//   S^T = K Q^T   (32 keys x 32 queries)   A operand: K rows, B operand: Q rows
//   O^T += V^T P^T (d_head x 32 queries)   A operand: V^T rows, read out of the key-major V
//                                           tile with the transposing LDS read,
//                                           B operand: P^T taken directly from the S^T
//                                           accumulator registers.
// In the 32x32 accumulator layout a lane holds one query column and 16 key rows
// rho = 8 (v/4) + 4 kh + v%4.  As a B operand of the second product a lane must supply 8
// consecutive contraction slots 8 kh .. 8 kh + 7 per 16-slot step.  Both fit together if
// accumulator row rho carries key pi(rho), pi swapping the bits "kh" and "v/4 & 1" inside each
// 16-block: then registers v = 8 s .. 8 s + 7 are keys 16 s + 8 kh .. + 7, the same run of keys
// a lane holds of its V^T row.  pi is applied for free when choosing which K row a lane loads.
// ---------------------------------------------------------------------------------------
typedef __bf16 att_bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 att_f16x8 __attribute__((ext_vector_type(8)));
typedef float att_f32x16 __attribute__((ext_vector_type(16)));
typedef short att_i16x4 __attribute__((ext_vector_type(4)));

template <typename T> struct AttMfma;
template <> struct AttMfma<bf16_t> {
    static __device__ __forceinline__ att_f32x16 run(uint4 a, uint4 b, att_f32x16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(att_bf16x8, a), __builtin_bit_cast(att_bf16x8, b), c, 0, 0, 0);
    }
};
template <> struct AttMfma<f16_t> {
    static __device__ __forceinline__ att_f32x16 run(uint4 a, uint4 b, att_f32x16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(att_f16x8, a), __builtin_bit_cast(att_f16x8, b), c, 0, 0, 0);
    }
};

// direct-to-LDS load of 16 bytes per lane (lane i lands at lds_base + 16 i); source: wave-uniform base + 32-bit byte offset per lane
__device__ __forceinline__ void att_load_to_lds(const void* sbase, uint32_t voff, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds_base), "v"(voff), "s"(sbase) : "memory");
}
__device__ __forceinline__ void att_load_to_lds(const void* sbase, int64_t off, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds_base), "v"((const char*)sbase + off) : "memory");
}

// Maximum over a lane and its partner in the other half of the wavefront: the swap hands every lane the lower half's value in one
// register and the upper half's in the other (a vector instruction; as an LDS permutation it cost a trip per tile).
__device__ __forceinline__ float att_max_halves(float x) {
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    const auto h = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    const uint32_t lower = h[0], upper = h[1];              // (as scalars: a bit cast of h[1] itself reads h[0])
    return fmaxf(__builtin_bit_cast(float, lower), __builtin_bit_cast(float, upper));
}

// Workgroup id -> (block of queries, pair of sequence and head).  The query blocks of one pair read the same
// keys and values; consecutive workgroup ids go to different XCDs, each with its own L2, so those blocks get ids that
// are congruent mod 8.  An XCD takes its pairs in groups of `group`, and in a group late query blocks (more keys under the
// causal mask) first.
__device__ __forceinline__ void att_place(int nqb, int n_pairs, int group, int& qb, int& pair) {
    const int pairs_xcd = (n_pairs + 7) >> 3, slot = blockIdx.x >> 3;
    const int first = slot / (group * nqb) * group, size = min(group, pairs_xcd - first);
    const int local = slot - first * nqb;
    qb = nqb - 1 - local / size;
    pair = (first + local % size) * 8 + (int)(blockIdx.x & 7);
}

// One workgroup = 128 queries of one (sequence, head); wavefront w owns queries 32 w .. 32 w + 31.
// Key tiles of 32 keys are brought into LDS once per workgroup (direct-to-LDS loads, a ring of four buffers,
// one barrier per tile) and shared by the four wavefronts; a wavefront skips the tiles past its
// diagonal.  K and V tiles: 32 rows of d_head elements, 16-byte chunks XOR-swizzled by swz(row).
// The transposing 8-byte LDS read works on groups of 16 lanes: lane 4 j + g of a group supplies the
// address of 4 consecutive elements, and lane 4 g + c receives element c of lanes g, 4 + g, 8 + g, 12 + g.
// Pointing lane 4 j + g at V[key0 + j][m0 + 4 g ..] therefore hands lane i the keys key0 .. key0 + 3 of
// column m0 + i: four consecutive contraction slots of its V^T row.
//
// What bounds it: the exponentials and the rest of the softmax take about as many cycles of the vector ALU as both products
// take of the matrix cores, so the two have to run side by side.  The first product is therefore one tile ahead: while tile t is
// exponentiated, the MFMAs of K Q^T of tile t + 1 run, and the maximum of tile t + 1 is found under the MFMAs of V^T P^T of tile t.
// The order of every sum is that of one tile after the other.  2 x 8192 queries, 40 heads of 128: 1690 us one tile after the other
// with banks met four times, 1380 now (1.0 PFLOP/s; matrix cores and vector ALU each busy half of the time); 32 heads of 64: 727 -> 670.
// Above d_head 64 a wavefront in its second product goes before its neighbour's exponentials (2 %; at 64 that costs 2 %).
template <typename T, int DH, bool FAR>      // FAR: rows lie too far apart for 32-bit offsets inside a tile
__global__ __launch_bounds__(256, 2) void attention_mfma_kernel(const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
                                                                 T* __restrict__ out, int seq, int64_t ld, int n_heads, int n_pairs, int group) {
    constexpr int KS = DH / 16;          // contraction steps of the first product
    constexpr int DT = (DH + 31) / 32;   // 32-row tiles of O^T (rows past DH are computed on padding and dropped)
    constexpr int DHP = DH <= 64 ? 64 : 128;   // LDS row pitch in elements: a power of two, so that the swizzle stays inside the row
    constexpr int KCH = DHP / 8;         // 16-byte chunk positions per LDS row
    constexpr int GCH = DH / 8;          // 16-byte chunks per row in memory
    constexpr int KTILE = 32 * DHP * 2, BUF = 2 * KTILE;                  // K tile, then V tile
    constexpr int KINSTR = KTILE / 1024 / 4;                              // direct-to-LDS loads per wavefront per tile and operand
    constexpr int NBUF = 4;                                               // ring of K / V tiles: loads run up to NBUF - 1 tiles ahead
    __shared__ __attribute__((aligned(1024))) char lds[NBUF * BUF];
    // Both reads of a tile should meet every bank once.  A transposing read of 32 lanes takes 64 bytes of each of four
    // consecutive rows: those go to different quarters of the banks (a row is all 64 banks, or half of them at a pitch of 128
    // bytes).  A 16-byte read of K takes one chunk of each row: rows that agree in their place among four differ by the next two bits.
    // (With the chunk index XORed by row & 7, all lanes of a transposing read met in a quarter of the banks.)
    auto swz = [](int row) { return DHP == 128 ? ((row & 3) << 2) | ((row >> 2) & 3) : ((row & 2) << 1) | ((row >> 2) & 3); };
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 31, kh = lane >> 5;
    const int nqb = (seq + 127) >> 7;
    int qb, pair;
    att_place(nqb, n_pairs, group, qb, pair);
    if (pair >= n_pairs) return;                             // padding of the last group of 8 (whole workgroup)
    const int head = pair % n_heads, sq = pair / n_heads;
    const int q0 = qb * 128 + wave * 32;
    const bool active = q0 < seq;                            // inactive wavefronts still load and synchronise
    const size_t base = (size_t)sq * seq * ld + (size_t)head * DH;
    const int qi = q0 + r;                                   // this lane's query
    const int qrow = min(qi, seq - 1);
    // key carried by accumulator row rho: swap bits 2 (kh of rho) and 3 inside each 16-block
    const int pr = (r & 0x13) | ((r & 4) << 1) | ((r & 8) >> 1);

    uint4 qf[KS];
#pragma unroll
    for (int c = 0; c < KS; ++c) qf[c] = *reinterpret_cast<const uint4*>(q + base + (size_t)qrow * ld + c * 16 + kh * 8);

    att_f32x16 o[DT];
#pragma unroll
    for (int d = 0; d < DT; ++d)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[d][v] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;
    constexpr float kLog2e = 1.4426950408889634f;

    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
    const int wg_last_q = min(qb * 128 + 127, seq - 1);
    const int wg_last_tile = wg_last_q >> 5;
    const int my_last_tile = active ? q0 >> 5 : -1;
    // transposing read: lane = 16 g16 + a; the group covers columns 16 (g16 & 1) .. + 15 and keys 8 (g16 >> 1) + 4 h + (a >> 2)
    const int g16 = lane >> 4, a16 = lane & 15;

    // loader plan: offsets inside a tile, the same for every tile that lies wholly inside the sequence
    using Off = std::conditional_t<FAR, int64_t, uint32_t>;
    Off ld_off[KINSTR];
    uint32_t ld_chunk[KINSTR];
    int ld_row[KINSTR];
#pragma unroll
    for (int x = 0; x < KINSTR; ++x) {                       // 1024 / (2 DHP) rows per instruction
        ld_row[x] = (wave * KINSTR + x) * (512 / DHP) + lane / KCH;
        int chunk = (lane % KCH) ^ swz(ld_row[x]);
        if (GCH < KCH && chunk >= GCH) chunk &= 7;           // padding positions of a row repeat a real chunk (finite, never used in a kept result)
        ld_chunk[x] = chunk * 16;
        ld_off[x] = (Off)ld_row[x] * (Off)ld * 2 + ld_chunk[x];
    }
    auto issue_tile = [&](int tile, int buf) {
        const int j0 = tile * 32;
        const T* kt = k + base + (size_t)j0 * ld;
        const T* vt = v + base + (size_t)j0 * ld;
        const int last = seq - 1 - j0;                       // rows past the end repeat the last one (masked keys)
#pragma unroll
        for (int x = 0; x < KINSTR; ++x) {
            const Off off = last >= 31 ? ld_off[x] : (Off)min(ld_row[x], last) * (Off)ld * 2 + ld_chunk[x];
            const uint32_t dst = lds0 + buf * BUF + (wave * KINSTR + x) * 1024;
            att_load_to_lds(kt, off, dst);
            att_load_to_lds(vt, off, dst + KTILE);
        }
    };
    // where this lane reads in a tile of K (one 16-byte chunk of row pr per step) and of V
    uint32_t k_at[KS], v_at[DT][2];
#pragma unroll
    for (int c = 0; c < KS; ++c) k_at[c] = pr * (DHP * 2) + (((2 * c + kh) ^ swz(pr)) * 16);
#pragma unroll
    for (int d = 0; d < DT; ++d)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int key = 8 * (g16 >> 1) + 4 * h + (a16 >> 2);                       // + 16 s2, which leaves swz() alone
            const int chunk = 4 * d + 2 * (g16 & 1) + ((a16 & 3) >> 1);
            v_at[d][h] = KTILE + key * (DHP * 2) + ((chunk ^ swz(key)) * 16) + 8 * (a16 & 1);
        }
    auto scores = [&](int buf) {                             // S^T = K Q^T of the tile in `buf`
        uint4 kf[KS];
#pragma unroll
        for (int c = 0; c < KS; ++c) kf[c] = *reinterpret_cast<const uint4*>(lds + buf * BUF + k_at[c]);
        att_f32x16 st;
#pragma unroll
        for (int v = 0; v < 16; ++v) st[v] = 0.f;
#pragma unroll
        for (int c = 0; c < KS; ++c) st = AttMfma<T>::run(kf[c], qf[c], st);
        return st;
    };
    auto mask = [&](int tile, att_f32x16& st) {              // only the diagonal tile has hidden keys; the branch is wave-uniform
        if (tile != my_last_tile) return;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            // accumulator row rho = 8 (v/4) + 4 kh + v%4 carries key j0 + pi(rho) = j0 + 16 (v/8) + 8 kh + v%8
            const int key = tile * 32 + 16 * (v >> 3) + 8 * kh + (v & 7);
            if (key > qi) st[v] = -INFINITY;
        }
    };
    auto tile_max = [&](const att_f32x16& st) {
        float tmax = st[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) tmax = fmaxf(tmax, st[v]);
        return att_max_halves(tmax);
    };
    att_f32x16 st;                                           // scores of the tile at hand, and their maximum
    float tmax = 0.f;

    // tile `tile` in buffer `cur` (= tile % NBUF): its scores are at hand
    auto process_tile = [&](int tile, int cur) {
        const float m_new = fmaxf(m_run, tmax);              // finite: key j0 <= q0 <= qi is always visible in tile 0
        // the running maximum of a query rarely moves after its first tiles: the accumulators are rescaled only when it
        // moved for some query of this wavefront
        if (__builtin_amdgcn_ballot_w64(m_new > m_run) != 0) {
            const float resc = __builtin_amdgcn_exp2f((m_run - m_new) * kLog2e);
            l_run *= resc;
#pragma unroll
            for (int d = 0; d < DT; ++d)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[d][v] *= resc;
            m_run = m_new;
        }
        // (of the tile after the last one the buffer holds other bytes, or none yet: their products are not used)
        att_f32x16 next = scores((cur + 1) % NBUF);
        const float m2 = m_new * kLog2e;
        float psum = 0.f;
        uint4 pf[2];
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
            Vec<T, 8> pv;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(st[8 * s2 + e], kLog2e, -m2));      // exp(st - m_new)
                psum += p;
                pv.v[e] = Fmt<T>::store(p);
            }
            pf[s2] = __builtin_bit_cast(uint4, pv);
        }
        l_run += psum;
        uint4 vf[DT][2];
#pragma unroll
        for (int d = 0; d < DT; ++d)
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2) {
                att_i16x4 half[2];
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    half[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) att_i16x4*)(lds + cur * BUF + v_at[d][h] + s2 * 16 * DHP * 2));
                vf[d][s2] = make_uint4(__builtin_bit_cast(uint2, half[0]).x, __builtin_bit_cast(uint2, half[0]).y,
                                       __builtin_bit_cast(uint2, half[1]).x, __builtin_bit_cast(uint2, half[1]).y);
            }
        // (held here, or the compiler moves the exponentials behind the branch below and away from those MFMAs)
        asm volatile("" : "+v"(pf[0].x), "+v"(pf[0].y), "+v"(pf[0].z), "+v"(pf[0].w), "+v"(pf[1].x), "+v"(pf[1].y), "+v"(pf[1].z), "+v"(pf[1].w), "+v"(l_run));
        mask(tile + 1, next);
        // ---- O^T += V^T P^T
        if constexpr (DH > 64) __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
            for (int d = 0; d < DT; ++d) o[d] = AttMfma<T>::run(vf[d][s2], pf[s2], o[d]);
        st = next;
        tmax = tile_max(st);
        if constexpr (DH > 64) __builtin_amdgcn_s_setprio(0);
    };

    // A tile is 8 - 16 KB and its MFMAs take a few hundred cycles, far less than a trip to memory, so several
    // tiles are kept in flight; direct-to-LDS loads complete in issue order, so "all but the loads of the younger
    // tile" is an exact wait for a tile.
#pragma unroll
    for (int t = 0; t < NBUF - 1; ++t)
        if (t <= wg_last_tile) issue_tile(t, t);
    // (the Q fragments were requested before the tiles; consuming them here puts the compiler's wait for them in front
    // of the loop instead of inside it, where it would also wait for every tile in flight)
#pragma unroll
    for (int c = 0; c < KS; ++c) asm volatile("" : : "v"(qf[c].x), "v"(qf[c].y), "v"(qf[c].z), "v"(qf[c].w));
    if (wg_last_tile >= 2) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(2 * 2 * KINSTR) : "memory");
    else if (wg_last_tile == 1) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(2 * KINSTR) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    st = scores(0);
    mask(0, st);
    tmax = tile_max(st);
    auto step = [&](int tile, auto cur_c) {                  // the buffer as a constant: its offset is part of the LDS instructions
        constexpr int cur = decltype(cur_c)::value;
        // own loads of the next tile landed; own reads of the buffer that is refilled below are done
        if (tile + 2 <= wg_last_tile) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"(2 * KINSTR) : "memory");
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __syncthreads();
        if (tile + NBUF - 1 <= wg_last_tile) issue_tile(tile + NBUF - 1, (cur + NBUF - 1) % NBUF);   // into the buffer of tile - 1
        if (tile <= my_last_tile) process_tile(tile, cur);
    };
    for (int tile = 0; tile <= wg_last_tile; tile += NBUF) {
        step(tile, std::integral_constant<int, 0>{});
        if (tile + 1 <= wg_last_tile) step(tile + 1, std::integral_constant<int, 1>{});
        if (tile + 2 <= wg_last_tile) step(tile + 2, std::integral_constant<int, 2>{});
        if (tile + 3 <= wg_last_tile) step(tile + 3, std::integral_constant<int, 3>{});
    }
    const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
    const float inv = 1.0f / l_tot;
    if (active && qi < seq) {
        T* op = out + base + (size_t)qi * ld;
#pragma unroll
        for (int d = 0; d < DT; ++d)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                if (d * 32 + 8 * g >= DH) continue;          // rows of the last O^T tile that lie past d_head
                Vec<T, 4> ov;
#pragma unroll
                for (int e = 0; e < 4; ++e) ov.v[e] = Fmt<T>::store(o[d][4 * g + e] * inv);
                store_vec<T, 4>(op + d * 32 + 8 * g + 4 * kh, ov);
            }
    }
}

// Pairs of (sequence, head) that an XCD takes together, long query blocks first.  More of them keep the compute units evenly
// busy to the end, fewer keep the keys and values of all of them in the XCD's L2: 8 up to 4096 queries, fewer beyond,
// in groups of about equal size (nqb: blocks of 128 queries).  2 x 2048 queries, 40 heads of 128: 136 us a pair at a time, 124 with 4, 110 with
// all ten of an XCD; 16 x 512, 32 heads of 80: 69, 58 with 4, 56 with 8, 70 with all 64; 2 x 8192, 40 of 128: 1438, 1380 with 4, 1422.
// float32, a pair at a time -> this: 2 x 2048, 12 heads of 64: 308 -> 199; 4 x 512, 32 of 80: 112 -> 88; 4 x 384, 32 of 64: 50 -> 46.
static int att_group(int n_pairs, int nqb) {
    const int pairs_xcd = (n_pairs + 7) / 8, target = nqb <= 32 ? 8 : std::max(1, 256 / nqb);
    const int groups = std::max(1, (2 * pairs_xcd + target) / (2 * target));
    return (pairs_xcd + groups - 1) / groups;
}

template <typename T>
static zo2_status launch_mfma_att(const T* q, const T* k, const T* v, T* out, int n_seq, int seq, int n_heads, int d_head,
                                  int64_t ld, hipStream_t st) {
    const int n_pairs = n_heads * n_seq, nqb = (seq + 127) / 128;
    const int group = att_group(n_pairs, nqb);
    const dim3 grid((unsigned)(8 * nqb) * (unsigned)((n_pairs + 7) / 8)), block(256);
    const bool far = ld >= (int64_t)1 << 25;       // 31 rows of 2^25 elements are 2 GB behind the first
#define ZO2_ATT16(DH)                                                                                                                       \
    if (far) hipLaunchKernelGGL((attention_mfma_kernel<T, DH, true>), grid, block, 0, st, q, k, v, out, seq, ld, n_heads, n_pairs, group); \
    else hipLaunchKernelGGL((attention_mfma_kernel<T, DH, false>), grid, block, 0, st, q, k, v, out, seq, ld, n_heads, n_pairs, group)
    if (d_head == 64) { ZO2_ATT16(64); }
    else if (d_head == 80) { ZO2_ATT16(80); }
    else { ZO2_ATT16(128); }
#undef ZO2_ATT16
    ZO2_HIP_LAUNCH_CHECK();
    return ZO2_OK;
}

// ---------------------------------------------------------------------------------------
// float32 on the matrix cores (v_mfma_f32_16x16x4_f32: float32 products and accumulation).  One wavefront = one workgroup =
// 16 QT queries of one (sequence, head); keys are visited 16 at a time, straight from L2 into registers, the next 16 on
// their way meanwhile: 8 KB (d_head 64) per 1024 QT cycles of MFMA, which the caches deliver without a trip through LDS,
// and without barriers small launches spread over as many compute units as they have groups of 16 queries.  The
// vector-ALU kernel has one wavefront per 64 queries, which walk their keys one by one: 62 us at 1 x 64 tokens (24 pairs of
// sequence and head) against 7 here, 365 us at 2 x 384 (128 pairs) against 46.
//   S^T = K Q^T    lane (r, kg) supplies key row r / query row r at the d_head positions 16 c + 4 kg .. + 3 with one 16-byte
//                  load: element t of it is contraction slot kg of issue t, the same positions for both operands;
//   O^T += V^T P^T  accumulator element e of S^T is key 4 kg + e of query r: contraction slot kg of issue e, where it is used
//                  as it stands.  Row r of O^T's tile 4 g + d is d_head position 64 g + 4 r + d, so that a lane's 16-byte
//                  load of a V row feeds four tiles and its results are four consecutive positions of the output.
// ---------------------------------------------------------------------------------------
typedef float att_f32x4 __attribute__((ext_vector_type(4)));
typedef float att_f32x2 __attribute__((ext_vector_type(2)));

template <int DH, int QT>
__global__ __launch_bounds__(64) void attention_f32_mfma_kernel(const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
                                                                float* __restrict__ out, int seq, int64_t ld, int n_heads, int n_pairs, int group) {
    static_assert(DH % 16 == 0 && DH % 64 != 48, "16-column tiles of the output: groups of four, then one or two");
    constexpr int DT = DH / 16, G4 = DH / 64, REM = DT % 4;      // tiles; groups of four; the rest
    const int lane = threadIdx.x, r = lane & 15, kg = lane >> 4;
    const int nqb = (seq + 16 * QT - 1) / (16 * QT);
    int qb, pair;
    att_place(nqb, n_pairs, group, qb, pair);
    if (pair >= n_pairs) return;
    const int head = pair % n_heads, sq = pair / n_heads;
    const int q0 = qb * 16 * QT;
    const size_t base = (size_t)sq * seq * ld + (size_t)head * DH;
    const float* kp = k + base + 4 * kg;
    const float* vp = v + base;

    att_f32x4 qf[QT][DT], o[QT][DT];
    float m_run[QT], l_run[QT];
#pragma unroll
    for (int t = 0; t < QT; ++t) {
        const float* qp = q + base + (size_t)min(q0 + 16 * t + r, seq - 1) * ld + 4 * kg;
#pragma unroll
        for (int c = 0; c < DT; ++c) {
            qf[t][c] = *reinterpret_cast<const att_f32x4*>(qp + 16 * c);
            o[t][c] = att_f32x4{0.f, 0.f, 0.f, 0.f};
        }
        m_run[t] = -INFINITY;
        l_run[t] = 0.f;
    }
    // rows past the end of the sequence repeat its last one: their keys are masked
    auto load_keys = [&](int j0, att_f32x4 (&kf)[DT], float (&vf)[4][DT]) {
        const float* kr = kp + (size_t)min(j0 + r, seq - 1) * ld;
#pragma unroll
        for (int c = 0; c < DT; ++c) kf[c] = *reinterpret_cast<const att_f32x4*>(kr + 16 * c);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float* vr = vp + (size_t)min(j0 + 4 * kg + e, seq - 1) * ld;
#pragma unroll
            for (int g = 0; g < G4; ++g) {
                const att_f32x4 x = *reinterpret_cast<const att_f32x4*>(vr + 64 * g + 4 * r);
#pragma unroll
                for (int d = 0; d < 4; ++d) vf[e][4 * g + d] = x[d];
            }
            if (REM == 2) {
                const att_f32x2 x = *reinterpret_cast<const att_f32x2*>(vr + 64 * G4 + 2 * r);
                vf[e][DT - 2] = x[0];
                vf[e][DT - 1] = x[1];
            }
            if (REM == 1) vf[e][DT - 1] = vr[64 * G4 + r];
        }
    };
    att_f32x4 kf[DT], kn[DT];
    float vf[4][DT], vn[4][DT];
    load_keys(0, kf, vf);
    const int tiles = (min(q0 + 16 * QT, seq) + 15) >> 4;
    for (int tile = 0; tile < tiles; ++tile) {
        const int j0 = tile * 16;
        load_keys(min(j0 + 16, seq - 1), kn, vn);
        att_f32x4 st[QT];
#pragma unroll
        for (int t = 0; t < QT; ++t) st[t] = att_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < DT; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int t = 0; t < QT; ++t) st[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][i], qf[t][c][i], st[t], 0, 0, 0);
#pragma unroll
        for (int t = 0; t < QT; ++t) {
            const int qi = q0 + 16 * t + r;
            float tmax = -INFINITY;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (j0 + 4 * kg + e > qi) st[t][e] = -INFINITY;
                tmax = fmaxf(tmax, st[t][e]);
            }
            tmax = fmaxf(tmax, __shfl_xor(tmax, 16, 64));
            tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
            // (-inf as long as every score so far was: their weights are 0, and exp(-inf + inf) must not come in)
            const float m_new = fmaxf(m_run[t], tmax), base = m_new == -INFINITY ? 0.f : m_new;
            if (__builtin_amdgcn_ballot_w64(m_new > m_run[t]) != 0) {
                const float resc = expf(m_run[t] - base);
                l_run[t] *= resc;
#pragma unroll
                for (int d = 0; d < DT; ++d) o[t][d] *= resc;
                m_run[t] = m_new;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                st[t][e] = expf(st[t][e] - base);
                l_run[t] += st[t][e];
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int d = 0; d < DT; ++d)
#pragma unroll
                for (int t = 0; t < QT; ++t) o[t][d] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[e][d], st[t][e], o[t][d], 0, 0, 0);
#pragma unroll
        for (int c = 0; c < DT; ++c) {
            kf[c] = kn[c];
#pragma unroll
            for (int e = 0; e < 4; ++e) vf[e][c] = vn[e][c];
        }
    }
#pragma unroll
    for (int t = 0; t < QT; ++t) {
        float l_tot = l_run[t] + __shfl_xor(l_run[t], 16, 64);
        l_tot += __shfl_xor(l_tot, 32, 64);
        const float inv = 1.0f / l_tot;
        const int qi = q0 + 16 * t + r;
        if (qi >= seq) continue;
        float* op = out + base + (size_t)qi * ld;
#pragma unroll
        for (int e = 0; e < 4; ++e) {                            // accumulator element e: tile row 4 kg + e
#pragma unroll
            for (int g = 0; g < G4; ++g)
                *reinterpret_cast<att_f32x4*>(op + 64 * g + 4 * (4 * kg + e)) =
                    att_f32x4{o[t][4 * g][e] * inv, o[t][4 * g + 1][e] * inv, o[t][4 * g + 2][e] * inv, o[t][4 * g + 3][e] * inv};
            if (REM == 2) *reinterpret_cast<att_f32x2*>(op + 64 * G4 + 2 * (4 * kg + e)) = att_f32x2{o[t][DT - 2][e] * inv, o[t][DT - 1][e] * inv};
            if (REM == 1) op[64 * G4 + 4 * kg + e] = o[t][DT - 1][e] * inv;
        }
    }
}

template <int DH, int QT>
static void launch_f32_att(const float* q, const float* k, const float* v, float* out, int n_seq, int seq, int n_heads, int64_t ld, hipStream_t st) {
    const int n_pairs = n_heads * n_seq, nqb = (seq + 16 * QT - 1) / (16 * QT);
    const dim3 grid((unsigned)(8 * nqb) * (unsigned)((n_pairs + 7) / 8)), block(64);
    hipLaunchKernelGGL((attention_f32_mfma_kernel<DH, QT>), grid, block, 0, st, q, k, v, out, seq, ld, n_heads, n_pairs, att_group(n_pairs, (seq + 127) / 128));
}

template <typename T>
static zo2_status launch_valu(const T* q, const T* k, const T* v, T* out, int n_seq, int seq, int n_heads, int d_head,
                              int64_t ld, hipStream_t st) {
    const dim3 grid((seq + 63) / 64, n_heads, n_seq), block(64);
    switch (d_head) {
#define ZO2_ATT_CASE(D) \
    case D: hipLaunchKernelGGL((attention_valu_kernel<T, D>), grid, block, 0, st, q, k, v, out, seq, ld); break;
        ZO2_ATT_CASE(8) ZO2_ATT_CASE(16) ZO2_ATT_CASE(32) ZO2_ATT_CASE(64) ZO2_ATT_CASE(80) ZO2_ATT_CASE(128)
#undef ZO2_ATT_CASE
        default:
            set_op_error("attention: d_head %d not supported (8, 16, 32, 64, 80, 128)", d_head);
            return ZO2_EINVAL;
    }
    ZO2_HIP_LAUNCH_CHECK();
    return ZO2_OK;
}

zo2_status attention_launch(int dtype, const void* q, const void* k, const void* v, void* out, int n_seq, int seq, int n_heads,
                            int d_head, int64_t ld, int vector_kernel, hipStream_t st) {
    if (n_seq == 0 || seq == 0) return ZO2_OK;
    ZO2_OP_CHECK(n_seq > 0 && seq > 0 && n_heads > 0 && d_head > 0, ZO2_EINVAL, "attention: bad shape");
    ZO2_OP_CHECK(q && k && v && out, ZO2_EINVAL, "attention: NULL buffer");
    ZO2_OP_CHECK(ld >= (int64_t)n_heads * d_head && ld % 8 == 0, ZO2_EINVAL, "attention: bad leading dimension");
    ZO2_OP_CHECK(n_seq <= 65535 && n_heads <= 65535 && (int64_t)n_seq * n_heads * ((seq + 127) / 128 + 1) < (int64_t)1 << 30, ZO2_EINVAL,
                 "attention: grid too large");
    {   // every kernel moves groups of 8 elements
        const uintptr_t align = 8 * (uintptr_t)zo2_dtype_size(dtype);
        ZO2_OP_CHECK(align != 0 && ((uintptr_t)q % align) == 0 && ((uintptr_t)k % align) == 0 && ((uintptr_t)v % align) == 0 &&
                     ((uintptr_t)out % align) == 0, ZO2_EINVAL, "attention: unknown dtype, or operands not aligned to 8 elements");
    }
    if (!vector_kernel && dtype != ZO2_F32 && (d_head == 64 || d_head == 80 || d_head == 128)) {
        if (dtype == ZO2_BF16)
            return launch_mfma_att<bf16_t>((const bf16_t*)q, (const bf16_t*)k, (const bf16_t*)v, (bf16_t*)out, n_seq, seq, n_heads, d_head, ld, st);
        return launch_mfma_att<f16_t>((const f16_t*)q, (const f16_t*)k, (const f16_t*)v, (f16_t*)out, n_seq, seq, n_heads, d_head, ld, st);
    }
    const bool f32_fits = (int64_t)(n_seq * (int64_t)n_heads + 8) * ((seq + 15) / 16) < (int64_t)1 << 25;      // its grid of 64-thread workgroups
    if (!vector_kernel && dtype == ZO2_F32 && f32_fits && (d_head == 16 || d_head == 32 || d_head == 64 || d_head == 80 || d_head == 128)) {
        // 16 queries per wavefront: a tile's loads take longer than its products, and more wavefronts per SIMD cover each other's.  32
        // read the keys half as often, which counts where there are wavefronts in any case (d_head 64, 32 heads, 32 -> 16 queries, us:
        // 4 x 384 63 -> 46, 2 x 1024 139 -> 128, 8 x 1024 422 against 428, 4 x 2048 749 against 784; 32 x 256 of 32 91 -> 88).
        // Beyond d_head 64 a wavefront's registers hold no more than 16.
        const bool wide = (int64_t)n_seq * n_heads * ((seq + 31) / 32) >= 32 * (int64_t)device_cu_count();
        const float *qf = (const float*)q, *kf = (const float*)k, *vf = (const float*)v;
        float* of = (float*)out;
#define ZO2_ATT_CASE(D, QT) launch_f32_att<D, QT>(qf, kf, vf, of, n_seq, seq, n_heads, ld, st)
        switch (d_head) {
            case 16: wide ? ZO2_ATT_CASE(16, 2) : ZO2_ATT_CASE(16, 1); break;
            case 32: wide ? ZO2_ATT_CASE(32, 2) : ZO2_ATT_CASE(32, 1); break;
            case 64: wide ? ZO2_ATT_CASE(64, 2) : ZO2_ATT_CASE(64, 1); break;
            case 80: ZO2_ATT_CASE(80, 1); break;
            case 128: ZO2_ATT_CASE(128, 1); break;
        }
#undef ZO2_ATT_CASE
        ZO2_HIP_LAUNCH_CHECK();
        return ZO2_OK;
    }
    ZO2_DISPATCH_COMPUTE(dtype, T, {
        return launch_valu<T>((const T*)q, (const T*)k, (const T*)v, (T*)out, n_seq, seq, n_heads, d_head, ld, st);
    });
    return ZO2_OK;
}

}  // namespace zo2
