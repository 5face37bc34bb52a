// Launch interface of the fused update + perturb kernel (K1).
#pragma once
#include "common.h"
#include "philox.h"

namespace zo2 {

struct K1Seg {
    int64_t off;          // element offset of the segment inside the theta buffer
    uint64_t e0;          // index, inside its tensor, of the segment's first element (multiple of 8)
    uint64_t n;           // elements
    uint32_t tensor_id;   // selects the random stream
    float scale;          // wire scale of the tensor (8-bit formats), else 1
    int64_t woff;         // with K1Args::packed_w: element offset of the segment inside w_plus / w_minus
};

struct K1Args {
    static constexpr int kMaxSeg = 16;
    void* theta;          // wire dtype; rewritten in place when an update is pending
    void* w_plus;         // compute dtype, addressed as w_plus[off - w_off0 + i]
    void* w_minus;        // may be nullptr: only W+ is written (single forward)
    int64_t w_off0;       // element offset (in theta's numbering) that maps to w_plus[0]
    int32_t nseg;
    uint32_t total_chunks;
    float c_imm;          // eta_prev * g_prev, used when c_ptr == nullptr
    int32_t stochastic;   // 1: theta' is stored with stochastic rounding (low-bit wire formats), 0: to nearest
    int32_t reverse;      // 1: the grid walks the chunks from the last to the first
    int32_t packed_w;     // 1: a segment's copies start at w_plus[seg.woff] (segments packed densely) instead of w_plus[off - w_off0]
    int32_t mixed;        // 1 (16-bit storage equal to the compute format, packed_w, update and perturb): segments with woff < 0 are only updated
    float eps;
    const float* c_ptr;   // device scalar holding eta_prev * g_prev (stays on the GPU between steps)
    PhiloxKeys k_prev, k_cur;
    uint32_t first_chunk[kMaxSeg];   // filled in by k1_launch: first workgroup of each segment (0xffffffff past nseg)
    K1Seg seg[kMaxSeg];
};

// The sweep of a round of several directions: any number of deferred updates, each stored before the next is applied, and the
// perturbed copies of up to kMaxDirs directions (or of none), with theta read and written once.
struct K1RoundArgs {
    static constexpr int kMaxUpdates = 16, kMaxDirs = 4;
    void* theta;
    void* w_plus[kMaxDirs];          // addressed as w_plus[j][off - w_off0 + i]
    void* w_minus[kMaxDirs];
    int64_t w_off0;
    const float* c_ptr;              // coefficients of the updates, in order
    int32_t n_upd, n_dir, nseg, stochastic;
    uint32_t total_chunks;
    float eps;
    PhiloxKeys k_upd[kMaxUpdates], k_dir[kMaxDirs];
    uint32_t first_chunk[K1Args::kMaxSeg];
    K1Seg seg[K1Args::kMaxSeg];      // (woff unused)
};
bool k1_round_applicable(int wire_dtype, int compute_dtype);
zo2_status k1_round_launch(K1RoundArgs& a, int wire_dtype, int compute_dtype, hipStream_t st);

// The perturbed (and updated) vectors of all blocks of a step in one launch, and with them those of the final LayerNorm: the same segments
// of every block, `theta_stride` elements and `tid_stride` tensors apart.  float32 and bfloat16, stored in the compute format; lengths in whole
// groups of eight.
struct K1VectorsArgs {
    struct List {
        void *theta, *w_plus, *w_minus;      // (copies packed: a segment's start at woff)
        int32_t nseg;
        uint32_t total_chunks;
        uint32_t first_chunk[K1Args::kMaxSeg];
        K1Seg seg[K1Args::kMaxSeg];
    } block, last;                           // of block 0; of the final LayerNorm
    int64_t theta_stride, w_stride;
    int32_t n_blocks, tid_stride;
    float eps;
    const float* c_ptr;
    PhiloxKeys k_prev, k_cur;
};
zo2_status k1_vectors_launch(K1VectorsArgs& a, int dtype, bool update, hipStream_t st);

// Enqueue K1 over the segments.  update: apply theta' = theta - c z_prev; perturb: write W+, W-.
zo2_status k1_launch(K1Args& a, int wire_dtype, int compute_dtype, bool update, bool perturb, hipStream_t st);
uint32_t k1_chunks(uint64_t n);

}  // namespace zo2
