// Launch interface of the projection GEMMs (QKV, attention output, FFN, LM head).
#pragma once
#include "common.h"

namespace zo2 {

struct GemmProblem {
    const void* X;          // [M, ldx] activations (compute dtype)
    const void* W;          // [N, ldw] weights, row n = output feature n
    const void* bias;       // [N] or nullptr
    const float* residual;  // [M, ldy] float32 or nullptr
    void* Y;                // [M, ldy] compute dtype or float32
    float out_scale;        // multiplies (acc + bias); 1/sqrt(d_head) for the query projection
    int32_t pad_;
    // cross-entropy mode (GemmArgs::ce_mode): nothing is stored to Y; per row and per 64-column span the
    // kernel writes max and sum(exp(y - max)), and the logit of the row's label.  The partial arrays are
    // span-major: span s of row m sits at [s * part_ld + m], s < 4 * ceil(N / 256).  No bias, relu, residual.
    const int32_t* labels;  // [M] device, -100 = ignored (partials are still written)
    float* part_max;        // [4 * ceil(N / 256), part_ld]
    float* part_sum;        // [4 * ceil(N / 256), part_ld]
    float* label_logit;     // [M]
};

struct GemmArgs {
    static constexpr int kMaxProblems = 24;      // q/k/v x two streams x four directions, or x two k pieces x two directions
    static constexpr int kMaxPieces = 12;        // problems x pieces of one direction's launch
    int32_t M, N, K;
    int64_t ldx, ldw, ldy;
    int64_t part_ld;        // cross-entropy mode: elements between consecutive spans of the partial arrays (>= M)
    int32_t relu;
    int32_t out_f32;        // Y is float32 instead of the compute dtype
    int32_t ce_mode;        // 1: LM-head + cross-entropy partials instead of an output matrix (256 x 256 kernel only)
    int32_t like_nprob;     // ce_mode: spans are added up as in a launch of this many problems (0: no matter)
    int32_t kpiece;         // float32 and 128 x 128 kernels: k per piece (K when the launch is not split), a multiple of 32 or 64 if there are several
    int32_t large_only;     // 1: not on the 128 x 128 kernel, whose wavefronts add a slab's k in two halves
    int32_t nprob;          // problems of identical shape, one per grid.z (the +/- streams, q/k/v)
    // Cycle stamps of one workgroup, for the measurement build of the 256 x 256 kernel only (-DZO2_GEMM_STAMPS: build.py
    // --gemm-stamps); NULL otherwise.  64 device words: s_memtime at the start of each tile, after the wait for its first
    // slab, after its k loop and after its epilogue (4 per tile, up to 14 tiles), then [60] cycles spent in the waits for
    // loads and [61] at the barriers in the middle of the slabs, [62] the number of tiles.
    unsigned long long* stamps;
    GemmProblem p[kMaxProblems];
};
static constexpr int kStampWorkgroup = 37;      // the workgroup that writes them

// Y = act((X W^T + bias) * out_scale) + residual for every problem; float32 accumulation.
// of_rows > M: rows of a matrix of that many, on the kernel that all of them at once would run on (the kernel, not its
// tiles' height, is what the order of a sum depends on: rows in chunks then have the bits of one launch).
zo2_status gemm_launch(const GemmArgs& a, int dtype, hipStream_t st, int of_rows = 0);
// the 256 x 256 x 64 kernel (bf16 / fp16, K % 128 == 0); gemm_launch picks it for large problems
zo2_status gemm_launch_256(const GemmArgs& a, int dtype, hipStream_t st);
// Split-k for launches that leave most compute units idle (few rows per stream): each problem is cut into `splits` pieces
// of K / splits along k, the pieces run as problems of their own into float32 partial sums
// ([nprob][splits][M][N] in `workspace`), and a second kernel adds a problem's pieces in order (deterministic) and applies
// bias, scale, ReLU and residual.  gemm_pick_splits: 1 (do not split), 2 or 4 for a launch of `nprob` problems.
int gemm_pick_splits(int M, int N, int K, int nprob, int dtype);
size_t gemm_splitk_workspace_bytes(int M, int N, int nprob, int splits);
// sum = false: the pieces stay in the workspace, the caller adds them and finishes the values.
zo2_status gemm_launch_splitk(const GemmArgs& a, int dtype, int splits, void* workspace, size_t workspace_bytes, hipStream_t st, bool sum = true);
// float32 (gemm_f32.hip): tiles of `rows` = 32, 64 or 128 rows; splits > 1: a.kpiece k per piece, Y = partial sums, a plane per piece
zo2_status gemm_launch_f32(const GemmArgs& a, int splits, int rows, hipStream_t st);
// Split-k for float32: any number of pieces that the workspace holds.
int gemm_f32_pick_splits(int M, int N, int K, int nprob, size_t workspace_bytes);
// sum = false: the pieces stay in the workspace ([problem][piece][M][N]), the caller adds them and finishes the values.
zo2_status gemm_launch_f32_splitk(const GemmArgs& a, int splits, void* workspace, size_t workspace_bytes, hipStream_t st, bool sum = true);
// What a block projection runs on: rows 0 the large-tile kernel (gemm_launch / gemm_launch_splitk), 64 or 128 (256 in
// gemm_launch_groups only) the 128 x 128
// kernel with tiles of that height (gemm_launch_mid_splitk); splits: pieces along k that the workspace holds.
struct GemmChoice { int rows, splits; };
GemmChoice gemm_choose(const GemmArgs& a, int dtype, size_t workspace_bytes);
// The launch that choice `k`, made for a.nprob / groups problems, stands for: the same sums for `groups` times as many problems at once
// (tile heights, which do not change a sum's order, are chosen anew).  Workspace: the pieces of all of them.
int gemm_groups_rows(const GemmArgs& a, int dtype, GemmChoice k);      // (k.rows not 0) that height
zo2_status gemm_launch_groups(const GemmArgs& a, int dtype, GemmChoice k, int groups, void* workspace, size_t workspace_bytes, hipStream_t st);
bool gemm256_is_forced();                 // a tile height or wavefront count is forced: the large-tile kernel is meant
zo2_status gemm_launch_mid_splitk(const GemmArgs& a, int dtype, int rows, int splits, void* workspace, size_t workspace_bytes, hipStream_t st, bool sum = true);
// 0 (default): the 256 x 256 kernel picks 256- or 128-row tiles per launch; 128 / 256: every launch uses that height
void gemm256_force_tile_rows(int rows);
void gemm256_force_waves(int waves);      // 0: chosen per launch; 4 or 8: every launch of 256-row tiles
bool gemm256_applicable(const GemmArgs& a, int dtype);
// How the large kernel runs a launch: tiles of rows[0] rows, and where it is two launches rows[1] for the problems from `probs` on, or
// for the tile columns (of 256) from `cols` on of every problem.
struct GemmTiles { int rows[2], probs, cols; };
GemmTiles gemm256_tiles(const GemmArgs& a);
int gemm_f32_tile_rows(int M, int N, int K, int nprob);      // of an uncut float32 launch
double gemm256_tile_cost(int rows);       // time of a tile of 256, 192 or 128 rows, in 256-row ones
// 128 x 128 (or 64 x 128) tiles with a deep ring of slabs, for launches of a few hundred rows
bool gemm_mid_applicable(const GemmArgs& a, int dtype);
zo2_status gemm_launch_mid(const GemmArgs& a, int dtype, int rows, int splits, hipStream_t st);

}  // namespace zo2
