// Launch interface of the projection for few tokens per step: both perturbation streams in one pass over the weights,
// with the perturbation generated in the weight-tile loader.
#pragma once
#include "common.h"
#include "philox.h"

namespace zo2 {

struct SkinnyProblem {
    const void* Xp;         // [M, ldx] activations of the "+" stream (compute dtype)
    const void* Xm;         // [M, ldx] activations of the "-" stream
    void* theta;            // [N, K] the weight as stored (dense, row n = output feature n); rewritten if an update is applied
    const void* bias_p;     // [N] perturbed bias of the "+" stream (compute dtype) or nullptr
    const void* bias_m;
    const float* res_p;     // [M, ldy] float32 residual or nullptr
    const float* res_m;
    void* Yp;               // [M, ldy] compute dtype or float32
    void* Ym;
    float out_scale;        // multiplies (acc + bias)
    uint32_t tensor_id;     // random stream of theta
};

struct SkinnyArgs {
    static constexpr int kMaxProblems = 3;
    int32_t M, N, K;        // M <= 256 rows per stream (float32: 96); K % 64 == 0; N % 4 == 0
    int64_t ldx, ldy;
    int32_t relu, out_f32, nprob;
    int32_t in_order;       // 1: one wavefront adds a slab's k in order, where two would share it (33 - 128 rows)
    int32_t onto_residual;  // 1: a projection whose pieces a LayerNorm's pass adds where it can: kernel and pieces are those that pay then, whoever adds them
    int32_t splits, k_per_split;     // filled in by skinny_launch: the k range is cut into `splits` pieces of k_per_split
    float eps;
    PhiloxKeys key;         // of the step seed
    // float32, and bfloat16 up to 32 rows (not in_order; refused elsewhere): an update that theta lacks, applied on the way (theta' = theta - c z_prev is
    // written back and used); c_ptr, the device scalar eta g, is nullptr where theta is up to date
    PhiloxKeys key_prev;
    const float* c_ptr;
    int32_t direct;         // filled in by skinny_launch: 1: the kernel finishes the outputs, nothing goes to partial
    float* partial;         // filled in by skinny_launch: [nprob][splits][2][M][N] float32 partial sums
    // cross-entropy mode (skinny_launch_ce, the LM head): per row and 64-column span max and sum(exp(y - max)) of the logits,
    // span-major, and the label's logit; the "-" stream's M rows behind the "+" stream's.  As in GemmProblem.
    const int32_t* labels;  // [M]
    float* part_max;        // [2 ceil(N / 128), part_ld], part_ld >= 2 M
    float* part_sum;
    float* label_logit;     // [2 M]
    int64_t part_ld;
    SkinnyProblem p[kMaxProblems];
};

// Y+- = act((X+- (theta +- eps z)^T + bias+-) * out_scale) + residual+- for every problem; the weights are read once
// and W+ = store(fma(+eps, z, theta)), W- = store(fma(-eps, z, theta)) exist only tile by tile in LDS.
// sum = false: the slices' sums stay where they are (a.partial, a.splits), the caller adds them and finishes the values.
zo2_status skinny_launch(SkinnyArgs& a, int dtype, void* workspace, size_t workspace_bytes, hipStream_t st, bool sum = true);
// The LM head on the same loader: one problem without bias, residual or output matrix; at most 128 rows.
zo2_status skinny_launch_ce(SkinnyArgs& a, int dtype, hipStream_t st);
size_t skinny_workspace_bytes(int M, int N, int K, int nprob);
// float32: the sums as they are, into out[2][M][N] (one problem, k in one piece)
zo2_status skinny_launch_sums(SkinnyArgs& a, float* out, hipStream_t st);
bool skinny_f32_applicable(int M, int N, int K);
// gemm_skinny_rows.hip: up to 96 rows; splits, k_per_split and partial are set.  ce: the LM head's partials
zo2_status skinny_rows_launch(const SkinnyArgs& a, int dtype, bool ce, hipStream_t st);
// gemm_skinny_few.hip: 16 bits, up to 32 rows; splits, k_per_split, direct (one piece) and partial are set
bool skinny_few_pays(const SkinnyArgs& a, int dtype);
void skinny_few_splits(const SkinnyArgs& a, int max_splits, int& splits, int& k_per_split);
zo2_status skinny_few_launch(const SkinnyArgs& a, int dtype, hipStream_t st);
bool skinny_applicable(int M, int N, int K, int dtype);
// W+ and W- of rows [n0, n0 + rows) of a dense [N, K] tensor, chunk by chunk with the loader's arithmetic (a test hook)
zo2_status skinny_perturbed_rows(int dtype, const void* theta, int64_t K, int64_t n0, int64_t rows, uint32_t tensor_id, uint64_t seed,
                                 float eps, void* w_plus, void* w_minus, hipStream_t st);

}  // namespace zo2
