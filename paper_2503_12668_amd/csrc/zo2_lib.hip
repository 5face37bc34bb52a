// libzo2: the training context (Alg. 2 + Alg. 3) and the C ABI.
//
// One zo2_step enqueues, without any host-side wait inside the block loop:
//   embedding gather (with on-the-fly update + perturb)  ->  for each decoder block
//   { [upload] -> K1 (update + perturb) -> dual forward -> [offload] }  ->  final LayerNorm
//   -> K1 on the LM-head weights -> LM head + cross-entropy -> g.
// Upload, compute and offload run on three HIP streams tied together by events only
// (Sec. 5.2); blocks cycle through a ring of equal slots carved out of the caller's arena
// (Sec. 5.3); each block crosses the host link once per direction per step because the
// update of iteration j-1 is applied when the block is visited in iteration j (Sec. 5.4).
#include <dlfcn.h>
#include <math.h>
#include <stdarg.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <vector>

#include "attention.h"
#include "common.h"
#include "gemm.h"
#include "gemm_skinny.h"
#include "k1.h"
#include "rowops.h"

namespace zo2 {

static thread_local char g_op_error[512] = "";
void set_op_error(const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_op_error, sizeof(g_op_error), fmt, ap);
    va_end(ap);
}

static inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Named ranges for profiler timelines (rocprofv3 --marker-trace): the tool's marker library is looked up at run time,
// once; without it the ranges cost one branch.  A range brackets the host-side enqueue of a phase of the step.
struct TraceRange {
    typedef int (*push_fn)(const char*);
    typedef int (*pop_fn)();
    static void lookup(push_fn& push, pop_fn& pop) {
        static push_fn p_push = nullptr;
        static pop_fn p_pop = nullptr;
        static std::once_flag once;
        std::call_once(once, [] {
            void* h = dlopen("librocprofiler-sdk-roctx.so.1", RTLD_NOW | RTLD_GLOBAL);     // what rocprofv3 listens to
            if (!h) h = dlopen("librocprofiler-sdk-roctx.so", RTLD_NOW | RTLD_GLOBAL);
            if (!h) h = dlopen("libroctx64.so.4", RTLD_NOW | RTLD_GLOBAL);                 // the older tools' library
            if (!h) h = dlopen("libroctx64.so", RTLD_NOW | RTLD_GLOBAL);
            if (!h) return;
            p_push = (push_fn)dlsym(h, "roctxRangePushA");
            p_pop = (pop_fn)dlsym(h, "roctxRangePop");
            if (!p_push || !p_pop) p_push = nullptr, p_pop = nullptr;
        });
        push = p_push;
        pop = p_pop;
    }
    pop_fn pop_;
    explicit TraceRange(const char* fmt, int arg = 0) : pop_(nullptr) {
        push_fn push;
        lookup(push, pop_);
        if (!push) { pop_ = nullptr; return; }
        char name[64];
        snprintf(name, sizeof(name), fmt, arg);
        push(name);
    }
    ~TraceRange() { if (pop_) pop_(); }
};
static constexpr int64_t kTensorAlign = 256;   // elements
static constexpr int kDefaultSweeps = 1;       // update + perturb sweeps per block when the budget leaves the choice
// Up to this many tokens per stream the projections perturb in their weight loader.  The line lies higher the wider the model
// is: the slices' partial sums grow with the tokens alone, and what is saved, the perturbed copies, with the weights.  Whole
// steps at the models' own depths in us, ordinary path -> loader (blocks of ffn 4 d): d 768 x 12: 16 tokens 906 -> 854, 24 918 -> 916,
// 32 917 -> 946; d 1024 x 24: 8 1841 -> 1724, 16 1856 -> 1819, 20 1865 -> 1895; d 1536 x 24: 24 2507 -> 2523, 44 2639 -> 2694; d 2048 x 24: 16
// 3377 -> 3014, 48 3507 -> 3394, 60 3523 -> 3521, 64 3535 -> 3550, 72 3676 -> 3789; d 2560 x 32: 64 8005 -> 5923, 128 8725 -> 7240; d 4096 x
// 32: 128 17236 -> 13609; d 5120 x 40: 128 32840 -> 25461.  (A model of few blocks gains more, by its head: d 2048 x 6: 64 1106 -> 1058.)
// Widths that are no multiple of 128 take 16 tokens more: the large kernel refuses them (8 blocks: d 832 32 710 -> 682, 64 733 -> 807; d 960
// 32 730 -> 701; d 1088 32 844 -> 844; d 1728 48 1270 -> 1153; d 2240 90 1636 -> 1581).  And where a matrix of the block has at most 2^19
// elements, which keeps its launches on the older kernels (gemm_choose), the line is 64: d 256 x 8, ffn 2048 64 641 -> 585, 100 660 ->
// 736; d 512, ffn 2048 64 698 -> 674, 80 689 -> 717; d 640 64 747 -> 744; d 704 64 938 -> 762; d 1024, ffn 512 64 790 -> 726.
static constexpr int kFuseAlways = 64;      // beyond this its workspace must fit into what the ordinary path needs; the line of contexts that keep_order()
// float32 (why: gemm_skinny_rows.hip).  By default 64 where a block's matrices are small (d 512, ffn 2048, 8 blocks: 64 tokens 779 -> 732, 96 845 -> 859), 32 where
// a launch has a workgroup or two (d 128, ffn 512: 16 468 -> 455, 48 471 -> 515, 64 497 -> 519; d 64: 16 443 -> 392, 64 438 -> 475; d 192, ffn 768: 64 558 -> 538).
static constexpr int kFuseF32 = 96;
static int fuse_f32_tokens(int64_t d, int64_t f) { return d * f <= 1 << 16 ? 32 : d * f <= 1 << 20 ? 64 : kFuseF32; }
static int fuse_max_tokens(int d, int f) {
    if ((int64_t)d * std::min(d, f) <= 1 << 19) return 64;
    return std::min(128, std::max(16, 16 + (d - 1536) * 11 / 128) + (d % 128 ? 16 : 0));
}

static bool config_ok(const zo2_config* c, char* why, size_t n) {
#define BAD(...) do { snprintf(why, n, __VA_ARGS__); return false; } while (0)
    if (!c) BAD("config is NULL");
    if (c->n_layers < 0 || c->d_model <= 0 || c->n_heads <= 0 || c->d_ffn <= 0 || c->vocab <= 0 || c->max_pos <= 0 || c->pos_offset < 0)
        BAD("non-positive model dimension");
    if (c->d_model % 8 || c->d_ffn % 8) BAD("d_model (%d) and d_ffn (%d) must be multiples of 8", c->d_model, c->d_ffn);
    if (c->d_model % c->n_heads) BAD("n_heads %d does not divide d_model %d", c->n_heads, c->d_model);
    const int dh = c->d_model / c->n_heads;
    if (!(dh == 8 || dh == 16 || dh == 32 || dh == 64 || dh == 80 || dh == 128)) BAD("head dimension %d not in {8,16,32,64,80,128}", dh);
    if (zo2_dtype_size(c->wire_dtype) == 0) BAD("unknown wire dtype %d", c->wire_dtype);
    if (!(c->compute_dtype == ZO2_F32 || c->compute_dtype == ZO2_BF16 || c->compute_dtype == ZO2_F16))
        BAD("compute dtype %d is not F32, BF16 or F16", c->compute_dtype);
    if (!(c->ln_eps > 0.f)) BAD("ln_eps must be positive");
    return true;
#undef BAD
}

static void block_tensor_elems(const zo2_config* c, int64_t n[ZO2_BLOCK_TENSORS]) {
    const int64_t d = c->d_model, f = c->d_ffn;
    const int64_t v[ZO2_BLOCK_TENSORS] = {d, d, d * d, d, d * d, d, d * d, d, d * d, d, d, d, f * d, f, d * f, d};
    for (int i = 0; i < ZO2_BLOCK_TENSORS; ++i) n[i] = v[i];
}

}  // namespace zo2

using namespace zo2;

// =========================================================================================
// context
// =========================================================================================
struct zo2_ctx {
    zo2_config cfg;
    zo2_device dev;
    std::vector<void*> host_bucket;
    void *h_tok, *h_pos, *h_flnw, *h_flnb, *h_lm;
    std::vector<float> scales;          // per tensor id
    char err[512];
    bool dead;
    size_t budget;

    // layout
    int64_t offs[ZO2_BLOCK_TENSORS + 1];
    int64_t tn[ZO2_BLOCK_TENSORS];
    size_t wsz, csz;                    // bytes per element: wire, compute
    size_t bucket_bytes;
    int64_t tok_elems, pos_elems, fln_off_b, fln_elems;   // final LN mini bucket: w at 0, b at fln_off_b
    int n_tensors;

    // persistent device region
    char *d_tok, *d_pos, *d_fln, *d_lm;
    float* d_state;                     // [4..7] result of a pass, [16 + k] coefficient eta g of deferred update k
    size_t persistent_bytes;

    // plan (depends on budget and batch x seq)
    bool planned, need_plan;
    int plan_T, plan_seq;
    bool resident;
    int sweeps;                         // update + perturb sweeps per block: 1 (whole-block scratch), 2 (per half) or 4 (per tensor group)
    int pb[5];                          // sweep p, issued at point p of the block's forward, covers tensors pb[p] .. pb[p + 1] - 1 (may be empty)
    int scratch_plan_forced;            // 0: the planner chooses; 1 / 2 / 4: that many sweeps per block
    int loader_fusion;                  // 0: for few tokens per step (fuse_max_tokens); 1: whenever the shapes allow; -1: never
    int split_k;                        // 0: projections that leave most compute units idle are split along k; -1: never
    bool fuse;                          // this plan: the projections of a block perturb in their weight loader (step passes only)
    char* sk_ws;                        // their workspace (float32 partial sums of the k slices)
    size_t sk_ws_bytes;
    size_t split_ws_bytes;              // the part that projections split along k may count on, whatever path the steps take
    int n_slots;
    char* slots;
    char *wp, *wm;                      // W+ / W- scratch in use (compute dtype)
    char *wps[2], *wms[2];              // the scratch sets; two when K1 of block l+1 may overlap the forwards of block l
    // Rounds of several directions on resident blocks, where the budget has room left for it: up to `wide` directions go through a
    // block together, with their own scratch sets, activations and partial sums.
    static constexpr int kMaxWide = K1RoundArgs::kMaxDirs;
    int wide;                            // 1: one after the other
    char *wide_wp[kMaxWide], *wide_wm[kMaxWide];
    char *wide_x, *wide_q, *wide_k, *wide_v, *wide_ctx, *wide_mid, *wide_ws;      // [direction][stream][token][...]
    size_t wide_ws_bytes;
    // The same for the head: up to `head_wide` directions, on their own copies of the vocabulary matrix, in the room that the blocks have left by then.
    int head_wide;
    char *head_wp[kMaxWide], *head_wm[kMaxWide];
    char *head_fln, *head_x;             // [direction][stream] copies of the final LayerNorm's vectors; its output
    float *head_pmax, *head_psum, *head_lab, *head_loss;
    bool overlap_k1;
    hipStream_t sk;                     // optional fourth stream for that overlap
    hipEvent_t ev_k1done[2], ev_fwd_done[2], ev_embed;
    int64_t scratch_elems;
    char *fln_wp, *fln_wm;
    float* h;
    char *x, *qb, *kb, *vb, *ctxb, *mid;
    float* logits;
    int logit_rows;                     // rows per sign per chunk
    bool fused_ce;                      // LM head writes cross-entropy partials instead of logits
    bool stochastic;                     // theta' is stored with stochastic rounding (low-bit wire formats)
    bool serial_streams;                 // ablation: upload, compute and offload of a block run one after the other
    int ns;                              // perturbation streams of the pass in progress: 2 (step) or 1 (evaluation)
    bool one_dir;                        // the pass in progress evaluates one direction
    bool vectors_at_once;                // the pass in progress has swept the vectors of all blocks ahead of them (sweep_vectors)
    int together, sums_left;             // facts about the last pass: directions that went through a block at once; sums that a LayerNorm's pass made
    RowSum left;                         // FC2's pieces that the next LayerNorm adds up (pieces 0: none)
    float *ce_pmax, *ce_psum, *ce_lab;  // [4 ceil(V/256), 2T] x 2 and [2T]
    int ce_parts;
    float* row_loss;
    int32_t *d_tokens, *d_labels;
    size_t bytes_used;
    bool blocks_on_device;

    // deferred updates (Sec. 5.4): none, one (the paper's case), or the directions of one round of the q-direction
    // estimator (zo2_step_extra), in the order in which they are applied.  Coefficient k sits at d_state[16 + k].
    static constexpr int kMaxPending = 16;
    int n_pend;
    uint64_t pend_seed[kMaxPending];
    bool apply_now;                      // the pass in progress applies them (false: a further direction at unchanged parameters)
    // Several directions in one pass (zo2_step_multi): every direction keeps its own residual stream; inside a module the
    // first direction applies the deferred updates, the later ones find the parameters final.
    float* hs[kMaxPending];              // residual streams of the directions (hs[0] is the only one of an ordinary pass)
    int plan_dirs, want_dirs;            // residual streams the plan holds / asked for
    bool dir_later;                      // the direction in progress is not the first of its pass
    // Streamed blocks with a write-back interval above one: updates already applied wherever parameters stay on the device
    // (embeddings, head) that the host copies of the blocks still lack.  Every upload of a block replays them, in order,
    // before anything else; coefficient k sits at d_state[32 + k].  Empty whenever the blocks are resident.
    static constexpr int kMaxStale = 32;
    int wb_interval;                     // a block is written back once its host copy would lack this many updates (1: after every update, as in Alg. 2)
    int n_stale;
    uint64_t stale_seed[kMaxStale];
    bool pass_writes_back;               // decided at the start of a pass

    // streams / events
    hipStream_t sc, su, so;
    std::vector<hipEvent_t> ev_up, ev_k1, ev_free, ev_read;
    std::vector<char> ev_free_valid, ev_read_valid;    // ev_read: the forwards that read the slot itself (loader fusion) are done
    hipEvent_t ev_step0, ev_c1, ev_u0, ev_u1, ev_o0, ev_o1;
    bool stat_u, stat_o;
    uint64_t bytes_up, bytes_down;
    float ms_c, ms_u, ms_o;

    uint32_t debug_delay_us[3];         // test aid: idle time inserted before each block's work on compute / upload / offload
    bool debug_poison;                  // test aid: a slot is filled with 0xFF bytes (NaN in every format) before each upload into it

    // optional per-kernel-class timing with events on the compute stream
    uint32_t prof_mask;
    std::vector<hipEvent_t> prof_ev;    // pairs (begin, end)
    std::vector<int> prof_cls;
    size_t prof_used;
    float prof_ms[ZO2_KERNEL_CLASSES];
    int32_t prof_launches[ZO2_KERNEL_CLASSES];

    // pinned staging
    int32_t* h_ids;                     // tokens then labels
    int h_ids_cap;
    float* h_result;
};

static zo2_status fail(zo2_ctx* c, zo2_status s, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(c->err, sizeof(c->err), fmt, ap);
    va_end(ap);
    if (s == ZO2_EHIP) c->dead = true;
    return s;
}
#define HIPCHK(c, call)                                                                        \
    do {                                                                                       \
        hipError_t e__ = (call);                                                               \
        if (e__ != hipSuccess) return fail(c, ZO2_EHIP, "%s failed: %s", #call, hipGetErrorString(e__)); \
    } while (0)
#define OPCHK(c, call)                                                       \
    do {                                                                     \
        zo2_status s__ = (call);                                             \
        if (s__ != ZO2_OK) return fail(c, s__, "%s", zo2_op_last_error());   \
    } while (0)

// Bracket one launch with a pair of events when its class is being profiled.
struct ProfScope {
    zo2_ctx* c;
    int cls;
    bool on;
    hipStream_t st;
    ProfScope(zo2_ctx* c_, int cls_, hipStream_t st_ = nullptr) : c(c_), cls(cls_), on((c_->prof_mask >> cls_) & 1u), st(st_ ? st_ : c_->sc) {
        if (!on) return;
        if (c->prof_used + 2 > c->prof_ev.size()) {
            hipEvent_t a, b;
            if (hipEventCreate(&a) != hipSuccess || hipEventCreate(&b) != hipSuccess) { on = false; return; }
            c->prof_ev.push_back(a);
            c->prof_ev.push_back(b);
        }
        (void)hipEventRecord(c->prof_ev[c->prof_used], st);
    }
    ~ProfScope() {
        if (!on) return;
        (void)hipEventRecord(c->prof_ev[c->prof_used + 1], st);
        c->prof_cls.push_back(cls);
        c->prof_used += 2;
    }
};
static void prof_reset(zo2_ctx* c) {
    c->prof_used = 0;
    c->prof_cls.clear();
    for (int i = 0; i < ZO2_KERNEL_CLASSES; ++i) { c->prof_ms[i] = 0.f; c->prof_launches[i] = 0; }
}
static void prof_collect(zo2_ctx* c) {   // after the compute stream has been synchronised
    for (size_t i = 0; i < c->prof_cls.size(); ++i) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, c->prof_ev[2 * i], c->prof_ev[2 * i + 1]) == hipSuccess) {
            c->prof_ms[c->prof_cls[i]] += ms;
            c->prof_launches[c->prof_cls[i]] += 1;
        }
    }
}
#define OPKS(c, cls, stream, call)                                           \
    do {                                                                     \
        zo2_status s__;                                                      \
        {                                                                    \
            ProfScope ps__(c, cls, stream);                                  \
            s__ = (call);                                                    \
        }                                                                    \
        if (s__ != ZO2_OK) return fail(c, s__, "%s", zo2_op_last_error());   \
    } while (0)
#define OPK(c, cls, call)                                                    \
    do {                                                                     \
        zo2_status s__;                                                      \
        {                                                                    \
            ProfScope ps__(c, cls);                                          \
            s__ = (call);                                                    \
        }                                                                    \
        if (s__ != ZO2_OK) return fail(c, s__, "%s", zo2_op_last_error());   \
    } while (0)

// Test aid for the scheduler: a kernel that idles for a bounded time on one stream, so that a test can make
// any of the three streams arbitrarily slow; with correct event dependencies the results cannot change.
__global__ void delay_kernel(unsigned long long ticks_100mhz) {
    const unsigned long long t0 = wall_clock64();
    while (wall_clock64() - t0 < ticks_100mhz) { __builtin_amdgcn_s_sleep(32); }
}
__global__ void poison_kernel(uint32_t* p, size_t n) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0xffffffffu;
}
static zo2_status debug_delay(zo2_ctx* c, int which, hipStream_t st) {
    const uint32_t us = c->debug_delay_us[which];
    if (us == 0) return ZO2_OK;
    hipLaunchKernelGGL(delay_kernel, dim3(1), dim3(1), 0, st, (unsigned long long)us * 100ull);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(c, ZO2_EHIP, "delay kernel: %s", hipGetErrorString(e));
    return ZO2_OK;
}

static inline uint32_t block_tid(int l, int k) { return (uint32_t)(2 + 16 * l + k); }
static inline uint32_t fln_tid(const zo2_ctx* c) { return (uint32_t)(2 + 16 * c->cfg.n_layers); }
static inline uint32_t lm_tid(const zo2_ctx* c) { return (uint32_t)(4 + 16 * c->cfg.n_layers); }

extern "C" size_t zo2_dtype_size(int32_t dt) {
    switch (dt) {
        case ZO2_F32: return 4;
        case ZO2_BF16: case ZO2_F16: return 2;
        case ZO2_FP8_E4M3: case ZO2_FP8_E5M2: return 1;
        default: return 0;
    }
}

extern "C" zo2_status zo2_block_tensor_offsets(const zo2_config* cfg, int64_t offs[ZO2_BLOCK_TENSORS + 1]) {
    char why[256];
    if (!offs || !config_ok(cfg, why, sizeof(why))) {
        set_op_error("%s", offs ? why : "offs is NULL");
        return ZO2_EINVAL;
    }
    int64_t n[ZO2_BLOCK_TENSORS];
    block_tensor_elems(cfg, n);
    int64_t o = 0;
    for (int i = 0; i < ZO2_BLOCK_TENSORS; ++i) {
        offs[i] = o;
        o += (n[i] + kTensorAlign - 1) / kTensorAlign * kTensorAlign;
    }
    offs[ZO2_BLOCK_TENSORS] = o;
    return ZO2_OK;
}

extern "C" const char* zo2_op_last_error(void) { return g_op_error; }
extern "C" const char* zo2_last_error(const zo2_ctx* c) { return c ? c->err : "context is NULL"; }

// ---------------------------------------------------------------------------------- init
extern "C" zo2_status zo2_init(zo2_ctx** out, const zo2_config* cfg, const zo2_host_weights* w, const zo2_device* dev) {
    if (!out) return ZO2_EINVAL;
    *out = nullptr;
    char why[256];
    if (!config_ok(cfg, why, sizeof(why))) { set_op_error("%s", why); return ZO2_EINVAL; }
    if (!w || !dev || !w->tok_emb || !w->pos_emb || !w->final_ln_w || !w->final_ln_b || (cfg->n_layers > 0 && !w->block_bucket)) {
        set_op_error("zo2_init: NULL weight or device argument");
        return ZO2_EINVAL;
    }
    if ((cfg->tied_lm_head != 0) != (w->lm_head == nullptr)) {
        set_op_error("zo2_init: lm_head must be NULL exactly when tied_lm_head = 1");
        return ZO2_EINVAL;
    }
    if (!dev->arena || ((uintptr_t)dev->arena & 255) || dev->arena_bytes == 0) {
        set_op_error("zo2_init: arena must be non-NULL and 256-byte aligned");
        return ZO2_EINVAL;
    }
    for (int l = 0; l < cfg->n_layers; ++l)
        if (!w->block_bucket[l]) { set_op_error("zo2_init: block_bucket[%d] is NULL", l); return ZO2_EINVAL; }

    zo2_ctx* c = new (std::nothrow) zo2_ctx();
    if (c) c->ns = 2;
    if (!c) { set_op_error("zo2_init: out of host memory"); return ZO2_ENOMEM; }
    c->cfg = *cfg;
    c->dev = *dev;
    c->err[0] = 0;
    c->dead = false;
    c->budget = dev->arena_bytes;
    c->host_bucket.assign(w->block_bucket, w->block_bucket + cfg->n_layers);
    c->h_tok = w->tok_emb; c->h_pos = w->pos_emb; c->h_flnw = w->final_ln_w; c->h_flnb = w->final_ln_b; c->h_lm = w->lm_head;
    c->n_tensors = 4 + 16 * cfg->n_layers + (cfg->tied_lm_head ? 0 : 1);
    c->scales.assign(c->n_tensors, 1.0f);
    const bool wire8 = zo2_dtype_size(cfg->wire_dtype) == 1;
    if (w->tensor_scale) {
        for (int i = 0; i < c->n_tensors; ++i) {
            const float s = w->tensor_scale[i];
            int ex = 0;
            if (!(s > 0.f) || !isfinite(s) || frexpf(s, &ex) != 0.5f || (!wire8 && s != 1.0f)) {
                set_op_error("zo2_init: tensor_scale[%d] = %g is invalid for this wire dtype (a power of two; 1 unless the format has 8 bits)", i, (double)s);
                delete c;
                return ZO2_EINVAL;
            }
            c->scales[i] = s;
        }
    }
    zo2_block_tensor_offsets(cfg, c->offs);
    block_tensor_elems(cfg, c->tn);
    c->wsz = zo2_dtype_size(cfg->wire_dtype);
    c->csz = zo2_dtype_size(cfg->compute_dtype);
    c->bucket_bytes = (size_t)c->offs[ZO2_BLOCK_TENSORS] * c->wsz;
    c->tok_elems = (int64_t)cfg->vocab * cfg->d_model;
    c->pos_elems = (int64_t)(cfg->max_pos + cfg->pos_offset) * cfg->d_model;
    c->fln_off_b = align_up(cfg->d_model, kTensorAlign);
    c->fln_elems = 2 * c->fln_off_b;
    c->sc = as_stream(dev->stream_compute);
    c->su = as_stream(dev->stream_upload);
    c->so = as_stream(dev->stream_offload);
    c->sk = as_stream(dev->stream_k1);
    c->overlap_k1 = false;
    c->planned = false;
    c->need_plan = false;
    c->blocks_on_device = false;
    c->n_pend = 0;
    c->apply_now = true;
    c->wb_interval = 1;
    c->n_stale = 0;
    c->pass_writes_back = true;
    c->h_ids = nullptr;
    c->h_ids_cap = 0;
    c->h_result = nullptr;
    c->plan_dirs = 0; c->want_dirs = 1; c->dir_later = false;
    for (float*& hp : c->hs) hp = nullptr;
    c->bytes_up = c->bytes_down = 0;
    c->ms_c = c->ms_u = c->ms_o = 0.f;
    c->bytes_used = 0;
    c->debug_delay_us[0] = c->debug_delay_us[1] = c->debug_delay_us[2] = 0;
    c->prof_mask = 0;
    prof_reset(c);
    c->n_slots = 0;
    c->resident = false;
    c->sweeps = 1;
    c->scratch_plan_forced = 0;
    c->loader_fusion = 0;
    c->split_k = 0;
    c->fuse = false;
    c->scratch_elems = 0;
    *out = c;   // from here on errors are reported through the context

    // persistent region: embeddings, final LayerNorm, LM head, state
    char* base = (char*)dev->arena;
    size_t off = 0;
    auto take = [&](size_t bytes) { char* p = base + off; off = align_up(off + bytes, 256); return p; };
    c->d_tok = take((size_t)c->tok_elems * c->wsz);
    c->d_pos = take((size_t)c->pos_elems * c->wsz);
    c->d_fln = take((size_t)c->fln_elems * c->wsz);
    c->d_lm = cfg->tied_lm_head ? nullptr : take((size_t)c->tok_elems * c->wsz);
    c->d_state = (float*)take(64 * sizeof(float));
    c->persistent_bytes = off;
    if (off > dev->arena_bytes) return fail(c, ZO2_ENOMEM, "arena of %zu bytes cannot hold the %zu bytes of embeddings", dev->arena_bytes, off);

    HIPCHK(c, hipMemcpy(c->d_tok, w->tok_emb, (size_t)c->tok_elems * c->wsz, hipMemcpyHostToDevice));
    HIPCHK(c, hipMemcpy(c->d_pos, w->pos_emb, (size_t)c->pos_elems * c->wsz, hipMemcpyHostToDevice));
    HIPCHK(c, hipMemset(c->d_fln, 0, (size_t)c->fln_elems * c->wsz));
    HIPCHK(c, hipMemcpy(c->d_fln, w->final_ln_w, (size_t)cfg->d_model * c->wsz, hipMemcpyHostToDevice));
    HIPCHK(c, hipMemcpy(c->d_fln + (size_t)c->fln_off_b * c->wsz, w->final_ln_b, (size_t)cfg->d_model * c->wsz, hipMemcpyHostToDevice));
    if (c->d_lm) HIPCHK(c, hipMemcpy(c->d_lm, w->lm_head, (size_t)c->tok_elems * c->wsz, hipMemcpyHostToDevice));
    HIPCHK(c, hipMemset(c->d_state, 0, 64 * sizeof(float)));
    HIPCHK(c, hipHostMalloc((void**)&c->h_result, (16 + 4 * zo2_ctx::kMaxPending) * sizeof(float), hipHostMallocDefault));
    hipEvent_t* evs[] = {&c->ev_step0, &c->ev_c1, &c->ev_u0, &c->ev_u1, &c->ev_o0, &c->ev_o1};
    for (hipEvent_t* e : evs) HIPCHK(c, hipEventCreate(e));
    hipEvent_t* evs2[] = {&c->ev_k1done[0], &c->ev_k1done[1], &c->ev_fwd_done[0], &c->ev_fwd_done[1], &c->ev_embed};
    for (hipEvent_t* e : evs2) HIPCHK(c, hipEventCreateWithFlags(e, hipEventDisableTiming));
    return ZO2_OK;
}

static zo2_status writeback_pass(zo2_ctx* c);

extern "C" void zo2_destroy(zo2_ctx* c) {
    if (!c) return;
    if (!c->dead) (void)writeback_pass(c);       // the caller's block buffers are left current (best effort: no status to report)
    hipStreamSynchronize(c->sc);
    hipStreamSynchronize(c->su);
    hipStreamSynchronize(c->so);
    if (c->sk) hipStreamSynchronize(c->sk);
    for (auto e : c->ev_up) hipEventDestroy(e);
    for (auto e : c->ev_k1) hipEventDestroy(e);
    for (auto e : c->ev_free) hipEventDestroy(e);
    for (auto e : c->ev_read) hipEventDestroy(e);
    for (auto e : c->prof_ev) hipEventDestroy(e);
    hipEvent_t evs[] = {c->ev_step0, c->ev_c1, c->ev_u0, c->ev_u1, c->ev_o0, c->ev_o1, c->ev_k1done[0], c->ev_k1done[1], c->ev_fwd_done[0], c->ev_fwd_done[1], c->ev_embed};
    if (c->h_result) for (hipEvent_t e : evs) hipEventDestroy(e);
    if (c->h_ids) hipHostFree(c->h_ids);
    if (c->h_result) hipHostFree(c->h_result);
    delete c;
}

extern "C" zo2_status zo2_set_resident_budget(zo2_ctx* c, size_t hbm_bytes) {
    if (!c) return ZO2_EINVAL;
    if (c->dead) return ZO2_ESTATE;
    if (hbm_bytes == 0) return fail(c, ZO2_EINVAL, "budget must be positive");
    c->budget = hbm_bytes < c->dev.arena_bytes ? hbm_bytes : c->dev.arena_bytes;
    c->need_plan = true;   // re-plan at the next step
    return ZO2_OK;
}

// ---------------------------------------------------------------------------------- sync to host
static zo2_status sync_blocks_to_host(zo2_ctx* c) {
    if (c->resident && c->blocks_on_device) {
        HIPCHK(c, hipStreamSynchronize(c->sc));
        for (int l = 0; l < c->cfg.n_layers; ++l)
            HIPCHK(c, hipMemcpy(c->host_bucket[l], c->slots + (size_t)l * c->bucket_bytes, c->bucket_bytes, hipMemcpyDeviceToHost));
    }
    return ZO2_OK;
}

extern "C" zo2_status zo2_sync_to_host(zo2_ctx* c) {
    if (!c) return ZO2_EINVAL;
    if (c->dead) return ZO2_ESTATE;
    { zo2_status s = writeback_pass(c); if (s != ZO2_OK) return s; }
    HIPCHK(c, hipStreamSynchronize(c->sc));
    HIPCHK(c, hipStreamSynchronize(c->so));
    const size_t d = c->cfg.d_model;
    HIPCHK(c, hipMemcpy(c->h_tok, c->d_tok, (size_t)c->tok_elems * c->wsz, hipMemcpyDeviceToHost));
    HIPCHK(c, hipMemcpy(c->h_pos, c->d_pos, (size_t)c->pos_elems * c->wsz, hipMemcpyDeviceToHost));
    HIPCHK(c, hipMemcpy(c->h_flnw, c->d_fln, d * c->wsz, hipMemcpyDeviceToHost));
    HIPCHK(c, hipMemcpy(c->h_flnb, c->d_fln + (size_t)c->fln_off_b * c->wsz, d * c->wsz, hipMemcpyDeviceToHost));
    if (c->d_lm) HIPCHK(c, hipMemcpy(c->h_lm, c->d_lm, (size_t)c->tok_elems * c->wsz, hipMemcpyDeviceToHost));
    return sync_blocks_to_host(c);
}

// ---------------------------------------------------------------------------------- planning
// The W+ / W- scratch holds the perturbed copies of the tensors one sweep of K1 writes.  The forward of a block needs
// them at four points: {ln1, q, k, v} before the QKV projection, {o} before the output projection, {ln2, fc1} before the
// first FFN projection, {fc2} before the second.  Three organisations: one sweep over the whole block at point 0; two
// sweeps (attention half at point 0, FFN half at point 2); four sweeps (one per group).  Fewer tensors per sweep = a
// smaller scratch, and the copies are consumed right after they are written, while they still sit in the memory-side
// cache; more sweeps = more, shorter launches.
static const int kSweepBounds[3][5] = {{0, 16, 16, 16, 16}, {0, 10, 10, 16, 16}, {0, 8, 10, 14, 16}};
static inline const int* sweep_bounds(int sweeps) { return kSweepBounds[sweeps == 1 ? 0 : sweeps == 2 ? 1 : 2]; }

// Under stochastic rounding of a low-bit master every stored parameter is a draw that turns over with a late digit of eta g:
// another order of the same products' sums moves l+ and l- by 1e-5 .. 2e-4 in 16 bits, g by a percent or two, and with it one in ten
// thousand stored bytes of an 8-bit master in two steps; parameters of a 16-bit one end two spacings apart.  Such a run is to give
// the same bits under every version of the kernels, so its 16-bit passes keep the order that sums have always had: one
// accumulator per wavefront along k, the large tiles' pieces, the loader path up to 64 tokens, logits for fewer than 256 tokens.
// (d 2048, 12 blocks, bf16: 1 x 16 tokens 1845 us where the order others take gives 1730, 5 x 37 2868 for 2570.)
static inline bool keep_order(const zo2_ctx* c) { return c->stochastic && c->wsz < 4 && c->cfg.compute_dtype != ZO2_F32; }

static zo2_status plan(zo2_ctx* c, int T, int batch, int seq) {
    const zo2_config& g = c->cfg;
    // a new layout starts from current host copies of the blocks (it may make them resident)
    { zo2_status s = writeback_pass(c); if (s != ZO2_OK) return s; }
    const size_t d = g.d_model, f = g.d_ffn, V = g.vocab;
    const size_t budget = c->budget;
    const size_t rows2 = 2 * (size_t)T;
    // logits chunk (float32 mode and shapes the fused LM-head + cross-entropy kernel does not take): up to 1/8 of the
    // budget, at least 128 rows per sign
    const bool fused_ce = (g.compute_dtype != ZO2_F32) && V >= 256 && (d % 128 == 0) && (V % 4 == 0) && (T >= 256 || !keep_order(c));
    const size_t ce_parts = 4 * ((V + 255) / 256);
    size_t lrows = budget / 8 / (V * 4) / 2;
    lrows = lrows / 128 * 128;
    if (lrows < 128) lrows = 128;
    if (lrows > (size_t)T) lrows = T;
    // few tokens per step: the block projections read the stored weights and perturb in their loader (16-bit storage
    // that is also the compute format, no wire scale)
    const bool f32 = g.compute_dtype == ZO2_F32;
    // (float32: the pieces go to the logits, which are idle until the head)
    const bool fuse_f32 = f32 && T <= kFuseF32 && (size_t)T * V >= (size_t)T * std::max(3 * d, f);
    const bool fuse_shapes = g.wire_dtype == g.compute_dtype && (f32 ? fuse_f32 : T <= 256) && d % 64 == 0 && f % 64 == 0 &&
                             (size_t)T * f * 2 < 0xffffffffull && std::max(d, f) < (size_t)1 << 22;
    size_t split_bytes = 0, fuse_bytes = 0;
    if (c->split_k >= 0 && g.compute_dtype != ZO2_F32) {      // split-k partial sums of the block projections (steps and single forwards)
        for (int ns_ = 1; ns_ <= 2; ++ns_) {
            const int shapes[4][3] = {{(int)d, (int)d, 3 * ns_}, {(int)d, (int)d, ns_}, {(int)f, (int)d, ns_}, {(int)d, (int)f, ns_}};      // N, K, problems
            for (const auto& sh : shapes)
                split_bytes = std::max(split_bytes, gemm_splitk_workspace_bytes(T, sh[0], sh[2], gemm_pick_splits(T, sh[0], sh[1], sh[2], g.compute_dtype)));
        }
    }
    if (fuse_shapes && !f32) {
        fuse_bytes = std::max(std::max(skinny_workspace_bytes(T, (int)d, (int)d, 3), skinny_workspace_bytes(T, (int)d, (int)d, 1)),
                              std::max(skinny_workspace_bytes(T, (int)f, (int)d, 1), skinny_workspace_bytes(T, (int)d, (int)f, 1)));
    }
    // above 64 tokens only where the slices' partial sums take no more than the logits that the head's partials replace, so
    // that no budget that holds the ordinary path is too small for this one
    const size_t freed = fused_ce && T < 256 ? 2 * std::min<size_t>(T, 128) * V * 4 - rows2 * (2 * ce_parts + 1) * 4 : 0;
    const bool few_tokens = f32 ? T <= fuse_f32_tokens((int64_t)d, (int64_t)f) : keep_order(c) ? T <= kFuseAlways
                                          : T <= fuse_max_tokens((int)d, (int)f) && (T <= kFuseAlways || fuse_bytes <= split_bytes + freed);
    const bool fuse = fuse_shapes && c->loader_fusion >= 0 && (c->loader_fusion == 1 || few_tokens) && (f32 || !c->sk);
    const size_t sk_ws_bytes = std::max(split_bytes, fuse ? fuse_bytes : 0);      // (float32: none)
    size_t act = 0;
    auto sz = [&](size_t bytes) { size_t o = act; act = align_up(act + bytes, 256); return o; };
    const int n_dirs = std::max(1, c->want_dirs);
    const size_t h_bytes = align_up(rows2 * d * 4, 256);
    const size_t o_h = sz(h_bytes * n_dirs), o_x = sz(rows2 * d * c->csz), o_q = sz(rows2 * d * c->csz), o_k = sz(rows2 * d * c->csz),
                 o_v = sz(rows2 * d * c->csz), o_ctx = sz(rows2 * d * c->csz), o_mid = sz(rows2 * f * c->csz),
                 o_logits = sz(fused_ce ? 0 : 2 * lrows * V * 4), o_rl = sz(rows2 * 4),
                 o_cpm = sz(fused_ce ? rows2 * ce_parts * 4 : 0), o_cps = sz(fused_ce ? rows2 * ce_parts * 4 : 0), o_cl = sz(fused_ce ? rows2 * 4 : 0), o_tok = sz((size_t)T * 4), o_lab = sz((size_t)T * 4),
                 o_fwp = sz((size_t)c->fln_elems * c->csz), o_fwm = sz((size_t)c->fln_elems * c->csz), o_skws = sz(sk_ws_bytes);
    const size_t act_bytes = act;

    const int64_t head_elems = (int64_t)align_up(c->tok_elems, kTensorAlign);
    auto scratch_for = [&](int sweeps) {
        const int* pb = sweep_bounds(sweeps);
        int64_t m = 0;
        for (int p = 0; p < 4; ++p) m = std::max(m, c->offs[pb[p + 1]] - c->offs[pb[p]]);
        return std::max(m, head_elems);
    };
    bool resident = false, two_sets = false;
    int sweeps = 1;
    int64_t scratch = 0;
    long slots = 0;
    // preference: two whole-block scratch sets (K1 of the next block overlaps this block's forwards) when a stream for
    // it was given, then the default organisation, then ever smaller scratch sets until 3 block slots fit
    const int forced = c->scratch_plan_forced;
    const int first = forced ? forced : kDefaultSweeps;
    // (in float32 steps on the loader path have no sweep that a stream of its own could take)
    for (int attempt = (c->sk && !forced && !fuse ? 0 : 1); attempt < 4; ++attempt) {
        two_sets = attempt == 0;
        sweeps = attempt == 0 ? 1 : attempt == 1 ? first : attempt == 2 ? std::max(first, 2) : 4;
        scratch = scratch_for(sweeps);
        const size_t fixed = c->persistent_bytes + act_bytes + (two_sets ? 4 : 2) * align_up((size_t)scratch * c->csz, 256);
        slots = fixed > budget ? -1 : (long)((budget - fixed) / align_up(c->bucket_bytes, 256));
        if (slots >= g.n_layers || slots >= 3 || forced) break;      // a forced organisation is not traded for a smaller one
    }
    if (g.n_layers > 0 && slots < g.n_layers && slots < 3)
        return fail(c, ZO2_EBUDGET, "budget of %zu bytes cannot hold embeddings + 3 block slots + scratch + activations for %d tokens", budget, T);
    resident = slots >= g.n_layers;
    const int n_slots = resident ? g.n_layers : (int)slots;

    // moving between resident and streamed (or resizing the ring) needs the host copy current
    if (c->planned && c->resident && c->blocks_on_device && !resident) {
        zo2_status s = sync_blocks_to_host(c);
        if (s != ZO2_OK) return s;
        c->blocks_on_device = false;
    }
    HIPCHK(c, hipStreamSynchronize(c->sc));
    HIPCHK(c, hipStreamSynchronize(c->su));
    HIPCHK(c, hipStreamSynchronize(c->so));
    if (c->sk) HIPCHK(c, hipStreamSynchronize(c->sk));

    char* base = (char*)c->dev.arena;
    size_t off = c->persistent_bytes;
    c->slots = base + off;
    off += (size_t)n_slots * align_up(c->bucket_bytes, 256);
    for (int k = 0; k < (two_sets ? 2 : 1); ++k) {
        c->wps[k] = base + off; off += align_up((size_t)scratch * c->csz, 256);
        c->wms[k] = base + off; off += align_up((size_t)scratch * c->csz, 256);
    }
    if (!two_sets) { c->wps[1] = c->wps[0]; c->wms[1] = c->wms[0]; }
    c->wp = c->wps[0]; c->wm = c->wms[0];
    c->overlap_k1 = two_sets;
    char* a0 = base + off;
    for (int j = 0; j < zo2_ctx::kMaxPending; ++j) c->hs[j] = j < n_dirs ? (float*)(a0 + o_h + (size_t)j * h_bytes) : nullptr;
    c->plan_dirs = n_dirs;
    c->h = c->hs[0]; c->x = a0 + o_x; c->qb = a0 + o_q; c->kb = a0 + o_k; c->vb = a0 + o_v; c->ctxb = a0 + o_ctx;
    c->mid = a0 + o_mid; c->logits = (float*)(a0 + o_logits); c->row_loss = (float*)(a0 + o_rl);
    c->d_tokens = (int32_t*)(a0 + o_tok); c->d_labels = (int32_t*)(a0 + o_lab);
    c->fln_wp = a0 + o_fwp; c->fln_wm = a0 + o_fwm;
    c->fuse = fuse; c->sk_ws = a0 + o_skws; c->sk_ws_bytes = sk_ws_bytes; c->split_ws_bytes = split_bytes;
    c->fused_ce = fused_ce; c->ce_parts = (int)ce_parts;
    c->ce_pmax = (float*)(a0 + o_cpm); c->ce_psum = (float*)(a0 + o_cps); c->ce_lab = (float*)(a0 + o_cl);
    off += act_bytes;
    c->bytes_used = off;
    // Room beyond that, up to the budget: the directions of a round go through a block together (block_forward_round).  Nothing depends
    // on it but time, so it is not counted as used and never takes the place of a slot.
    c->wide = 1;
    if (n_dirs > 1 && resident && !fuse && !two_sets && !c->sk && sweeps == 1 && !forced && k1_round_applicable(g.wire_dtype, g.compute_dtype)) {
        for (int w = std::min(n_dirs, (int)zo2_ctx::kMaxWide); w > 1 && c->wide == 1; --w) {
            size_t at = align_up(off, 256);
            auto take = [&](size_t bytes) { char* p = base + at; at += align_up(bytes, 256); return p; };
            const size_t set = (size_t)c->offs[ZO2_BLOCK_TENSORS] * c->csz, row = rows2 * w * c->csz;
            char *wp[zo2_ctx::kMaxWide] = {}, *wm[zo2_ctx::kMaxWide] = {};
            for (int j = 0; j < w; ++j) { wp[j] = take(set); wm[j] = take(set); }      // (evenly spaced: see norm() in block_forward_round)
            char *x = take(row * d), *q = take(row * d), *k = take(row * d), *v = take(row * d), *ctx = take(row * d), *mid = take(row * f), *ws = take(w * split_bytes);
            if (at > budget) continue;
            c->wide = w;
            for (int j = 0; j < w; ++j) { c->wide_wp[j] = wp[j]; c->wide_wm[j] = wm[j]; }
            c->wide_x = x; c->wide_q = q; c->wide_k = k; c->wide_v = v; c->wide_ctx = ctx; c->wide_mid = mid; c->wide_ws = ws;
            c->wide_ws_bytes = w * split_bytes;
        }
    }
    c->head_wide = 1;
    if (n_dirs > 1 && resident && fused_ce && !fuse && !two_sets && !c->sk && !forced && k1_round_applicable(g.wire_dtype, g.compute_dtype)) {
        for (int w = std::min(n_dirs, (int)zo2_ctx::kMaxWide); w > 1 && c->head_wide == 1; --w) {
            size_t at = align_up(off, 256);
            auto take = [&](size_t bytes) { char* p = base + at; at += align_up(bytes, 256); return p; };
            char *wp[zo2_ctx::kMaxWide] = {}, *wm[zo2_ctx::kMaxWide] = {};
            for (int j = 0; j < w; ++j) { wp[j] = take((size_t)head_elems * c->csz); wm[j] = take((size_t)head_elems * c->csz); }
            char *fln = take(2 * w * align_up((size_t)c->fln_elems * c->csz, 256)), *x = take(rows2 * w * d * c->csz), *pmax = take(rows2 * w * ce_parts * 4),
                 *psum = take(rows2 * w * ce_parts * 4), *lab = take(rows2 * w * 4), *loss = take(rows2 * w * 4);
            if (at > budget) continue;
            c->head_wide = w;
            for (int j = 0; j < w; ++j) { c->head_wp[j] = wp[j]; c->head_wm[j] = wm[j]; }
            c->head_fln = fln; c->head_x = x; c->head_pmax = (float*)pmax; c->head_psum = (float*)psum; c->head_lab = (float*)lab; c->head_loss = (float*)loss;
        }
    }
    c->logit_rows = (int)lrows;
    c->scratch_elems = scratch;
    c->sweeps = sweeps;
    for (int p = 0; p < 5; ++p) c->pb[p] = sweep_bounds(sweeps)[p];
    if (c->bucket_bytes % 256) return fail(c, ZO2_EINVAL, "internal: bucket size not aligned");

    // events per slot
    while ((int)c->ev_up.size() < n_slots) {
        hipEvent_t e1, e2, e3, e4;
        HIPCHK(c, hipEventCreateWithFlags(&e1, hipEventDisableTiming));
        HIPCHK(c, hipEventCreateWithFlags(&e2, hipEventDisableTiming));
        HIPCHK(c, hipEventCreateWithFlags(&e3, hipEventDisableTiming));
        HIPCHK(c, hipEventCreateWithFlags(&e4, hipEventDisableTiming));
        c->ev_up.push_back(e1); c->ev_k1.push_back(e2); c->ev_free.push_back(e3); c->ev_read.push_back(e4);
    }
    c->ev_free_valid.assign(c->ev_up.size(), 0);
    c->ev_read_valid.assign(c->ev_up.size(), 0);

    if (resident && !(c->planned && c->resident && c->blocks_on_device && c->n_slots == n_slots)) {
        for (int l = 0; l < g.n_layers; ++l)
            HIPCHK(c, hipMemcpy(c->slots + (size_t)l * c->bucket_bytes, c->host_bucket[l], c->bucket_bytes, hipMemcpyHostToDevice));
        c->blocks_on_device = true;
    }
    if (!resident) c->blocks_on_device = false;
    c->resident = resident;
    c->n_slots = n_slots;
    c->plan_T = T;
    c->plan_seq = seq;
    c->planned = true;
    c->need_plan = false;

    if (c->h_ids_cap < 2 * T) {
        if (c->h_ids) hipHostFree(c->h_ids);
        c->h_ids = nullptr;
        HIPCHK(c, hipHostMalloc((void**)&c->h_ids, (size_t)2 * T * sizeof(int32_t), hipHostMallocDefault));
        c->h_ids_cap = 2 * T;
    }
    return ZO2_OK;
}

extern "C" zo2_status zo2_get_plan(const zo2_ctx* c, int32_t* n_slots, int32_t* resident, size_t* bytes_used) {
    if (!c) return ZO2_EINVAL;
    if (n_slots) *n_slots = c->n_slots;
    if (resident) *resident = c->resident ? 1 : 0;
    if (bytes_used) *bytes_used = c->planned ? c->bytes_used : c->persistent_bytes;
    return ZO2_OK;
}

extern "C" zo2_status zo2_get_scratch_plan(const zo2_ctx* c, int32_t* sweeps_per_block, int64_t* scratch_elems, int32_t* scratch_sets) {
    if (!c) return ZO2_EINVAL;
    if (sweeps_per_block) *sweeps_per_block = c->planned ? c->sweeps : 0;
    if (scratch_elems) *scratch_elems = c->planned ? c->scratch_elems : 0;
    if (scratch_sets) *scratch_sets = c->planned ? (c->overlap_k1 ? 2 : 1) : 0;
    return ZO2_OK;
}

extern "C" zo2_status zo2_get_pass_facts(const zo2_ctx* c, int32_t* directions_together, int32_t* sums_in_layernorm) {
    if (!c) return ZO2_EINVAL;
    if (directions_together) *directions_together = c->together;
    if (sums_in_layernorm) *sums_in_layernorm = c->sums_left;
    return ZO2_OK;
}

extern "C" zo2_status zo2_set_scratch_plan(zo2_ctx* c, int32_t mode) {
    if (!c) return ZO2_EINVAL;
    if (c->dead) return ZO2_ESTATE;
    if (mode != 0 && mode != 1 && mode != 2 && mode != 4) return fail(c, ZO2_EINVAL, "zo2_set_scratch_plan: %d sweeps per block (0, 1, 2 or 4)", mode);
    c->scratch_plan_forced = mode;
    c->need_plan = true;   // re-plan at the next step
    return ZO2_OK;
}

extern "C" zo2_status zo2_set_loader_fusion(zo2_ctx* c, int32_t mode) {
    if (!c) return ZO2_EINVAL;
    if (c->dead) return ZO2_ESTATE;
    if (mode < -1 || mode > 1) return fail(c, ZO2_EINVAL, "zo2_set_loader_fusion: mode %d (-1, 0 or 1)", mode);
    c->loader_fusion = mode;
    c->need_plan = true;   // re-plan at the next step
    return ZO2_OK;
}

extern "C" zo2_status zo2_set_split_k(zo2_ctx* c, int32_t mode) {
    if (!c) return ZO2_EINVAL;
    if (c->dead) return ZO2_ESTATE;
    if (mode < -1 || mode > 0) return fail(c, ZO2_EINVAL, "zo2_set_split_k: mode %d (-1 or 0)", mode);
    c->split_k = mode;
    c->need_plan = true;   // re-plan at the next step
    return ZO2_OK;
}

extern "C" zo2_status zo2_set_writeback_interval(zo2_ctx* c, int32_t updates) {
    if (!c) return ZO2_EINVAL;
    if (c->dead) return ZO2_ESTATE;
    if (updates < 1 || updates > zo2_ctx::kMaxStale - zo2_ctx::kMaxPending)
        return fail(c, ZO2_EINVAL, "zo2_set_writeback_interval: %d (1 .. %d)", updates, zo2_ctx::kMaxStale - zo2_ctx::kMaxPending);
    c->wb_interval = updates;
    return ZO2_OK;
}

extern "C" zo2_status zo2_get_writeback_state(const zo2_ctx* c, int32_t* interval, int32_t* lacking) {
    if (!c || !interval || !lacking) return ZO2_EINVAL;
    *interval = c->wb_interval;
    *lacking = c->n_stale;
    return ZO2_OK;
}

extern "C" zo2_status zo2_get_loader_fusion(const zo2_ctx* c, int32_t* active) {
    if (!c || !active) return ZO2_EINVAL;
    *active = (c->planned && c->fuse) ? 1 : 0;
    return ZO2_OK;
}

extern "C" zo2_status zo2_set_profiling(zo2_ctx* c, uint32_t class_mask) {
    if (!c) return ZO2_EINVAL;
    c->prof_mask = class_mask & ((1u << ZO2_KERNEL_CLASSES) - 1);
    return ZO2_OK;
}

extern "C" zo2_status zo2_get_kernel_times(const zo2_ctx* c, float ms[ZO2_KERNEL_CLASSES], int32_t launches[ZO2_KERNEL_CLASSES]) {
    if (!c) return ZO2_EINVAL;
    for (int i = 0; i < ZO2_KERNEL_CLASSES; ++i) {
        if (ms) ms[i] = c->prof_ms[i];
        if (launches) launches[i] = c->prof_launches[i];
    }
    return ZO2_OK;
}

extern "C" zo2_status zo2_debug_set_slot_poison(zo2_ctx* c, int32_t enabled) {
    if (!c) return ZO2_EINVAL;
    c->debug_poison = enabled != 0;
    return ZO2_OK;
}

extern "C" zo2_status zo2_debug_set_stream_delay(zo2_ctx* c, int32_t which, uint32_t microseconds) {
    if (!c || which < 0 || which > 2 || microseconds > 100000u) return ZO2_EINVAL;
    c->debug_delay_us[which] = microseconds;
    return ZO2_OK;
}

extern "C" zo2_status zo2_set_wire_rounding(zo2_ctx* c, int32_t stochastic) {
    if (!c) return ZO2_EINVAL;
    if (c->dead) return ZO2_ESTATE;
    c->need_plan = c->need_plan || c->stochastic != (stochastic != 0);      // see keep_order
    c->stochastic = stochastic != 0;
    return ZO2_OK;
}

extern "C" zo2_status zo2_set_stream_overlap(zo2_ctx* c, int32_t enabled) {
    if (!c) return ZO2_EINVAL;
    if (c->dead) return ZO2_ESTATE;
    c->serial_streams = enabled == 0;
    return ZO2_OK;
}

extern "C" zo2_status zo2_get_step_stats(const zo2_ctx* c, float* ms_c, float* ms_u, float* ms_o, uint64_t* up, uint64_t* down) {
    if (!c) return ZO2_EINVAL;
    if (ms_c) *ms_c = c->ms_c;
    if (ms_u) *ms_u = c->ms_u;
    if (ms_o) *ms_o = c->ms_o;
    if (up) *up = c->bytes_up;
    if (down) *down = c->bytes_down;
    return ZO2_OK;
}

// ---------------------------------------------------------------------------------- K1 helpers
static inline float* coef_slot(const zo2_ctx* c, int k) { return c->d_state + 16 + k; }
// does the fused sweep (update + perturb) of the pass in progress carry an update?  It carries the last deferred one;
// the earlier ones of a round of several directions are applied by update-only sweeps in front of it.
static inline bool fused_update(const zo2_ctx* c) { return c->apply_now && c->n_pend > 0; }

// pend: index of the deferred update this sweep applies; -1 = the last one (the fused sweep's)
static void k1_common(const zo2_ctx* c, K1Args& a, uint64_t seed, float eps, int pend = -1) {
    memset(&a, 0, sizeof(a));
    const int k = pend >= 0 ? pend : (c->n_pend > 0 ? c->n_pend - 1 : 0);
    a.c_ptr = coef_slot(c, k);
    a.c_imm = 0.f;
    a.stochastic = c->stochastic ? 1 : 0;
    a.eps = eps;
    a.k_prev = philox_keys(c->n_pend > 0 ? c->pend_seed[k] : 0);
    a.k_cur = philox_keys(seed);
}

// one whole tensor held contiguously at `theta`
static zo2_status k1_tensor(zo2_ctx* c, void* theta, int64_t n, uint32_t tid, bool perturb, void* wp, void* wm,
                            uint64_t seed, float eps, hipStream_t st = nullptr, int pend = -1) {
    if (!st) st = c->sc;
    K1Args a;
    k1_common(c, a, seed, eps, pend);
    a.theta = theta; a.w_plus = wp; a.w_minus = c->ns == 2 ? wm : nullptr; a.w_off0 = 0; a.nseg = 1;
    a.seg[0].off = 0; a.seg[0].e0 = 0; a.seg[0].n = (uint64_t)n; a.seg[0].tensor_id = tid; a.seg[0].scale = c->scales[tid];
    OPKS(c, ZO2_KC_K1, st, k1_launch(a, c->cfg.wire_dtype, c->cfg.compute_dtype, pend >= 0 || fused_update(c), perturb, st));
    return ZO2_OK;
}

// tensors [t0, t1) of block l whose bucket sits at `bucket`; W+- go to the scratch, tensor t0 at its start (fc2.b, if it is not
// negative, at element fc2_bias_at)
static zo2_status k1_block(zo2_ctx* c, int l, char* bucket, int t0, int t1, bool perturb, uint64_t seed, float eps,
                           hipStream_t st = nullptr, int pend = -1, int64_t fc2_bias_at = -1) {
    if (!st) st = c->sc;
    if (fc2_bias_at < 0) fc2_bias_at = c->offs[15] - c->offs[t0];
    K1Args a;
    k1_common(c, a, seed, eps, pend);
    a.theta = bucket; a.w_plus = c->wp; a.w_minus = c->ns == 2 ? c->wm : nullptr; a.w_off0 = c->offs[t0]; a.nseg = t1 - t0;
    a.reverse = perturb ? 1 : 0;      // end with the tensors the next projection reads (see k1_kernel)
    for (int k = t0; k < t1; ++k) {
        K1Seg& s = a.seg[k - t0];
        s.off = c->offs[k]; s.e0 = 0; s.n = (uint64_t)c->tn[k]; s.tensor_id = block_tid(l, k); s.scale = c->scales[s.tensor_id];
        s.woff = k == 15 && perturb ? fc2_bias_at : c->offs[k] - a.w_off0;
    }
    a.packed_w = 1;
    OPKS(c, ZO2_KC_K1, st, k1_launch(a, c->cfg.wire_dtype, c->cfg.compute_dtype, pend >= 0 || fused_update(c), perturb, st));
    return ZO2_OK;
}

// update-only sweep over block l with an explicit coefficient (device scalar) and seed: replays an update the block's
// host copy lacks
static inline float* stale_slot(const zo2_ctx* c, int k) { return c->d_state + 32 + k; }
static zo2_status k1_block_replay(zo2_ctx* c, int l, char* bucket, const float* coef, uint64_t seed_prev, hipStream_t st) {
    if (!st) st = c->sc;
    K1Args a;
    k1_common(c, a, 0, 0.f, -1);
    a.c_ptr = coef;
    a.k_prev = philox_keys(seed_prev);
    a.theta = bucket; a.w_plus = nullptr; a.w_minus = nullptr; a.w_off0 = 0; a.nseg = ZO2_BLOCK_TENSORS;
    for (int k = 0; k < ZO2_BLOCK_TENSORS; ++k) {
        K1Seg& s = a.seg[k];
        s.off = c->offs[k]; s.e0 = 0; s.n = (uint64_t)c->tn[k]; s.tensor_id = block_tid(l, k); s.scale = c->scales[s.tensor_id];
    }
    OPKS(c, ZO2_KC_K1, st, k1_launch(a, c->cfg.wire_dtype, c->cfg.compute_dtype, true, false, st));
    return ZO2_OK;
}
static zo2_status stale_updates_block(zo2_ctx* c, int l, char* bucket, hipStream_t st = nullptr) {
    if (c->resident) return ZO2_OK;
    for (int k = 0; k < c->n_stale; ++k) {
        zo2_status s = k1_block_replay(c, l, bucket, stale_slot(c, k), c->stale_seed[k], st);
        if (s != ZO2_OK) return s;
    }
    return ZO2_OK;
}

// the final LayerNorm's two vectors
static zo2_status k1_final_ln(zo2_ctx* c, bool perturb, uint64_t seed, float eps, int pend = -1) {
    K1Args a;
    k1_common(c, a, seed, eps, pend);
    a.theta = c->d_fln; a.w_off0 = 0; a.nseg = 2;
    if (perturb) { a.w_plus = c->fln_wp; a.w_minus = c->ns == 2 ? c->fln_wm : nullptr; }
    for (int k = 0; k < 2; ++k) {
        a.seg[k].off = k * c->fln_off_b; a.seg[k].e0 = 0; a.seg[k].n = (uint64_t)c->cfg.d_model;
        a.seg[k].tensor_id = fln_tid(c) + k; a.seg[k].scale = c->scales[fln_tid(c) + k];
    }
    OPK(c, ZO2_KC_K1, k1_launch(a, c->cfg.wire_dtype, c->cfg.compute_dtype, pend >= 0 || fused_update(c), perturb, c->sc));
    return ZO2_OK;
}

// Deferred updates 0 .. n_pend - 2 of a module, in order, as update-only sweeps: after a round of several directions
// they precede the fused sweep, which applies the last one together with the new perturbation.
static zo2_status earlier_updates_tensor(zo2_ctx* c, void* theta, int64_t n, uint32_t tid, hipStream_t st = nullptr) {
    if (!c->apply_now) return ZO2_OK;
    for (int k = 0; k + 1 < c->n_pend; ++k) {
        zo2_status s = k1_tensor(c, theta, n, tid, false, nullptr, nullptr, 0, 0.f, st, k);
        if (s != ZO2_OK) return s;
    }
    return ZO2_OK;
}
static zo2_status earlier_updates_block(zo2_ctx* c, int l, char* bucket, hipStream_t st = nullptr) {
    if (c->dir_later) return ZO2_OK;          // the first direction of the pass has brought the block up to date
    { zo2_status s = stale_updates_block(c, l, bucket, st); if (s != ZO2_OK) return s; }      // what the host copy lacks comes first, whatever the pass
    if (!c->apply_now) return ZO2_OK;
    for (int k = 0; k + 1 < c->n_pend; ++k) {
        zo2_status s = k1_block(c, l, bucket, 0, ZO2_BLOCK_TENSORS, false, 0, 0.f, st, k);
        if (s != ZO2_OK) return s;
    }
    return ZO2_OK;
}

// ---------------------------------------------------------------------------------- block forward
// float32: the logits chunk, idle until the head, takes the partial sums; only the part of it that every budget provides is
// counted on, so that the split - and with it the order of the sums - does not depend on the plan
static size_t f32_split_workspace(const zo2_ctx* c, int T) { return 2 * (size_t)std::min(T, 128) * c->cfg.vocab * sizeof(float); }
static int f32_pieces(const zo2_ctx* c, const GemmArgs& ga) { return gemm_f32_pick_splits(ga.M, ga.N, ga.K, ga.nprob, f32_split_workspace(c, ga.M)); }

// A block projection: split along k when the launch would leave most compute units idle (few rows per stream).
// left: a projection onto the residual stream that is split leaves its pieces in the workspace, described here but for the biases, for
// the pass of the LayerNorm behind it; pieces = 0 where there is nothing left to add.
static zo2_status block_gemm(zo2_ctx* c, GemmArgs ga, RowSum* left = nullptr) {
    const int dt = c->cfg.compute_dtype;
    ga.large_only = keep_order(c);
    const bool sum = left == nullptr;
    auto leave = [&](const void* part, int pieces) {
        if (left && pieces > 1) *left = RowSum{(const float*)part, pieces, (int64_t)ga.M * ga.N, (int64_t)pieces * ga.M * ga.N, nullptr, nullptr};
    };
    if (left) left->pieces = 0;
    if (dt == ZO2_F32 && c->split_k >= 0) {
        const int pieces = f32_pieces(c, ga);
        leave(c->logits, pieces);
        return gemm_launch_f32_splitk(ga, pieces, c->logits, f32_split_workspace(c, ga.M), c->sc, sum);
    }
    if (c->split_k >= 0 && dt != ZO2_F32) {
        const GemmChoice k = gemm_choose(ga, dt, c->split_ws_bytes);
        if (k.rows || k.splits > 1) leave(c->sk_ws, k.splits);
        if (k.rows) return gemm_launch_mid_splitk(ga, dt, k.rows, k.splits, c->sk_ws, c->sk_ws_bytes, c->sc, sum);
        if (k.splits > 1) return gemm_launch_splitk(ga, dt, k.splits, c->sk_ws, c->sk_ws_bytes, c->sc, sum);
    }
    return gemm_launch(ga, dt, c->sc);
}

// Pieces of a projection onto the residual stream can wait for the LayerNorm behind it, whose pass adds them up in the order that the
// sum's own pass would take.  That saves a launch (370 rows of 2048: 5.8 + 5.0 -> 6.1 us), but a workgroup per row is
// the slower way where there are rows enough (1026 of 2560: 16.0 + 6.5 -> 23.9); the line is drawn between the two.
static inline bool may_leave_sum(const zo2_ctx* c, int T) {
    return c->sweeps == 1 && reduce_layernorm_applicable(c->cfg.d_model) && (int64_t)c->ns * T * c->cfg.d_model <= (int64_t)1 << 20;
}
// FC2's pieces wait for the next block's first LayerNorm, or the final one.  Between the two comes the next block's sweep, so the
// perturbed FC2 biases must outlive it: odd blocks keep them behind the block's other copies (`after`: elements of one block's copies),
// where the scratch has room for that.
static inline bool may_leave_fc2(const zo2_ctx* c, int T, int64_t after, int64_t more) {
    return c->one_dir && !c->overlap_k1 && may_leave_sum(c, T) && after + more <= c->scratch_elems;
}
static inline int64_t fc2_bias_room(const zo2_ctx* c) { return (c->tn[15] + kTensorAlign - 1) / kTensorAlign * kTensorAlign; }
// h += pieces that the block before left, if any; x = LayerNorm(h)
static zo2_status sum_and_norm(zo2_ctx* c, const void* wp, const void* bp, const void* wm, const void* bm, int T) {
    const zo2_config& g = c->cfg;
    if (c->left.pieces > 0) ++c->sums_left;
    if (c->left.pieces > 0) OPK(c, ZO2_KC_LN, reduce_layernorm(g.compute_dtype, c->left, c->h, wp, bp, wm, bm, c->x, c->ns * T, T, g.d_model, g.ln_eps, c->sc));
    else OPK(c, ZO2_KC_LN, layernorm(g.compute_dtype, c->h, wp, bp, wm, bm, c->x, c->ns * T, T, g.d_model, g.ln_eps, c->sc));
    c->left.pieces = 0;
    return ZO2_OK;
}

// A single forward whose parameters are stored in the compute format has nothing to perturb and nothing to convert: it reads
// them where they lie, and a sweep only comes before it where an update is pending.  (Copies cost 33 us a block and 63 for the
// vocabulary matrix at d 2048: an evaluation of 8 blocks, 16 x 256 tokens, nothing pending, 4473 -> 4077 us; right behind a step, whose
// update the sweeps still apply, 4606 -> 4451.)
static inline bool reads_in_place(const zo2_ctx* c) { return c->ns == 1 && c->cfg.wire_dtype == c->cfg.compute_dtype && !c->overlap_k1; }

struct PhaseView {       // where tensor k's perturbed copies are inside the scratch, or the tensor itself
    const zo2_ctx* c;
    int64_t off0;
    const char* bucket;      // nullptr: copies
    const char* P(int k) const { return bucket ? bucket + (size_t)c->offs[k] * c->csz : c->wp + (size_t)(c->offs[k] - off0) * c->csz; }
    const char* M(int k) const { return bucket ? P(k) : c->wm + (size_t)(c->offs[k] - off0) * c->csz; }
};

static zo2_status block_forward(zo2_ctx* c, int l, char* bucket, int batch, int seq, uint64_t seed, float eps, hipEvent_t k1_done,
                                bool k1_enqueued = false) {
    const zo2_config& g = c->cfg;
    const int T = batch * seq, d = g.d_model, f = g.d_ffn, dh = d / g.n_heads;
    const int dt = g.compute_dtype;
    const size_t cs = c->csz;
    const size_t half_d = (size_t)T * d * cs, half_f = (size_t)T * f * cs;
    const bool f32 = dt == ZO2_F32;
    const int ns = c->ns;                 // 2: both perturbation streams (rows 0..T-1 and T..2T-1); 1: a single forward
    const bool in_place = reads_in_place(c);
    // (read in place, the biases stay where they are for as long as the block does)
    const bool leave_fc2 = !k1_enqueued && (in_place ? c->resident && may_leave_fc2(c, T, 0, 0) : may_leave_fc2(c, T, c->offs[ZO2_BLOCK_TENSORS], fc2_bias_room(c)));
    const int64_t bias2_at = !in_place && leave_fc2 && (l & 1) ? c->offs[ZO2_BLOCK_TENSORS] : -1;
    auto phase = [&](int p) -> zo2_status {
        if (in_place) {
            if (p > 0) return ZO2_OK;
            if (fused_update(c)) { const zo2_status s = k1_block(c, l, bucket, 0, ZO2_BLOCK_TENSORS, false, seed, eps); if (s != ZO2_OK) return s; }
            if (k1_done) HIPCHK(c, hipEventRecord(k1_done, c->sc));
            return ZO2_OK;
        }
        if (k1_enqueued || c->pb[p + 1] == c->pb[p]) return ZO2_OK;
        zo2_status s = k1_block(c, l, bucket, c->pb[p], c->pb[p + 1], true, seed, eps, nullptr, -1, bias2_at);
        // the block's parameters are final after its last sweep: the offload may start (streamed mode)
        if (s == ZO2_OK && c->pb[p + 1] == ZO2_BLOCK_TENSORS && k1_done) HIPCHK(c, hipEventRecord(k1_done, c->sc));
        return s;
    };
    // the scratch holds the tensors of the last sweep issued at or before point p, the first of them at its start
    auto view = [&](int p) {
        int q = p;
        while (c->pb[q + 1] == c->pb[q]) --q;       // sweep 0 is never empty
        return PhaseView{c, c->offs[c->pb[q]], in_place ? bucket : nullptr};
    };
    GemmArgs ga;

    // ---- attention half: h += O(Attn(LN1(h)))
    if (!k1_enqueued) { zo2_status s = earlier_updates_block(c, l, bucket); if (s != ZO2_OK) return s; }
    { zo2_status s = phase(0); if (s != ZO2_OK) return s; }
    PhaseView w = view(0);
    { zo2_status s = sum_and_norm(c, w.P(0), w.P(1), w.M(0), w.M(1), T); if (s != ZO2_OK) return s; }
    memset(&ga, 0, sizeof(ga));
    ga.M = T; ga.N = d; ga.K = d; ga.ldx = d; ga.ldw = d; ga.ldy = d; ga.relu = 0; ga.out_f32 = f32; ga.nprob = 3 * ns;
    char* outs[3] = {c->qb, c->kb, c->vb};
    for (int s = 0; s < ns; ++s)
        for (int t = 0; t < 3; ++t) {
            GemmProblem& p = ga.p[s * 3 + t];
            p.X = c->x + s * half_d;
            p.W = s ? w.M(2 + 2 * t) : w.P(2 + 2 * t);
            p.bias = s ? w.M(3 + 2 * t) : w.P(3 + 2 * t);
            p.residual = nullptr;
            p.Y = outs[t] + s * half_d;
            p.out_scale = t == 0 ? 1.0f / sqrtf((float)dh) : 1.0f;
        }
    OPK(c, ZO2_KC_GEMM, block_gemm(c, ga));
    OPK(c, ZO2_KC_ATTN, attention_launch(dt, c->qb, c->kb, c->vb, c->ctxb, ns * batch, seq, g.n_heads, dh, d, 0, c->sc));
    { zo2_status s = phase(1); if (s != ZO2_OK) return s; }
    w = view(1);
    memset(&ga, 0, sizeof(ga));
    ga.M = T; ga.N = d; ga.K = d; ga.ldx = d; ga.ldw = d; ga.ldy = d; ga.relu = 0; ga.out_f32 = 1; ga.nprob = ns;
    for (int s = 0; s < ns; ++s) {
        GemmProblem& p = ga.p[s];
        p.X = c->ctxb + s * half_d; p.W = s ? w.M(8) : w.P(8); p.bias = s ? w.M(9) : w.P(9);
        p.residual = c->h + (size_t)s * T * d; p.Y = c->h + (size_t)s * T * d; p.out_scale = 1.0f;
    }
    // in pieces and with one sweep per block (no other one between the two): the LayerNorm's pass adds them up
    const bool leave_o = may_leave_sum(c, T) || (f32 && c->sweeps == 1 && reduce_layernorm_applicable(d));
    OPK(c, ZO2_KC_GEMM, block_gemm(c, ga, leave_o ? &c->left : nullptr));
    c->left.bias = w.P(9); c->left.bias2 = w.M(9);

    // ---- FFN half: h += FC2(ReLU(FC1(LN2(h))))
    { zo2_status s = phase(2); if (s != ZO2_OK) return s; }
    w = view(2);
    { zo2_status s = sum_and_norm(c, w.P(10), w.P(11), w.M(10), w.M(11), T); if (s != ZO2_OK) return s; }
    memset(&ga, 0, sizeof(ga));
    ga.M = T; ga.N = f; ga.K = d; ga.ldx = d; ga.ldw = d; ga.ldy = f; ga.relu = 1; ga.out_f32 = f32; ga.nprob = ns;
    for (int s = 0; s < ns; ++s) {
        GemmProblem& p = ga.p[s];
        p.X = c->x + s * half_d; p.W = s ? w.M(12) : w.P(12); p.bias = s ? w.M(13) : w.P(13);
        p.residual = nullptr; p.Y = c->mid + s * half_f; p.out_scale = 1.0f;
    }
    OPK(c, ZO2_KC_GEMM, block_gemm(c, ga));
    { zo2_status s = phase(3); if (s != ZO2_OK) return s; }
    w = view(3);
    memset(&ga, 0, sizeof(ga));
    ga.M = T; ga.N = d; ga.K = f; ga.ldx = f; ga.ldw = f; ga.ldy = d; ga.relu = 0; ga.out_f32 = 1; ga.nprob = ns;
    const char *bias2_p = bias2_at < 0 ? w.P(15) : c->wp + (size_t)bias2_at * cs, *bias2_m = bias2_at < 0 ? w.M(15) : c->wm + (size_t)bias2_at * cs;
    for (int s = 0; s < ns; ++s) {
        GemmProblem& p = ga.p[s];
        p.X = c->mid + s * half_f; p.W = s ? w.M(14) : w.P(14); p.bias = s ? bias2_m : bias2_p;
        p.residual = c->h + (size_t)s * T * d; p.Y = c->h + (size_t)s * T * d; p.out_scale = 1.0f;
    }
    OPK(c, ZO2_KC_GEMM, block_gemm(c, ga, leave_fc2 ? &c->left : nullptr));
    c->left.bias = bias2_p; c->left.bias2 = bias2_m;
    return ZO2_OK;
}

// A resident block under `n` directions j0 .. j0 + n - 1 of a round at once: one sweep applies the deferred updates (the first
// group's) and writes the perturbed copies of all of them, and a projection of all directions is one launch.  Everything is
// computed by the kernels, and added up in the order, that one direction alone would take, so the results are the same bits.
// (OPT-1.3B shape, 4 x 128 tokens, four directions, a block in us, one after the other -> together: sweeps 295 -> 176, QKV 141 -> 132, output
// 78 -> 65, FC1 149 -> 120, FC2 218 -> 164, attention 28 -> 18, LayerNorm 46 -> 28; a round
// of 8 blocks 9530 -> 7640.)
static zo2_status block_forward_round(zo2_ctx* c, int l, char* bucket, int batch, int seq, const uint64_t* seeds, int j0, int n, bool update, float eps) {
    const zo2_config& g = c->cfg;
    const int T = batch * seq, d = g.d_model, f = g.d_ffn, dh = d / g.n_heads, dt = g.compute_dtype;
    const size_t cs = c->csz, half_d = (size_t)T * d * cs, half_f = (size_t)T * f * cs;
    {
        K1RoundArgs a;
        memset(&a, 0, sizeof(a));
        a.theta = bucket; a.c_ptr = coef_slot(c, 0); a.n_upd = update ? c->n_pend : 0; a.n_dir = n; a.nseg = ZO2_BLOCK_TENSORS;
        a.stochastic = c->stochastic ? 1 : 0; a.eps = eps;
        for (int u = 0; u < a.n_upd; ++u) a.k_upd[u] = philox_keys(c->pend_seed[u]);
        for (int j = 0; j < n; ++j) { a.w_plus[j] = c->wide_wp[j]; a.w_minus[j] = c->wide_wm[j]; a.k_dir[j] = philox_keys(seeds[j0 + j]); }
        for (int k = 0; k < ZO2_BLOCK_TENSORS; ++k) {
            K1Seg& s = a.seg[k];
            s.off = c->offs[k]; s.e0 = 0; s.n = (uint64_t)c->tn[k]; s.tensor_id = block_tid(l, k); s.scale = c->scales[s.tensor_id];
        }
        OPK(c, ZO2_KC_K1, k1_round_launch(a, g.wire_dtype, dt, c->sc));
    }
    auto W = [&](int j, int s, int k) { return (const void*)((s ? c->wide_wm[j] : c->wide_wp[j]) + (size_t)c->offs[k] * cs); };
    const int64_t step = c->wide_wm[0] - c->wide_wp[0];
    const bool h_joined = n == 1 || c->hs[j0 + 1] - c->hs[j0] == (int64_t)2 * T * d;
    auto norm = [&](int k) -> zo2_status {
        if (h_joined && layernorm_sets_applicable(dt, d, c->wide_x, W(0, 0, k), W(0, 0, k + 1), step)) {
            OPK(c, ZO2_KC_LN, layernorm_sets(dt, c->hs[j0], W(0, 0, k), W(0, 0, k + 1), step, c->wide_x, 2 * n * T, T, d, g.ln_eps, c->sc));
            return ZO2_OK;
        }
        for (int j = 0; j < n; ++j)
            OPK(c, ZO2_KC_LN, layernorm(dt, c->hs[j0 + j], W(j, 0, k), W(j, 0, k + 1), W(j, 1, k), W(j, 1, k + 1), c->wide_x + 2 * j * half_d, 2 * T, T, d, g.ln_eps, c->sc));
        return ZO2_OK;
    };
    // one projection of every direction: out[t] = X W_(tensor + 2 t)^T, t < np
    auto project = [&](int np, int tensor, int N, int K, const char* X, char* const* out, bool relu, bool to_h) -> zo2_status {
        GemmArgs ga;
        memset(&ga, 0, sizeof(ga));
        ga.M = T; ga.N = N; ga.K = K; ga.ldx = K; ga.ldw = K; ga.ldy = N; ga.relu = relu; ga.out_f32 = to_h; ga.large_only = keep_order(c);
        auto fill = [&](GemmProblem& p, int j, int s, int t) {
            const size_t row = (size_t)(2 * j + s) * T;
            p.X = X + row * K * cs; p.W = W(j, s, tensor + 2 * t); p.bias = W(j, s, tensor + 2 * t + 1);
            float* h = c->hs[j0 + j] + (size_t)s * T * d;
            p.residual = to_h ? h : nullptr; p.Y = to_h ? (void*)h : (void*)(out[t] + row * N * cs);
            p.out_scale = np == 3 && t == 0 ? 1.0f / sqrtf((float)dh) : 1.0f;
        };
        // what one direction's launch would run on: the sums' order
        for (int s = 0; s < 2; ++s)
            for (int t = 0; t < np; ++t) fill(ga.p[s * np + t], 0, s, t);
        ga.nprob = 2 * np;
        const GemmChoice k = gemm_choose(ga, dt, c->split_k >= 0 ? c->split_ws_bytes : 0);
        const GemmChoice choice = c->split_k >= 0 ? k : GemmChoice{k.rows, 1};
        for (int j = 0; j < n; ++j)
            for (int s = 0; s < 2; ++s)
                for (int t = 0; t < np; ++t) fill(ga.p[(2 * j + s) * np + t], j, s, t);
        ga.nprob = 2 * np * n;
        OPK(c, ZO2_KC_GEMM, gemm_launch_groups(ga, dt, choice, n, c->wide_ws, c->wide_ws_bytes, c->sc));
        return ZO2_OK;
    };
#define ROUND(call) { const zo2_status s_ = (call); if (s_ != ZO2_OK) return s_; }
    char* qkv[3] = {c->wide_q, c->wide_k, c->wide_v};
    char* mid[1] = {c->wide_mid};
    ROUND(norm(0));
    ROUND(project(3, 2, d, d, c->wide_x, qkv, false, false));
    // (grids have a limit, which one direction keeps: per direction beyond it)
    const int at_once = (int64_t)2 * n * batch <= 65535 && (int64_t)2 * n * batch * g.n_heads * ((seq + 127) / 128 + 1) < (int64_t)1 << 30 ? n : 1;
    for (int j = 0; j < n; j += at_once) {
        const size_t at = 2 * j * half_d;
        OPK(c, ZO2_KC_ATTN, attention_launch(dt, c->wide_q + at, c->wide_k + at, c->wide_v + at, c->wide_ctx + at, 2 * at_once * batch, seq, g.n_heads, dh, d, 0, c->sc));
    }
    ROUND(project(1, 8, d, d, c->wide_ctx, nullptr, false, true));
    ROUND(norm(10));
    ROUND(project(1, 12, f, d, c->wide_x, mid, true, false));
    ROUND(project(1, 14, d, f, c->wide_mid, nullptr, false, true));
#undef ROUND
    return ZO2_OK;
}

// The same block for a step of few tokens: K1 applies the pending update (theta' is final after it), or leaves that of the matrices to the projections
// (block_updates_in_loader: final behind FC2), and perturbs the block's ten one-dimensional tensors into a densely packed scratch; the six projections
// read theta' itself and perturb in their weight loader, both streams per pass over the weights (gemm_skinny.hip).
static const int kVecTensors[10] = {0, 1, 3, 5, 7, 9, 10, 11, 13, 15};      // ln1.w ln1.b q.b k.b v.b o.b ln2.w ln2.b fc1.b fc2.b

// The last deferred update can be applied by the same loader, so that a matrix is read and written once: always in float32, in bfloat16 up to 32
// tokens.  With more the loader, bound by the vector ALU, takes longer for the second draw than a sweep of its own, which leaves the block in the
// memory-side cache (sweep -> loader, both with skinny_rows_kernel, us: d 2048, 12 blocks, 16 tokens 1526 -> 1485, 48 1702 -> 1686; d 4096, 4 blocks, 20 1499 -> 1365, 64 1717 -> 1748;
// d 5120, 3 blocks, 90 2159 -> 2252; d 768 766 -> 767).  float16 stays with the sweep, whose compiled roundings every update has to share (embed_kernel),
// and so does stochastic rounding, a third draw.
static inline bool updates_in_loader(const zo2_ctx* c, int T) {
    const int dt = c->cfg.compute_dtype;
    return fused_update(c) && (dt == ZO2_F32 || (dt == ZO2_BF16 && T <= 32 && !c->stochastic));
}
// A streamed block that goes back to its host buffer is swept all the same: it is final, and its offload starts, a sweep behind its upload and not behind its
// FC2, and the link, not the kernels, is what such a step waits for (3 slots, us a step, swept -> updated in the loader: bfloat16, 16 tokens, d 768,
// 8 blocks 2760 -> 2800, d 2048 18270 -> 18326; float32, 64 tokens, d 768, 10 blocks 6515 -> 6597).  The tables and the head never leave.
static inline bool block_updates_in_loader(const zo2_ctx* c, int T) { return updates_in_loader(c, T) && (c->resident || !c->pass_writes_back); }
static void loader_applies(const zo2_ctx* c, SkinnyArgs& sa) {
    sa.key_prev = philox_keys(c->pend_seed[c->n_pend - 1]);
    sa.c_ptr = coef_slot(c, c->n_pend - 1);
}

static int64_t place_vectors(const zo2_ctx* c, int64_t* voff) {      // where a block's copies of its vectors stand; returns their elements
    int64_t o = 0;
    for (const int k : kVecTensors) {
        voff[k] = o;
        o += (c->tn[k] + kTensorAlign - 1) / kTensorAlign * kTensorAlign;
    }
    return o;
}
// The vectors of resident blocks have no reason to wait for their block: one launch ahead of the first sweeps those of all and the final
// LayerNorm's, where no sweep of the matrices would take them along and the scratch holds them (12 blocks: 4.7 -> 0.5 us a
// block; steps, us: d 2048, 16 tokens, bf16 1497 -> 1464; d 768, 64 tokens, float32 1290 -> 1252).  (float16: embed_kernel says why its
// roundings stay in the instance they are in.)
static bool vectors_at_once(const zo2_ctx* c, int T) {
    int64_t voff[ZO2_BLOCK_TENSORS];
    return c->fuse && c->ns == 2 && c->resident && c->one_dir && !c->overlap_k1 && c->cfg.compute_dtype != ZO2_F16 && c->cfg.n_layers >= 2 && c->cfg.n_layers < 65535 &&
           (!fused_update(c) || updates_in_loader(c, T)) && (int64_t)c->cfg.n_layers * place_vectors(c, voff) <= c->scratch_elems;
}
static zo2_status sweep_vectors(zo2_ctx* c, uint64_t seed, float eps) {
    for (int l = 0; l < c->cfg.n_layers; ++l) { zo2_status s = earlier_updates_block(c, l, c->slots + (size_t)l * c->bucket_bytes); if (s != ZO2_OK) return s; }
    for (int k = 0; c->apply_now && k + 1 < c->n_pend; ++k) { zo2_status s = k1_final_ln(c, false, 0, 0.f, k); if (s != ZO2_OK) return s; }
    K1Args common;
    k1_common(c, common, seed, eps);
    K1VectorsArgs a;
    memset(&a, 0, sizeof(a));
    int64_t voff[ZO2_BLOCK_TENSORS];
    a.w_stride = place_vectors(c, voff);
    a.theta_stride = c->offs[ZO2_BLOCK_TENSORS]; a.n_blocks = c->cfg.n_layers; a.tid_stride = (int32_t)(block_tid(1, 0) - block_tid(0, 0));
    a.eps = eps; a.c_ptr = common.c_ptr; a.k_prev = common.k_prev; a.k_cur = common.k_cur;
    a.block.theta = c->slots; a.block.w_plus = c->wps[0]; a.block.w_minus = c->wms[0];
    for (const int k : kVecTensors) a.block.seg[a.block.nseg++] = K1Seg{c->offs[k], 0, (uint64_t)c->tn[k], block_tid(0, k), 1.0f, voff[k]};
    a.last.theta = c->d_fln; a.last.w_plus = c->fln_wp; a.last.w_minus = c->fln_wm; a.last.nseg = 2;
    for (int k = 0; k < 2; ++k) a.last.seg[k] = K1Seg{k * c->fln_off_b, 0, (uint64_t)c->cfg.d_model, fln_tid(c) + k, 1.0f, k * c->fln_off_b};
    OPK(c, ZO2_KC_K1, k1_vectors_launch(a, c->cfg.compute_dtype, fused_update(c), c->sc));
    return ZO2_OK;
}
static zo2_status block_forward_fused(zo2_ctx* c, int l, char* bucket, int batch, int seq, uint64_t seed, float eps, hipEvent_t k1_done) {
    const zo2_config& g = c->cfg;
    const int T = batch * seq, d = g.d_model, f = g.d_ffn, dh = d / g.n_heads;
    const int dt = g.compute_dtype;
    const size_t cs = c->csz;
    const bool f32 = dt == ZO2_F32, loader_updates = block_updates_in_loader(c, T);
    const size_t half_d = (size_t)T * d * cs, half_f = (size_t)T * f * cs;
    int64_t voff[ZO2_BLOCK_TENSORS] = {0};
    const int64_t vec_elems = place_vectors(c, voff);
    const bool leave_fc2 = may_leave_fc2(c, T, vec_elems, vec_elems);
    {
        const int64_t base = c->vectors_at_once ? l * vec_elems : leave_fc2 && (l & 1) ? vec_elems : 0;
        for (const int k : kVecTensors) voff[k] += base;
    }
    if (!c->vectors_at_once) {
        { zo2_status s = earlier_updates_block(c, l, bucket); if (s != ZO2_OK) return s; }
        auto is_vec = [](int k) { for (const int v : kVecTensors) if (v == k) return true; return false; };
        // the matrices have no part in the sweep where no update is pending, or where the loader applies it
        const bool update = fused_update(c), sweep_matrices = update && !loader_updates;
        K1Args a, m;                               // (float32: the matrices in a launch of their own, which only updates)
        k1_common(c, a, seed, eps);
        a.theta = bucket; a.w_plus = c->wp; a.w_minus = c->wm; a.packed_w = 1; a.mixed = sweep_matrices && !f32; a.nseg = 0;
        m = a;
        for (int k = 0; k < ZO2_BLOCK_TENSORS; ++k) {
            if (!sweep_matrices && !is_vec(k)) continue;
            K1Args& to = f32 && !is_vec(k) ? m : a;
            K1Seg& sg = to.seg[to.nseg++];
            sg.off = c->offs[k]; sg.e0 = 0; sg.n = (uint64_t)c->tn[k]; sg.tensor_id = block_tid(l, k); sg.scale = 1.0f;
            sg.woff = is_vec(k) ? voff[k] : -1;
        }
        OPK(c, ZO2_KC_K1, k1_launch(a, g.wire_dtype, g.compute_dtype, update, true, c->sc));
        if (m.nseg) OPK(c, ZO2_KC_K1, k1_launch(m, g.wire_dtype, g.compute_dtype, true, false, c->sc));
    }
    if (k1_done && !loader_updates) HIPCHK(c, hipEventRecord(k1_done, c->sc));      // the block's parameters are final: the offload may start
    auto VP = [&](int k) { return (const void*)(c->wp + (size_t)voff[k] * cs); };
    auto VM = [&](int k) { return (const void*)(c->wm + (size_t)voff[k] * cs); };
    auto TH = [&](int k) { return (void*)(bucket + (size_t)c->offs[k] * cs); };
    void* ws = f32 ? (void*)c->logits : c->sk_ws;
    const size_t ws_bytes = f32 ? f32_split_workspace(c, T) : c->sk_ws_bytes;
    SkinnyArgs sa;
    auto common = [&](int N, int K, int ldx, int ldy, int relu, int out_f32, int nprob) {
        memset(&sa, 0, sizeof(sa));
        sa.M = T; sa.N = N; sa.K = K; sa.ldx = ldx; sa.ldy = ldy; sa.relu = relu; sa.out_f32 = out_f32; sa.nprob = nprob; sa.eps = eps;
        sa.key = philox_keys(seed); sa.in_order = keep_order(c);
        if (loader_updates) loader_applies(c, sa);
    };

    // ---- attention half: h += O(Attn(LN1(h)))
    { zo2_status s = sum_and_norm(c, VP(0), VP(1), VM(0), VM(1), T); if (s != ZO2_OK) return s; }
    common(d, d, d, d, 0, 0, 3);
    char* outs[3] = {c->qb, c->kb, c->vb};
    for (int t = 0; t < 3; ++t) {
        SkinnyProblem& p = sa.p[t];
        p.Xp = c->x; p.Xm = c->x + half_d; p.theta = TH(2 + 2 * t); p.bias_p = VP(3 + 2 * t); p.bias_m = VM(3 + 2 * t);
        p.Yp = outs[t]; p.Ym = outs[t] + half_d; p.out_scale = t == 0 ? 1.0f / sqrtf((float)dh) : 1.0f; p.tensor_id = block_tid(l, 2 + 2 * t);
    }
    OPK(c, ZO2_KC_GEMM, skinny_launch(sa, dt, ws, ws_bytes, c->sc));
    OPK(c, ZO2_KC_ATTN, attention_launch(dt, c->qb, c->kb, c->vb, c->ctxb, 2 * batch, seq, g.n_heads, dh, d, 0, c->sc));
    common(d, d, d, d, 0, 1, 1);
    sa.onto_residual = 1;
    {
        SkinnyProblem& p = sa.p[0];
        p.Xp = c->ctxb; p.Xm = c->ctxb + half_d; p.theta = TH(8); p.bias_p = VP(9); p.bias_m = VM(9);
        p.res_p = c->h; p.res_m = c->h + (size_t)T * d; p.Yp = c->h; p.Ym = c->h + (size_t)T * d; p.out_scale = 1.0f; p.tensor_id = block_tid(l, 8);
    }
    // the output projection's slices are summed by the pass that makes FFN half's LayerNorm: h += FC2(ReLU(FC1(LN2(h))))
    const bool sum_with_ln = reduce_layernorm_applicable(d);
    OPK(c, ZO2_KC_GEMM, skinny_launch(sa, dt, ws, ws_bytes, c->sc, !sum_with_ln));
    if (sum_with_ln) {
        const RowSum rs = {sa.partial, sa.splits, 2 * (int64_t)T * d, (int64_t)T * d, VP(9), VM(9)};
        ++c->sums_left;
        OPK(c, ZO2_KC_LN, reduce_layernorm(dt, rs, c->h, VP(10), VP(11), VM(10), VM(11), c->x, 2 * T, T, d, g.ln_eps, c->sc));
    } else {
        OPK(c, ZO2_KC_LN, layernorm(dt, c->h, VP(10), VP(11), VM(10), VM(11), c->x, 2 * T, T, d, g.ln_eps, c->sc));
    }
    common(f, d, d, f, 1, 0, 1);
    {
        SkinnyProblem& p = sa.p[0];
        p.Xp = c->x; p.Xm = c->x + half_d; p.theta = TH(12); p.bias_p = VP(13); p.bias_m = VM(13);
        p.Yp = c->mid; p.Ym = c->mid + half_f; p.out_scale = 1.0f; p.tensor_id = block_tid(l, 12);
    }
    OPK(c, ZO2_KC_GEMM, skinny_launch(sa, dt, ws, ws_bytes, c->sc));
    common(d, f, f, d, 0, 1, 1);
    sa.onto_residual = 1;
    {
        SkinnyProblem& p = sa.p[0];
        p.Xp = c->mid; p.Xm = c->mid + half_f; p.theta = TH(14); p.bias_p = VP(15); p.bias_m = VM(15);
        p.res_p = c->h; p.res_m = c->h + (size_t)T * d; p.Yp = c->h; p.Ym = c->h + (size_t)T * d; p.out_scale = 1.0f; p.tensor_id = block_tid(l, 14);
    }
    OPK(c, ZO2_KC_GEMM, skinny_launch(sa, dt, ws, ws_bytes, c->sc, !leave_fc2));
    if (leave_fc2) c->left = RowSum{sa.partial, sa.splits, 2 * (int64_t)T * d, (int64_t)T * d, VP(15), VM(15)};
    if (k1_done && loader_updates) HIPCHK(c, hipEventRecord(k1_done, c->sc));
    return ZO2_OK;
}

// A sweep of a round over one tensor or two: all deferred updates (updates = true), and the copies of directions j0 .. j0 + n - 1.
static zo2_status k1_round_tables(zo2_ctx* c, void* theta, const K1Seg* seg, int nseg, bool updates, const uint64_t* seeds, int n, char* const* wp, char* const* wm, float eps) {
    K1RoundArgs a;
    memset(&a, 0, sizeof(a));
    a.theta = theta; a.c_ptr = coef_slot(c, 0); a.n_upd = updates ? c->n_pend : 0; a.n_dir = n; a.nseg = nseg;
    a.stochastic = c->stochastic ? 1 : 0; a.eps = eps;
    for (int u = 0; u < a.n_upd; ++u) a.k_upd[u] = philox_keys(c->pend_seed[u]);
    for (int j = 0; j < n; ++j) { a.w_plus[j] = wp[j]; a.w_minus[j] = wm[j]; a.k_dir[j] = philox_keys(seeds[j]); }
    for (int k = 0; k < nseg; ++k) { a.seg[k] = seg[k]; a.seg[k].scale = c->scales[seg[k].tensor_id]; }
    OPK(c, ZO2_KC_K1, k1_round_launch(a, c->cfg.wire_dtype, c->cfg.compute_dtype, c->sc));
    return ZO2_OK;
}
static inline K1Seg whole_tensor(int64_t off, int64_t n, uint32_t tid) { return K1Seg{off, 0, (uint64_t)n, tid, 1.0f, 0}; }

// The head under directions j0 .. j0 + n - 1 of a round: final LayerNorm, vocabulary matrix and row losses of all of them in one launch each.
// Row losses of direction j0 + j: head_loss + 2 j T.  (Vocabulary 50272, d 2048, 4 x 128 tokens, four directions, in us, one after the
// other -> together: sweeps of the matrix 579, three of them in front of the gather -> 367; logits 977, four launches of 3.1 rounds of tiles
// each -> 755; a step of 8 blocks 7294 -> 6779.)
static zo2_status head_round(zo2_ctx* c, int T, const uint64_t* seeds, int j0, int n, bool update, float eps) {
    const zo2_config& g = c->cfg;
    const int d = g.d_model, dt = g.compute_dtype;
    const size_t cs = c->csz, half_d = (size_t)T * d * cs;
    const int64_t set = (int64_t)align_up((size_t)c->fln_elems * cs, 256);      // from one copy of the final LayerNorm's vectors to the next
    char *fp[zo2_ctx::kMaxWide], *fm[zo2_ctx::kMaxWide];
    for (int j = 0; j < n; ++j) { fp[j] = c->head_fln + 2 * j * set; fm[j] = fp[j] + set; }
    const K1Seg ln[2] = {whole_tensor(0, d, fln_tid(c)), whole_tensor(c->fln_off_b, d, fln_tid(c) + 1)};
    { zo2_status s = k1_round_tables(c, c->d_fln, ln, 2, update, seeds + j0, n, fp, fm, eps); if (s != ZO2_OK) return s; }
    const size_t b = (size_t)c->fln_off_b * cs;
    if ((n == 1 || c->hs[j0 + 1] - c->hs[j0] == (int64_t)2 * T * d) && layernorm_sets_applicable(dt, d, c->head_x, fp[0], fp[0] + b, set)) {
        OPK(c, ZO2_KC_LN, layernorm_sets(dt, c->hs[j0], fp[0], fp[0] + b, set, c->head_x, 2 * n * T, T, d, g.ln_eps, c->sc));
    } else {
        for (int j = 0; j < n; ++j)
            OPK(c, ZO2_KC_LN, layernorm(dt, c->hs[j0 + j], fp[j], fp[j] + b, fm[j], fm[j] + b, c->head_x + 2 * j * half_d, 2 * T, T, d, g.ln_eps, c->sc));
    }
    const K1Seg table = whole_tensor(0, c->tok_elems, g.tied_lm_head ? 0u : lm_tid(c));
    { zo2_status s = k1_round_tables(c, g.tied_lm_head ? c->d_tok : c->d_lm, &table, 1, update, seeds + j0, n, c->head_wp, c->head_wm, eps); if (s != ZO2_OK) return s; }
    GemmArgs ga;
    memset(&ga, 0, sizeof(ga));
    ga.M = T; ga.N = g.vocab; ga.K = d; ga.ldx = d; ga.ldw = d; ga.ldy = g.vocab; ga.out_f32 = 1; ga.nprob = 2 * n; ga.ce_mode = 1; ga.like_nprob = 2; ga.part_ld = 2 * (int64_t)n * T;
    for (int i = 0; i < 2 * n; ++i) {
        GemmProblem& p = ga.p[i];
        p.X = c->head_x + i * half_d; p.W = i & 1 ? c->head_wm[i / 2] : c->head_wp[i / 2]; p.out_scale = 1.0f; p.labels = c->d_labels;
        p.part_max = c->head_pmax + (size_t)i * T; p.part_sum = c->head_psum + (size_t)i * T; p.label_logit = c->head_lab + (size_t)i * T;
    }
    OPK(c, ZO2_KC_GEMM, gemm_launch(ga, dt, c->sc));
    OPK(c, ZO2_KC_CE, ce_combine(c->head_pmax, c->head_psum, c->head_lab, c->d_labels, 2 * n * T, c->ce_parts, 2 * (int64_t)n * T, 0, T, c->head_loss, c->sc, keep_order(c), 2 * T));
    return ZO2_OK;
}

// ---------------------------------------------------------------------------------- streaming (Alg. 3)
// U(W_i): runs on the upload stream once the slot's previous occupant has left it.
static zo2_status enqueue_upload(zo2_ctx* c, int l) {
    const int s = l % c->n_slots;
    if (c->ev_free_valid[s]) HIPCHK(c, hipStreamWaitEvent(c->su, c->ev_free[s], 0));
    // with the perturbation in the projections' loader, or no perturbation at all, the forwards read the slot itself: its next occupant also waits for them
    if (c->ev_read_valid[s]) HIPCHK(c, hipStreamWaitEvent(c->su, c->ev_read[s], 0));
    if (!c->stat_u) { HIPCHK(c, hipEventRecord(c->ev_u0, c->su)); c->stat_u = true; }
    { zo2_status ds = debug_delay(c, 1, c->su); if (ds != ZO2_OK) return ds; }
    if (c->debug_poison) {      // whoever reads the slot before the copy below has landed computes NaN
        hipLaunchKernelGGL(poison_kernel, dim3(1024), dim3(256), 0, c->su, (uint32_t*)(c->slots + (size_t)s * c->bucket_bytes), c->bucket_bytes / 4);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(c, ZO2_EHIP, "poison kernel: %s", hipGetErrorString(e));
    }
    HIPCHK(c, hipMemcpyAsync(c->slots + (size_t)s * c->bucket_bytes, c->host_bucket[l], c->bucket_bytes, hipMemcpyHostToDevice, c->su));
    HIPCHK(c, hipEventRecord(c->ev_up[s], c->su));
    c->bytes_up += c->bucket_bytes;
    return ZO2_OK;
}

// O(W_i): the updated block goes back as soon as its K1 pass is done (the forwards behind it write only
// scratch; those that read the slot itself keep its next occupant waiting, ev_read); without a pending update nothing changed.
static zo2_status enqueue_offload(zo2_ctx* c, int l, bool changed) {
    const int s = l % c->n_slots;
    if (changed) {
        HIPCHK(c, hipStreamWaitEvent(c->so, c->ev_k1[s], 0));
        if (!c->stat_o) { HIPCHK(c, hipEventRecord(c->ev_o0, c->so)); c->stat_o = true; }
        { zo2_status ds = debug_delay(c, 2, c->so); if (ds != ZO2_OK) return ds; }
        HIPCHK(c, hipMemcpyAsync(c->host_bucket[l], c->slots + (size_t)s * c->bucket_bytes, c->bucket_bytes, hipMemcpyDeviceToHost, c->so));
        HIPCHK(c, hipEventRecord(c->ev_free[s], c->so));
        c->bytes_down += c->bucket_bytes;
    } else {
        HIPCHK(c, hipStreamWaitEvent(c->so, c->ev_k1[s], 0));
        HIPCHK(c, hipEventRecord(c->ev_free[s], c->so));
    }
    c->ev_free_valid[s] = 1;
    return ZO2_OK;
}

// Brings the host copies of streamed blocks up to date: every block travels once, takes the updates its host copy lacks
// and goes back.  Nothing to do when the blocks are resident or nothing is lacking.
static zo2_status writeback_pass(zo2_ctx* c) {
    if (!c->planned || c->resident || c->n_stale == 0) return ZO2_OK;
    const zo2_config& g = c->cfg;
    TraceRange range("zo2 write-back");
    c->stat_u = c->stat_o = true;   // no span statistics
    int next_upload = 0;
    for (; next_upload < c->n_slots && next_upload < g.n_layers; ++next_upload) {
        zo2_status s = enqueue_upload(c, next_upload);
        if (s != ZO2_OK) return s;
    }
    for (int l = 0; l < g.n_layers; ++l) {
        const int sl = l % c->n_slots;
        HIPCHK(c, hipStreamWaitEvent(c->sc, c->ev_up[sl], 0));
        { zo2_status s = stale_updates_block(c, l, c->slots + (size_t)sl * c->bucket_bytes); if (s != ZO2_OK) return s; }
        HIPCHK(c, hipEventRecord(c->ev_k1[sl], c->sc));
        c->ev_read_valid[sl] = 0;
        zo2_status s = enqueue_offload(c, l, true);
        if (s != ZO2_OK) return s;
        if (next_upload < g.n_layers) {
            s = enqueue_upload(c, next_upload++);
            if (s != ZO2_OK) return s;
        }
    }
    HIPCHK(c, hipStreamSynchronize(c->sc));
    HIPCHK(c, hipStreamSynchronize(c->su));
    HIPCHK(c, hipStreamSynchronize(c->so));
    c->n_stale = 0;
    return ZO2_OK;
}

// ---------------------------------------------------------------------------------- one pass over the model
// ns = 2: Alg. 2's iteration (update, perturb both ways, dual forward, g).  ns = 1: the same walk with a
// single unperturbed forward (evaluation): the pending update is still applied on the way, W+ = theta' (in place: reads_in_place).
// extra: a further direction of the current round (ns = 2): nothing deferred is applied, the parameters stay as
// they are, and the pass's own (seed, eta g) joins the deferred updates instead of replacing them.
// One pass over the model.  seeds[0 .. ndirs - 1]: the directions evaluated in this pass (ndirs > 1: zo2_step_multi; every
// module - embedding, each block while it sits in its slot, head - runs the dual forward of all directions before the
// pass moves on, so a streamed block travels once for all of them).  Results of direction j: pass_result(c, j).
static inline float* pass_result(const zo2_ctx* c, int j) { return j == 0 ? c->h_result : c->h_result + 16 + 4 * (j - 1); }
static zo2_status model_pass(zo2_ctx* c, const char* who, const int32_t* tokens, const int32_t* labels, int32_t batch, int32_t seq,
                             const uint64_t* seeds, int ndirs, float eps, float lr, int ns, bool extra = false) {
    const uint64_t seed = seeds[0];
    const zo2_config& g = c->cfg;
    if (batch <= 0 || seq <= 0 || seq > g.max_pos) return fail(c, ZO2_EINVAL, "%s: batch %d, seq %d (max_pos %d)", who, batch, seq, g.max_pos);
    if ((int64_t)batch * seq > (1 << 24)) return fail(c, ZO2_EINVAL, "%s: too many tokens", who);
    c->ns = ns;
    c->one_dir = ndirs == 1;
    c->left = RowSum{};
    c->together = 1;
    c->sums_left = 0;
    const int T = batch * seq;
    for (int i = 0; i < T; ++i) {
        if (tokens[i] < 0 || tokens[i] >= g.vocab) return fail(c, ZO2_EINVAL, "%s: token %d at %d outside [0, %d)", who, tokens[i], i, g.vocab);
        if (labels[i] != -100 && (labels[i] < 0 || labels[i] >= g.vocab)) return fail(c, ZO2_EINVAL, "%s: label %d at %d invalid", who, labels[i], i);
    }
    const int held = c->want_dirs;
    const bool stands = c->planned && !c->need_plan && c->plan_T == T && c->plan_seq == seq;
    c->want_dirs = std::max(c->want_dirs, ndirs);
    if (!stands || (c->plan_dirs < ndirs && !c->overlap_k1)) {
        zo2_status s = plan(c, T, batch, seq);
        if (s != ZO2_OK) return s;
    }
    // (asked of this call's plan: the one before it may have been for a step without a sweep, or there was none)
    if (c->overlap_k1 && ndirs > 1) {
        c->want_dirs = held;
        c->need_plan = !stands;
        return fail(c, ZO2_ESTATE, "%s: not available with the sweep kernel on a stream of its own", who);
    }
    const int d = g.d_model, dt = g.compute_dtype;
    c->apply_now = !extra;
    c->dir_later = false;
    // direction j of the pass: its residual stream; only the first direction of a pass applies deferred updates
    auto set_dir = [&](int j) {
        c->h = c->hs[j];
        c->dir_later = j > 0;
        c->apply_now = j == 0 ? !extra : false;
    };
    const bool upd = fused_update(c);
    // streamed blocks: does this pass write them back?  Their host copies lack n_stale updates already; this pass adds the
    // deferred ones it applies.  (The list of lacking updates must keep room for a whole round of the next pass.)
    const int lack = c->resident ? 0 : c->n_stale + (upd ? c->n_pend : 0);
    c->pass_writes_back = c->resident || lack >= c->wb_interval || lack > zo2_ctx::kMaxStale - zo2_ctx::kMaxPending;
    const bool changed = upd || (!c->resident && c->n_stale > 0);
    c->bytes_up = c->bytes_down = 0;
    c->stat_u = c->stat_o = false;
    prof_reset(c);

    memcpy(c->h_ids, tokens, (size_t)T * 4);
    memcpy(c->h_ids + T, labels, (size_t)T * 4);
    HIPCHK(c, hipEventRecord(c->ev_step0, c->sc));
    HIPCHK(c, hipMemcpyAsync(c->d_tokens, c->h_ids, (size_t)T * 4, hipMemcpyHostToDevice, c->sc));
    HIPCHK(c, hipMemcpyAsync(c->d_labels, c->h_ids + T, (size_t)T * 4, hipMemcpyHostToDevice, c->sc));

    // U(W_1..): prefetch as many blocks as there are slots; overlaps the embedding
    int next_upload = 0;
    const bool serial = c->serial_streams && !c->overlap_k1;   // the ablation is defined for the three-stream schedule
    if (!c->resident && !serial)
        for (; next_upload < c->n_slots && next_upload < g.n_layers; ++next_upload) {
            zo2_status s = enqueue_upload(c, next_upload);
            if (s != ZO2_OK) return s;
        }

    TraceRange step_range(ns == 2 ? (extra ? "zo2_step_extra" : "zo2_step") : "zo2_eval");
    // DualForward(Embedding)
    // (a head of several directions sweeps the tables once, with all deferred updates; the gather makes them for the rows it reads)
    const bool round_head = ndirs > 1 && ns == 2 && c->head_wide > 1;
    if (!round_head) {   // earlier directions of the last round: the tables first, the gather then sees them
        zo2_status s = earlier_updates_tensor(c, c->d_tok, c->tok_elems, 0);
        if (s == ZO2_OK) s = earlier_updates_tensor(c, c->d_pos, c->pos_elems, 1);
        if (s != ZO2_OK) return s;
    }
    EmbedArgs ea;
    memset(&ea, 0, sizeof(ea));
    ea.tok_emb = c->d_tok; ea.pos_emb = c->d_pos; ea.tokens = c->d_tokens; ea.h = c->h;
    ea.T = T; ea.seq = seq; ea.d = d; ea.pos_offset = g.pos_offset; ea.eps = eps; ea.single = ns == 1; ea.stochastic = c->stochastic ? 1 : 0;
    ea.scale_tok = c->scales[0]; ea.scale_pos = c->scales[1]; ea.n_upd = !upd ? 0 : round_head ? c->n_pend : 1;
    const int first_upd = c->n_pend - ea.n_upd;
    ea.c_ptr = coef_slot(c, first_upd);
    for (int u = 0; u < ea.n_upd; ++u) ea.k_upd[u] = philox_keys(c->pend_seed[first_upd + u]);
    for (int j = 0; j < ndirs; ++j) {      // every direction gathers before the tables are updated in place below
        ea.h = c->hs[j];
        ea.k_cur = philox_keys(seeds[j]);
        OPK(c, ZO2_KC_EMBED, embed_gather(ea, g.wire_dtype, dt, c->sc));
    }
    if (upd && round_head) {
        const K1Seg pos = whole_tensor(0, c->pos_elems, 1), tok = whole_tensor(0, c->tok_elems, 0);
        { zo2_status s = k1_round_tables(c, c->d_pos, &pos, 1, true, nullptr, 0, nullptr, nullptr, 0.f); if (s != ZO2_OK) return s; }
        if (!g.tied_lm_head) { zo2_status s = k1_round_tables(c, c->d_tok, &tok, 1, true, nullptr, 0, nullptr, nullptr, 0.f); if (s != ZO2_OK) return s; }
    } else if (upd) {
        { zo2_status s = k1_tensor(c, c->d_pos, c->pos_elems, 1, false, nullptr, nullptr, seed, eps); if (s != ZO2_OK) return s; }
        if (!g.tied_lm_head) { zo2_status s = k1_tensor(c, c->d_tok, c->tok_elems, 0, false, nullptr, nullptr, seed, eps); if (s != ZO2_OK) return s; }
    }

    // DualForward(W_1 .. W_N).  With a fourth stream and two scratch sets, K1 of block l runs on that
    // stream as soon as the forwards of block l-2 have released its scratch set, i.e. under the
    // forwards of block l-1 (K1 is bound by the vector ALU and HBM, the forwards by the matrix cores).
    if (c->overlap_k1) HIPCHK(c, hipEventRecord(c->ev_embed, c->sc));
    c->vectors_at_once = vectors_at_once(c, T);
    if (c->vectors_at_once) { zo2_status s = sweep_vectors(c, seed, eps); if (s != ZO2_OK) return s; }
    for (int l = 0; l < g.n_layers; ++l) {
        TraceRange block_range("block %d", l);
        const int sl = c->resident ? l : l % c->n_slots;
        char* bucket = c->slots + (size_t)sl * c->bucket_bytes;
        const int sb = l & 1;
        c->wp = c->wps[sb];
        c->wm = c->wms[sb];
        if (c->overlap_k1) {
            if (l >= 2) HIPCHK(c, hipStreamWaitEvent(c->sk, c->ev_fwd_done[sb], 0));
            if (!c->resident) HIPCHK(c, hipStreamWaitEvent(c->sk, c->ev_up[sl], 0));  // C(W_i) after U(W_i)
            { zo2_status s = earlier_updates_block(c, l, bucket, c->sk); if (s != ZO2_OK) return s; }
            { zo2_status s = k1_block(c, l, bucket, 0, ZO2_BLOCK_TENSORS, true, seed, eps, c->sk); if (s != ZO2_OK) return s; }
            HIPCHK(c, hipEventRecord(c->ev_k1done[sb], c->sk));
            if (!c->resident) HIPCHK(c, hipEventRecord(c->ev_k1[sl], c->sk));
            HIPCHK(c, hipStreamWaitEvent(c->sc, c->ev_k1done[sb], 0));
            zo2_status s = block_forward(c, l, bucket, batch, seq, seed, eps, nullptr, true);
            if (s != ZO2_OK) return s;
            HIPCHK(c, hipEventRecord(c->ev_fwd_done[sb], c->sc));
        } else {
            if (!c->resident && serial) {      // ablation of Sec. 5.2: nothing overlaps, U(W_i) starts when O(W_{i-1}) is done
                zo2_status us = enqueue_upload(c, next_upload++);
                if (us != ZO2_OK) return us;
                HIPCHK(c, hipStreamSynchronize(c->su));
            }
            if (!c->resident) HIPCHK(c, hipStreamWaitEvent(c->sc, c->ev_up[sl], 0));  // C(W_i) after U(W_i)
            { zo2_status ds = debug_delay(c, 0, c->sc); if (ds != ZO2_OK) return ds; }
            const bool fused_block = c->fuse && ns == 2, reads_slot = fused_block || reads_in_place(c);
            const bool together = ndirs > 1 && c->wide > 1;
            if (together) c->together = std::min(c->wide, ndirs);
            for (int j = 0; together && j < ndirs; j += c->wide) {
                zo2_status s = block_forward_round(c, l, bucket, batch, seq, seeds, j, std::min(c->wide, ndirs - j), upd && j == 0, eps);
                if (s != ZO2_OK) return s;
            }
            for (int j = 0; !together && j < ndirs; ++j) {
                set_dir(j);
                // the slot is read by every direction's sweep: it is released (offload, next occupant) after the last one
                hipEvent_t k1_done = (c->resident || j + 1 < ndirs) ? nullptr : c->ev_k1[sl];
                zo2_status s = fused_block ? block_forward_fused(c, l, bucket, batch, seq, seeds[j], eps, k1_done)
                                           : block_forward(c, l, bucket, batch, seq, seeds[j], eps, k1_done);
                if (s != ZO2_OK) { set_dir(0); return s; }
            }
            set_dir(0);
            if (!c->resident) {
                if (reads_slot) HIPCHK(c, hipEventRecord(c->ev_read[sl], c->sc));
                c->ev_read_valid[sl] = reads_slot ? 1 : 0;
            }
        }
        if (!c->resident && serial) {
            HIPCHK(c, hipStreamSynchronize(c->sc));
            zo2_status s = enqueue_offload(c, l, changed && c->pass_writes_back);
            if (s != ZO2_OK) return s;
            HIPCHK(c, hipStreamSynchronize(c->so));
        } else if (!c->resident) {
            zo2_status s = enqueue_offload(c, l, changed && c->pass_writes_back);                             // O(W_i) after its update
            if (s != ZO2_OK) return s;
            if (next_upload < g.n_layers) {                                        // U(W_{i+n}) into the slot O(W_i) frees
                s = enqueue_upload(c, next_upload++);
                if (s != ZO2_OK) return s;
            }
        }
    }

    // DualForward(LM head): final LayerNorm, (tied) vocabulary matrix, loss
    TraceRange head_range("lm_head + loss");
    for (int j = 0; j < ndirs; ++j) {
        const uint64_t seed = seeds[j];
        set_dir(j);
        if (round_head) {
            const int in_group = j % c->head_wide;
            if (in_group == 0) { zo2_status s = head_round(c, T, seeds, j, std::min(c->head_wide, ndirs - j), upd && j == 0, eps); if (s != ZO2_OK) { set_dir(0); return s; } }
            OPK(c, ZO2_KC_CE, loss_epilogue(c->head_loss + (size_t)2 * in_group * T, c->d_labels, T, eps, lr, ns, c->d_state + 4, coef_slot(c, j), c->sc));
            HIPCHK(c, hipMemcpyAsync(pass_result(c, j), c->d_state + 4, 4 * sizeof(float), hipMemcpyDeviceToHost, c->sc));
            continue;
        }
        for (int k = 0; !c->vectors_at_once && c->apply_now && k + 1 < c->n_pend; ++k) { zo2_status s = k1_final_ln(c, false, 0, 0.f, k); if (s != ZO2_OK) return s; }
        if (!c->vectors_at_once) { zo2_status s = k1_final_ln(c, true, seed, eps); if (s != ZO2_OK) return s; }
        const size_t boff = (size_t)c->fln_off_b * c->csz;
        { zo2_status s = sum_and_norm(c, c->fln_wp, c->fln_wp + boff, c->fln_wm, c->fln_wm + boff, T); if (s != ZO2_OK) return s; }
        // few tokens: the sweep only updates the vocabulary matrix, the head perturbs it in its loader (c->fuse rules overlap_k1 out)
        const char *head_wp = nullptr, *head_wm = nullptr;      // the vocabulary matrix of the ordinary head
        const bool loader_head = c->fuse && ns == 2 && c->fused_ce && T <= 128;
        const bool loader_logits = c->fuse && ns == 2 && dt == ZO2_F32 && c->logit_rows >= T && skinny_f32_applicable(T, g.vocab, d);      // float32: written
        if (loader_logits) {
            char* table = g.tied_lm_head ? c->d_tok : c->d_lm;
            const uint32_t tid = g.tied_lm_head ? 0u : lm_tid(c);
            if (!g.tied_lm_head) { zo2_status es = earlier_updates_tensor(c, c->d_lm, c->tok_elems, tid); if (es != ZO2_OK) return es; }
            SkinnyArgs sa;
            memset(&sa, 0, sizeof(sa));
            sa.M = T; sa.N = g.vocab; sa.K = d; sa.ldx = d; sa.nprob = 1; sa.eps = eps; sa.key = philox_keys(seed);
            sa.p[0].Xp = c->x; sa.p[0].Xm = c->x + (size_t)T * d * c->csz; sa.p[0].theta = table; sa.p[0].tensor_id = tid;
            if (updates_in_loader(c, T)) loader_applies(c, sa);
            OPK(c, ZO2_KC_GEMM, skinny_launch_sums(sa, c->logits, c->sc));
            // (both streams' rows lie together: 64 each, 50272 logits, 12.3 + 12.3 -> 13.2 us)
            OPK(c, ZO2_KC_CE, cross_entropy_rows(c->logits, g.vocab, c->d_labels, 2 * T, 0, T, g.vocab, c->row_loss, c->sc));
        } else if (loader_head) {
            char* table = g.tied_lm_head ? c->d_tok : c->d_lm;
            const uint32_t tid = g.tied_lm_head ? 0u : lm_tid(c);
            if (!g.tied_lm_head) { zo2_status es = earlier_updates_tensor(c, c->d_lm, c->tok_elems, tid); if (es != ZO2_OK) return es; }
            SkinnyArgs sa;
            memset(&sa, 0, sizeof(sa));
            if (updates_in_loader(c, T)) loader_applies(c, sa);
            else { zo2_status s = k1_tensor(c, table, c->tok_elems, tid, false, nullptr, nullptr, seed, eps); if (s != ZO2_OK) return s; }
            sa.M = T; sa.N = g.vocab; sa.K = d; sa.ldx = d; sa.nprob = 1; sa.eps = eps; sa.key = philox_keys(seed);
            sa.p[0].Xp = c->x; sa.p[0].Xm = c->x + (size_t)T * d * c->csz; sa.p[0].theta = table; sa.p[0].tensor_id = tid;
            sa.labels = c->d_labels; sa.part_max = c->ce_pmax; sa.part_sum = c->ce_psum; sa.label_logit = c->ce_lab; sa.part_ld = 2 * (int64_t)T;
            OPK(c, ZO2_KC_GEMM, skinny_launch_ce(sa, dt, c->sc));
            OPK(c, ZO2_KC_CE, ce_combine(c->ce_pmax, c->ce_psum, c->ce_lab, c->d_labels, 2 * T, 2 * ((g.vocab + 127) / 128), 2 * (int64_t)T, 0, T, c->row_loss, c->sc));
        } else {
            const int sb = g.n_layers & 1;
            c->wp = c->wps[sb];
            c->wm = c->wms[sb];
            head_wp = c->wp;
            head_wm = c->wm;
            hipStream_t st = c->sc;
            if (c->overlap_k1) {      // the vocabulary matrix is swept under the last block's forwards
                st = c->sk;
                HIPCHK(c, hipStreamWaitEvent(c->sk, c->ev_embed, 0));                  // the gather read the table before its update
                if (g.n_layers >= 2) HIPCHK(c, hipStreamWaitEvent(c->sk, c->ev_fwd_done[sb], 0));
            }
            if (!g.tied_lm_head) { zo2_status es = earlier_updates_tensor(c, c->d_lm, c->tok_elems, lm_tid(c), st); if (es != ZO2_OK) return es; }
            char* table = g.tied_lm_head ? c->d_tok : c->d_lm;
            const bool in_place = reads_in_place(c);
            if (!in_place || fused_update(c)) {
                zo2_status s = k1_tensor(c, table, c->tok_elems, g.tied_lm_head ? 0u : lm_tid(c), !in_place, c->wp, c->wm, seed, eps, st);
                if (s != ZO2_OK) return s;
            }
            if (in_place) head_wp = table;
            if (c->overlap_k1) {
                HIPCHK(c, hipEventRecord(c->ev_k1done[sb], c->sk));
                HIPCHK(c, hipStreamWaitEvent(c->sc, c->ev_k1done[sb], 0));
            }
        }
        if (loader_head || loader_logits) {
        } else if (c->fused_ce) {
            // logits are never written: the GEMM epilogue reduces each 64-column span to (max, sum exp) and picks the label's logit
            GemmArgs ga;
            memset(&ga, 0, sizeof(ga));
            ga.M = T; ga.N = g.vocab; ga.K = d; ga.ldx = d; ga.ldw = d; ga.ldy = g.vocab; ga.relu = 0; ga.out_f32 = 1; ga.nprob = ns; ga.ce_mode = 1; ga.part_ld = 2 * (int64_t)T;
            for (int s = 0; s < ns; ++s) {
                GemmProblem& p = ga.p[s];
                p.X = c->x + (size_t)s * T * d * c->csz; p.W = s ? head_wm : head_wp; p.bias = nullptr; p.residual = nullptr; p.Y = nullptr;
                p.out_scale = 1.0f; p.labels = c->d_labels;
                p.part_max = c->ce_pmax + (size_t)s * T; p.part_sum = c->ce_psum + (size_t)s * T;
                p.label_logit = c->ce_lab + (size_t)s * T;
            }
            OPK(c, ZO2_KC_GEMM, gemm_launch(ga, dt, c->sc));
            OPK(c, ZO2_KC_CE, ce_combine(c->ce_pmax, c->ce_psum, c->ce_lab, c->d_labels, ns * T, c->ce_parts, 2 * (int64_t)T, 0, T, c->row_loss, c->sc, keep_order(c)));
        } else {
            const int R = c->logit_rows;
            for (int r0 = 0; r0 < T; r0 += R) {
                const int rows = std::min(R, T - r0);
                GemmArgs ga;
                memset(&ga, 0, sizeof(ga));
                ga.M = rows; ga.N = g.vocab; ga.K = d; ga.ldx = d; ga.ldw = d; ga.ldy = g.vocab; ga.relu = 0; ga.out_f32 = 1; ga.nprob = ns;
                ga.large_only = keep_order(c);
                for (int s = 0; s < ns; ++s) {
                    GemmProblem& p = ga.p[s];
                    p.X = c->x + ((size_t)s * T + r0) * d * c->csz; p.W = s ? head_wm : head_wp; p.bias = nullptr; p.residual = nullptr;
                    p.Y = c->logits + (size_t)s * R * g.vocab; p.out_scale = 1.0f;
                }
                // (the kernel of all T rows: R is the budget's, and the budget is not to show in a loss)
                OPK(c, ZO2_KC_GEMM, gemm_launch(ga, dt, c->sc, T));
                for (int s = 0; s < ns; ++s)
                    OPK(c, ZO2_KC_CE, cross_entropy_rows(c->logits + (size_t)s * R * g.vocab, g.vocab, c->d_labels, rows, s * T + r0, T, g.vocab, c->row_loss, c->sc, keep_order(c)));
            }
        }
        // eta g of this pass: deferred update 0 of a new round (every older one has been applied on the way), or one more of
        // the current round
        if (j == 0 && !c->resident && upd && !c->pass_writes_back)      // the coefficients of the updates the blocks' host copies now lack, before slot 0 is rewritten
            HIPCHK(c, hipMemcpyAsync(stale_slot(c, c->n_stale), coef_slot(c, 0), (size_t)c->n_pend * sizeof(float), hipMemcpyDeviceToDevice, c->sc));
        OPK(c, ZO2_KC_CE, loss_epilogue(c->row_loss, c->d_labels, T, eps, lr, ns, c->d_state + 4, coef_slot(c, extra ? c->n_pend : j), c->sc));
        HIPCHK(c, hipMemcpyAsync(pass_result(c, j), c->d_state + 4, 4 * sizeof(float), hipMemcpyDeviceToHost, c->sc));
    }
    set_dir(0);
    HIPCHK(c, hipEventRecord(c->ev_c1, c->sc));
    if (c->stat_u) HIPCHK(c, hipEventRecord(c->ev_u1, c->su));
    if (c->stat_o) HIPCHK(c, hipEventRecord(c->ev_o1, c->so));
    HIPCHK(c, hipStreamSynchronize(c->sc));
    if (c->overlap_k1) HIPCHK(c, hipStreamSynchronize(c->sk));
    if (!c->resident) {
        HIPCHK(c, hipStreamSynchronize(c->su));
        HIPCHK(c, hipStreamSynchronize(c->so));
    }
    prof_collect(c);
    // statistics only: a failed query leaves the figure at zero
    c->ms_c = c->ms_u = c->ms_o = 0.f;
    (void)hipEventElapsedTime(&c->ms_c, c->ev_step0, c->ev_c1);
    if (c->stat_u) (void)hipEventElapsedTime(&c->ms_u, c->ev_u0, c->ev_u1);
    if (c->stat_o) (void)hipEventElapsedTime(&c->ms_o, c->ev_o0, c->ev_o1);

    c->apply_now = true;
    c->dir_later = false;
    if (!c->resident) {
        if (c->pass_writes_back) {
            if (changed) c->n_stale = 0;          // the host copies are current again
        } else if (upd) {
            for (int k = 0; k < c->n_pend; ++k) c->stale_seed[c->n_stale++] = c->pend_seed[k];
        }
    }
    if (ns == 1) {
        c->n_pend = 0;            // the pending updates have been applied to every module on the way
        return ZO2_OK;
    }
    if (ndirs > 1) {          // a new round of ndirs directions; a non-finite loss in any of them drops the whole round
        for (int j = 0; j < ndirs; ++j) {
            const float* r = pass_result(c, j);
            if (!(isfinite(r[0]) && isfinite(r[1]) && isfinite(r[2]))) {
                c->n_pend = 0;
                return fail(c, ZO2_ENONFINITE, "%s: non-finite loss in direction %d (l+ %g, l- %g)", who, j, (double)r[0], (double)r[1]);
            }
        }
        c->n_pend = ndirs;
        for (int j = 0; j < ndirs; ++j) c->pend_seed[j] = seeds[j];
        return ZO2_OK;
    }
    const bool finite = isfinite(c->h_result[0]) && isfinite(c->h_result[1]) && isfinite(c->h_result[2]);
    if (extra) {
        if (finite) c->pend_seed[c->n_pend++] = seed;
    } else {
        c->n_pend = finite ? 1 : 0;
        c->pend_seed[0] = seed;
    }
    // a non-finite g must never reach the parameters: this direction's update is dropped
    if (!finite) return fail(c, ZO2_ENONFINITE, "%s: non-finite loss (l+ %g, l- %g)", who, (double)c->h_result[0], (double)c->h_result[1]);
    return ZO2_OK;
}

// ---------------------------------------------------------------------------------- step
extern "C" zo2_status zo2_step(zo2_ctx* c, const int32_t* tokens, const int32_t* labels, int32_t batch, int32_t seq,
                               uint64_t seed, float eps, float lr, float* loss_plus, float* loss_minus, float* gout) {
    if (!c) return ZO2_EINVAL;
    if (c->dead) return ZO2_ESTATE;
    if (!tokens || !labels || !loss_plus || !loss_minus || !gout) return fail(c, ZO2_EINVAL, "zo2_step: NULL argument");
    if (!(eps != 0.f) || !isfinite(eps) || !isfinite(lr)) return fail(c, ZO2_EINVAL, "zo2_step: eps must be non-zero and finite, lr finite");
    const zo2_status s = model_pass(c, "zo2_step", tokens, labels, batch, seq, &seed, 1, eps, lr, 2);
    if (s == ZO2_OK || s == ZO2_ENONFINITE) {
        *loss_plus = c->h_result[0];
        *loss_minus = c->h_result[1];
        *gout = c->h_result[2];
    }
    return s;
}

// A further direction of the current round (q-direction form of the estimator): same parameters, same arithmetic,
// nothing applied; its update joins the deferred ones.
extern "C" zo2_status zo2_step_extra(zo2_ctx* c, const int32_t* tokens, const int32_t* labels, int32_t batch, int32_t seq,
                                     uint64_t seed, float eps, float lr, float* loss_plus, float* loss_minus, float* gout) {
    if (!c) return ZO2_EINVAL;
    if (c->dead) return ZO2_ESTATE;
    if (!tokens || !labels || !loss_plus || !loss_minus || !gout) return fail(c, ZO2_EINVAL, "zo2_step_extra: NULL argument");
    if (!(eps != 0.f) || !isfinite(eps) || !isfinite(lr)) return fail(c, ZO2_EINVAL, "zo2_step_extra: eps must be non-zero and finite, lr finite");
    if (c->n_pend < 1) return fail(c, ZO2_ESTATE, "zo2_step_extra: no round in progress (call zo2_step first)");
    if (c->n_pend >= zo2_ctx::kMaxPending) return fail(c, ZO2_ESTATE, "zo2_step_extra: at most %d directions per round", zo2_ctx::kMaxPending);
    const zo2_status s = model_pass(c, "zo2_step_extra", tokens, labels, batch, seq, &seed, 1, eps, lr, 2, true);
    if (s == ZO2_OK || s == ZO2_ENONFINITE) {
        *loss_plus = c->h_result[0];
        *loss_minus = c->h_result[1];
        *gout = c->h_result[2];
    }
    return s;
}

// A whole round of n_dirs directions in one pass: the results and the state it leaves equal those of zo2_step(seeds[0])
// followed by zo2_step_extra(seeds[1]) ... bit for bit, but every module is visited once - a streamed block is uploaded
// once and runs the dual forwards of all directions while it sits in its slot.
extern "C" zo2_status zo2_step_multi(zo2_ctx* c, const int32_t* tokens, const int32_t* labels, int32_t batch, int32_t seq,
                                     int32_t n_dirs, const uint64_t* seeds, float eps, float lr, float* results) {
    if (!c) return ZO2_EINVAL;
    if (c->dead) return ZO2_ESTATE;
    if (!tokens || !labels || !seeds || !results) return fail(c, ZO2_EINVAL, "zo2_step_multi: NULL argument");
    if (n_dirs < 1 || n_dirs > zo2_ctx::kMaxPending) return fail(c, ZO2_EINVAL, "zo2_step_multi: %d directions (1 .. %d)", n_dirs, zo2_ctx::kMaxPending);
    if (!(eps != 0.f) || !isfinite(eps) || !isfinite(lr)) return fail(c, ZO2_EINVAL, "zo2_step_multi: eps must be non-zero and finite, lr finite");
    const zo2_status s = model_pass(c, "zo2_step_multi", tokens, labels, batch, seq, seeds, n_dirs, eps, lr, 2);
    if (s == ZO2_OK || s == ZO2_ENONFINITE)
        for (int j = 0; j < n_dirs; ++j) {
            const float* r = pass_result(c, j);
            results[3 * j] = r[0]; results[3 * j + 1] = r[1]; results[3 * j + 2] = r[2];
        }
    return s;
}

// ---------------------------------------------------------------------------------- evaluation (single forward)
extern "C" zo2_status zo2_eval(zo2_ctx* c, const int32_t* tokens, const int32_t* labels, int32_t batch, int32_t seq, float* loss) {
    if (!c) return ZO2_EINVAL;
    if (c->dead) return ZO2_ESTATE;
    if (!tokens || !labels || !loss) return fail(c, ZO2_EINVAL, "zo2_eval: NULL argument");
    const uint64_t no_seed = 0;
    const zo2_status s = model_pass(c, "zo2_eval", tokens, labels, batch, seq, &no_seed, 1, 0.f, 0.f, 1);
    if (s == ZO2_OK) *loss = c->h_result[0];
    return s;
}

// ---------------------------------------------------------------------------------- the deferred update as data
// What Sec. 5.4 carries from one iteration to the next: (seed, c = eta * g).  Together with the parameters
// (zo2_sync_to_host) this is the whole training state, so it is what a checkpoint has to hold.
extern "C" zo2_status zo2_pending_count(zo2_ctx* c, int32_t* n) {
    if (!c) return ZO2_EINVAL;
    if (c->dead) return ZO2_ESTATE;
    if (!n) return fail(c, ZO2_EINVAL, "zo2_pending_count: NULL argument");
    *n = c->n_pend;
    return ZO2_OK;
}

extern "C" zo2_status zo2_get_pending_at(zo2_ctx* c, int32_t i, uint64_t* seed, float* step) {
    if (!c) return ZO2_EINVAL;
    if (c->dead) return ZO2_ESTATE;
    if (!seed || !step) return fail(c, ZO2_EINVAL, "zo2_get_pending_at: NULL argument");
    if (i < 0 || i >= c->n_pend) return fail(c, ZO2_EINVAL, "zo2_get_pending_at: index %d of %d", i, c->n_pend);
    HIPCHK(c, hipMemcpyAsync(c->h_result + 8, coef_slot(c, i), sizeof(float), hipMemcpyDeviceToHost, c->sc));
    HIPCHK(c, hipStreamSynchronize(c->sc));
    *seed = c->pend_seed[i];
    *step = c->h_result[8];
    return ZO2_OK;
}

extern "C" zo2_status zo2_add_pending(zo2_ctx* c, uint64_t seed, float step) {
    if (!c) return ZO2_EINVAL;
    if (c->dead) return ZO2_ESTATE;
    if (!isfinite(step)) return fail(c, ZO2_EINVAL, "zo2_add_pending: step must be finite");
    if (c->n_pend >= zo2_ctx::kMaxPending) return fail(c, ZO2_ESTATE, "zo2_add_pending: at most %d deferred updates", zo2_ctx::kMaxPending);
    c->h_result[8] = step;
    HIPCHK(c, hipMemcpyAsync(coef_slot(c, c->n_pend), c->h_result + 8, sizeof(float), hipMemcpyHostToDevice, c->sc));
    HIPCHK(c, hipStreamSynchronize(c->sc));
    c->pend_seed[c->n_pend++] = seed;
    return ZO2_OK;
}

extern "C" zo2_status zo2_get_pending(zo2_ctx* c, int32_t* has_pending, uint64_t* seed, float* step) {
    if (!c) return ZO2_EINVAL;
    if (c->dead) return ZO2_ESTATE;
    if (!has_pending || !seed || !step) return fail(c, ZO2_EINVAL, "zo2_get_pending: NULL argument");
    if (c->n_pend > 1) return fail(c, ZO2_ESTATE, "zo2_get_pending: %d updates are deferred; read them with zo2_get_pending_at", c->n_pend);
    *has_pending = c->n_pend;
    *seed = 0;
    *step = 0.f;
    return c->n_pend ? zo2_get_pending_at(c, 0, seed, step) : ZO2_OK;
}

extern "C" zo2_status zo2_set_pending(zo2_ctx* c, int32_t has_pending, uint64_t seed, float step) {
    if (!c) return ZO2_EINVAL;
    if (c->dead) return ZO2_ESTATE;
    if (has_pending && !isfinite(step)) return fail(c, ZO2_EINVAL, "zo2_set_pending: step must be finite");
    c->n_pend = 0;
    return has_pending ? zo2_add_pending(c, seed, step) : ZO2_OK;
}

// ---------------------------------------------------------------------------------- flush
extern "C" zo2_status zo2_flush(zo2_ctx* c) {
    if (!c) return ZO2_EINVAL;
    if (c->dead) return ZO2_ESTATE;
    if (c->n_pend == 0) return writeback_pass(c);
    const zo2_config& g = c->cfg;
    if (!c->planned) return fail(c, ZO2_EINVAL, "zo2_flush: nothing to flush");
    c->apply_now = true;
    const int np = c->n_pend;       // every module takes all deferred updates, in order, while it is on the device
    for (int k = 0; k < np; ++k) { zo2_status s = k1_tensor(c, c->d_tok, c->tok_elems, 0, false, nullptr, nullptr, 0, 0.f, nullptr, k); if (s != ZO2_OK) return s; }
    for (int k = 0; k < np; ++k) { zo2_status s = k1_tensor(c, c->d_pos, c->pos_elems, 1, false, nullptr, nullptr, 0, 0.f, nullptr, k); if (s != ZO2_OK) return s; }
    c->bytes_up = c->bytes_down = 0;
    c->stat_u = c->stat_o = true;   // no span statistics for a flush
    int next_upload = 0;
    if (!c->resident)
        for (; next_upload < c->n_slots && next_upload < g.n_layers; ++next_upload) {
            zo2_status s = enqueue_upload(c, next_upload);
            if (s != ZO2_OK) return s;
        }
    for (int l = 0; l < g.n_layers; ++l) {
        if (c->resident) {
            for (int k = 0; k < np; ++k) {
                zo2_status s = k1_block(c, l, c->slots + (size_t)l * c->bucket_bytes, 0, ZO2_BLOCK_TENSORS, false, 0, 0.f, nullptr, k);
                if (s != ZO2_OK) return s;
            }
        } else {
            const int sl = l % c->n_slots;
            HIPCHK(c, hipStreamWaitEvent(c->sc, c->ev_up[sl], 0));
            { zo2_status s = stale_updates_block(c, l, c->slots + (size_t)sl * c->bucket_bytes); if (s != ZO2_OK) return s; }
            for (int k = 0; k < np; ++k) {
                zo2_status s = k1_block(c, l, c->slots + (size_t)sl * c->bucket_bytes, 0, ZO2_BLOCK_TENSORS, false, 0, 0.f, nullptr, k);
                if (s != ZO2_OK) return s;
            }
            HIPCHK(c, hipEventRecord(c->ev_k1[sl], c->sc));
            zo2_status s = enqueue_offload(c, l, true);
            if (s != ZO2_OK) return s;
            if (next_upload < g.n_layers) {
                s = enqueue_upload(c, next_upload++);
                if (s != ZO2_OK) return s;
            }
        }
    }
    for (int k = 0; k < np; ++k) { zo2_status s = k1_final_ln(c, false, 0, 0.f, k); if (s != ZO2_OK) return s; }
    if (c->d_lm)
        for (int k = 0; k < np; ++k) { zo2_status s = k1_tensor(c, c->d_lm, c->tok_elems, lm_tid(c), false, nullptr, nullptr, 0, 0.f, nullptr, k); if (s != ZO2_OK) return s; }
    HIPCHK(c, hipStreamSynchronize(c->sc));
    HIPCHK(c, hipStreamSynchronize(c->su));
    HIPCHK(c, hipStreamSynchronize(c->so));
    c->n_pend = 0;
    c->n_stale = 0;
    return ZO2_OK;
}

// =========================================================================================
// kernel-level entry points
// =========================================================================================
extern "C" zo2_status zo2_op_philox_words(uint64_t seed, uint32_t tensor_id, uint64_t e0, uint64_t n, uint32_t* out, void* stream) {
    return philox_words(seed, tensor_id, e0, n, out, as_stream(stream));
}
extern "C" zo2_status zo2_op_gaussian(uint64_t seed, uint32_t tensor_id, uint64_t e0, uint64_t n, float* out, void* stream) {
    return gaussian(seed, tensor_id, e0, n, out, as_stream(stream));
}

extern "C" zo2_status zo2_op_update_perturb(void* theta, int32_t wire_dtype, void* w_plus, void* w_minus, int32_t compute_dtype,
                                            uint32_t tensor_id, uint64_t e0, uint64_t n, int32_t has_pending, uint64_t seed_prev,
                                            float cval, uint64_t seed, float eps, float scale, int32_t stochastic, void* stream) {
    if (n == 0) return ZO2_OK;
    const size_t ws = zo2_dtype_size(wire_dtype), cs = zo2_dtype_size(compute_dtype);
    ZO2_OP_CHECK(ws != 0 && cs != 0, ZO2_EINVAL, "update_perturb: unknown dtype");
    ZO2_OP_CHECK(w_plus != nullptr || w_minus == nullptr, ZO2_EINVAL, "update_perturb: W- without W+");
    ZO2_OP_CHECK(((uintptr_t)theta % (8 * ws)) == 0 && ((uintptr_t)w_plus % (8 * cs)) == 0 && ((uintptr_t)w_minus % (8 * cs)) == 0,
                 ZO2_EINVAL, "update_perturb: pointers must be aligned to 8 elements");
    K1Args a;
    memset(&a, 0, sizeof(a));
    a.theta = theta; a.w_plus = w_plus; a.w_minus = w_minus; a.w_off0 = 0; a.nseg = 1;
    a.c_imm = cval; a.c_ptr = nullptr; a.eps = eps; a.stochastic = stochastic != 0;
    a.k_prev = philox_keys(seed_prev); a.k_cur = philox_keys(seed);
    a.seg[0].off = 0; a.seg[0].e0 = e0; a.seg[0].n = n; a.seg[0].tensor_id = tensor_id; a.seg[0].scale = scale;
    return k1_launch(a, wire_dtype, compute_dtype, has_pending != 0, w_plus != nullptr, as_stream(stream));
}

// One block bucket, all 16 tensors in one grid: the launch the context issues per decoder block.
extern "C" zo2_status zo2_op_update_perturb_block(const zo2_config* cfg, int32_t layer, void* bucket, void* w_plus, void* w_minus,
                                                  int32_t has_pending, uint64_t seed_prev, float cval, uint64_t seed, float eps,
                                                  const float* host_scales, int32_t stochastic, void* stream) {
    char why[256];
    ZO2_OP_CHECK(config_ok(cfg, why, sizeof(why)), ZO2_EINVAL, "update_perturb_block: %s", why);
    ZO2_OP_CHECK(layer >= 0 && bucket != nullptr, ZO2_EINVAL, "update_perturb_block: bad layer or NULL bucket");
    ZO2_OP_CHECK(w_plus != nullptr || w_minus == nullptr, ZO2_EINVAL, "update_perturb_block: W- without W+");
    const size_t ws = zo2_dtype_size(cfg->wire_dtype), cs = zo2_dtype_size(cfg->compute_dtype);
    ZO2_OP_CHECK(((uintptr_t)bucket % (8 * ws)) == 0 && ((uintptr_t)w_plus % (8 * cs)) == 0 && ((uintptr_t)w_minus % (8 * cs)) == 0,
                 ZO2_EINVAL, "update_perturb_block: pointers must be aligned to 8 elements");
    int64_t offs[ZO2_BLOCK_TENSORS + 1], tn[ZO2_BLOCK_TENSORS];
    zo2_block_tensor_offsets(cfg, offs);
    block_tensor_elems(cfg, tn);
    K1Args a;
    memset(&a, 0, sizeof(a));
    a.theta = bucket; a.w_plus = w_plus; a.w_minus = w_minus; a.w_off0 = 0; a.nseg = ZO2_BLOCK_TENSORS;
    a.c_imm = cval; a.c_ptr = nullptr; a.eps = eps; a.stochastic = stochastic != 0;
    a.k_prev = philox_keys(seed_prev); a.k_cur = philox_keys(seed);
    for (int k = 0; k < ZO2_BLOCK_TENSORS; ++k) {
        K1Seg& sg = a.seg[k];
        sg.off = offs[k]; sg.e0 = 0; sg.n = (uint64_t)tn[k]; sg.tensor_id = block_tid(layer, k); sg.scale = host_scales ? host_scales[k] : 1.0f;
    }
    return k1_launch(a, cfg->wire_dtype, cfg->compute_dtype, has_pending != 0, w_plus != nullptr, as_stream(stream));
}

extern "C" zo2_status zo2_op_convert(const void* src, int32_t sdt, float sscale, void* dst, int32_t ddt, float dscale, uint64_t n, void* stream) {
    return convert(src, sdt, sscale, dst, ddt, dscale, n, as_stream(stream));
}

extern "C" zo2_status zo2_op_gemm(int32_t dtype, int32_t M, int32_t N, int32_t K, const void* X, int64_t ldx, const void* W, int64_t ldw,
                                  const void* bias, const float* residual, void* Y, int32_t out_dtype, int64_t ldy, float out_scale,
                                  int32_t relu, void* stream) {
    ZO2_OP_CHECK(out_dtype == ZO2_F32 || out_dtype == dtype, ZO2_EINVAL, "gemm: output dtype must be F32 or the input dtype");
    GemmArgs a;
    memset(&a, 0, sizeof(a));
    a.M = M; a.N = N; a.K = K; a.ldx = ldx; a.ldw = ldw; a.ldy = ldy; a.relu = relu; a.out_f32 = out_dtype == ZO2_F32; a.nprob = 1;
    a.p[0].X = X; a.p[0].W = W; a.p[0].bias = bias; a.p[0].residual = residual; a.p[0].Y = Y; a.p[0].out_scale = out_scale;
    return gemm_launch(a, dtype, as_stream(stream));
}

// zo2_op_gemm on the 256 x 256 kernel with one workgroup's cycle stamps (measurement build only)
extern "C" zo2_status zo2_op_gemm_phases(int32_t dtype, int32_t M, int32_t N, int32_t K, const void* X, int64_t ldx, const void* W, int64_t ldw,
                                         const float* residual, void* Y, int32_t out_dtype, int64_t ldy, uint64_t* stamps, void* stream) {
#ifdef ZO2_GEMM_STAMPS
    ZO2_OP_CHECK(stamps != nullptr, ZO2_EINVAL, "gemm_phases: stamps is NULL");
    ZO2_OP_CHECK(out_dtype == ZO2_F32 || out_dtype == dtype, ZO2_EINVAL, "gemm_phases: output dtype must be F32 or the input dtype");
    GemmArgs a;
    memset(&a, 0, sizeof(a));
    a.M = M; a.N = N; a.K = K; a.ldx = ldx; a.ldw = ldw; a.ldy = ldy; a.out_f32 = out_dtype == ZO2_F32; a.nprob = 1;
    a.p[0].X = X; a.p[0].W = W; a.p[0].residual = residual; a.p[0].Y = Y; a.p[0].out_scale = 1.0f;
    a.stamps = reinterpret_cast<unsigned long long*>(stamps);
    return gemm_launch_256(a, dtype, as_stream(stream));
#else
    (void)dtype; (void)M; (void)N; (void)K; (void)X; (void)ldx; (void)W; (void)ldw; (void)residual; (void)Y; (void)out_dtype; (void)ldy; (void)stamps; (void)stream;
    set_op_error("zo2_op_gemm_phases: this library was built without cycle stamps (build.py --gemm-stamps builds libzo2_stamps.so)");
    return ZO2_ESTATE;
#endif
}

extern "C" size_t zo2_op_gemm_split_k_workspace_bytes(int32_t M, int32_t N, int32_t splits) { return gemm_splitk_workspace_bytes(M, N, 1, splits); }

extern "C" int32_t zo2_op_gemm_split_k_pieces(int32_t dtype, int32_t M, int32_t N, int32_t K, int32_t nprob) { return gemm_pick_splits(M, N, K, nprob, dtype); }

extern "C" zo2_status zo2_op_gemm_split_k(int32_t dtype, int32_t M, int32_t N, int32_t K, const void* X, int64_t ldx, const void* W, int64_t ldw,
                                          const void* bias, const float* residual, void* Y, int32_t out_dtype, int64_t ldy, float out_scale,
                                          int32_t relu, int32_t splits, void* workspace, size_t workspace_bytes, void* stream) {
    if (M == 0 || N == 0) return ZO2_OK;
    ZO2_OP_CHECK(out_dtype == ZO2_F32 || out_dtype == dtype, ZO2_EINVAL, "gemm: output dtype must be F32 or the input dtype");
    GemmArgs a;
    memset(&a, 0, sizeof(a));
    a.M = M; a.N = N; a.K = K; a.ldx = ldx; a.ldw = ldw; a.ldy = ldy; a.relu = relu; a.out_f32 = out_dtype == ZO2_F32; a.nprob = 1;
    a.p[0].X = X; a.p[0].W = W; a.p[0].bias = bias; a.p[0].residual = residual; a.p[0].Y = Y; a.p[0].out_scale = out_scale;
    return gemm_launch_splitk(a, dtype, splits, workspace, workspace_bytes, as_stream(stream));
}

extern "C" zo2_status zo2_op_gemm_choice(int32_t dtype, int32_t M, int32_t N, int32_t K, int32_t nprob, size_t workspace_bytes, int32_t* rows, int32_t* pieces) {
    ZO2_OP_CHECK((dtype == ZO2_BF16 || dtype == ZO2_F16) && M > 0 && N > 0 && K > 0 && nprob >= 1 && nprob <= GemmArgs::kMaxProblems && rows && pieces, ZO2_EINVAL,
                 "gemm_choice: 16-bit dtypes and positive sizes");
    GemmArgs a;
    memset(&a, 0, sizeof(a));
    a.M = M; a.N = N; a.K = K; a.ldx = K; a.ldw = K; a.ldy = N; a.nprob = nprob;
    const GemmChoice k = gemm_choose(a, dtype, workspace_bytes);
    *rows = k.rows;
    *pieces = k.splits;
    return ZO2_OK;
}

extern "C" zo2_status zo2_op_gemm_group_rows(int32_t dtype, int32_t M, int32_t N, int32_t K, int32_t nprob, int32_t groups, size_t workspace_bytes, int32_t* rows) {
    ZO2_OP_CHECK((dtype == ZO2_BF16 || dtype == ZO2_F16) && M > 0 && N > 0 && K > 0 && nprob >= 1 && groups >= 1 && (int64_t)nprob * groups <= GemmArgs::kMaxProblems && rows,
                 ZO2_EINVAL, "gemm_group_rows: 16-bit dtypes and positive sizes");
    GemmArgs a;
    memset(&a, 0, sizeof(a));
    a.M = M; a.N = N; a.K = K; a.ldx = K; a.ldw = K; a.ldy = N; a.nprob = nprob;
    const GemmChoice k = gemm_choose(a, dtype, workspace_bytes);
    a.nprob = nprob * groups;
    *rows = k.rows ? gemm_groups_rows(a, dtype, k) : 0;
    return ZO2_OK;
}

extern "C" zo2_status zo2_op_gemm_tiles(int32_t dtype, int32_t M, int32_t N, int32_t K, int32_t nprob, int32_t rows[2], int32_t* problems, int32_t* columns) {
    ZO2_OP_CHECK((dtype == ZO2_F32 || dtype == ZO2_BF16 || dtype == ZO2_F16) && M > 0 && N > 0 && K > 0 && nprob >= 1 && nprob <= GemmArgs::kMaxProblems && rows && problems &&
                 columns, ZO2_EINVAL, "gemm_tiles: compute dtypes and positive sizes");
    GemmArgs a;
    memset(&a, 0, sizeof(a));
    a.M = M; a.N = N; a.K = K; a.ldx = K; a.ldw = K; a.ldy = N; a.out_f32 = 1; a.nprob = nprob;
    ZO2_OP_CHECK(dtype == ZO2_F32 || gemm256_applicable(a, dtype), ZO2_EINVAL, "gemm_tiles: not a shape of the large tiles");
    const GemmTiles t = dtype == ZO2_F32 ? GemmTiles{{gemm_f32_tile_rows(M, N, K, nprob), 0}, 0, 0} : gemm256_tiles(a);
    rows[0] = t.rows[0]; rows[1] = t.rows[1];
    *problems = t.probs; *columns = t.cols * 256;
    return ZO2_OK;
}

extern "C" zo2_status zo2_op_gemm_wide128(int32_t dtype, int32_t M, int32_t N, int32_t K, const void* X, int64_t ldx, const void* W, int64_t ldw,
                                          const void* bias, const float* residual, void* Y, int32_t out_dtype, int64_t ldy, float out_scale,
                                          int32_t relu, int32_t rows, int32_t pieces, void* workspace, size_t workspace_bytes, void* stream) {
    if (M == 0 || N == 0) return ZO2_OK;
    ZO2_OP_CHECK(out_dtype == ZO2_F32 || out_dtype == dtype, ZO2_EINVAL, "gemm: output dtype must be F32 or the input dtype");
    GemmArgs a;
    memset(&a, 0, sizeof(a));
    a.M = M; a.N = N; a.K = K; a.ldx = ldx; a.ldw = ldw; a.ldy = ldy; a.relu = relu; a.out_f32 = out_dtype == ZO2_F32; a.nprob = 1;
    a.p[0].X = X; a.p[0].W = W; a.p[0].bias = bias; a.p[0].residual = residual; a.p[0].Y = Y; a.p[0].out_scale = out_scale;
    ZO2_OP_CHECK(pieces >= 1, ZO2_EINVAL, "gemm: %d pieces", pieces);
    return gemm_launch_mid_splitk(a, dtype, rows, pieces, workspace, workspace_bytes, as_stream(stream));
}

extern "C" size_t zo2_op_gemm_perturbed_workspace_bytes(int32_t M, int32_t N, int32_t K) { return skinny_workspace_bytes(M, N, K, 1); }

extern "C" zo2_status zo2_op_gemm_perturbed(int32_t dtype, int32_t M, int32_t N, int32_t K, const void* X_plus, const void* X_minus, int64_t ldx,
                                            const void* theta, uint32_t tensor_id, uint64_t seed, float eps, const void* bias_plus,
                                            const void* bias_minus, const float* residual_plus, const float* residual_minus, void* Y_plus,
                                            void* Y_minus, int32_t out_dtype, int64_t ldy, float out_scale, int32_t relu, void* workspace,
                                            size_t workspace_bytes, void* stream) {
    if (M == 0 || N == 0) return ZO2_OK;
    ZO2_OP_CHECK(dtype == ZO2_BF16 || dtype == ZO2_F16, ZO2_EINVAL, "skinny gemm: needs 16-bit dtype");
    ZO2_OP_CHECK(out_dtype == ZO2_F32 || out_dtype == dtype, ZO2_EINVAL, "gemm_perturbed: output dtype must be F32 or the input dtype");
    SkinnyArgs a;
    memset(&a, 0, sizeof(a));
    a.M = M; a.N = N; a.K = K; a.ldx = ldx; a.ldy = ldy; a.relu = relu; a.out_f32 = out_dtype == ZO2_F32; a.nprob = 1; a.eps = eps;
    a.key = philox_keys(seed);
    SkinnyProblem& p = a.p[0];
    p.Xp = X_plus; p.Xm = X_minus; p.theta = const_cast<void*>(theta); p.bias_p = bias_plus; p.bias_m = bias_minus; p.res_p = residual_plus; p.res_m = residual_minus;
    p.Yp = Y_plus; p.Ym = Y_minus; p.out_scale = out_scale; p.tensor_id = tensor_id;
    return skinny_launch(a, dtype, workspace, workspace_bytes, as_stream(stream));
}

extern "C" zo2_status zo2_op_perturbed_rows(int32_t dtype, const void* theta, int64_t K, int64_t n0, int64_t rows, uint32_t tensor_id,
                                            uint64_t seed, float eps, void* w_plus, void* w_minus, void* stream) {
    return skinny_perturbed_rows(dtype, theta, K, n0, rows, tensor_id, seed, eps, w_plus, w_minus, as_stream(stream));
}

extern "C" zo2_status zo2_op_attention(int32_t dtype, const void* q, const void* k, const void* v, void* out, int32_t n_seq,
                                       int32_t seq, int32_t n_heads, int32_t d_head, int64_t ld, int32_t vector_kernel, void* stream) {
    return attention_launch(dtype, q, k, v, out, n_seq, seq, n_heads, d_head, ld, vector_kernel, as_stream(stream));
}

extern "C" zo2_status zo2_op_set_gemm_tile_rows(int32_t rows) {
    ZO2_OP_CHECK(rows == 0 || rows == 128 || rows == 256, ZO2_EINVAL, "zo2_op_set_gemm_tile_rows: %d (0, 128 or 256)", rows);
    gemm256_force_tile_rows(rows);
    return ZO2_OK;
}

extern "C" zo2_status zo2_op_set_gemm_wavefronts(int32_t waves) {
    ZO2_OP_CHECK(waves == 0 || waves == 4 || waves == 8, ZO2_EINVAL, "zo2_op_set_gemm_wavefronts: %d (0, 4 or 8)", waves);
    gemm256_force_waves(waves);
    return ZO2_OK;
}

extern "C" zo2_status zo2_op_layernorm(int32_t dtype, const float* x, const void* w, const void* b, const void* w2, const void* b2, void* y,
                                       int32_t rows, int32_t rows_first, int32_t d, float eps, void* stream) {
    return layernorm(dtype, x, w, b, w2, b2, y, rows, rows_first, d, eps, as_stream(stream));
}

extern "C" zo2_status zo2_op_cross_entropy_rows(const float* logits, int64_t ld, const int32_t* labels, int32_t rows, int32_t vocab,
                                                float* row_loss, void* stream) {
    return cross_entropy_rows(logits, ld, labels, rows, 0, rows > 0 ? rows : 1, vocab, row_loss, as_stream(stream));
}

extern "C" size_t zo2_op_lm_head_ce_workspace_bytes(int32_t M, int32_t N) {
    if (M <= 0 || N <= 0) return 0;
    const size_t parts = 4 * (((size_t)N + 255) / 256);
    return (2 * parts + 1) * (size_t)M * sizeof(float);
}

static zo2_status lm_head_ce_on(int32_t dtype, int32_t M, int32_t N, int32_t K, const void* X, int64_t ldx, const void* W, int64_t ldw,
                                const int32_t* labels, float* row_loss, void* workspace, hipStream_t st) {
    const int parts = 4 * ((N + 255) / 256);
    float* pmax = (float*)workspace;
    float* psum = pmax + (size_t)parts * M;
    float* lab = psum + (size_t)parts * M;
    GemmArgs ga;
    memset(&ga, 0, sizeof(ga));
    ga.M = M; ga.N = N; ga.K = K; ga.ldx = ldx; ga.ldw = ldw; ga.ldy = N; ga.out_f32 = 1; ga.nprob = 1; ga.ce_mode = 1; ga.part_ld = M;
    ga.p[0].X = X; ga.p[0].W = W; ga.p[0].out_scale = 1.0f; ga.p[0].labels = labels;
    ga.p[0].part_max = pmax; ga.p[0].part_sum = psum; ga.p[0].label_logit = lab;
    const zo2_status s = gemm_launch(ga, dtype, st);
    if (s != ZO2_OK) return s;
    return ce_combine(pmax, psum, lab, labels, M, parts, M, 0, M, row_loss, st);
}

extern "C" zo2_status zo2_op_lm_head_ce(int32_t dtype, int32_t M, int32_t N, int32_t K, const void* X, int64_t ldx, const void* W,
                                        int64_t ldw, const int32_t* labels, float* row_loss, void* workspace, size_t workspace_bytes,
                                        void* stream) {
    if (M == 0) return ZO2_OK;
    ZO2_OP_CHECK(X && W && labels && row_loss && workspace, ZO2_EINVAL, "lm_head_ce: NULL argument");
    ZO2_OP_CHECK(dtype == ZO2_BF16 || dtype == ZO2_F16, ZO2_EINVAL, "lm_head_ce: dtype must be BF16 or F16");
    ZO2_OP_CHECK(M >= 256 && N >= 256 && K > 0 && K % 128 == 0 && N % 4 == 0, ZO2_EINVAL,
                 "lm_head_ce: needs M, N >= 256, K %% 128 == 0, N %% 4 == 0 (got %d x %d x %d)", M, N, K);
    ZO2_OP_CHECK(((uintptr_t)workspace & 255) == 0 && workspace_bytes >= zo2_op_lm_head_ce_workspace_bytes(M, N) && M > 0 && N > 0,
                 ZO2_EINVAL, "lm_head_ce: workspace too small or not 256-byte aligned");
    return lm_head_ce_on(dtype, M, N, K, X, ldx, W, ldw, labels, row_loss, workspace, as_stream(stream));
}

// ---------------------------------------------------------------------------------- LM head + cross-entropy without a workspace
// For callers that cannot allocate device memory: the partials live in a fixed array inside the library's
// code object.  Every GPU the library runs on holds its own copy of the array at its own address; in host
// code the array's name is only a handle for hipGetSymbolAddress, never a device address.
static __device__ __align__(256) unsigned char scratch[ZO2_STATIC_SCRATCH_BYTES];

static constexpr int kMaxStaticDevices = 64;
static void* g_static_scratch[kMaxStaticDevices];      // per device: where `scratch` lives there (NULL: not asked yet)
static std::mutex g_static_scratch_lock;

// The address of `scratch` on the current device, looked up once per device.
static zo2_status static_scratch_address(void** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) { set_op_error("lm_head_ce_static: hipGetDevice failed: %s", hipGetErrorString(e)); return ZO2_EHIP; }
    ZO2_OP_CHECK(dev >= 0 && dev < kMaxStaticDevices, ZO2_EINVAL, "lm_head_ce_static: device index %d beyond %d", dev, kMaxStaticDevices);
    std::lock_guard<std::mutex> guard(g_static_scratch_lock);
    if (!g_static_scratch[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            set_op_error("lm_head_ce_static: hipGetSymbolAddress failed: %s", hipGetErrorString(e));
            return ZO2_EHIP;
        }
        g_static_scratch[dev] = p;
    }
    *out = g_static_scratch[dev];
    return ZO2_OK;
}

extern "C" zo2_status zo2_op_lm_head_ce_static(int32_t dtype, int32_t M, int32_t N, int32_t K, const void* X, int64_t ldx, const void* W,
                                               int64_t ldw, const int32_t* labels, float* row_loss, void* stream) {
    if (M == 0) return ZO2_OK;
    ZO2_OP_CHECK(X && W && labels && row_loss, ZO2_EINVAL, "lm_head_ce_static: NULL argument");
    ZO2_OP_CHECK(dtype == ZO2_BF16 || dtype == ZO2_F16, ZO2_EINVAL, "lm_head_ce_static: dtype must be BF16 or F16");
    ZO2_OP_CHECK(M >= 256 && N >= 256 && K > 0 && K % 128 == 0 && N % 4 == 0, ZO2_EINVAL,
                 "lm_head_ce_static: needs M, N >= 256, K %% 128 == 0, N %% 4 == 0 (got %d x %d x %d)", M, N, K);
    const size_t need = zo2_op_lm_head_ce_workspace_bytes(M, N);
    ZO2_OP_CHECK(need <= (size_t)ZO2_STATIC_SCRATCH_BYTES, ZO2_EINVAL,
                 "lm_head_ce_static: %d rows x %d columns need %zu bytes of partials, the built-in buffer holds %zu; "
                 "use zo2_op_lm_head_ce with a workspace", M, N, need, (size_t)ZO2_STATIC_SCRATCH_BYTES);
    void* ws = nullptr;
    const zo2_status s = static_scratch_address(&ws);
    if (s != ZO2_OK) return s;
    // every partial and label logit the second kernel reads is written by the first in the same call: nothing in the
    // buffer has to start at zero, and what an earlier (larger) call left behind is never read
    return lm_head_ce_on(dtype, M, N, K, X, ldx, W, ldw, labels, row_loss, ws, as_stream(stream));
}
