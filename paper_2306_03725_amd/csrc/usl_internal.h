// Internal declarations shared by the host layer and the kernel files of libusl.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "../../include/usl.h"
#include "k_lanes.h"

// Largest slice of LDS one workgroup uses to hold activation rows.  gfx950 has 160 KiB per
// compute unit; 128 KiB is one float32 row of 32768 features.
static constexpr int USL_ROW_LDS_BYTES = 128 * 1024;

struct usl_ctx {
    int64_t m;
    int32_t d, k, max_b;
    int storage;  // usl_dtype
    hipStream_t stream;
    int device;        // -1 until the first launch
    int num_cu;
    char err[512];

    // --- device scratch, allocated on first use, freed by usl_destroy ---
    double* bce_partials;     size_t bce_partials_cap;   // per-block loss sums
    uint32_t* sel_hist;       // radix-select histograms + state
    uint8_t* prune_flags;     // [m*k] 1 = slot removed by the current redistribution
    uint32_t* tie_counts;     size_t tie_counts_cap;
    int64_t* counter64;       // small device counter (validate)
    // transposed (column-major) connectivity for backward_input
    uint32_t* csc_ptr;        size_t csc_ptr_cap;     // [nwin*d+1] start of each (window, feature) list
    uint32_t* csc_cursor;     size_t csc_cursor_cap;  // [splits][nwin*d] counts, then places; [splits][nwin*chunks] sums of the counts
    uint32_t* csc_order;      size_t csc_order_cap;   // [nwin*d] features of each chunk of a window by falling list length
    uint32_t* csc_slot;       // [m*k] flat slot j*k+t, grouped by (label window, feature)
    float* csc_w;             // [m*k] W of that slot (refreshed by every backward_input)
    bool print_done;          // inside usl_train_step: the fingerprint of idx has been compared
    uint64_t* idx_print;      // fingerprints of idx when each of the three kinds of lists was built (USL_PRINT_*), and the stale word:
                              // 1 = a later call found idx changed
    const int32_t* idx_to_check;  // idx whose fingerprint the next weight gather compares (NULL right after a build)
    int csc_win_labels;       // labels per window the lists were built with
    int csc_chunk;            // features that were put into the order of their lists' lengths together
    const int32_t* csc_built_for;  // idx pointer the lists were built from (NULL = stale)
    // bank-aware order in which a label's slots are visited by the LDS gathers (performance only)
    uint8_t* slot_order;      size_t slot_order_cap;   // [m][padded k] slot read at step s
    const int32_t* slot_order_for; // idx pointer it was computed from (NULL = stale)
    // the step of a small layer (k_step_small.hip)
    float* small_sums;        size_t small_sums_cap;   // [workgroups][b][d] of the input gradient
    uint16_t* small_order;    size_t small_order_cap;  // [m*k] a workgroup's connections in the order of their columns; looked at before use
    bool part_of_batch;            // usl_predict's chunks: the sums are taken in the order of a whole batch's, however short the chunk
    bool no_order;                 // label-subset context: idx is new on every call, an order would not pay
    void* xi;                 size_t xi_cap;   // activations interleaved for the LDS gathers (k_products.hip)
    bool xi_keep;                  // inside usl_train_step: the copy that forward makes serves the weight gradient
    const void* xi_of;             // x that xi holds (only set inside usl_train_step), else NULL
    int xi_q, xi_row_bytes;        // ... its instances per group and bytes per row
    uint32_t* tgt_bits;       size_t tgt_bits_cap;   // [max_b / 32][m] bit i % 32 of word [i / 32][j]: j is a target of instance i.  All zero between calls
    bool tgt_bits_set;             // a call has set bits and not come to the kernel that takes them back
    void* xr;                 size_t xr_cap;   // activations in the layout of the backward kernel, where that is another one
    float* gT;                size_t gT_cap;   // [tiles][m][32] upstream gradient, one 128-byte piece per (tile of 32 instances, label)
    uint8_t* nz_flags;        size_t nz_flags_cap;   // [tiles][m] 1 = that 32-instance piece of gT is not all zero
    // label-subset calls: a child context sized for the subset, and the subset's rows of idx / W
    usl_ctx* sub;
    int32_t* sub_idx;         size_t sub_idx_cap;
    void* sub_W;              size_t sub_W_cap;
    float* predict_out;       size_t predict_out_cap;   // [chunk][m] scores of usl_predict, one chunk of instances at a time
    uint64_t* topk_cand;      size_t topk_cand_cap;  // [b][segments][kk] packed (score, label) keys
    uint32_t* topk_done;           // behind them: the count of a prediction's forward (k_count.h; 0 between calls)
    bool topk_done_clear;          // it has been cleared
    float* gw_part;           size_t gw_part_cap;   // [groups][m*k] partial weight gradients of a split batch
    int gw_parts_most;             // groups that it has room for (0: not known yet)
    float* gxT;               size_t gxT_cap;  // [tiles][d][32] input gradient in the same layout
    // per-instance lists of the nonzero entries of g (k_sparse_grad.hip)
    uint32_t* nz_state;       size_t nz_state_cap;   // [0] = 1: gradient is dense, lists abandoned; entries of every instance, a line each (k_sparse_grad.hip)
    uint32_t* nz_bits;        size_t nz_bits_cap;    // [max_b][m / 32] bit j % 32 of word j / 32: g of label j is not zero (forward with the squared hinge)
    int32_t* nz_lab;          size_t nz_lab_cap;     // [max_b][m/32] label of an entry
    float* nz_val;            size_t nz_val_cap;     // [max_b][m/32] its gradient
    const float* nz_lists_of; // g that has just been looked at (only set inside usl_train_step), else NULL
    bool nz_lists_tried;      // ... and whether lists were built for it (else only the dense kernels run)
    uint32_t* hint_host;      // pinned: serial of the last finished look at a gradient, above one bit: it was dense
    uint32_t* hint_dev;       // the same word as the device addresses it
    uint32_t hint_seen, probe_serial;
    int sparse_streak;        // looks in a row that found the sample sparse
    // the register-list forms (k_backward_input_lds.hip): [0] lists of 68 slots per lane from windows of up to 32768
    // labels, for usl_backward_input; [1] lists of 36 or 32 slots from shorter windows, for the kernel of usl_train_step
    // and usl_backward that computes both gradients from the same gathers
    struct usl_lf {
        void* mem;            size_t mem_cap;      // holds count .. pos
        uint32_t* count;                           // [nwin*d] list lengths
        uint32_t* where;                           // [nwin*d] where a feature's list starts among its workgroup's entries
        uint16_t* feat;                            // [wg][2][1024] feature of a lane's list
        uint32_t* caps;                            // [wg][16] slots the wavefronts visit
        uint32_t* ov_base;                         // [wg+1] start of a workgroup's overflow entries, [wg] their number; the same two for all its entries
        uint32_t* ovr;                             // [wg][2][1024] a lane's lists' share of the overflow entries held in LDS
        uint16_t* lab;                             // [wg][slots / 8][1024][8] label within the window
        uint32_t* slot;                            // flat slot j*k+t (where the weight lives): [0] [wg][slots][1024]; [1] [m*k], by place
        uint32_t* ent;                             // [m*k] entries grouped by (workgroup, feature), before the bank-aware order (k_lf_plan)
        uint32_t* ovoff;                           // [nwin*d] where a list's overflow starts in its workgroup's
        void* ov;                                  // overflow entries
        float* stage;         size_t stage_cap;    // [1] only: per part of the batch the weight gradient by place, [m*k]; behind them per part
                                                   // the sums of the overflow entries that LDS does not hold
        uint32_t* pos;                             // [1] only: [m*k] where a slot's weight gradient is in stage
        float* partial;       size_t partial_cap;  // [nwin or chains of windows][rows of a pass][d]
        int most_parts;       size_t most_rows;    // [1] only: what the largest need of any batch is (0: not known yet)
        const int32_t* built_for;                  // idx pointer the lists were built from (NULL = stale)
    } lf[2];
};

#define USL_FAIL(ctx, code, ...)                                   \
    do {                                                           \
        snprintf((ctx)->err, sizeof((ctx)->err), __VA_ARGS__);     \
        return (code);                                             \
    } while (0)

#define USL_HIP(ctx, call)                                                              \
    do {                                                                                \
        hipError_t e_ = (call);                                                         \
        if (e_ != hipSuccess)                                                           \
            USL_FAIL(ctx, USL_EHIP, "%s failed: %s", #call, hipGetErrorString(e_));     \
    } while (0)

#define USL_TRY(expr)                     \
    do {                                  \
        usl_status s_ = (expr);           \
        if (s_ != USL_OK) return s_;      \
    } while (0)

// Makes the device current on first use and reads its compute-unit count.
usl_status usl_prepare_device(usl_ctx* ctx);
// Grows *buf to at least `bytes` (old contents are dropped).
usl_status usl_reserve(usl_ctx* ctx, void** buf, size_t* cap, size_t bytes);
// The per-block loss sums of every loss kernel, for max_b instances: no later call has to grow them (growing frees and
// allocates, which waits for the stream).  usl_forward_blocks: workgroups that forward may have when it sums the loss.
usl_status usl_reserve_loss_partials(usl_ctx* ctx);
static inline size_t usl_forward_blocks(const usl_ctx* c) { return (size_t)((c->m + 255) / 256) + (size_t)c->num_cu * 32; }
usl_status usl_check_launch(usl_ctx* ctx, const char* what);

// Proposal rounds of a bank-aware order (k_matching.h), of forward's slots and of the register lists; 0 = stored order.
// None for a layer whose steps gather so little that the order cannot pay for its making, a chain of waits of 40 to 90 us
// whatever the size: at m = 1024, d = 64, k = 8, b = 16 a step on new connectivity takes 107 us instead of 160, a later one
// 33.6 instead of 33.4; at m = 1024, b = 128 there is no difference between later steps; at m = 4096, d = 256, k = 16,
// b = 32 (the line) it is 45.0 and 44.3, at m = 31k, d = 1024, k = 32, b = 128 already 109 and 102.
static inline int usl_order_rounds(const usl_ctx* c) {
    if (const char* e = getenv("USL_TUNE_ROUNDS")) return atoi(e);
    return (double)c->m * c->k * c->max_b < (double)(1 << 21) ? 0 : 3;
}

// K = padded fan-in, unit = bytes per column of the rows that will be gathered (4, 8 or 16; 2: single bfloat16)
usl_status usl_build_slot_order(usl_ctx* ctx, const int32_t* idx, int K, int unit);

// Kernel launchers (one per file).  All take validated arguments.
usl_status usl_launch_forward(usl_ctx* ctx, const void* x, const int32_t* idx, const void* W,
                              float* out, int32_t b);
// forward and loss in one: out receives the gradient of the loss by the scores.  A later kernel of the same step has to
// turn *sum into the loss and take the targets' bits back (usl_launch_adam and usl_launch_adam_staged do).  Also compares the
// fingerprint of idx if lists for it stand (ctx->print_done says so).  marks_clear (may be null): the squared hinge's nonzeros are to be
// marked for usl_sparse_lists, and this [m][k] array, 16-byte aligned, to be cleared.  usl_forward_loss_applies: else forward and loss are called one
// after the other.
struct usl_targets {
    const int64_t* off;    // nullptr: none
    const int32_t* lab;
    uint32_t* bits;        // usl_ctx::tgt_bits
    int64_t m;
    int b;
};
struct usl_loss_sum {
    const double* partials;   // the loss = scale * the sum of n partial sums; nullptr: nothing left to add up
    size_t n;
    float scale;
    float* loss;
    usl_targets targets;      // whose bits have to go
};
bool usl_forward_loss_applies(const usl_ctx* ctx, const void* x, const int32_t* idx, const void* W, int32_t b);
usl_status usl_launch_forward_loss(usl_ctx* ctx, const void* x, const int32_t* idx, const void* W, float* g, int32_t b, int loss_kind,
                                   const int64_t* tgt_off, const int32_t* tgt_lab, float scale, float* loss, usl_loss_sum* sum, float* marks_clear);
// dense = the caller knows that g holds (almost) no exact zeros: the zero-skipping tests are left out
usl_status usl_launch_backward_weight(usl_ctx* ctx, const float* g, const void* x,
                                      const int32_t* idx, float* grad_W, int32_t b, bool dense = false);
usl_status usl_launch_backward_input(usl_ctx* ctx, const float* g, const int32_t* idx,
                                     const void* W, float* grad_x, int32_t b);
// The products over the nonzero entries of g only (k_sparse_grad.hip).  usl_sparse_compact builds the lists (or
// finds g dense); *gate is a device word, 0 = the lists stand and the sparse kernels do the work, 1 = the dense
// kernels have to.  Dense kernels that are handed the gate leave at once when it reads 0.
bool usl_sparse_supported(const usl_ctx* ctx);
bool usl_sparse_expected(usl_ctx* ctx);
usl_status usl_sparse_compact(usl_ctx* ctx, const float* g, int32_t b, const uint32_t** gate);
// The same lists from the marks that forward left (ctx->nz_bits; usl_sparse_marks_ready before it): no look and no pass over g.
usl_status usl_sparse_marks_ready(usl_ctx* ctx);
static constexpr size_t USL_NZ_STATE_LINE = 32;   // words; the number of entries of instance i (below) and what else its line counts (above)
__host__ __device__ constexpr size_t usl_nz_count_at(size_t i) { return (i + 1) * USL_NZ_STATE_LINE; }
static inline size_t usl_sparse_mark_words(const usl_ctx* c) { return (size_t)((c->m + 31) / 32); }   // of an instance
usl_status usl_sparse_lists(usl_ctx* ctx, const float* g, int32_t b, const uint32_t** gate);
usl_status usl_sparse_backward_weight(usl_ctx* ctx, const void* x, const int32_t* idx, float* grad_W, int32_t b, bool cleared = false);
usl_status usl_sparse_backward_input(usl_ctx* ctx, const int32_t* idx, const void* W, float* grad_x, int32_t b);
// backward_input in pieces, for callers that produce gT / nz_flags / the nonzero count themselves, one group of
// at most usl_bwd_input_group_rows() instances at a time
int usl_bwd_input_group_rows(void);
usl_status usl_bwd_input_prepare(usl_ctx* ctx, const int32_t* idx, int32_t b);
usl_status usl_bwd_input_gather_w(usl_ctx* ctx, const void* W, const uint32_t* gate, bool begin);
usl_status usl_bwd_input_begin_group(usl_ctx* ctx);
usl_status usl_bwd_input_group(usl_ctx* ctx, float* grad_x_rows, int32_t rows, uint64_t sampled_labels,
                               const uint32_t* gate);
// The same product with the lists of each (label window, 2048 features) held in registers and the rows of g staged
// through LDS (k_backward_input_lds.hip); applies to shapes with about 32 connections per (window, feature).
bool usl_bwi_lds_applies(const usl_ctx* ctx);
usl_status usl_bwi_lds_run(usl_ctx* ctx, const float* g, const int32_t* idx, const void* W, float* grad_x, int32_t b,
                           const uint32_t* gate);
// Both backward products from one pass of gathers through register lists of half the length (k_backward_input_lds.hip):
// grad_W[m][k] and grad_x[b][d] from g[b][m] and x[b][d]; for every layer of up to 65536 features whose partial sums of 64
// instances fit the allowance.
bool usl_both_lds_applies(const usl_ctx* ctx);
// Sums of the input gradient that are still to be added up: out[i][c] = sum over the sets of partial[set][i][c], n4 groups of four values a
// set, rows of dp values (d rounded up to a multiple of 4).  vec: rows of out are 16-byte aligned and dp = d.
struct usl_window_sums {
    const float4* partial;
    int sets;
    size_t n4;
    int d, dp;
    bool vec;
    float* out;
    unsigned blocks;   // of 256 lanes, a multiple of 8; 0: nothing to do
    int at_once;       // windows whose loads of a lane go out together
};
// Where k_both_lds left the weight gradient: slot f's is the sum over p < parts of stage[p * part_stride + pos[f]].
// stale: device word, not 0 = the lists were built from other contents of idx.
struct usl_staged {
    const float* stage;
    const uint32_t* pos;
    const uint32_t* stale;
    int parts;
    size_t part_stride;
    usl_window_sums sums;   // the kernel that picks up the weight gradient adds these up beside it
};
usl_status usl_both_lds_run(usl_ctx* ctx, const float* g, const void* x, const int32_t* idx, const void* W, float* grad_x,
                            int32_t b, const uint32_t* gate, usl_staged* out);
// x in rows of *stride elements, 16-byte aligned: by itself (Q = 1), or interleaved by Q instances ([group][column][Q],
// *stride elements from group to group); x itself where it is that already, else a copy in scratch.
usl_status usl_activation_rows(usl_ctx* ctx, const void* x, int32_t b, int Q, const void** rows, size_t* stride);
// grad_W[f] = the staged gradient of slot f (behind a zero gate: nothing, the kernels over the listed nonzeros wrote grad_W)
usl_status usl_launch_unstage(usl_ctx* ctx, const usl_staged& st, const uint32_t* gate, float* grad_W);
usl_status usl_launch_adam_staged(usl_ctx* ctx, void* W, const usl_staged& st, const uint32_t* gate, float* grad_W, float* m1, float* m2,
                                  float lr, float beta1, float beta2, float eps, float inv_c1, float inv_c2, const usl_loss_sum& sum);
// In ctx->idx_print: the sums of a fingerprint for each kind of lists (they are built and kept side by side), then the stale word.
enum { USL_PRINT_COLUMNS = 0, USL_PRINT_ONE_PRODUCT = 1, USL_PRINT_BOTH_PRODUCTS = 2, USL_PRINT_STALE = 3 * 64, USL_PRINT_WORDS = USL_PRINT_STALE + 8 };
static inline uint32_t* usl_stale_word(usl_ctx* c) { return reinterpret_cast<uint32_t*>(c->idx_print + USL_PRINT_STALE); }
// Records (store = 1) the fingerprint of idx for lists of the kind `which`, or compares with the recorded one (store = 0)
// and raises the stale word on a difference.
usl_status usl_idx_fingerprint(usl_ctx* ctx, const int32_t* idx, int which, int store);
usl_status usl_idx_print_ready(usl_ctx* ctx);   // allocates ctx->idx_print, for kernels that record a fingerprint themselves
static inline uint32_t* usl_nz_cells(usl_ctx* c) { return reinterpret_cast<uint32_t*>(c->counter64) + 4; }
// Loss and gradient in place on zg[b][m], which also leaves the gradient in c->gT (tile-major) with
// its piece flags and sampled nonzero count (usl_bwd_input_prepare must have run); *sampled_labels
// receives the number of labels the count covers.
// One call per group of instances [row0, row0 + rows) (row0 a multiple of 32); the call for the last group also
// sums the loss over the whole batch of b instances.
usl_status usl_launch_loss_tiles(usl_ctx* ctx, int loss_kind, float* zg, const int64_t* tgt_off,
                                 const int32_t* tgt_lab, float scale, float* loss, int32_t b,
                                 uint64_t* sampled_labels, int32_t row0, int32_t rows);
// loss_kind: 0 = binary cross-entropy, 1 = squared hinge
usl_status usl_launch_loss(usl_ctx* ctx, int loss_kind, const float* out, const int64_t* tgt_off,
                           const int32_t* tgt_lab, float scale, float* g, float* loss, int32_t b);
// the same loss through the static scratch array (no allocation); usl_noalloc_setup runs once per device
usl_status usl_noalloc_setup(usl_ctx* ctx);
usl_status usl_launch_loss_noalloc(usl_ctx* ctx, int loss_kind, const float* out, const int64_t* tgt_off,
                                   const int32_t* tgt_lab, float scale, float* g, float* loss, int32_t b);
// The whole training step of a small layer in two launches (k_step_small.hip).
bool usl_step_small_applies(const usl_ctx* ctx);
usl_status usl_launch_step_small(usl_ctx* ctx, const void* x, const int32_t* idx, void* W, float* m1, float* m2, const int64_t* tgt_off,
                                 const int32_t* tgt_lab, int loss_kind, float scale, float lr, float beta1, float beta2, float eps, float inv_c1,
                                 float inv_c2, float* g, float* grad_W, float* grad_x, float* loss, int32_t b);
usl_status usl_launch_adam(usl_ctx* ctx, void* W, const float* grad_W, float* m1, float* m2,
                           float lr, float beta1, float beta2, float eps, float inv_c1,
                           float inv_c2, const usl_loss_sum& sum);
usl_status usl_launch_redistribute(usl_ctx* ctx, int32_t* idx, void* W, float* m1, float* m2,
                                   int64_t n, uint64_t seed, uint64_t epoch);
usl_status usl_launch_redistribute_rows(usl_ctx* ctx, int32_t* idx, void* W, float* m1, float* m2,
                                        int32_t per_row, uint64_t seed, uint64_t epoch);
usl_status usl_launch_init_indices(usl_ctx* ctx, int32_t* idx, uint64_t seed);
usl_status usl_launch_topk(usl_ctx* ctx, const float* out, int32_t b, int32_t kk, int32_t* top_lab,
                           float* top_val);
usl_status usl_launch_precision_hits(usl_ctx* ctx, const int32_t* top_lab, const int64_t* tgt_off,
                                     const int32_t* tgt_lab, int32_t b, int32_t kk, int64_t* hits);
int usl_topk_max(void);
usl_status usl_reserve_topk(usl_ctx* ctx);
usl_status usl_launch_topk_merge(usl_ctx* ctx, int nseg, int32_t b, int32_t kk, int32_t* top_lab, float* top_val);
// usl_predict of one instance: the best labels from the forward kernel's workgroups (out: scratch, not to be read afterwards).  *done = false: not such a call.
usl_status usl_launch_predict_few(usl_ctx* ctx, const void* x, const int32_t* idx, const void* W, float* out, int32_t b, int32_t kk,
                                  int32_t* top_lab, float* top_val, bool* done);
static inline int usl_forward_few_blocks(const usl_ctx* c) { return c->num_cu * 2; }   // workgroups of its forward at most
// dst_idx[q][:] = idx[rows[q]][:] and (if W) dst_W[q][:] = W[rows[q]][:], q < n; row ids are clamped into [0, m)
usl_status usl_launch_gather_rows(usl_ctx* ctx, const int32_t* idx, const void* W, const int32_t* rows,
                                  int64_t n, int32_t* dst_idx, void* dst_W);  // largest kk usl_launch_topk takes
usl_status usl_launch_validate(usl_ctx* ctx, const int32_t* idx, int64_t* n_bad_host);
usl_status usl_launch_philox(usl_ctx* ctx, const uint32_t* ctr, uint32_t key0, uint32_t key1,
                             uint32_t* out, int64_t n);

// ---- small device helpers -------------------------------------------------------------------
__device__ __forceinline__ float usl_bf16_to_f32(uint16_t v) {
    return __uint_as_float((uint32_t)v << 16);
}
__device__ __forceinline__ uint16_t usl_f32_to_bf16(float f) {  // nearest, ties to even
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)((u >> 16) | 0x0040u);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
// The losses of one score z against its target y, 0 or 1: l and the gradient by z times scale.  (In the forward kernel the
// arithmetic counts: with the division of the standard library the step took 2 to 4 % longer where rows are short.)
// 0, binary cross-entropy: l = max(z,0) - z*y + log(1 + exp(-|z|));  dl/dz = sigmoid(z) - y
// 1, squared hinge: s = 2y-1, l = max(0, 1 - s*z)^2;                 dl/dz = -2*s*max(0, 1 - s*z)  (exact zeros)
struct usl_loss_of { float g, l; };
__device__ __forceinline__ usl_loss_of usl_loss_one(int kind, float z, float y, float scale) {
    usl_loss_of o;
    if (kind == 0) {
        const float e = __expf(-fabsf(z)), p = 1.f + e;   // p in [1, 2]
        // 1 / p: the hardware's estimate and a Newton step; the bits of the correctly rounded division for each of the
        // 2^23 + 1 values of p (compared on the device)
        const float r0 = __builtin_amdgcn_rcpf(p), r = fmaf(r0, fmaf(-p, r0, 1.f), r0);
        const float sig = z >= 0.f ? r : e * r;
        o.g = scale * (sig - y);
        o.l = fmaxf(z, 0.f) - (y != 0.f ? z : 0.f) + __logf(p);
    } else {
        const float sgn = 2.f * y - 1.f;
        const float margin = fmaxf(0.f, fmaf(-sgn, z, 1.f));
        o.g = scale * (-2.f * sgn * margin);
        o.l = margin * margin;
    }
    return o;
}
// The same in parts, for kernels that are bound by this arithmetic: l = lin + ln(2) * log2, so that many scores' logarithms are scaled at once.  p lies in
// [1, 2], so the hardware's logarithm needs neither the scaling of denormal numbers nor the tests for infinities that the standard library's has around it (12 of 27
// instructions a score; steps at m = 200k, d = 8k, k = 32, b = 64, bfloat16 214.5 us, now 210.5; m = 670k, d = 16k, b = 32 556.4 and 551.0; at the larger
// sizes the gain is within what two runs of one side differ by).  g has the bits of usl_loss_one's.
struct usl_loss_parts { float g, lin, log2; };
__device__ __forceinline__ usl_loss_parts usl_loss_in_parts(int kind, float z, float y, float scale) {
    usl_loss_parts o;
    if (kind == 0) {
        const float e = __expf(-fabsf(z)), p = 1.f + e;
        const float r0 = __builtin_amdgcn_rcpf(p), r = fmaf(r0, fmaf(-p, r0, 1.f), r0);
        const bool up = z >= 0.f;
        o.g = scale * ((up ? r : e * r) - y);
        o.lin = (up ? z : 0.f) - (y != 0.f ? z : 0.f);
        o.log2 = __builtin_amdgcn_logf(p);
    } else {
        const usl_loss_of one = usl_loss_one(1, z, y, scale);
        o.g = one.g;
        o.lin = one.l;
        o.log2 = 0.f;
    }
    return o;
}
__device__ __forceinline__ float usl_to_f32(float v) { return v; }
__device__ __forceinline__ float usl_to_f32(uint16_t v) { return usl_bf16_to_f32(v); }
template <typename TS> __device__ __forceinline__ float usl_load_f32(const TS* p, size_t i);
template <> __device__ __forceinline__ float usl_load_f32<float>(const float* p, size_t i) {
    return p[i];
}
template <> __device__ __forceinline__ float usl_load_f32<uint16_t>(const uint16_t* p, size_t i) {
    return usl_bf16_to_f32(p[i]);
}
// Fingerprint of idx: mixed 16-byte groups at up to 4096 evenly spaced places, 64 consecutive ones to a sum (64 KiB read, every load in
// flight at once).  store = 1 records the sums when lists are built; store = 0 compares on a later call and raises the stale
// word when the contents are no longer those the lists were built from: a new tensor at a recycled address, a checkpoint copied
// in, ...  A single edited entry can slip through the sample; wholesale replacement cannot.
// A sum for each wavefront, so that a check can be spread: one workgroup takes 10 us for the 4096 lines of a large idx, sixteen hide
// beside the activations (usl_train_step at m = 200k, k = 32: 15.1 and 5.5 us with them).
static constexpr int USL_PRINT_SUMS = 64;
template <int N>   // sums first, first + step, ... (N of them) by one wavefront
__device__ __forceinline__ void usl_idx_fingerprint_sums(const uint32_t* __restrict__ idx, size_t n_words, uint64_t* __restrict__ print, int which,
                                                         int store, int first, int step) {
    const size_t groups = n_words / 4;
    const size_t samples = groups < 4096 ? groups : 4096;
    const size_t stride = samples ? groups / samples : 1;   // >= 1
    const int lane = threadIdx.x & 63;
    uint4 v[N];
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const size_t s = (size_t)(first + q * step) * 64 + lane;
        v[q] = s < samples ? reinterpret_cast<const uint4*>(idx)[s * stride] : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const size_t s = (size_t)(first + q * step) * 64 + lane, at = s * stride;
        uint64_t a = ((uint64_t)v[q].x << 32 | v[q].y) ^ (at * 0x9E3779B97F4A7C15ull);
        uint64_t b2 = ((uint64_t)v[q].z << 32 | v[q].w) + (at << 7);
        a ^= a >> 31; a *= 0xD6E8FEB86659FD93ull; a ^= a >> 29;
        b2 ^= b2 >> 33; b2 *= 0xC2B2AE3D27D4EB4Full; b2 ^= b2 >> 30;
        uint64_t h = s < samples ? a + (b2 << 1 | b2 >> 63) : 0;
        if (first + q * step == 0)   // the ragged tail
            for (size_t w = groups * 4 + lane; w < n_words; w += 64) h += (uint64_t)idx[w] * 0xFF51AFD7ED558CCDull;
        for (int o = 32; o > 0; o >>= 1) h += __shfl_down(h, o);
        if (lane == 0) {
            uint64_t* at_sum = print + which * USL_PRINT_SUMS + first + q * step;
            if (store) *at_sum = h;
            else if (*at_sum != h) *reinterpret_cast<uint32_t*>(print + USL_PRINT_STALE) = 1u;
        }
    }
}
__device__ __forceinline__ void usl_idx_fingerprint_block(const uint32_t* __restrict__ idx, size_t n_words,
                                                      uint64_t* __restrict__ print, int which, int store) {   // 1024 lanes
    usl_idx_fingerprint_sums<USL_PRINT_SUMS / 16>(idx, n_words, print, which, store, (int)(threadIdx.x >> 6), 16);
}
