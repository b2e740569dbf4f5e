/*
 * frameft.h -- C ABI of the FrameFT adapter hot path on MI355X (gfx950).
 *
 * FrameFT fine-tunes a frozen weight W0 (m x n, m = d_out, n = d_in) as
 *     W' = W0 + s * P_out C P_in^T,          s = alpha / sqrt(m n)
 * (paper Sec. 3.1, update equation; Algorithm 1).  P_in (n x k rho_n) and
 * P_out (m x k rho_m) are real Parseval tight fusion frames generated by
 * Spectral Tetris, root-of-unity modulation and realification (Sec. 3.2 and
 * the appendix "Fusion Frames Construction: an example"); C is a sparse fp32
 * coefficient matrix whose support is shared across layers (Sec. 3.3).
 *
 * The library computes, for a batch of T tokens stored one per row:
 *   forward   Y  = beta * Y  + s * P_out C P_in^T x            (per token x)
 *   backward  dX = beta * dX + s * P_in C^T P_out^T g          (per token g)
 *             dC = s * (P_out^T G^T X P_in) on the support of C
 *                  (Appendix A: grad f(C) = P_m^T grad f(W) P_n)
 *   merge     W  = beta * W  + s * P_out C P_in^T            (Algorithm 1, steps 5-6)
 * W0 x itself is the caller's GEMM; the library computes the adapter branch.
 *
 * Conventions shared by every call
 *   - Frame column (coefficient) index, "canonical": i*rho + 2r + s for
 *     subspace i (0..k-1), Spectral Tetris row r (0..rho/2-1) and real part
 *     s (0: image of [Re; Im], 1: image of [-Im; Re]); i.e. P = [P_1..P_k].
 *     Real coordinate 2j / 2j+1 is the real / imaginary part of complex
 *     coordinate j.  Rows of C index P_out columns, columns of C index P_in
 *     columns.
 *   - Activations are row-major, one token per row: element (t, i) of X is
 *     at X[t*ldx + i].  W is row-major m x n (nn.Linear.weight layout).
 *   - Tensors are caller-owned device memory; `stream` is a hipStream_t
 *     (NULL = default stream).  Hot-path calls are asynchronous on `stream`,
 *     never allocate, never synchronise, and write nothing when they return
 *     an error.  Calls that share a plan must be ordered on one stream: they
 *     share the plan's workspace.
 *   - bf16 activations: 16-byte aligned base pointers and leading dimensions
 *     that are multiples of 8 elements; fp32: multiples of 4 (plans with a
 *     lift, below: element alignment and any leading dimension).  Arithmetic
 *     accumulates in fp32; bf16 results are rounded to nearest even.
 *   - Supported frames on the GPU: every tight (k, rho, d) with 2k a multiple
 *     of 8 and at most 4096 (k a power of 4 times at most 64 beyond 512 wide),
 *     and also 2k a multiple of 4 up to 128 when k rho != d.  With k rho = d
 *     the frame is block diagonal with square 2k x 2k blocks.  Any other tight
 *     frame -- redundant (k rho > d, C of size k rho_m x k rho_n) or with a
 *     non-integer d / rho -- is P = L^T Pv: Pv the block frame of dimension
 *     k rho and L a sparse lift that places each Spectral Tetris row at the
 *     positions j mod k of its block (modulation sees j only mod k).  Calls on
 *     plans with such a frame lift their inputs into fp32 staging rows of
 *     width k rho (plan workspace), run the kernels there in fp32 and lift the
 *     results back; batched calls and plan groups do not take them
 *     (FF_EUNSUPPORTED).
 */
#ifndef FRAMEFT_H
#define FRAMEFT_H

#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

typedef enum ff_status {
    FF_OK = 0,
    FF_EINVAL = 1,        /* bad argument: null pointer, size, alignment, index out of range */
    FF_ENOTFF = 2,        /* (k, rho, d) does not give a tight fusion frame */
    FF_EUNSUPPORTED = 3,  /* valid request that the GPU path does not implement */
    FF_ENOMEM = 4,        /* device or host allocation failed (ff_framegen, ff_plan_create only) */
    FF_EDEVICE = 5        /* no usable device, or a HIP call / kernel launch failed */
} ff_status;

typedef enum ff_dtype { FF_F32 = 0, FF_BF16 = 1 } ff_dtype;

typedef struct ff_frame ff_frame;  /* immutable; shareable by every layer of that width (Sec. 3.4, "Memory Overhead") */
typedef struct ff_plan ff_plan;    /* (frame_in, frame_out, support) + device index tables and workspace */

/* Name of a status code.  Never NULL. */
const char* ff_status_string(int status);
/* Detail message of the last failing call on this thread ("" if none). */
const char* ff_last_error(void);
/* ABI version, currently 1. */
int ff_abi_version(void);

/*
 * ff_tff_host -- host construction of the real (k, rho, d) tight fusion frame
 * (Sec. 3.2 construction), any tight case including redundant ones (k rho > d).
 * Writes columns col0 .. col0+ncols-1 (canonical order) of the d x (k rho)
 * matrix P in fp64, row-major d x ncols, into the host buffer `out`.
 * Errors: FF_EINVAL (odd or non-positive sizes, column range outside
 * [0, k rho), out == NULL), FF_ENOTFF (construction not tight).  Needs no GPU.
 */
ff_status ff_tff_host(int64_t d, int64_t k, int64_t rho, int64_t col0, int64_t ncols, double* out);

/*
 * ff_framegen -- generate the frame TFF(k, rho, d) (Algorithm 1, step 2) and
 * place its device form on the current HIP device.  *out receives a new frame
 * (release with ff_frame_destroy).  Errors: FF_EINVAL, FF_ENOTFF,
 * FF_EUNSUPPORTED (a block width 2k outside the supported set above),
 * FF_ENOMEM, FF_EDEVICE.  On error *out is set to NULL.
 */
ff_status ff_framegen(int64_t d, int64_t k, int64_t rho, ff_frame** out);

/*
 * ff_frame_export -- copy back the frame as the kernels use it (fp32 block,
 * read from the device) and expand columns col0 .. col0+ncols-1 of P into
 * the host buffer `out`, fp64 row-major d x ncols.  Synchronises the device.
 */
ff_status ff_frame_export(const ff_frame* f, int64_t col0, int64_t ncols, double* out);

/* Frame geometry: d, k, rho; any pointer may be NULL. */
ff_status ff_frame_info(const ff_frame* f, int64_t* d, int64_t* k, int64_t* rho);

/* Release a frame.  Plans made from it keep it alive until they are destroyed. */
void ff_frame_destroy(ff_frame* f);

/*
 * ff_plan_create -- prepare the coefficient support G of Algorithm 1 (shared
 * by every layer that uses these frames, Sec. 3.3) for repeated calls.
 *   f_in, f_out : frames of the input (n) and output (m) spaces.
 *   nnz         : number of support entries, 0 <= nnz <= (k rho_m)(k rho_n).
 *   rows, cols  : host arrays of nnz canonical indices, rows[e] in [0, k rho_m),
 *                 cols[e] in [0, k rho_n), pairwise distinct ("user order").
 * Coefficient layout.  Algorithm 1 places the coefficient vector into C through
 * G ("rearrange") without fixing the order of the vector; the plan fixes it and
 * may pad it.  Every c_vals and dC array of later calls is a plan-layout array
 * of L = ff_plan_query(FF_Q_COEF_SLOTS) >= nnz fp32 slots: slot j holds the
 * coefficient of support entry user_index[j] as reported by ff_plan_order, or
 * nothing when user_index[j] == -1 (padding).  Padding slots of c_vals must
 * hold zero (as in ELLPACK-style padded formats: the kernels multiply them in);
 * overwriting backward calls set the padding slots of dC to zero and
 * accumulating calls leave them unchanged, so gradient steps keep them zero.  Keep the trainable coefficients in
 * plan layout; convert with c_plan[j] = c_user[user_index[j]] (j not padding)
 * and dC_user[user_index[j]] = dC_plan[j].  The layout follows the kernels'
 * entry streams, so that coefficient reads need no index.
 *   max_tokens  : largest T any later call will pass.
 *   max_batch   : largest `count` of later batched calls (>= 1).
 * Allocates all device workspace here (FF_Q_WORKSPACE_BYTES), whichever activation
 * type the calls will have.  It belongs to one call at a time, and each plan
 * holds its own: plans whose bf16 calls pass a side's coefficients through memory
 * (all but those with FF_Q_FAST128 and those of frames with k rho != d) take 2
 * bytes for every coefficient of the wider side (of both with frames in several
 * radix-4 stages) and token of the longest call of max_batch adapters, up to 128
 * MiB, beside the partial sums of dC.  An MLP projection 4096 <-> 11008 with
 * 50,000 entries and 4096 tokens holds 104 MiB, a 28672 -> 8192 one with 200,000
 * and 8192 tokens 211 MiB: let layers of one shape share a plan (max_batch, or
 * calls one after the other) where their supports agree, and ask for no more
 * tokens than are used where they do not.
 * Errors: FF_EINVAL (range, duplicate entry, null pointer), FF_ENOMEM,
 * FF_EDEVICE.  On error *out is NULL.
 */
ff_status ff_plan_create(const ff_frame* f_in, const ff_frame* f_out, int64_t nnz,
                         const int32_t* rows, const int32_t* cols, int64_t max_tokens,
                         int64_t max_batch, ff_plan** out);

void ff_plan_destroy(ff_plan* p);

/*
 * ff_plan_order -- the plan's coefficient layout: user_index (host array of L =
 * ff_plan_query(FF_Q_COEF_SLOTS) int64) receives, for every slot j, the user
 * index e of the support entry stored there (rows[e], cols[e]), or -1 for a
 * padding slot.  Each e in 0..nnz-1 appears exactly once.
 */
ff_status ff_plan_order(const ff_plan* p, int64_t* user_index);

typedef enum ff_plan_query_key {
    FF_Q_TOKENS_PER_TILE_F32 = 0,   /* tokens per workgroup tile, fp32 activations */
    FF_Q_TOKENS_PER_TILE_BF16 = 1,  /* tokens per workgroup tile, bf16 activations */
    FF_Q_WORKSPACE_BYTES = 2,       /* device workspace held by the plan */
    FF_Q_NNZ = 3,
    FF_Q_FAST128 = 4,               /* 1 if bf16 calls use the fused kernels for 128-wide frame blocks */
    FF_Q_COEF_SLOTS = 5,            /* L: length of every c_vals / dC array (nnz plus padding) */
    FF_Q_SAVED_FLOATS = 6,          /* length of a c_saved array (0: the plan needs none) */
    FF_Q_BWD_TILE_TOKENS = 7,       /* tokens per workgroup tile of the fused 128-wide backward
                                       (16 or 8; 0 without that path) */
    FF_Q_RADIX_IN = 8,              /* 4 if the input frame's block is applied in factored form
                                       (radix-4 stage plus a DFT of size k/4), 1 if densely */
    FF_Q_RADIX_OUT = 9,             /* the same for the output frame */
    FF_Q_GEN_CHUNKS = 10,           /* input-side chunks of a generic-kernel tile (1: the whole
                                       input side at once; more when the support is dense) */
    FF_Q_GEN_TILE_TOKENS_F32 = 11,  /* most tokens per generic-kernel tile with those chunks, fp32 */
    FF_Q_GEN_TILE_TOKENS_BF16 = 12, /* the same, bf16 activations */
    FF_Q_GEN_TOKEN_GROUPS = 13      /* 1 if bf16 forwards on the generic kernels keep four tokens
                                       of a coefficient together in their tiles (frames whose blocks
                                       are applied directly, up to 128 wide, or in one radix-4
                                       stage); their tiles are then a multiple of four tokens */
} ff_plan_query_key;
ff_status ff_plan_query(const ff_plan* p, int key, int64_t* value);

/*
 * ff_adapter_fwd -- Y = beta * Y + scale * P_out C P_in^T x for the T token rows
 * of X (Sec. 3.1 update equation applied to an input).
 *   act      : FF_F32 or FF_BF16, dtype of X and Y.
 *   X        : device, T x n, leading dimension ldx >= n.
 *   c_vals   : device, L fp32 coefficient slots in plan layout (ff_plan_order),
 *              16-byte aligned.
 *   scale    : s = alpha / sqrt(m n), passed by the caller.
 *   beta     : 0 overwrites Y (Y is not read), otherwise Y is read and scaled.
 *   Y        : device, T x m, leading dimension ldy >= m.
 * T = 0 is a no-op.  Errors: FF_EINVAL (T > max_tokens, bad pointers,
 * dimensions or alignment), FF_EDEVICE (launch failure).
 */
ff_status ff_adapter_fwd(const ff_plan* p, int64_t T, int act, const void* X, int64_t ldx,
                         const float* c_vals, float scale, float beta, void* Y, int64_t ldy,
                         void* stream);

/*
 * ff_adapter_bwd -- backward of ff_adapter_fwd for upstream gradient G (T x m):
 *   dX = beta_dx * dX + scale * P_in C^T P_out^T g       (skipped if dX == NULL)
 *   dC = [dC +] scale * sum_t u_t[rows[e]] z_t[cols[e]],  u = P_out^T g, z = P_in^T x
 *        (Appendix A, grad f(C) = P_m^T grad f(W) P_n; skipped if dC == NULL;
 *        added to the existing dC when accumulate_dc != 0, else overwritten)
 * X may be NULL when dC == NULL.  dC is fp32, L slots in plan layout
 * (padding slots zeroed, or unchanged when accumulating), and is reduced
 * deterministically (same inputs give bitwise-equal dC).  c_vals is in plan
 * layout.
 */
ff_status ff_adapter_bwd(const ff_plan* p, int64_t T, int act, const void* X, int64_t ldx,
                         const void* G, int64_t ldg, const float* c_vals, float scale,
                         float beta_dx, void* dX, int64_t lddx, int accumulate_dc, float* dC,
                         void* stream);

/*
 * ff_adapter_bwd_noalloc -- ff_adapter_bwd for callers that cannot allocate
 * device memory or use a plan's workspace (code under HIP graph capture, tight
 * serving loops, harnesses that forbid allocation).  Arguments, results
 * (bitwise those of ff_adapter_bwd) and errors are those of ff_adapter_bwd;
 * the backward's scratch (the coefficients in its own order, the dC partial
 * sums and, where the coefficients of a side pass through memory, those of some
 * tokens at a time) lives instead in a 96 MiB array that the library's code object
 * holds on every device it runs on, until the process ends.  Nothing is allocated
 * and no memset node is issued: the scratch is cleared by a fill kernel where
 * it must start at zero.
 *   Limit: a call needing more than 32 MiB of coefficients and partial sums
 *   (a row of them per tile, at most one per compute unit on the generic
 *   kernels) returns FF_EINVAL and writes nothing (the q_proj layer, 4096 x 4096
 *   with 10,000 coefficients, needs about 13 MB at 4096 bf16 tokens); split the
 *   tokens over several calls with accumulate_dc = 1.
 *   All calls on one device share that array: calls that overlap in time on
 *   one device (different streams, threads or processes' streams without an
 *   ordering between them) race and give undefined results.
 */
ff_status ff_adapter_bwd_noalloc(const ff_plan* p, int64_t T, int act, const void* X, int64_t ldx,
                                 const void* G, int64_t ldg, const float* c_vals, float scale,
                                 float beta_dx, void* dX, int64_t lddx, int accumulate_dc, float* dC,
                                 void* stream);

/*
 * ff_adapter_fwd_save / ff_adapter_bwd_saved -- the forward and backward of a
 * training step that uses the same coefficients in both.  The forward also
 * writes c_saved: the coefficients in the backward's own slot order, which the
 * backward otherwise rebuilds from c_vals with a reordering pass of its own.
 *   c_saved : device, ff_plan_query(FF_Q_SAVED_FLOATS) fp32, 16-byte aligned,
 *             owned by the caller; one per adapter, since a plan is shared by
 *             many layers.  Its contents are opaque.
 * ff_adapter_bwd_saved takes the c_saved written by ff_adapter_fwd_save with
 * the same c_vals, which must not change in between; otherwise the arguments,
 * results and errors are those of ff_adapter_fwd / ff_adapter_bwd.  The saved
 * copy is used by bf16 calls on plans that report FF_Q_FAST128; elsewhere
 * FF_Q_SAVED_FLOATS is 0, c_saved may be NULL and the calls are the plain ones.
 */
ff_status ff_adapter_fwd_save(const ff_plan* p, int64_t T, int act, const void* X, int64_t ldx,
                              const float* c_vals, float scale, float beta, void* Y, int64_t ldy,
                              float* c_saved, void* stream);
ff_status ff_adapter_bwd_saved(const ff_plan* p, int64_t T, int act, const void* X, int64_t ldx,
                               const void* G, int64_t ldg, const float* c_vals, const float* c_saved,
                               float scale, float beta_dx, void* dX, int64_t lddx, int accumulate_dc,
                               float* dC, void* stream);

/*
 * ff_merge_delta -- W = beta * W + scale * P_out C P_in^T (Algorithm 1, steps
 * 5-6; with scale < 0 it un-merges: the adapter hot-swap of Sec. 3.4, "Storage efficiency").  W: device,
 * m x n row-major with leading dimension ldw >= n, dtype w_dtype.  beta = 0
 * writes the dense delta dW without reading W.
 */
ff_status ff_merge_delta(const ff_plan* p, const float* c_vals, float scale, int w_dtype,
                         float beta, void* W, int64_t ldw, void* stream);

/*
 * Plan groups -- adapters that share one frame pair but each have their own
 * support of C, run together: per-layer random masks (Sec. 4.6, the sparsity
 * pattern ablation compares one mask shared across layers with a mask per
 * layer) and multi-tenant serving, where one backbone carries many users'
 * adapters that are hot-swapped or applied per request (Sec. 3.4, "Storage
 * efficiency").
 *   ff_plan_group_create : plans[i] (host array of `count` distinct plans)
 *       serves adapter i.  All plans must use the same two frame objects and
 *       the same kernel path (FF_Q_FAST128 and the generic tile geometry
 *       agree whenever the supports have similar sizes; FF_Q_BWD_TILE_TOKENS
 *       may differ); otherwise FF_EUNSUPPORTED.  The plans must outlive the group,
 *       and a plan in a group must not be used by another call concurrently
 *       (group calls use the plan's own workspace).  Allocates a small device
 *       table.  Errors: FF_EINVAL, FF_EUNSUPPORTED, FF_ENOMEM, FF_EDEVICE.
 *   ff_adapter_fwd_group / ff_adapter_bwd_group : ff_adapter_fwd_batched /
 *       ff_adapter_bwd_batched with adapter i running plans[i]: c_vals[i] and
 *       dC[i] are in plans[i]'s layout.  T (<= every plan's max_tokens) sizes
 *       the launch; `tokens`, if not NULL, is a DEVICE array of `count` int32
 *       token counts (each clamped to [0, T]) so that requests of different
 *       lengths share a launch: adapter i then reads and writes only its first
 *       tokens[i] rows (dC sums over those rows; 0 rows give dC = 0).
 *   Results per adapter equal those of the single calls on its own plan: bit for
 *   bit on plans that report FF_Q_FAST128, and
 *   elsewhere up to the rounding of the activation type, since the kernels that
 *   take a bf16 call depend on its number of tokens there.
 */
typedef struct ff_plan_group ff_plan_group;
ff_status ff_plan_group_create(int64_t count, const ff_plan* const* plans, ff_plan_group** out);
void ff_plan_group_destroy(ff_plan_group* g);
ff_status ff_adapter_fwd_group(const ff_plan_group* g, int64_t T, const int32_t* tokens, int act,
                               const void* const* X, int64_t ldx, const float* const* c_vals, float scale,
                               float beta, void* const* Y, int64_t ldy, void* stream);
ff_status ff_adapter_bwd_group(const ff_plan_group* g, int64_t T, const int32_t* tokens, int act,
                               const void* const* X, int64_t ldx, const void* const* G, int64_t ldg,
                               const float* const* c_vals, float scale, float beta_dx, void* const* dX,
                               int64_t lddx, int accumulate_dc, float* const* dC, void* stream);

/*
 * ff_coef_to_plan / ff_coef_to_user -- move a coefficient vector between the
 * caller's support order (entry e at (rows[e], cols[e]) as passed to
 * ff_plan_create) and the plan layout of every c_vals / dC argument; this is
 * the "rearrange" of Algorithm 1, step 4, run on the device so that a training
 * loop can keep C and dC in its own order without host round trips.
 *   ff_coef_to_plan : c_plan[j] = c_user[user_index[j]], and 0 in padding slots
 *                     (user_index as reported by ff_plan_order).
 *                     c_user: device, nnz fp32, 4-byte aligned.
 *                     c_plan: device, ff_plan_query(FF_Q_COEF_SLOTS) fp32, 16-byte aligned.
 *   ff_coef_to_user : c_user[e] = c_plan[slot of e], or c_user[e] += that value
 *                     when accumulate != 0 (gradient accumulation in user order).
 * Both run asynchronously on `stream`, allocate nothing, and need the two
 * arrays not to overlap.  Errors: FF_EINVAL (NULL, misaligned or overlapping
 * arrays, wrong device), FF_EDEVICE (launch failure).
 */
ff_status ff_coef_to_plan(const ff_plan* p, const float* c_user, float* c_plan, void* stream);
ff_status ff_coef_to_user(const ff_plan* p, const float* c_plan, float* c_user, int accumulate, void* stream);

/*
 * Batched forms for many adapters that share frames and support but own their
 * activations and coefficient values (one layer stack).  X, Y, G, dX, c_vals
 * and dC are DEVICE arrays of `count` device pointers (1 <= count <=
 * max_batch); every other argument is shared.  Semantics per adapter are those
 * of the single calls, including the alignment of each pointer (the pointed-to
 * arrays cannot be checked from the host: misaligned pointers are undefined
 * behaviour).  dX / dC arrays may be NULL to skip that output.
 */
ff_status ff_adapter_fwd_batched(const ff_plan* p, int64_t count, int64_t T, int act,
                                 const void* const* X, int64_t ldx, const float* const* c_vals,
                                 float scale, float beta, void* const* Y, int64_t ldy,
                                 void* stream);
ff_status ff_adapter_bwd_batched(const ff_plan* p, int64_t count, int64_t T, int act,
                                 const void* const* X, int64_t ldx, const void* const* G,
                                 int64_t ldg, const float* const* c_vals, float scale,
                                 float beta_dx, void* const* dX, int64_t lddx, int accumulate_dc,
                                 float* const* dC, void* stream);

/*
 * ff_adamw_step -- one AdamW step on a coefficient vector (the optimizer the
 * paper trains C with, Appendix G): decoupled weight decay, then the
 * bias-corrected Adam step, at step number `step` (1 for the first):
 *     c <- c (1 - lr weight_decay)
 *     m <- beta1 m + (1 - beta1) g,   v <- beta2 v + (1 - beta2) g^2
 *     c <- c - lr (m / (1 - beta1^step)) / (sqrt(v / (1 - beta2^step)) + eps)
 * c, m, v (updated in place) and g are device fp32 arrays of n elements,
 * 4-byte aligned (16-byte aligned ones move in 16-byte accesses); any common
 * layout works, so plan-layout arrays (c_vals, dC) can be stepped directly:
 * their padding slots hold zeros and stay zero.  m and v start at zero.
 * Asynchronous on `stream`; allocates nothing.  Errors: FF_EINVAL (NULL or
 * misaligned array, step < 1, betas outside [0, 1), eps <= 0, negative or
 * non-finite lr / weight_decay), FF_EDEVICE.
 */
ff_status ff_adamw_step(int64_t n, float* c, const float* g, float* m, float* v, float lr, float beta1,
                        float beta2, float eps, float weight_decay, int64_t step, void* stream);
/* The same for `count` equally long vectors (one layer stack) in one launch: c, g, m,
 * v are DEVICE arrays of `count` device pointers, each 16-byte aligned. */
ff_status ff_adamw_step_batched(int64_t count, int64_t n, float* const* c, const float* const* g,
                                float* const* m, float* const* v, float lr, float beta1, float beta2,
                                float eps, float weight_decay, int64_t step, void* stream);
/* Learning rate of optimizer step `step` (0 for the first) under the linear schedule
 * with warmup of Appendix G: base_lr * step / warmup during the warmup, then falling
 * linearly to 0 at step `total`.  Host function. */
double ff_lr_linear_warmup(int64_t step, int64_t warmup, int64_t total, double base_lr);

/*
 * ff_time_next_kernel -- instrumentation for benchmarks.  Arms this thread so
 * that the next hot-path call records the hipEvent_t `ev_start` just before and
 * `ev_stop` just after its main kernel (the fused forward, the fused backward,
 * or the merge), on that call's stream; the arming is then cleared.  Where a call
 * passes a side's coefficients through memory, that is the launches from the first
 * analysis to the last synthesis, two to four for every part that the call is split
 * into.  The reordering of the coefficients and the reduction of dC lie outside.
 * Passing NULL for both disarms.  Results are unaffected.
 */
ff_status ff_time_next_kernel(void* ev_start, void* ev_stop);

#ifdef __cplusplus
}
#endif

#endif /* FRAMEFT_H */
