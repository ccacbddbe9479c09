// Host side of libfle: argument validation, epilogue grammar, kernel planning and the C ABI.
// This translation unit makes no HIP call, so everything it decides is testable without a GPU.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>

#include "fle_plan.h"

namespace fle {

static thread_local char g_error[512] = "";
// The calling thread's most recent plan; its text is only formatted when fle_last_plan asks for it.
enum LastPlan { LAST_NONE, LAST_GEMM, LAST_ATTENTION, LAST_CHAIN };
static thread_local LastPlan g_last = LAST_NONE;
static thread_local Plan g_plan;
static thread_local AttnPlan g_attn_plan;
static thread_local ChainPlan g_chain_plan;
static void remember(const Plan &plan) { g_plan = plan; g_last = LAST_GEMM; }
static void remember(const AttnPlan &plan) { g_attn_plan = plan; g_last = LAST_ATTENTION; }
static void remember(const ChainPlan &plan) { g_chain_plan = plan; g_last = LAST_CHAIN; }
static thread_local int g_forced = V_AUTO;
static thread_local int g_split = 0;

fle_status fail(fle_status s, const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_error, sizeof g_error, fmt, ap);
    va_end(ap);
    return s;
}

static inline bool is_row_op(int k) { return k == FLE_LAYERNORM || k == FLE_SOFTMAX || k == FLE_LOGSUMEXP; }
static inline size_t esize(int dtype) { return dtype == FLE_F32 ? 4 : 2; }
static inline bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }
static inline size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Half-open byte ranges [a, a+na) and [b, b+nb) intersect.
static bool overlaps(const void *a, size_t na, const void *b, size_t nb) {
    if (!a || !b || na == 0 || nb == 0) return false;
    uintptr_t pa = reinterpret_cast<uintptr_t>(a), pb = reinterpret_cast<uintptr_t>(b);
    return pa < pb + nb && pb < pa + na;
}

static size_t span_bytes(int64_t rows, int64_t cols, int64_t ld, size_t es) {
    if (rows <= 0 || cols <= 0) return 0;
    return (static_cast<size_t>(rows - 1) * static_cast<size_t>(ld) + static_cast<size_t>(cols)) * es;
}

// Grouped problems with at most this many rows per group on average read nearly every W panel once: their W
// copies carry the non-temporal hint (32 groups of 4096 x 4096, 512 rows in all: 187 -> 174 us back to back,
// 249 -> 185 us from cold caches; at 128 rows per group the hint costs 3 % back to back, so the limit is 64).
static const int64_t kGroupedStreamRows = 64;

// What an automatic plan may be changed to after the first choice (see below).
enum Refine { REFINE_NONE, REFINE_TILES, REFINE_ALL };
static fle_status make_plan_core(const fle_problem *p, int forced, int forced_split, Plan *plan, const fle_groups *grp, bool stage_f32 = false, int min_split = 1, Refine refine = REFINE_NONE, bool small = false);
static void plan_copies(const fle_problem *p, Plan *plan, bool x_ours, bool refine);

// Time of a GEMM kernel on 2-byte or fp8 operands, in microseconds between one launch and the next:
//     start + rounds (steps (step + step_full u) + fixed + fixed_full u) [+ split + 8 S M N bytes of slabs at slab_bw TB/s]
// over its workgroups (u: share of the chip's slots that they fill, 1 at most; rounds: workgroups / slots, at least 1,
// between that and the next whole number as much as `smooth` says) and the K steps of one of them.  Fitted to calls on new
// operands at 1120 random shapes: 1 .. 8192 rows, 128 .. 32768 columns, K = 128 .. 16384 (2-byte) and 150 shapes of fp8 (which the
// same constants fit), relative error 6 % (128 tiles) to 15 % (dot products) in the mean square.
struct KernelTime {
    double start, step, step_full, fixed, fixed_full, smooth, slab_bw, split;
    int slots, k_step;  // k_step: bytes of a row
};
static const KernelTime kTiled256 = {2.9, 1.06, 0.49, 11.0, 20.0, 0.435, 9.8, 0.0, 256, 128};
// Tiles of 256 columns by 160, 192 and 224 rows, and what they are compared with, unsplit: fitted to the same 620 random shapes (130 ..
// 33000 rows, 256 .. 24000 columns, 2-byte operands), 6 - 9 %.
static const KernelTime kRows160 = {3.0, 0.769, 0.283, 10.0, 2.5, 0.268, 1.0, 0.0, 256, 128};
static const KernelTime kRows192 = {2.2, 0.822, 0.312, 12.9, 1.9, 0.226, 1.0, 0.0, 256, 128};
static const KernelTime kRows224 = {2.3, 0.874, 0.383, 15.2, 2.1, 0.238, 1.0, 0.0, 256, 128};
static const KernelTime kRows256 = {2.5, 0.994, 0.376, 16.7, 2.5, 0.236, 1.0, 0.0, 256, 128};
static const KernelTime kSquare128 = {5.2, 0.582, 0.323, 1.7, 5.9, 0.458, 1.0, 0.0, 512, 128};
static const KernelTime kTiled128 = {5.5, 0.58, 0.47, 3.0, 4.4, 0.51, 9.6, 0.1, 512, 128};
static const KernelTime kDeep128 = {4.9, 0.31, 0.264, 4.8, 1.6, 0.45, 10.0, 0.0, 256, 128};
// Block-scaled fp8 (200 shapes, 13 and 12 %): the scales of a step come from as many cache lines as the tile has rows, and the
// two-stage tile waits for the registers that hold them.
static const KernelTime kTiled128Mx = {3.9, 0.36, 1.12, 3.7, 1.9, 0.51, 6.9, 0.95, 512, 128};
static const KernelTime kDeep128Mx = {7.2, 0.40, 0.29, 0.2, 0.75, 0.45, 5.2, 0.8, 256, 128};
static const KernelTime kGeneral16 = {4.0, 0.65, 2.15, 0.0, 0.0, 0.9, 6.0, 0.0, 1024, 512};
static const KernelTime kGeneral32 = {4.1, 1.08, 6.0, 0.0, 0.2, 0.89, 8.0, 0.0, 1024, 512};
static const KernelTime kDot = {1.2, 0.26, 2.12, 1.9, 3.3, 1.0, 8.0, 0.0, 1024, 1024};  // and 0.9 us per row of x
static const KernelTime kThin16 = {2.0, 0.17, 0.86, 2.5, 3.9, 0.83, 6.0, 0.0, 1024, 256};
static const KernelTime kThin32 = {5.0, 0.26, 1.09, 0.0, 6.5, 0.66, 6.0, 0.0, 1024, 256};
// skinny kernel: rows of x at once x 2-byte elements of a K step (64 .. 256 rows on a step of 256: 32 in turn)
static const KernelTime kSkinny32x64 = {3.3, 0.378, 0.041, 1.36, 2.22, 0.41, 3.6, 2.3, 256, 128};
static const KernelTime kSkinny32x128 = {4.35, 0.72, 0.20, 0.45, 1.74, 0.5, 3.4, 2.0, 256, 256};
static const KernelTime kSkinny32x256 = {4.35, 1.64, 0.125, 0.0, 2.5, 0.31, 6.0, 2.1, 256, 512};
static const KernelTime kSkinny64x128 = {2.75, 0.87, 0.135, 3.34, 1.45, 0.33, 7.9, 2.0, 256, 256};
static const KernelTime kSkinny64x256 = {4.0, 1.81, 0.25, 2.0, 2.2, 0.86, 3.4, 1.6, 256, 512};
static const KernelTime kSkinny128x256 = {4.0, 2.6, 0.5, 4.5, 3.5, 0.3, 6.0, 1.0, 256, 512};
static const KernelTime kSkinny256x256 = {5.4, 4.48, 0.99, 7.9, 3.3, 0.41, 12.0, 0.0, 256, 512};

// Whether the split-K reduction takes the row reduction along (reduce_rows): one of them, rows of up to 8192 columns, and not
// more than 512 KB of slabs per row, which one workgroup reads.  us, in two passes and in one, bf16 with LayerNorm: 128 x 4096 x 4096
// in four ranges 26.4 / 22.2, 2048 x 1024 x 2048 in two 30.9 / 24.0, 512 x 8192 x 2048 in two 47.3 / 38.2, 1 x 8192 x 4096 in eight
// 24.8 / 22.7.
static bool reduces_rows(const DevEpilogue &e, int64_t M, int64_t N, int64_t split) {
    return split > 1 && e.row_kind >= 0 && e.row2_kind < 0 && M <= (int64_t(1) << 20) && N <= 8192 && split * N <= 131072;
}

static double kernel_us(const KernelTime &k, int64_t tiles, int64_t k_bytes, int64_t split, int64_t M, int64_t N) {
    const double rounds = double(tiles * split) / k.slots, u = rounds < 1.0 ? rounds : 1.0;
    const double turns = rounds <= 1.0 ? 1.0 : std::ceil(rounds) * (1.0 - k.smooth) + rounds * k.smooth;
    const int64_t steps = ((k_bytes + k.k_step - 1) / k.k_step + split - 1) / split;
    double t = k.start + turns * (double(steps) * (k.step + k.step_full * u) + k.fixed + k.fixed_full * u);
    t = std::max(t, k.start + double(N) * double(k_bytes) / 6.0e6);  // (W comes from memory once)
    if (split <= 1) return t;
    // (two launches one behind the other, whatever they do: 2 x 377 x 896 in fp8, two ranges, 10 us)
    return std::max(t + k.split + 8.0e-6 * double(split) * double(M) * double(N) / k.slab_bw, 10.0);
}

// Operands that only the general kernel can read (a K, a leading dimension or an address that is no whole number of
// 16-byte chunks) are copied into the workspace first, rows aligned and K filled up with zeros to a whole K step, where
// the copies and another kernel together cost less: the general kernel reads every operand element from global memory
// for 16 outputs or so and does about 40 TFLOP/s on such rows, the copies move every element twice at some 4.5 TB/s
// and the tiled kernel does ten to thirty times as much (bf16 2047 x 4099 x 3071: 1204 -> 93 us, 65 x 4099 x 3071:
// 77 -> 28, 33 x 32641 x 8001: 596 -> 298; fp32 513 x 4099 x 3071: 303 -> 165).  Everything that the plan brings with it counts: the
// slabs of a split K that fp32 operands need (6525 x 5819 x 169, 608 MB of them: 390 us against 298 on the general kernel; 2000 x
// 2000 x 201: 48 against 42; 2048 x 16385 x 257: 373 against 424), and values staged in fp32 where the general kernel
// stages 2 bytes.  The workspace may grow by 2 GiB at most.  x_ours: x stands for the normalised copy (and needs no other).
static void plan_copies(const fle_problem *p, Plan *plan, bool x_ours, bool refine) {
    if (plan->variant != V_GENERAL || p->M < 1 || p->K < 1) return;
    const int64_t es = int64_t(esize(p->dtype)), chunk = 16 / es, M = p->M, N = p->N, K = p->K;
    auto whole = [&](const void *a, int64_t ld) { return aligned(a, 16) && ld % chunk == 0 && ld < (int64_t(1) << 22) / es; };
    const bool ragged = K % chunk != 0;
    const bool cx = !x_ours && (ragged || !whole(p->x, p->ldx)), cw = ragged || !whole(p->w, p->ldw);
    if (!cx && !cw) return;
    fle_problem q = *p;
    q.K = ragged ? (K + 128 / es - 1) / (128 / es) * (128 / es) : K;
    // (stand-ins for the copies: aligned, overlapping nothing)
    if (cx || ragged) { q.x = reinterpret_cast<const void *>(uintptr_t(1) << 62); q.ldx = q.K; }
    if (cw) { q.w = reinterpret_cast<const void *>(uintptr_t(3) << 61); q.ldw = q.K; }
    Plan alt;
    // Nothing is further off than on the general kernel.  Its row partials are 16 columns wide, the others' up to 128 or 256,
    // and a staged 2-byte value is rounded relative to its distance from its partial's maximum or mean: these plans stage
    // in fp32 (fp16 33 x 8001 x 3001 softmax, error against float64: general 2.5e-4, staged in fp16 3.2e-4).  Its four
    // waves sum a quarter of K each: fp32 operands run with K split at least in four, or on the dot-product kernel
    // (513 x 2049 x 1025 with LayerNorm: 1.6e-7 against 1.8e-7 with three).
    if (make_plan_core(&q, V_AUTO, 0, &alt, nullptr, true, 1, refine ? REFINE_TILES : REFINE_NONE) != FLE_OK || alt.variant == V_GENERAL) return;
    if (p->dtype == FLE_F32 && alt.split_k < 4 && !(alt.variant == V_THIN && alt.bm == 8) &&
        (make_plan_core(&q, V_AUTO, 0, &alt, nullptr, true, 4) != FLE_OK || alt.variant == V_GENERAL || alt.split_k < 4)) return;
    const size_t bx = cx ? size_t(M) * size_t(q.K) * size_t(es) : 0, bw = cw ? size_t(N) * size_t(q.K) * size_t(es) : 0;
    const size_t off_x = alt.ws_total, off_w = round_up(off_x + bx, 256), total = round_up(off_w + bw, 256);
    if (total > plan->ws_total + (size_t(1) << 31)) return;
    const double copy = 3.0 + 2.0 * double(bx + bw) / 4.5e6;
    double run = alt.time_us;
    if (run <= 0.0) {  // skinny and thin kernels: W at 5 TB/s, fp32 skinny products at 58 TFLOP/s (64 x 8192 x 4128: 74 us), slabs
        run = 5.0 + double(N) * double(q.K) * double(es) / 5.0e6;
        if (alt.variant == V_SKINNY && p->dtype == FLE_F32) run = std::max(run, 2.0 * double(M) * double(N) * double(q.K) / 58.0e6);
        if (alt.split_k > 1) run += 4.0 + 8.0 * double(alt.split_k) * double(M) * double(N) / 6.0e6;
    }
    if (alt.staging == ST_WS && plan->staging == ST_OUT && p->dtype != FLE_F32) run += 4.0 * double(M) * double(N) / 4.5e6;
    // What the estimates leave out: another launch and its start on the copies' side, by kernel, and the way of a 2-byte result to
    // memory on the general kernel's.  Measured at 794 shapes near the line, us on copies / on the general kernel: bf16 1626 x
    // 412 x 205 15.3 / 9.3, fp16 7565 x 83 x 391 22.5 / 13.0, but 7579 x 1329 x 49 with LayerNorm 42 / 58; 5 x 1098 x 1081 (thin) 10.3 /
    // 7.1, 8 x 2581 x 7725 30 / 39; fp32 6 x 732 x 1061 12.1 / 7.0, 4205 x 1241 x 245 63 / 53.  Of the 236 that these terms keep on the
    // general kernel 186 are over 5 % faster there, 8 over 5 % slower (27 % at most).
    const bool f32 = p->dtype == FLE_F32;
    const double start = alt.variant == V_THIN ? 5.0 : alt.variant != V_TILED ? 0.0 : f32 ? (x_ours ? 0.0 : 3.0) : alt.split_k == 1 ? 4.0 : 0.0;
    if (copy + run + start >= plan->time_us + (f32 ? 0.0 : 4.0 * double(M) * double(N) / 4.5e6)) return;
    *plan = alt;
    plan->copy_x = cx;
    plan->copy_w = cw;
    plan->ws_xc_off = off_x;
    plan->ws_wc_off = off_w;
    plan->ws_total = total;
}

// A list that starts with FLE_LAYERNORM_PRE: the rest of the list is planned as a problem of its own, first on x as
// it is.  If that gives the dot-product kernel for a few rows, the kernel normalises in its own sweep and nothing else
// changes.  Otherwise a pass writes the normalised rows into the workspace and the rest is planned again for that
// copy (contiguous and aligned whatever x looks like).
fle_status make_plan(const fle_problem *p, int forced, int forced_split, Plan *plan, const fle_groups *grp, int allow) {
    const bool again = (allow & PLAN_REFINE) != 0, small = (allow & PLAN_SMALL) != 0;
    const Refine refine = again ? REFINE_ALL : REFINE_NONE;
    const bool copies = (allow & PLAN_COPIES) && forced == V_AUTO && forced_split == 0 && !grp;  // (a caller's own split, 1 for none among them, is kept)
    if (!p) return fail(FLE_ERR_NULL, "problem is NULL");
    bool ln_pre = false;
    if (p->n_ops > 0 && p->n_ops <= FLE_MAX_OPS && p->ops)
        for (int i = 0; i < p->n_ops; ++i)
            if (p->ops[i].kind == FLE_LAYERNORM_PRE) {
                if (i != 0) return fail(FLE_ERR_UNSUPPORTED, "op %d: the LayerNorm of x must be the first entry of the list", i);
                ln_pre = true;
            }
    if (!ln_pre) {
        const fle_status s = make_plan_core(p, forced, forced_split, plan, grp, false, 1, refine, small);
        if (s == FLE_OK && copies) plan_copies(p, plan, false, again);
        return s;
    }
    const fle_op &op = p->ops[0];
    if (grp) return fail(FLE_ERR_UNSUPPORTED, "op 0: grouped problems take no LayerNorm of x");
    if (p->dtype == FLE_F8E4M3) return fail(FLE_ERR_UNSUPPORTED, "op 0: fp8 operands take no LayerNorm of x");
    if (!(op.alpha >= 0.0f && std::isfinite(op.alpha))) return fail(FLE_ERR_OP, "op 0: layernorm eps must be finite and >= 0");
    if (p->K < 1) return fail(FLE_ERR_SHAPE, "op 0: a LayerNorm of x needs K >= 1");
    fle_problem q = *p;
    q.ops = p->ops + 1;
    q.n_ops = p->n_ops - 1;
    fle_status s = make_plan_core(&q, forced, forced_split, plan, nullptr, false, 1, again && q.M <= 4 ? REFINE_TILES : refine, small);  // (the dot-product kernel saves the pass)
    if (s != FLE_OK && !(s == FLE_ERR_UNSUPPORTED && forced != V_AUTO)) return s;  // (a forced kernel may only fit the copy)
    const size_t es = p->dtype == FLE_F32 ? 4 : 2;
    if (!aligned(op.p0, es) || !aligned(op.p1, es)) return fail(FLE_ERR_ALIGN, "op 0: gamma/beta not aligned to the element size");
    if (p->M > 0 && p->out) {
        const size_t ob = (plan->epi.row_kind == FLE_LOGSUMEXP || plan->epi.row2_kind == FLE_LOGSUMEXP) ? size_t(p->M) * es : span_bytes(p->M, p->N, p->ldo, es);
        if (overlaps(p->out, ob, op.p0, size_t(p->K) * es) || overlaps(p->out, ob, op.p1, size_t(p->K) * es)) return fail(FLE_ERR_UNSUPPORTED, "op 0: out overlaps gamma or beta");
    }
    const bool fused = s == FLE_OK && plan->variant == V_THIN && plan->bm == 8 && p->M <= 4;  // (8 fp32 rows with the extra sums need more than 256 registers)
    if (!fused) {
        q.x = reinterpret_cast<const void *>(uintptr_t(256));  // stands for the copy: aligned, rows contiguous, overlapping nothing
        q.ldx = p->K;
        s = make_plan_core(&q, forced, forced_split, plan, nullptr, false, 1, refine, small);
        if (s != FLE_OK) return s;
        if (copies) plan_copies(&q, plan, true, again);
        plan->ws_xhat_off = plan->ws_total;
        plan->ws_total = round_up(plan->ws_total + size_t(p->M) * size_t(plan->k_run) * es, 256);
    }
    plan->ln_pre = fused ? LN_PRE_FUSED : LN_PRE_PASS;
    plan->ln_gamma = op.p0;
    plan->ln_beta = op.p1;
    plan->ln_eps = op.alpha;
    return FLE_OK;
}

// stage_f32: what a row reduction stages between its two passes is held in fp32 in the workspace, whatever the dtype.
// min_split > 1 (fp32 operands): a plan with K split at least so often, or the general kernel if there is none.
// refine: REFINE_TILES keeps a dot-product, thin or skinny kernel that the first choice gave.
// small: see PLAN_SMALL.
static fle_status make_plan_core(const fle_problem *p, int forced, int forced_split, Plan *plan, const fle_groups *grp, bool stage_f32, int min_split, Refine refine, bool small) {
    if (!p) return fail(FLE_ERR_NULL, "problem is NULL");
    std::memset(plan, 0, sizeof *plan);
    if (p->dtype != FLE_F32 && p->dtype != FLE_BF16 && p->dtype != FLE_F16 && p->dtype != FLE_F8E4M3)
        return fail(FLE_ERR_OP, "dtype %d is not FLE_F32, FLE_BF16, FLE_F16 or FLE_F8E4M3", p->dtype);
    const bool f8 = p->dtype == FLE_F8E4M3;
    const int64_t M = p->M, N = p->N, K = p->K;
    const int64_t kLimit = int64_t(1) << 40;
    if (M < 0 || N < 1 || K < 0) return fail(FLE_ERR_SHAPE, "need M >= 0, N >= 1, K >= 0 (got %lld, %lld, %lld)", (long long)M, (long long)N, (long long)K);
    if (M > kLimit || N > (int64_t(1) << 30) || K > (int64_t(1) << 30)) return fail(FLE_ERR_SHAPE, "size too large");
    if (p->n_ops < 0 || p->n_ops > FLE_MAX_OPS) return fail(FLE_ERR_OP, "n_ops %d outside 0..%d", p->n_ops, FLE_MAX_OPS);
    if (p->n_ops > 0 && !p->ops) return fail(FLE_ERR_NULL, "ops is NULL with n_ops %d", p->n_ops);

    const int64_t G = grp ? grp->n_groups : 0;
    if (grp) {
        if (G < 1 || G > 65536) return fail(FLE_ERR_SHAPE, "n_groups %lld outside 1..65536", (long long)G);
        if (grp->w_group_stride < 0 || grp->b_group_stride < 0 || grp->w_group_stride > kLimit || grp->b_group_stride > kLimit) return fail(FLE_ERR_SHAPE, "group strides must be >= 0");
        if (M > 0 && !grp->row_offsets) return fail(FLE_ERR_NULL, "row_offsets is NULL");
        if (!aligned(grp->row_offsets, 8)) return fail(FLE_ERR_ALIGN, "row_offsets is not aligned to 8 bytes");
    }
    plan->groups = int32_t(G);

    DevEpilogue &e = plan->epi;
    e.row_kind = -1;
    e.row2_kind = -1;
    e.dtype = f8 ? int32_t(FLE_BF16) : p->dtype;  // fp8 problems: everything but x and W is bf16
    e.bias = p->b;
    plan->op_dtype = p->dtype;
    plan->k_run = K;
    const size_t es = esize(e.dtype);      // bytes per element of b, residual / store operands, gamma, beta, out
    const size_t xs = f8 ? 1 : es;         // bytes per element of x and W
    for (int i = 0; i < p->n_ops; ++i) {
        const fle_op &op = p->ops[i];
        if (op.kind < FLE_BIAS || op.kind > FLE_LAYERNORM_PRE) return fail(FLE_ERR_OP, "op %d: unknown kind %d", i, op.kind);
        if (op.kind == FLE_LAYERNORM_PRE) return fail(FLE_ERR_UNSUPPORTED, "op %d: the LayerNorm of x must be the first entry of the list", i);
        if (op.kind == FLE_MXSCALE) {  // not an epilogue op: says how x and W are to be read
            if (i != 0) return fail(FLE_ERR_UNSUPPORTED, "op %d: the block scales of x and W must be the first entry of the list", i);
            if (!f8) return fail(FLE_ERR_UNSUPPORTED, "op %d: block scales need FLE_F8E4M3 operands", i);
            if (grp) return fail(FLE_ERR_UNSUPPORTED, "op %d: grouped problems take no block scales", i);
            if (K % 128 != 0) return fail(FLE_ERR_UNSUPPORTED, "op %d: block scales need K to be a multiple of 128 (got %lld)", i, (long long)K);
            if ((!op.p0 || !op.p1) && M > 0 && K > 0) return fail(FLE_ERR_NULL, "op %d: a block-scale pointer is NULL", i);
            if (!aligned(op.p0, 4) || !aligned(op.p1, 4)) return fail(FLE_ERR_ALIGN, "op %d: block scales must be 4-byte aligned", i);
            plan->mx = 1;
            plan->x_scale = op.p0;
            plan->w_scale = op.p1;
            continue;
        }
        if (e.row_kind == FLE_LOGSUMEXP || e.row2_kind == FLE_LOGSUMEXP) return fail(FLE_ERR_UNSUPPORTED, "op %d follows logsumexp, which must be last", i);
        DevOp d{op.kind, op.alpha, op.p0, op.p1, op.ld};
        if (is_row_op(op.kind)) {
            if (e.row2_kind >= 0) return fail(FLE_ERR_UNSUPPORTED, "op %d: a third row reduction in one list is not supported", i);
            if (e.row_kind >= 0 && grp) return fail(FLE_ERR_UNSUPPORTED, "op %d: grouped problems take one row reduction", i);
            if (op.kind == FLE_LAYERNORM && !(op.alpha >= 0.0f && std::isfinite(op.alpha))) return fail(FLE_ERR_OP, "op %d: layernorm eps must be finite and >= 0", i);
            if (e.row_kind >= 0) { e.row2_kind = op.kind; e.row2 = d; }
            else { e.row_kind = op.kind; e.row = d; }
            continue;
        }
        if (op.kind == FLE_BIAS && !p->b && M > 0) return fail(FLE_ERR_NULL, "op %d: bias listed but b is NULL", i);
        if (op.kind == FLE_SCALE && !std::isfinite(op.alpha)) return fail(FLE_ERR_OP, "op %d: scale factor is not finite", i);
        if (op.kind == FLE_RESIDUAL || op.kind == FLE_STORE) {
            const char *what = op.kind == FLE_STORE ? "store" : "residual";
            if (!op.p0 && M > 0) return fail(FLE_ERR_NULL, "op %d: %s pointer is NULL", i, what);
            if (op.ld < N) return fail(FLE_ERR_SHAPE, "op %d: %s ld %lld < N %lld", i, what, (long long)op.ld, (long long)N);
            if (op.ld > kLimit) return fail(FLE_ERR_SHAPE, "op %d: %s ld too large", i, what);
            if (op.kind == FLE_STORE && e.row_kind >= 0) return fail(FLE_ERR_UNSUPPORTED, "op %d: a store after the row op is not supported", i);
        }
        if (e.row_kind < 0) e.pre[e.n_pre++] = d;
        else if (e.row2_kind < 0) e.post[e.n_post++] = d;
        else e.post2[e.n_post2++] = d;
    }
    const bool lse = e.row_kind == FLE_LOGSUMEXP || e.row2_kind == FLE_LOGSUMEXP;  // out is [M]
    if (p->ldx < K || p->ldw < K) return fail(FLE_ERR_SHAPE, "ldx %lld / ldw %lld smaller than K %lld", (long long)p->ldx, (long long)p->ldw, (long long)K);
    if (!lse && p->ldo < N) return fail(FLE_ERR_SHAPE, "ldo %lld < N %lld", (long long)p->ldo, (long long)N);
    if (p->ldx > kLimit || p->ldw > kLimit || p->ldo > kLimit) return fail(FLE_ERR_SHAPE, "leading dimension too large");
    if (M > 0) {
        if (!p->out) return fail(FLE_ERR_NULL, "out is NULL");
        if (K > 0 && (!p->x || !p->w)) return fail(FLE_ERR_NULL, "x or w is NULL");
        // element alignment is the only hard requirement
        if (!aligned(p->x, xs) || !aligned(p->w, xs) || !aligned(p->out, es) || !aligned(p->b, es)) return fail(FLE_ERR_ALIGN, "a pointer is not aligned to its element size");
        const size_t out_bytes = lse ? size_t(M) * es : span_bytes(M, N, p->ldo, es);
        const size_t w_bytes = span_bytes(N, K, p->ldw, xs) + (grp ? size_t(G - 1) * size_t(grp->w_group_stride) * xs : 0);
        const size_t b_bytes = size_t(N) * es + (grp ? size_t(G - 1) * size_t(grp->b_group_stride) * es : 0);
        if (overlaps(p->out, out_bytes, p->x, span_bytes(M, K, p->ldx, xs)) || overlaps(p->out, out_bytes, p->w, w_bytes) || overlaps(p->out, out_bytes, p->b, b_bytes))
            return fail(FLE_ERR_UNSUPPORTED, "out overlaps x, w or b");
        if (plan->mx && (overlaps(p->out, out_bytes, plan->x_scale, size_t(M) * size_t(K / 32)) || overlaps(p->out, out_bytes, plan->w_scale, size_t(N) * size_t(K / 32)) ||
                         overlaps(p->workspace, p->workspace_bytes, plan->x_scale, size_t(M) * size_t(K / 32)) || overlaps(p->workspace, p->workspace_bytes, plan->w_scale, size_t(N) * size_t(K / 32))))
            return fail(FLE_ERR_UNSUPPORTED, "out or the workspace overlaps the block scales");
        if (grp && (overlaps(p->out, out_bytes, grp->row_offsets, size_t(G + 1) * 8) || overlaps(p->workspace, p->workspace_bytes, grp->row_offsets, size_t(G + 1) * 8)))
            return fail(FLE_ERR_UNSUPPORTED, "out or the workspace overlaps row_offsets");
        for (int i = 0; i < p->n_ops; ++i) {
            const fle_op &op = p->ops[i];
            if (op.kind == FLE_RESIDUAL) {
                if (!aligned(op.p0, es)) return fail(FLE_ERR_ALIGN, "op %d: residual pointer not aligned to its element size", i);
                const bool same = op.p0 == p->out && op.ld == p->ldo && !lse;
                if (!same && overlaps(p->out, out_bytes, op.p0, span_bytes(M, N, op.ld, es))) return fail(FLE_ERR_UNSUPPORTED, "op %d: out overlaps the residual without being identical to it", i);
            } else if (op.kind == FLE_STORE) {
                if (!aligned(op.p0, es)) return fail(FLE_ERR_ALIGN, "op %d: store pointer not aligned to its element size", i);
                const size_t t_bytes = span_bytes(M, N, op.ld, es);
                bool clash = overlaps(op.p0, t_bytes, p->out, out_bytes) || overlaps(op.p0, t_bytes, p->x, span_bytes(M, K, p->ldx, xs)) ||
                             overlaps(op.p0, t_bytes, p->w, w_bytes) || overlaps(op.p0, t_bytes, p->b, b_bytes) ||
                             overlaps(op.p0, t_bytes, p->workspace, p->workspace_bytes) || (grp && overlaps(op.p0, t_bytes, grp->row_offsets, size_t(G + 1) * 8));
                for (int j = 0; j < p->n_ops && !clash; ++j) {
                    const fle_op &o2 = p->ops[j];
                    if (j == i) continue;
                    if (o2.kind == FLE_RESIDUAL || o2.kind == FLE_STORE) clash = overlaps(op.p0, t_bytes, o2.p0, span_bytes(M, N, o2.ld, es));
                    else if (o2.kind == FLE_LAYERNORM) clash = overlaps(op.p0, t_bytes, o2.p0, size_t(N) * es) || overlaps(op.p0, t_bytes, o2.p1, size_t(N) * es);
                }
                if (clash) return fail(FLE_ERR_UNSUPPORTED, "op %d: the store target overlaps another operand, out or the workspace", i);
            } else if (op.kind == FLE_LAYERNORM) {
                if (!aligned(op.p0, es) || !aligned(op.p1, es)) return fail(FLE_ERR_ALIGN, "op %d: gamma/beta not aligned to the element size", i);
                if (overlaps(p->out, out_bytes, op.p0, size_t(N) * es) || overlaps(p->out, out_bytes, op.p1, size_t(N) * es)) return fail(FLE_ERR_UNSUPPORTED, "op %d: out overlaps gamma or beta", i);
            }
        }
        if (p->workspace && overlaps(p->out, out_bytes, p->workspace, p->workspace_bytes)) return fail(FLE_ERR_UNSUPPORTED, "out overlaps the workspace");
    }

    // ---- kernel variant
    const int asked = forced;
    const bool f32 = p->dtype == FLE_F32;
    // The tiled kernels copy 16-byte chunks and read / write groups of 4 consecutive columns.
    const int64_t chunk = 16 / int64_t(xs);                  // x / W elements per 16-byte chunk: 16 fp8, 8 bf16, 4 fp32
    const size_t vec4 = 4 * es;                              // alignment of a 4-column group
    const int64_t ld_max = (int64_t(1) << 22) / int64_t(es); // 32-bit byte offsets inside a 256-row tile (epilogue operands)
    const int64_t ldx_max = (int64_t(1) << 22) / int64_t(xs);  // (x and W)
    bool res_ok = true, post_res_alias_out = false;
    for (int i = 0; i < e.n_pre; ++i) {
        if ((e.pre[i].kind == FLE_RESIDUAL || e.pre[i].kind == FLE_STORE) && !(aligned(e.pre[i].p0, vec4) && e.pre[i].ld % 4 == 0 && e.pre[i].ld < ld_max)) res_ok = false;
    }
    for (int i = 0; i < e.n_post; ++i)
        if (e.post[i].kind == FLE_RESIDUAL && e.post[i].p0 == p->out) post_res_alias_out = true;
    for (int i = 0; i < e.n_post2; ++i)
        if (e.post2[i].kind == FLE_RESIDUAL && e.post2[i].p0 == p->out) post_res_alias_out = true;
    // x and W rows must be whole, aligned 16-byte chunks; everything the epilogue touches may be ragged
    // (the kernel then has an element-wise epilogue)
    const bool tiled_ok = K >= chunk && K % chunk == 0 && aligned(p->x, 16) && aligned(p->w, 16) && p->ldx % chunk == 0 && p->ldw % chunk == 0 &&
                          p->ldx < ldx_max && p->ldw < ldx_max && (!grp || grp->w_group_stride % chunk == 0);
    const bool vec_epi = N % 4 == 0 && (lse || (aligned(p->out, vec4) && p->ldo % 4 == 0)) && aligned(p->b, vec4) && res_ok && (!grp || grp->b_group_stride % 4 == 0);
    if (grp) {
        // Grouped problems run on the tiled kernels only, one workgroup per tile over the whole K.  A group's
        // tile rows start at its first row, so with rows spread over G groups about G / 2 tile rows are
        // partly empty: the 256 tile only pays when groups hold several hundred rows.
        if (forced != V_AUTO && forced != V_TILED && forced != V_TILED_256 && forced != V_TILED_128) return fail(FLE_ERR_UNSUPPORTED, "grouped problems run on the tiled kernels only");
        if (forced_split > 1) return fail(FLE_ERR_UNSUPPORTED, "grouped problems are not split along K");
        if (!tiled_ok) return fail(FLE_ERR_UNSUPPORTED, "a grouped problem needs x and W rows made of whole, 16-byte aligned chunks (K, the leading dimensions and the W group stride multiples of 16 bytes)");
        if (forced == V_AUTO || forced == V_TILED) {
            auto cost = [&](int tile) -> double {
                const double wgs = (double(M) / tile + 0.5 * double(G)) * double((N + tile - 1) / tile);
                const double slots = tile == 128 ? 512.0 : 256.0;
                const double per_step = p->dtype == FLE_F32 ? (tile == 256 ? 7.8 : 3.9) : (tile == 256 ? 1.45 : 0.85);
                return (wgs > slots ? wgs / slots : 1.0) * per_step;
            };
            bool big = cost(256) < cost(128);
            // 2-byte operands: the other tile where the fitted times put it ahead (the 256 tile by 5 %, the 128 tile by 10 %), over the tile rows of groups whose sizes scatter about
            // their mean m as a router's do (exponentially: 1 / (1 - e^(-tile / m)) of them a group).  Over 60 random calls on these two
            // tiles 0.7 % behind the better one of each and none slower than before, by steps alone 4.5 %: 5774 rows, 8 groups, 2496 x 1920 111 us on 256, 81 on 128;
            // 8053, 32, 2560 x 3840 239 and 284; over 102 calls of all sizes 1.024 times as fast.  (Not in front of a row reduction: its partials are as wide as the tile's wave, and a
            // value staged in 2 bytes is rounded relative to them.)
            if (!f8 && p->dtype != FLE_F32 && e.row_kind < 0 && M > 0) {
                auto fitted = [&](KernelTime k, int tile) {
                    k.smooth = 0.4;
                    return kernel_us(k, std::llround(double(G) / (1.0 - std::exp(-double(tile) * double(G) / double(M)))) * ((N + tile - 1) / tile), K * int64_t(xs), 1, M, N);
                };
                const double t256 = fitted(kRows256, 256), t128 = fitted(kSquare128, 128);
                if (big ? t128 < 0.9 * t256 : t256 < 0.95 * t128) big = !big;
            }
            forced = M > 128 && N > 128 && big ? V_TILED_256 : V_TILED_128;
        }
        forced_split = 1;
    }
    if (f8) {  // fp8 operands exist on the tiled kernels only
        if (forced != V_AUTO && forced != V_TILED && forced != V_TILED_256 && forced != V_TILED_128 && forced != V_DEEP_128) return fail(FLE_ERR_UNSUPPORTED, "fp8 problems run on the tiled kernels only");
        if (!tiled_ok) return fail(FLE_ERR_UNSUPPORTED, "an fp8 problem needs x and W rows made of whole, 16-byte aligned chunks (K and the leading dimensions multiples of 16 elements, K >= 16)");
        if (forced == V_AUTO) forced = V_TILED;
    }
    // (grouped: the deep tile where rows spread over the groups leave one workgroup per CU)
    bool grouped_deep = false;
    if (grp && asked == V_AUTO && forced == V_TILED_128 && !f32 && M > G * kGroupedStreamRows) {
        const int64_t tiles = (M / 128 + (G + 1) / 2) * ((N + 127) / 128), kb = K * int64_t(xs);
        grouped_deep = tiles <= 512 && kernel_us(kDeep128, tiles, kb, 1, M, N) < 0.97 * kernel_us(kTiled128, tiles, kb, 1, M, N);
    }
    const bool automatic = asked == V_AUTO && forced_split == 0 && !grp && min_split <= 1 && !f32 && M > 0 && refine != REFINE_NONE;
    int variant = forced, forced_tile = 0, deep = grouped_deep ? 1 : 0;
    if (variant == V_TILED_256 || variant == V_TILED_128) {
        forced_tile = variant == V_TILED_256 ? 256 : 128;
        variant = V_TILED;
    }
    if (variant == V_DEEP_128) {
        if (f32) return fail(FLE_ERR_UNSUPPORTED, "the deep form of the 128 tile takes no fp32 operands");
        deep = 1;
        forced_tile = 128;
        variant = V_TILED;
    }
    int rows = 0;  // rows of a tile of 256 columns, where they are not 256
    if (variant == V_ROWS_160 || variant == V_ROWS_192 || variant == V_ROWS_224) {
        if (f32 || f8) return fail(FLE_ERR_UNSUPPORTED, "tiles of 160, 192 or 224 rows take 2-byte operands");
        rows = variant == V_ROWS_160 ? 160 : variant == V_ROWS_192 ? 192 : 224;
        forced_tile = 256;
        variant = V_TILED;
    }
    int forced_bk = 0;
    bool forced_seq = false;
    if (variant == V_SKINNY_128 || variant == V_SKINNY_256 || variant == V_SKINNY_SEQ) {
        forced_bk = variant == V_SKINNY_128 ? 128 : 256;
        forced_seq = variant == V_SKINNY_SEQ;
        variant = V_SKINNY;
    }
    const bool skinny_ok = !f8 && tiled_ok && vec_epi && M <= 256 && K % (f32 ? 32 : 64) == 0;  // a K step is at least 128 bytes of every row
    const bool thin_ok = !f8 && tiled_ok && M >= 1 && M <= 32;  // element-wise epilogue: nothing else needs alignment

    // Tile and split of K of the tiled kernel together, by a coarse time model (microseconds) fitted
    // to measured runs.  bf16: a K step (128 bytes of every row) costs a 256 tile 1.45, a 128 tile 0.85
    // with two workgroups per CU and 0.6 alone.  fp32: the matrix pipe bounds a K step at 7.8 / 3.9 /
    // 1.95.  Filling the pipeline and the epilogue cost about 15 us (256 tile) or 6 us;
    // workgroups beyond the 256 (512) that are resident at once wait for a second round; a split adds
    // a launch and 8 S M N bytes of slab traffic at about 6 TB/s (the slabs mostly stay in the
    // last-level cache).
    const int64_t tiled_steps = (K * int64_t(xs) + 127) / 128;
    auto tiled_cost = [&](int tile, int64_t sp) -> double {
        const int64_t tiles = ((M + tile - 1) / tile) * ((N + tile - 1) / tile), wgs = tiles * sp;
        const int64_t slots = tile == 128 ? 512 : 256, rounds = (wgs + slots - 1) / slots;
        // (a 256 tile whose K is split over no more workgroups than there are CUs measured 1.3 per step: 768 .. 2048 x
        // 4096 x 16384 with K split in 2 or 4 came out 10 - 26 % ahead of the 128 tile where 1.45 said the opposite)
        const double per_step = f32 ? (tile == 256 ? 7.8 : wgs > 256 ? 3.9 : 1.95) : (tile == 256 ? (sp > 1 && wgs <= 256 ? 1.3 : 1.45) : wgs > 256 ? 0.85 : 0.6);
        // in K steps; two co-resident 128 tiles hide part of each other's epilogue
        const double fixed = f32 ? (tile == 256 ? 1.5 : 3.5) : (tile == 256 ? 10.5 : wgs > 256 ? 7.0 : 8.0);
        double t = double(rounds) * (double((tiled_steps + sp - 1) / sp) + fixed) * per_step;
        if (sp > 1) t += 4.0 + 8.0 * double(sp) * double(M) * double(N) / 6.0e6;
        return t;
    };
    int best_tile = 0, best_split = 1;
    double best = 0.0;
    static const int kSplits[] = {1, 2, 3, 4, 6, 8, 12, 16};
    // fp32 operands with K split at least in four: the 128 tile (the 256 tile at best level: 6525 x 5819 x 192 in four 372
    // us against 360, 2047 x 4099 x 3072 439 against 568, 8191 x 2049 x 544 243 against 273).  Over several rounds the
    // workgroups of two rounds overlap and a step of all 512 costs 3.57; 4096 x 4097 x 160: 153 us, estimated 168;
    // 4096 x 4097 x 1056 359, 383; 513 x 4099 x 3072 194, in six 144, 193 and 141; 2048 x 16385 x 288 368, 363.
    auto split_cost = [&](int64_t sp) -> double {
        const double wgs = double((M + 127) / 128) * double((N + 127) / 128) * double(sp), rounds = wgs / 512.0, steps = double((tiled_steps + sp - 1) / sp);
        const double t = wgs <= 256.0 ? (steps + 3.5) * 1.95 : (rounds <= 1.0 ? 1.0 : rounds <= 2.0 ? 2.0 : rounds) * steps * 3.57;
        return t + 7.0 + 4.0 + 8.0 * double(sp) * double(M) * double(N) / 6.0e6;
    };
    if (min_split > 1) {
        for (int sp : kSplits) {
            if (!tiled_ok || M < 1 || sp < min_split || sp > tiled_steps) continue;
            if (sp > min_split && (sp * 4 > tiled_steps || int64_t(sp) * M * (N + 3) * 4 > (int64_t(128) << 20))) continue;
            const double t = split_cost(sp);
            if (!best_tile || t < best) { best = t; best_tile = 128; best_split = sp; }
        }
    } else if (tiled_ok && M > 0) {
        for (int tile = 128; tile <= 256; tile += 128) {
            if (forced_tile ? tile != forced_tile : (tile == 256 && !(M > 128 && N > 128))) continue;
            for (int sp : kSplits) {
                if (forced_split > 0 ? sp != 1 : (sp > 1 && (sp * 4 > tiled_steps || int64_t(sp) * M * (N + 3) * 4 > (int64_t(128) << 20)))) continue;
                const double t = tiled_cost(tile, sp);
                if (!best_tile || t < best) { best = t; best_tile = tile; best_split = sp; }
            }
        }
    }
    const bool split_found = min_split > 1 && best_tile;
    if (!best_tile) best_tile = forced_tile ? forced_tile : 128;
    if (variant == V_AUTO) {
        // W is worth streaming: always for a small M; up to 128 rows when W (256 MB or more) cannot stay in the
        // Infinity Cache anyway (measured: 128 x 32768 x 8192 124 us against 156 us tiled; at 134 MB the tiled
        // kernel wins warm and cold; 8 sub-blocks are slower than the tiled kernel everywhere)
        // A few rows against a whole weight matrix (a perceptron layer at batch 1 .. 32): the thin kernels, where
        // they measured faster than what follows.  Dot-product form: fp32 up to 8 rows from 512 x 1024 weights on
        // (4096^2 at one row: 16 us against 33 us general; 1024 x 32768: 46 against 110); 2-byte dtypes up to 4
        // rows while the skinny kernel would need a split of K and a second launch (4096^2: 8.5-9.6 us against
        // 12.5), i.e. up to 2^24 weights (any size for a single row: 32768 x 8192 85 us against 91), with rows of
        // 2048 or more beyond 2^22.  MFMA form: 2-byte dtypes, 5 .. 32 rows,
        // 2^20 .. 2^23 weights (2048^2 at 16 rows: 7.9 us against 10.4).
        const int64_t nk = N * K;
        const bool gemv_auto = thin_ok && M <= (f32 ? 8 : 4) && nk >= (int64_t(1) << 19) &&
                               (f32 || ((M == 1 || nk <= (int64_t(1) << 24)) && (nk <= (int64_t(1) << 22) || K >= 2048)));
        const bool thin_auto = thin_ok && !f32 && M > 4 && nk >= (int64_t(1) << 20) && nk <= (int64_t(1) << 23);
        if ((gemv_auto || thin_auto) && forced_split <= 1 && min_split <= 1) variant = V_THIN;
        // (fp32 operands keep the matrix pipe about as busy as the memory system: worth it from 2^24 weights on,
        // 2^25 up to 16 rows where the general kernel's 16 x 16 tiles are as fast; 8192^2 at 16 rows 83 -> 60 us)
        // 65 .. 128 rows of a 2-byte dtype: the skinny kernel with 64 rows at once on a 128-wide K step.  Measured with
        // the weights coming from memory, as they do when a layer is used once per pass: 128 x 16384 x 4096 42.5 us
        // against 77.0 us for the 128 tile with K split, 128 x 4096 x 16384 50.4 against 74.4, 128 x 4096 x 4096 20.7
        // against 28.2; in a back-to-back loop, where up to 256 MB of weights stay in the Infinity Cache for the
        // tiled kernel's cacheable copies, within 12 % either way.  (192 .. 256 rows: 20 - 35 % faster from memory
        // but 35 - 50 % slower back to back; left to the tuned table.)
        else if (skinny_ok && !f32 && M > 64 && M <= 128 && K % 128 == 0 && N >= 2048 && N * K >= (int64_t(1) << 22) && forced_split <= 1) {
            variant = V_SKINNY;
            forced_bk = 128;
        }
        else if (skinny_ok && ((M <= 64 && N >= 2048 && N * K >= (int64_t(1) << (f32 ? (M <= 16 ? 25 : 24) : 22))) || (!f32 && M <= 128 && K % 256 == 0 && N >= 8192 && N * K >= (int64_t(1) << 27)))) variant = V_SKINNY;
        else {
            // The general kernel: about 4 us of launch and latency, then either its throughput (55 TFLOP/s on
            // fp32 operands, 70 on bf16, 40 on rows that are no whole chunks) or, for few workgroups and a long K, the serial chain of one
            // workgroup (1.25 us per 256 of K; up to 4 workgroups per CU are resident).
            const int64_t gt = (M <= 16 || ((M + 31) / 32) * ((N + 31) / 32) < 128) ? 16 : 32;
            const int64_t gw = ((M + gt - 1) / gt) * ((N + gt - 1) / gt);
            const double chain = double((gw + 1023) / 1024) * double((K + 255) / 256) * 1.25;
            const double rate = 2.0 * double(M) * double(N) * double(K) / (tiled_ok ? (f32 ? 55.0e6 : 70.0e6) : 40.0e6);
            const double general = 4.0 + (chain > rate ? chain : rate);
            // a forced split only exists on the tiled and skinny kernels
            variant = (tiled_ok && M > 0 && (min_split > 1 ? split_found : best < general || forced_split > 1)) ? V_TILED : V_GENERAL;
            plan->time_us = variant == V_TILED ? best : general;
        }
    }
    if (variant == V_SKINNY && !skinny_ok) return fail(FLE_ERR_UNSUPPORTED, "the skinny kernel needs M <= 256, K a multiple of 128 bytes and everything the tiled kernel needs");
    if (variant == V_TILED && !tiled_ok) return fail(FLE_ERR_UNSUPPORTED, "the tiled MFMA kernel needs x and W rows made of whole, 16-byte aligned chunks (K and the leading dimensions multiples of 16 bytes)");
    if (variant == V_THIN && !thin_ok) return fail(FLE_ERR_UNSUPPORTED, "the thin kernel needs M <= 32 and everything the tiled kernel needs of x and W");
    if (variant == V_THIN && forced_split > 1) return fail(FLE_ERR_UNSUPPORTED, "the thin kernel does not split K");
    if (variant != V_TILED && variant != V_GENERAL && variant != V_SKINNY && variant != V_THIN) return fail(FLE_ERR_OP, "unknown forced variant %d", variant);
    plan->edge = 0;
    int auto_split = 0;  // chosen with the tile (tiled kernel); 0: decided below
    // The skinny kernel fills the chip by a split of K as long as every workgroup keeps at least 512 of K.  Its W tiles go to
    // the 8 XCDs in turn and one workgroup fills a CU, so the count is that of the XCD with most of them (80 x 5248 x
    // 4992, 41 W tiles: 36 workgroups for the 32 CUs of the first XCD took 37 us, a split less 23).
    auto skinny_tiles = [&](int64_t bm) -> int64_t { return (M + bm - 1) / bm * (((N + 127) / 128 + 7) / 8 * 8); };
    bool more_ranges = false;
    auto skinny_split = [&](int64_t bm, int64_t bk) -> int64_t {
        const int64_t steps = K / bk, min_steps = 512 / bk > 2 ? 512 / bk : 2;
        auto ranges = [&](int64_t tiles, int64_t workgroups) -> int64_t {
            int64_t s = 1;
            if (tiles * 2 <= workgroups) {
                s = workgroups / tiles;
                if (s > steps / min_steps) s = steps / min_steps;
                if (s > 16) s = 16;
            }
            return s < 1 ? 1 : s;
        };
        const int64_t s = ranges(skinny_tiles(bm), 256);
        // A range less is a longer chain of fp32 sums, which is what fp32 results are off by: where the count by XCD gives fewer
        // ranges than the W tiles would, two workgroups per CU in turn (35 x 5308 x 4736 in two ranges 64 us and 9.6e-7 off float64,
        // in three 83 and 7.7e-7, in five 58 and 6.0e-7; 20 x 6196 x 16256 in four 114 and 1.2e-6, in five 156 and 1.1e-6, in ten 130 and 7.7e-7).
        // (A workspace that has no room for their slabs gets the count by W tiles.)
        if (f32) {
            const int64_t by_tiles = ranges((M + bm - 1) / bm * ((N + 127) / 128), 256);
            if (s < by_tiles) {
                const int64_t more = refine == REFINE_NONE ? 0 : ranges(skinny_tiles(bm), 512);
                if (more > by_tiles) more_ranges = true;
                return std::max(by_tiles, more);
            }
        }
        return s;
    };
    auto general_tile = [&]() -> int { return (M <= 16 || ((M + 31) / 32) * ((N + 31) / 32) < 128) ? 16 : 32; };
    int skinny_bm = 0, skinny_bk = 0;
    if (variant == V_SKINNY) {
        // The widest K step that fits two stages: 512-byte runs per W row stream at 6.0 TB/s where 128- and 256-byte runs
        // reach 4.5 TB/s.  forced 64 keeps the narrow ring for comparison.
        int bk = forced_bk ? forced_bk : 256;  // in 2-byte elements; fp32 operands take half as many for the same bytes
        if (forced == V_SKINNY) bk = 64;
        const int per = f32 ? 2 : 1;
        while (bk > 64 && K % (bk / per) != 0) bk /= 2;
        // Row blocks of 32.  More than 32 rows: one block of 64, 128 or 256 rows whose 32-row sub-blocks take
        // turns on a 256-wide W stage (automatic choice; with fewer than 64 W tiles the chip is not full and
        // more, smaller workgroups do better), or, on request, 64 rows at once on a 128-wide K step; a forced
        // 256-wide K step keeps blocks of 32 (one workgroup each) for comparison.
        skinny_bm = 32;
        if (f32) { /* row blocks of 32 only */ }
        else if (M > 32 && forced_bk == 128 && bk == 128) skinny_bm = 64;
        else if (M > 32 && bk == 256 && (forced_seq || (forced == V_AUTO && N >= 8192))) skinny_bm = M <= 64 ? 64 : M <= 128 ? 128 : 256;
        skinny_bk = bk / per;
    }
    // ---- second look at an automatic choice on 2-byte and fp8 operands.  The rules above know neither the deep tile
    // nor the streaming kernels outside the sizes that they were drawn up for; kernel_us compares every kernel that can
    // run the problem with the first choice, which stays unless another is so much ahead that the fits' error does
    // not turn it round: 3 % between 128 tiles (5 % with block scales), 8 % otherwise, 12 % to leave a 256 tile or to go to the general kernel, 15 % between
    // forms of the skinny kernel, 40 % to leave a thin kernel for a split of K and its second launch,
    // unless it has few workgroups with a long chain each (24 x 384 x 6016 20.7 us, in 16 ranges 11.9).  Of 1185 random calls
    // on 2-byte and fp8 operands, with every kind of list, 453 change hands: they take 12 % less time, and 9 of them are over 3 %
    // slower than the first choice (6301 x 299 x 2752 with LayerNorm 38.9 -> 48.2 us, the others 1.14 times at most); 80 x 5248 x 4992 37.7
    // -> 22.4 us, 1024 x 4096 x 4096 54 -> 39.
    if (automatic && tiled_ok) {
        const int64_t kb = K * int64_t(xs);
        struct { int variant, bm, bk, tile, deep; int64_t split; double us; bool f32; int rows; } pick = {variant, skinny_bm, skinny_bk, best_tile, 0, best_split, 0.0, false, 0};
        auto tiles_of = [&](int64_t bm, int64_t bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
        auto skinny_time = [&](int bm, int bk) -> const KernelTime & {
            if (bm == 32) return bk == 256 ? kSkinny32x256 : bk == 128 ? kSkinny32x128 : kSkinny32x64;
            return bm == 64 ? (bk == 128 ? kSkinny64x128 : kSkinny64x256) : bm == 128 ? kSkinny128x256 : kSkinny256x256;
        };
        auto skinny_us = [&](int bm, int bk) { return kernel_us(skinny_time(bm, bk), skinny_tiles(bm), kb, skinny_split(bm, bk), M, N); };
        const bool dot = M <= 4;
        const double us_general = kernel_us(general_tile() == 16 ? kGeneral16 : kGeneral32, tiles_of(general_tile(), general_tile()), kb, 1, M, N);
        const double us_thin = kernel_us(dot ? kDot : M <= 16 ? kThin16 : kThin32, (N + 15) / 16, kb, 1, M, N) + (dot ? 0.9 * double(M) : 0.0);
        const KernelTime &tiled128 = plan->mx ? kTiled128Mx : kTiled128;
        const double first_product = variant == V_TILED ? kernel_us(best_tile == 256 ? kTiled256 : tiled128, tiles_of(best_tile, best_tile), kb, best_split, M, N)
                             : variant == V_SKINNY ? skinny_us(skinny_bm, skinny_bk) : variant == V_THIN ? us_thin : us_general;
        const bool from256 = variant == V_TILED && best_tile == 256;
        // A row reduction's values are staged in 2 bytes, rounded relative to their partial's maximum or mean: in a wider partial
        // further off (fp16 softmax, error against float64 in the first choice's partials, in this one's, staged in fp32: 28 x 8320 x
        // 640, 16 and 32 columns, 2.54e-4, 2.69e-4, 2.13e-4; 79 x 10112 x 2176, 32 and 256, 2.74e-4, 3.21e-4, 2.19e-4).  A plan with
        // wider partials than the first choice's stages in fp32 instead, for 4 bytes more per value over both passes (117 x
        // 23232 x 4096 78.1 us, 61.0 staged in 2 bytes, 61.5 in fp32).  So does every plan behind a first choice whose split reduces
        // its rows over the slabs: nothing of that is staged, and the result is rounded once.
        const bool rounds = (e.row_kind == FLE_LAYERNORM || e.row_kind == FLE_SOFTMAX) && !post_res_alias_out && !lse && !stage_f32;
        auto partial = [&](int v, int tile, int64_t sp) { return sp > 1 ? (reduces_rows(e, M, N, sp) ? 0 : 256) : v == V_TILED ? tile / 2 : v == V_SKINNY ? 32 : 16; };
        const int64_t first_split = variant == V_TILED ? best_split : variant == V_SKINNY ? skinny_split(skinny_bm, skinny_bk) : 1;
        const int first_partial = small && first_split > 1 ? 256 : partial(variant, best_tile, first_split);
        // (behind such a first choice, fp32 against 2 bytes on the same kernel at 45 shapes: 932 x 2752 1.0 us, 2366 x 1152 1.7, 4355 x 896 1.5, 2277 x
        // 1536 1.8, 4920 x 1920 2.0, 2303 x 3712 4.3, 5940 x 2816 11; with 4.5 the first went back to its split, 36.7 us in 2 bytes, 37.7 in fp32, 38.4 split)
        const double f32_us = 4.0 * double(M) * double(N) / (first_partial == 0 ? 9.0e6 : 4.5e6);
        // What LayerNorm or softmax adds (a logsumexp reads partials only): a pass over the row, every wave of which combines the row's
        // partials 64 at a time (LayerNorm, 16 x 21760 x 256 in fp16: 1360 partials of 16 columns 24.1 us, 680 of 32 16.3; with 400 -
        // 500 of 16 the width makes no difference), or, behind a split, a workgroup per row over the slabs: that gains on
        // two passes up to about a million values (161 x 704 x 832 14.6 us unsplit, 11.5 in four ranges; 932 x 2752 x 4544 41.5
        // unsplit, 47.3 in two).  The margins are shares of the product's time, which alone is fitted.
        auto row_pass = [&](int v, int tile, int64_t sp) -> double {
            if (e.row_kind != FLE_LAYERNORM && e.row_kind != FLE_SOFTMAX) return 0.0;
            const int cols = partial(v, tile, sp);
            if (cols == 0) return 1.0 + std::min(2.9, double(M) * double(N) / 4.0e5);
            return 3.9 + (e.row_kind == FLE_LAYERNORM ? 0.4 * std::max(0.0, double(N / cols / 64) - 8.0) : 0.0);
        };
        const double first = first_product + row_pass(variant, best_tile, first_split);
        pick.us = first;
        auto offer = [&](double us, double margin, int v, int bm, int bk, int tile, int dp, int64_t sp) {
            const int64_t ranges = v == V_SKINNY ? skinny_split(bm, bk) : sp;
            if (variant == V_THIN && (dot || K <= 4 * N) && ranges > 1 && us >= 0.6 * us_thin) return;  // (by the products alone)
            const bool in_f32 = rounds && partial(v, tile, ranges) > first_partial;
            us += row_pass(v, tile, ranges);
            if (in_f32) us += f32_us;
            if (us < first - (1.0 - margin) * first_product && us < pick.us) { pick.variant = v; pick.bm = bm; pick.bk = bk; pick.tile = tile; pick.deep = dp; pick.split = sp; pick.us = us; pick.f32 = in_f32; pick.rows = 0; }
        };
        const bool all = refine == REFINE_ALL && !f8;
        if (all) {
            // (a call with a row reduction keeps the tiled kernel: 512 x 1024 x 256 with LayerNorm 15.0 us, 13.1 here)
            if (e.row_kind < 0 || variant != V_TILED) offer(us_general, 0.88, V_GENERAL, 0, 0, best_tile, 0, 1);
            if (thin_ok) offer(us_thin, 0.92, V_THIN, 0, 0, best_tile, 0, 1);
            if (skinny_ok) {
                auto skinny = [&](int bm, int bk) {  // (narrow W under many ranges of K is slower than fitted: 136 x 128 x 6656 21.5 us, estimated 11.8)
                    if (K % bk == 0 && (N >= 1024 || skinny_split(bm, bk) == 1)) offer(skinny_us(bm, bk), variant == V_SKINNY ? 0.85 : 0.92, V_SKINNY, bm, bk, best_tile, 0, 1);
                };
                for (int bk = 256; bk >= 64; bk /= 2) skinny(32, bk);
                if (M > 32) {
                    skinny(64, 128);
                    skinny(M <= 64 ? 64 : M <= 128 ? 128 : 256, 256);
                }
            }
        }
        if (refine == REFINE_ALL || variant == V_TILED) {
            const double margin = from256 ? 0.88 : variant == V_TILED ? (plan->mx ? 0.95 : 0.97) : 0.92;
            const KernelTime &deep128 = plan->mx ? kDeep128Mx : kDeep128;
            for (int sp : kSplits) {
                if (sp > 1 && (sp * 3 > tiled_steps || int64_t(sp) * M * (N + 3) * 4 > (int64_t(128) << 20))) continue;
                if (tiles_of(128, 128) * sp <= 512) offer(kernel_us(deep128, tiles_of(128, 128), kb, sp, M, N), margin, V_TILED, 0, 0, 128, 1, sp);
            }
        }
        // Tiles of fewer rows, where 256 or 128 leave CUs idle in the last round or rows empty in the last tile.  They stand back 3 %
        // behind the choice so far, its product at a time fitted with theirs where it is unsplit on one of those tiles.  Of 614 random
        // shapes 169 change hands, 1.12 times as fast in the geometric mean (565 x 18816 x 14464 443 -> 301 us, 7232 x 1088 x 3712
        // 80 -> 63, 540 x 16256 x 640 34.8 -> 26.9), 3 of them over 3 % slower; over all shapes the best kernel of each would gain 3.4 %,
        // this gains 3.3.  (The older fits put a 256 tile of several rounds 10 % too high and gave 32768 x 2048 x 2048 away.)
        if ((refine == REFINE_ALL || variant == V_TILED) && !f8 && M > 128 && N > 128) {
            double at = pick.us;
            if (pick.variant == V_TILED && pick.split == 1 && !pick.deep) {
                const int64_t tiles = tiles_of(pick.tile, pick.tile);
                const bool big = pick.tile == 256;
                at = std::min(at, at - kernel_us(big ? kTiled256 : kTiled128, tiles, kb, 1, M, N) + kernel_us(big ? kRows256 : kSquare128, tiles, kb, 1, M, N));
            }
            const bool in_f32 = rounds && partial(V_TILED, 256, 1) > first_partial;
            const double behind = row_pass(V_TILED, 256, 1) + (in_f32 ? f32_us : 0.0);
            double least = 0.97 * at;
            for (int high = 160; high <= 224; high += 32) {
                const double us = kernel_us(high == 160 ? kRows160 : high == 192 ? kRows192 : kRows224, tiles_of(high, 256), kb, 1, M, N) + behind;
                if (us < least) {
                    least = us;
                    pick = {V_TILED, 0, 0, 256, 0, 1, us, in_f32, high};
                }
            }
        }
        plan->refined = pick.us < first || pick.rows;
        variant = pick.variant;
        skinny_bm = pick.bm;
        skinny_bk = pick.bk;
        best_tile = pick.tile;
        best_split = int(pick.split);
        deep = pick.deep;
        rows = pick.rows;
        stage_f32 = stage_f32 || pick.f32;
    }
    plan->variant = variant;
    if (variant == V_SKINNY) {
        plan->bm = skinny_bm;
        plan->bn = 128;
        plan->bk = skinny_bk;
        plan->part_cols = 32;  // one partial per wave tile
    } else if (variant == V_THIN) {
        // few rows: dot products on row-contiguous loads (the vector ALU keeps up with HBM to 4 rows of a 2-byte
        // dtype, 8 of fp32); else the 16x16 MFMA
        plan->bm = M <= (f32 ? 8 : 4) ? 8 : M <= 16 ? 16 : 32;
        plan->bn = 16;
        plan->bk = int32_t(64 / es);  // MFMA form: one step is 64 bytes of every row
        if (plan->bm == 8) {
            // dot-product form: the field holds the W rows per wave instead.  One row of x against many long rows
            // of W: one W row per wave and 16 waves per workgroup keep more loads in flight (fp32 8192^2: 53 ->
            // 47 us; bf16 32768 x 8192: 91 -> 85 us); with more x rows or few W rows 4 per wave are faster.
            plan->bk = (M == 1 && N >= 4096 && K >= 2048) ? 1 : 4;
        }
        plan->part_cols = 16;
    } else if (variant == V_TILED) {
        plan->bm = plan->bn = best_tile;
        if (rows) plan->bm = rows;
        plan->deep = deep;
        plan->bk = f32 ? 32 : f8 ? 128 : 64;
        plan->part_cols = plan->bn / 2;  // one partial per wave column
        plan->edge = vec_epi ? 0 : 1;
        auto_split = best_split;
    } else {
        // 32 x 32 tiles; 16 x 16 when those would give fewer than 128 workgroups (tiny, latency-bound problems)
        plan->bm = plan->bn = general_tile();  // (up to 16 rows a 32-row tile would be half empty)
        plan->bk = 16;
        plan->part_cols = 16;
    }
    plan->tiles_m = (M + plan->bm - 1) / plan->bm;
    if (grp) {  // every group may end in a partly filled tile row; the kernel finds the actual count
        plan->tiles_m = M / plan->bm + G;
        if (plan->tiles_m > M) plan->tiles_m = M;
        plan->w_stream = (plan->bm == 128 && M <= G * kGroupedStreamRows) ? 1 : 0;
    }
    plan->tiles_n = (N + plan->bn - 1) / plan->bn;
    if (plan->tiles_m * plan->tiles_n > (int64_t(1) << 31) - 1) return fail(FLE_ERR_SHAPE, "too many tiles for one launch");

    // ---- split K: few tiles and a long K leave most of the chip idle, so several workgroups share
    // a tile, each over its own K range, writing fp32 slabs that a reduction pass sums in slab order
    // (deterministic).
    plan->split_k = 1;
    if (variant != V_GENERAL && variant != V_THIN && M > 0) {
        const int64_t steps = variant == V_TILED ? tiled_steps : K / plan->bk;
        int64_t s = 1;
        if (forced_split > 0) s = forced_split;
        else if (auto_split > 0) s = auto_split;
        else {
            s = skinny_split(plan->bm, plan->bk);
            if (s < min_split) s = min_split;
            if (more_ranges) plan->refined = 1;
        }
        if (s > steps) s = steps;
        if (s > 64) s = 64;
        if (s < 1) s = 1;
        plan->split_k = int32_t(s);
        if (s > 1) plan->part_cols = 256;  // the reduction pass owns the partials
        plan->one_pass = reduces_rows(e, M, N, s) ? 1 : 0;
    }

    // ---- staging and workspace (of one pass over the slabs as of two: what a call needs does not hang on the number of passes)
    size_t off = 0;
    plan->staging = ST_NONE;
    plan->stage_rel = 0;
    if (e.row_kind >= 0) {
        plan->np = int32_t((N + plan->part_cols - 1) / plan->part_cols);
        plan->ws_part_off = off;
        off = round_up(off + size_t(M) * size_t(plan->np) * 2 * sizeof(float), 256);
        if (e.row_kind != FLE_LOGSUMEXP) {
            // Staged in out itself unless a trailing residual aliases out (or out is the [M] vector of a logsumexp
            // that comes second).  A 2-byte dtype stages v minus the
            // statistic of v's partial (its mean for LayerNorm, its maximum for softmax), which the finalize pass
            // adds back in fp32: the rounding error of the staged value is then relative to the distance from that
            // statistic, not to v itself (a row of mean 100 and deviation 0.01 keeps its deviations; exp() of a
            // distance d <= 0 is off by at most |d| 2^-9, negligible where the probability is not).
            const bool in_out = !post_res_alias_out && !lse && !(stage_f32 && p->dtype != FLE_F32);
            plan->staging = in_out ? ST_OUT : ST_WS;
            plan->stage_rel = (in_out && p->dtype != FLE_F32) ? 1 : 0;
            if (!in_out) {
                plan->ws_y_off = off;
                off = round_up(off + size_t(M) * size_t(N) * sizeof(float), 256);
            }
        }
    }
    if (e.row2_kind >= 0) {  // the values between the two row reductions, fp32 [M,N]
        plan->ws_mid_off = off;
        off = round_up(off + size_t(M) * size_t(N) * sizeof(float), 256);
    }
    if (plan->split_k > 1) {
        plan->ws_slab_off = off;
        off = round_up(off + size_t(plan->split_k) * size_t(M) * size_t((N + 3) / 4 * 4) * sizeof(float), 256);
    }
    plan->ws_total = M > 0 ? off : 0;
    return FLE_OK;
}

}  // namespace fle

using namespace fle;

static const char *dtype_name(int dtype) { return dtype == FLE_F32 ? "f32" : dtype == FLE_F16 ? "f16" : dtype == FLE_F8E4M3 ? "f8" : "bf16"; }

static void format_plan(const AttnPlan &plan, char *buf, size_t n) {
    const bool few = plan.splits > 0;
    snprintf(buf, n, "variant=%s_%s D=%d queries=%d ranges=%d workspace=%zu", few ? "decode_attention" : "flash_attention", dtype_name(plan.dtype), plan.D, few ? 32 : 128,
             few ? plan.splits : 1, plan.ws_bytes);
}

static void format_plan(const ChainPlan &plan, char *buf, size_t n) {
    snprintf(buf, n, "variant=%s_%s weights=%s layers=%d workgroups=%d ahead_kb=%d", plan.ahead_kb ? "perceptron_lds" : "mlp_chain", dtype_name(plan.dtype), dtype_name(plan.w_dtype),
             plan.n_layers, plan.workgroups, plan.ahead_kb ? plan.ahead_kb : 4);
}

static void format_plan(const Plan &plan, char *buf, size_t n) {
    const char *dt = plan.mx ? "f8mx" : dtype_name(plan.op_dtype);
    // (operands of any layout: the general path, which may run another kernel on aligned copies)
    snprintf(buf, n, "variant=%s%s_%s_%s%s%s tile=%dx%dx%d tiles=%lldx%lld split_k=%d row_op=%d np=%d staging=%s workspace=%zu%s%s%s",
             plan.copy_x || plan.copy_w ? "general+copies:" : "", plan.variant == V_TILED ? (plan.groups ? "grouped_tiled" : "tiled") : plan.variant == V_SKINNY ? "skinny" : plan.variant == V_THIN ? "thin" : "general", dt,
             plan.variant == V_THIN && plan.bm == 8 ? "dot" : "mfma",
             plan.edge ? "+edge" : "", plan.deep ? "+deep" : plan.w_stream ? "+wstream" : "", plan.bm, plan.bn, plan.bk, (long long)plan.tiles_m, (long long)plan.tiles_n, plan.split_k, plan.epi.row_kind,
             plan.np, plan.staging == ST_OUT ? "out" : plan.staging == ST_WS ? "workspace_f32" : "none", plan.ws_total,
             plan.ln_pre == LN_PRE_FUSED ? " ln_pre=fused" : plan.ln_pre == LN_PRE_PASS ? " ln_pre=pass" : "", plan.one_pass ? " reduction=one_pass" : "",
             plan.copy_x && plan.copy_w ? " copies=x,w" : plan.copy_x ? " copies=x" : plan.copy_w ? " copies=w" : "");
}

static bool workspace_does(const fle_problem *p, const Plan &plan) {
    return plan.ws_total == 0 || (p->workspace && p->workspace_bytes >= plan.ws_total && aligned(p->workspace, 256));
}

// A plan that copies operands or that is not the first choice needs a workspace where the plan without may need none (or
// less): a caller's workspace that does not do for it (too small, missing, misaligned, over an operand) gets the plan without.
static bool extras_fit(const fle_problem *p, const Plan &plan) {
    if ((!plan.copy_x && !plan.copy_w && !plan.refined) || plan.ws_total == 0) return true;
    if (!workspace_does(p, plan)) return false;
    const size_t es = esize(p->dtype), xs = p->dtype == FLE_F8E4M3 ? 1 : es;
    auto over = [&](const void *a, size_t n) { return overlaps(p->workspace, plan.ws_total, a, n); };
    if (over(p->x, span_bytes(p->M, p->K, p->ldx, xs)) || over(p->w, span_bytes(p->N, p->K, p->ldw, xs)) || over(p->b, size_t(p->N) * es)) return false;
    for (int i = 0; i < p->n_ops; ++i) {
        const fle_op &op = p->ops[i];
        if (op.kind == FLE_RESIDUAL && over(op.p0, span_bytes(p->M, p->N, op.ld, es))) return false;
        const size_t aff = size_t(op.kind == FLE_LAYERNORM_PRE ? p->K : p->N) * es;
        if ((op.kind == FLE_LAYERNORM || op.kind == FLE_LAYERNORM_PRE) && (over(op.p0, aff) || over(op.p1, aff))) return false;
    }
    return true;
}

static fle_status plan_for_run(const fle_problem *p, int forced, int forced_split, Plan *plan) {
    fle_status s = make_plan(p, forced, forced_split, plan);
    if (s == FLE_OK && p->M > 0 && !extras_fit(p, *plan)) s = make_plan(p, forced, forced_split, plan, nullptr, PLAN_REFINE);
    if (s == FLE_OK && p->M > 0 && !extras_fit(p, *plan)) s = make_plan(p, forced, forced_split, plan, nullptr, 0);
    if (s == FLE_OK && p->M > 0 && plan->one_pass && !workspace_does(p, *plan)) {  // (no room for the slabs either)
        Plan less;
        if (make_plan(p, forced, forced_split, &less, nullptr, PLAN_REFINE | PLAN_SMALL) == FLE_OK && workspace_does(p, less) && extras_fit(p, less)) *plan = less;
    }
    return s;
}

static fle_status check_workspace(const fle_problem *p, const Plan &plan) {
    if (plan.ws_total == 0) return FLE_OK;
    if (!p->workspace) return fail(FLE_ERR_WORKSPACE, "workspace is NULL but %zu bytes are needed", plan.ws_total);
    if (p->workspace_bytes < plan.ws_total) return fail(FLE_ERR_WORKSPACE, "workspace has %zu bytes, %zu needed", p->workspace_bytes, plan.ws_total);
    if (reinterpret_cast<uintptr_t>(p->workspace) % 256 != 0) return fail(FLE_ERR_ALIGN, "workspace must be 256-byte aligned");
    return FLE_OK;
}

// ------------------------------------------------------------------ attention
// Elements spanned by B sequences of T tokens of HD elements with token stride ld and sequence stride sb,
// or 0 if the two strides make tokens of different sequences collide.
static int64_t attention_extent(int64_t B, int64_t T, int64_t HD, int64_t ld, int64_t sb) {
    const bool seq_major = sb >= (T - 1) * ld + HD, token_major = sb >= HD && ld >= (B - 1) * sb + HD;
    if (B > 1 && !seq_major && !token_major) return 0;
    return (B - 1) * sb + (T - 1) * ld + HD;
}

static fle_status check_attention(const fle_attention *p) {
    if (!p) return fail(FLE_ERR_NULL, "attention problem is NULL");
    if (p->dtype != FLE_BF16 && p->dtype != FLE_F16) return fail(FLE_ERR_UNSUPPORTED, "attention takes FLE_BF16 or FLE_F16 (got dtype %d)", p->dtype);
    if (p->B < 0 || p->H < 1 || p->T < 1 || p->Tk < 0) return fail(FLE_ERR_SHAPE, "need B >= 0, H >= 1, T >= 1, Tk >= 0 (got %lld, %lld, %lld, %lld)", (long long)p->B, (long long)p->H, (long long)p->T, (long long)p->Tk);
    if (p->D != 32 && p->D != 64 && p->D != 128 && p->D != 256) return fail(FLE_ERR_UNSUPPORTED, "head dimension %lld is not 32, 64, 128 or 256", (long long)p->D);
    if (p->causal < 0) return fail(FLE_ERR_OP, "causal must be 0, 1 or a group size (got %d)", p->causal);
    if (p->B > 65535 || p->H > 65535) return fail(FLE_ERR_SHAPE, "B and H are limited to 65535");
    const int64_t Tk = p->Tk > 0 ? p->Tk : p->T;
    if (p->T > (int64_t(1) << 24) || Tk > (int64_t(1) << 24)) return fail(FLE_ERR_SHAPE, "T and Tk are limited to 2^24");
    if (p->causal && Tk < p->T) return fail(FLE_ERR_SHAPE, "a causal mask needs Tk >= T (got Tk = %lld, T = %lld)", (long long)Tk, (long long)p->T);
    if ((p->T + 127) / 128 * p->H * p->B >= (int64_t(1) << 31)) return fail(FLE_ERR_SHAPE, "B * H * T / 128 is limited to 2^31 workgroups");
    const int64_t HD = p->H * p->D;
    const int64_t kLimit = int64_t(1) << 40;
    if (p->ldq < HD || p->ldk < HD || p->ldv < HD || p->ldo < HD) return fail(FLE_ERR_SHAPE, "a token stride is smaller than H*D = %lld", (long long)HD);
    if (p->ldq > kLimit || p->ldk > kLimit || p->ldv > kLimit || p->ldo > kLimit) return fail(FLE_ERR_SHAPE, "token stride too large");
    if (p->sbq < 0 || p->sbk < 0 || p->sbv < 0 || p->sbo < 0 || p->sbq > kLimit || p->sbk > kLimit || p->sbv > kLimit || p->sbo > kLimit)
        return fail(FLE_ERR_SHAPE, "sequence strides must be >= 0 (0 = packed)");
    // the kernel addresses the Q, K and V of one sequence with 32-bit byte offsets
    if ((p->T + 256) * p->ldq * 2 >= (int64_t(1) << 31) || (Tk + 64) * (p->ldk > p->ldv ? p->ldk : p->ldv) * 2 >= (int64_t(1) << 31))
        return fail(FLE_ERR_SHAPE, "one sequence's Q, K or V spans 2 GiB or more");
    if (!(p->scale >= 0.0f) || std::isinf(p->scale)) return fail(FLE_ERR_OP, "scale must be finite and > 0 (or 0 for 1/sqrt(D))");
    if (p->B == 0) return FLE_OK;
    if (!p->q || !p->k || !p->v || !p->o) return fail(FLE_ERR_NULL, "q, k, v or o is NULL");
    if (!aligned(p->q, 16) || !aligned(p->k, 16) || !aligned(p->v, 16)) return fail(FLE_ERR_ALIGN, "q, k and v must be 16-byte aligned");
    if (p->ldq % 8 || p->ldk % 8 || p->ldv % 8 || p->sbq % 8 || p->sbk % 8 || p->sbv % 8) return fail(FLE_ERR_ALIGN, "the strides of q, k and v must be multiples of 8 elements");
    if (!aligned(p->o, 8) || p->ldo % 4 || p->sbo % 4) return fail(FLE_ERR_ALIGN, "o must be 8-byte aligned and its strides multiples of 4 elements");
    const int64_t eq = attention_extent(p->B, p->T, HD, p->ldq, p->sbq > 0 ? p->sbq : p->T * p->ldq);
    const int64_t ek = attention_extent(p->B, Tk, HD, p->ldk, p->sbk > 0 ? p->sbk : Tk * p->ldk);
    const int64_t ev = attention_extent(p->B, Tk, HD, p->ldv, p->sbv > 0 ? p->sbv : Tk * p->ldv);
    const int64_t eo = attention_extent(p->B, p->T, HD, p->ldo, p->sbo > 0 ? p->sbo : p->T * p->ldo);
    if (!eq || !ek || !ev || !eo) return fail(FLE_ERR_SHAPE, "token and sequence strides make sequences collide");
    const size_t no = size_t(eo) * 2;
    if (overlaps(p->o, no, p->q, size_t(eq) * 2) || overlaps(p->o, no, p->k, size_t(ek) * 2) || overlaps(p->o, no, p->v, size_t(ev) * 2))
        return fail(FLE_ERR_UNSUPPORTED, "o overlaps q, k or v");
    return FLE_OK;
}

// Up to 32 queries per sequence can run on either kernel: the one of 128 queries per workgroup, of whose four waves one has
// work then, or the one whose waves share out the keys, which keeps twice the LDS per workgroup and needs enough keys for its
// waves, or enough workgroups, to make that good.  Measured at 1100 shapes of 8 .. 2000 heads (8, 12, 16 or 25 a sequence), 1, 2, 5 and 16 queries,
// 64 .. 6000 keys, bf16, new K and V in each call, as a decoding step meets them; us on the kernel of 128 queries / on the other.  By these
// bounds the calls with heads of 64, 128 and 256 take 1.0, 1.4 and 0.7 % longer than on the better kernel each (2.0, 2.4 and 1.3 % by
// 512 keys for heads of 64, 192 heads or ranges over 768 keys for 128, 256 and 512 keys for 256).  K and V that a call before left in the
// Infinity Cache are found there by the kernel of 128 queries only, as the other reads past it: repeated calls over less than 256 MB run up to 1.25
// times as fast on it from 320 heads on (768 heads of 64 over 1024 keys 34 / 38, new ones 44 / 38).  A little more than one head
// per CU gives either kernel the same uneven share: level on new K and V, 1.2 - 1.4 times as fast on repeated ones on the kernel of 128 queries (not so
// 264 - 320 heads of 64 over 1900 keys and more with 12 or 25 heads a sequence, 300 over 2293 44.6 / 38.0; with 8, 264 over 3000 54.9 / 56.4).
static bool sharing_keys_pays(const fle_attention *p, int64_t heads, int64_t Tk, int splits) {
    switch (p->D) {
    case 32:   // (512 heads over 128 keys 5.2 / 5.9, over 512 9.2 / 10.5, over 1024 22.3 / 21.2; 288 over 858 13.2 / 11.2; 256 over 256 6.1 / 6.0; 900 over 32 5.9 / 4.7)
        return heads > 768 || Tk >= (heads <= 256 ? 256 : 768);
    case 64:   // (256 heads over 512 keys 12.3 / 10.8, at most 256 over 256 - 383 1.05 - 1.15 times; 264 over 512 13.0 / 14.6, over 8000 139 / 143; 321 - 384 over
               // 2000 - 6000 1.10 times, 352 over 1514 36.0 / 33.8; 396 over 3924 78.0 / 71.7; 420 over 1430 32.1 / 30.1; 512 over 512 16.2 / 16.7, over 700 20.2 / 19.7; 768 over 600
               // 27.4 / 24.6; 2048 over 512 51 / 52, over 600 60.9 / 57.7, over 1024 101 / 99, 4096 188 / 193)
        if (heads <= 256) return Tk >= 256;
        return heads > 320 && heads <= 2048 && Tk >= (heads >= 512 ? 600 : heads > 384 ? 1000 : 1500);
    case 128:  // (128 heads over 512 keys 13.0 / 14.4, in ranges 16.9 at 800, 23.9 on the other; 176 over 730 23.6 / 19.5; 256 over 600 21.7 / 18.0; 264 over 700 24.2 / 24.9,
               // over 6000 166 / 167; 304 over 1024 35.6 / 35.0; 336 over 600 24.5 / 24.0; 512 over 64 7.4 / 8.1, over 504 27.4 / 25.6; 925 over 390 39.6 / 37.8; 1225
               // over 426 55.5 / 52.2)
        if (heads > 256) return heads > 320 && Tk >= 384;
        return (heads >= 192 && Tk >= 256) || (heads >= 144 && Tk >= 512) || splits > 1;  // (ranges are first taken over 513 keys)
    default:   // one workgroup per CU there, two here (300 heads over 32 keys 15.5 / 8.4, 32 queries 17.7 / 15.9; up to 256 heads: 64 over 32 8.3 / 6.6, over 64 8.6 /
               // 9.2, 192 over 88, three blocks of 32 keys against two of 64, 12.3 / 11.3; in ranges 8 over 209 15.9 / 13.1, 84 over 195 17.0 / 15.0, 48 over 187 13.9 / 13.9; 16 queries, 24 over 235 16.5 / 15.7, 224 over 174 17.7 / 19.9, 160
               // over 246 19.7 / 22.9, 60 over 289 21.4 / 19.4; 32 queries over 256 17 / 22, over 512 31 / 25)
        return heads > 256 || (p->T <= 8 && (Tk <= 32 || (Tk > 64 && Tk <= 96))) || (splits > 1 && Tk >= (p->T <= 8 ? 192 : p->T <= 16 ? 288 : 512));
    }
}

// How attention runs (see above for up to 32 queries per sequence).  With a workspace (max_splits > 1) the
// keys are also cut into ranges, by a coarse time model in microseconds fitted to measured runs: a block step of a
// workgroup (32 KB; 16 KB at head dimension 32) takes 1.2 (1.8 at 256) while the memory system is idle and 3.0 when all
// 512 (1024) resident workgroups ask for theirs, a workgroup starts and ends in 4, the pass that puts s ranges together
// costs 4 + 0.4 s.  (One sequence of 16 heads of 128 over 8192 keys: see the kernel for the gain; 20 x 16 heads over 1000
// keys, one range 37 us, two 43, three 38; 3 x 8 heads of 256 over 650 keys, 1, 4, 8, 16 ranges: 41, 20, 16, 19 us.)
static AttnPlan plan_attention(const fle_attention *p, int max_splits) {
    AttnPlan plan = {p->dtype, int32_t(p->D), 0, 0};
    if (p->T > 32 || p->B == 0) return plan;
    const int64_t Tk = p->Tk > 0 ? p->Tk : p->T, heads = p->B * p->H, waves = p->D == 256 ? 1 : p->D == 128 ? 2 : 4;
    const int64_t blocks = (Tk + 31) / 32, slots = p->D == 32 ? 1024 : 512;
    double best = 0.0;
    for (int64_t s = 1; s <= max_splits && s <= 64 && (s == 1 || s * waves <= blocks); ++s) {
        const int64_t wgs = heads * s, rounds = (wgs + slots - 1) / slots, last = wgs - (rounds - 1) * slots;
        const double steps = double(((blocks + s - 1) / s + waves - 1) / waves), busy = 3.0 * double(last) / double(slots), idle = p->D == 256 ? 1.8 : 1.2;
        const double t = double(rounds - 1) * (4.0 + 3.0 * steps) + 4.0 + (busy > idle ? busy : idle) * steps + (s > 1 ? 4.0 + 0.4 * double(s) : 0.0);
        if (s == 1 || t < best) {
            best = t;
            plan.splits = int32_t(s);
        }
        if (s == 1 && t < 14.0) break;  // a second launch costs the host as much as could be gained (8 heads of 128 over 500 keys: 11.8 -> 15.5 us with four ranges)
    }
    if (!sharing_keys_pays(p, heads, Tk, plan.splits)) plan.splits = 0;
    if (plan.splits > 1) plan.ws_bytes = size_t(plan.splits) * size_t(heads * p->T) * size_t(p->D + 2) * sizeof(float);
    return plan;
}

// The three stages of an attention block and where their intermediates sit in the workspace.
struct BlockParts {
    fle_problem proj, outp;
    fle_attention att;
    fle_op proj_ops[1], out_ops[2];
    Plan proj_plan, out_plan;
    size_t qkv_off, a_off, sub_off, total;
};

static fle_status plan_block(const fle_attention_block *p, BlockParts *bp, int allow = PLAN_REFINE) {
    if (!p) return fail(FLE_ERR_NULL, "attention block is NULL");
    if (p->dtype != FLE_BF16 && p->dtype != FLE_F16) return fail(FLE_ERR_UNSUPPORTED, "attention takes FLE_BF16 or FLE_F16 (got dtype %d)", p->dtype);
    if (p->B < 0 || p->T < 1 || p->C < 1 || p->H < 1) return fail(FLE_ERR_SHAPE, "need B >= 0, T >= 1, C >= 1, H >= 1");
    if (p->B > 65535 || p->T > (int64_t(1) << 24) || p->C > (int64_t(1) << 24)) return fail(FLE_ERR_SHAPE, "size too large");
    if (p->C % p->H) return fail(FLE_ERR_SHAPE, "C = %lld is not a multiple of H = %lld", (long long)p->C, (long long)p->H);
    const int64_t D = p->C / p->H, rows = p->B * p->T, C = p->C;
    std::memset(bp, 0, sizeof *bp);
    bp->qkv_off = 0;
    bp->a_off = round_up(size_t(rows) * size_t(3 * C) * 2, 256);
    bp->sub_off = bp->a_off + round_up(size_t(rows) * size_t(C) * 2, 256);
    char *ws = reinterpret_cast<char *>(p->workspace);
    char *qkv = ws ? ws + bp->qkv_off : nullptr, *a = ws ? ws + bp->a_off : nullptr;

    fle_problem &pj = bp->proj;
    pj.M = rows; pj.N = 3 * C; pj.K = C; pj.dtype = p->dtype;
    pj.x = p->x; pj.ldx = C; pj.w = p->w_qkv; pj.ldw = C; pj.b = p->b_qkv;
    pj.out = qkv;
    pj.ldo = 3 * C;
    if (p->b_qkv) { bp->proj_ops[0].kind = FLE_BIAS; pj.n_ops = 1; }
    pj.ops = bp->proj_ops;
    pj.stream = p->stream;

    fle_attention &at = bp->att;
    at.dtype = p->dtype; at.causal = p->causal; at.B = p->B; at.H = p->H; at.T = p->T; at.D = D;
    at.q = qkv; at.k = qkv ? qkv + C * 2 : nullptr; at.v = qkv ? qkv + 2 * C * 2 : nullptr;
    at.ldq = at.ldk = at.ldv = 3 * C;
    at.o = a; at.ldo = C; at.scale = 0.0f; at.stream = p->stream;

    fle_problem &po = bp->outp;
    po.M = rows; po.N = C; po.K = C; po.dtype = p->dtype;
    po.x = a; po.ldx = C; po.w = p->w_o; po.ldw = C; po.b = p->b_o;
    po.out = p->out; po.ldo = C;
    int n = 0;
    if (p->b_o) bp->out_ops[n++].kind = FLE_BIAS;
    if (p->residual) { bp->out_ops[n].kind = FLE_RESIDUAL; bp->out_ops[n].p0 = p->residual; bp->out_ops[n].ld = C; ++n; }
    po.ops = bp->out_ops; po.n_ops = n;
    po.stream = p->stream;

    if (D != 32 && D != 64 && D != 128 && D != 256) return fail(FLE_ERR_UNSUPPORTED, "head dimension C / H = %lld is not 32, 64, 128 or 256", (long long)D);
    if (rows > 0 && (!p->x || !p->w_qkv || !p->w_o || !p->out)) return fail(FLE_ERR_NULL, "x, w_qkv, w_o or out is NULL");
    if (rows > 0) {
        // the output projection checks out against its own operands; the first stage's are checked here
        const size_t n_out = size_t(rows) * size_t(C) * 2;
        if (overlaps(p->out, n_out, p->w_qkv, size_t(3 * C) * size_t(C) * 2) || overlaps(p->out, n_out, p->b_qkv, size_t(3 * C) * 2))
            return fail(FLE_ERR_UNSUPPORTED, "out overlaps w_qkv or b_qkv");
        if (overlaps(p->out, n_out, p->x, n_out) && !(p->out == p->x && p->residual == p->x))
            return fail(FLE_ERR_UNSUPPORTED, "out overlaps x (allowed only when x is also the residual, exactly)");
    }
    fle_status s;
    if (ws) {
        s = make_plan(&pj, V_AUTO, 0, &bp->proj_plan, nullptr, allow);
        if (s == FLE_OK) s = check_attention(&at);
        if (s == FLE_OK) s = make_plan(&po, V_AUTO, 0, &bp->out_plan, nullptr, allow);
        if (s != FLE_OK) return s;
        if (rows > 0 && overlaps(p->out, size_t(rows) * size_t(C) * 2, ws, p->workspace_bytes)) return fail(FLE_ERR_UNSUPPORTED, "out overlaps the workspace");
    } else {
        // No workspace yet (validation, sizing): the intermediates get a stand-in address that is never
        // dereferenced; the plans of the two projections do not depend on where qkv and a will live.
        fle_problem t1 = pj, t2 = po;
        t1.out = reinterpret_cast<void *>(uintptr_t(256));
        t2.x = reinterpret_cast<const void *>(uintptr_t(256));
        s = make_plan(&t1, V_AUTO, 0, &bp->proj_plan, nullptr, allow);
        if (s == FLE_OK) s = make_plan(&t2, V_AUTO, 0, &bp->out_plan, nullptr, allow);
        if (s != FLE_OK) return s;
    }
    const size_t sub = bp->proj_plan.ws_total > bp->out_plan.ws_total ? bp->proj_plan.ws_total : bp->out_plan.ws_total;
    bp->total = bp->sub_off + round_up(sub, 256);
    pj.workspace = ws ? ws + bp->sub_off : nullptr; pj.workspace_bytes = round_up(sub, 256);
    po.workspace = pj.workspace; po.workspace_bytes = pj.workspace_bytes;
    return FLE_OK;
}

// ------------------------------------------------------------------ perceptron chain
static const size_t kChainSyncBytes = 2560;  // the barrier state at the start of the workspace: 20 lines of 128 bytes
static fle_status check_chain(const fle_chain *p, size_t *act_bytes) {
    if (!p) return fail(FLE_ERR_NULL, "chain is NULL");
    if (p->dtype != FLE_F32 && p->dtype != FLE_BF16 && p->dtype != FLE_F16) return fail(FLE_ERR_OP, "dtype %d is not FLE_F32, FLE_BF16 or FLE_F16", p->dtype);
    if (p->n_layers < 1 || p->n_layers > FLE_CHAIN_MAX_LAYERS) return fail(FLE_ERR_SHAPE, "n_layers %d outside 1..%d", p->n_layers, FLE_CHAIN_MAX_LAYERS);
    if (!p->layers || !p->x || !p->out) return fail(FLE_ERR_NULL, "layers, x or out is NULL");
    if (p->w_dtype != p->dtype && !(p->dtype == FLE_F32 && (p->w_dtype == FLE_BF16 || p->w_dtype == FLE_F16)))
        return fail(FLE_ERR_UNSUPPORTED, "w_dtype %d must equal dtype %d, or be a 2-byte dtype under FLE_F32", p->w_dtype, p->dtype);
    const size_t es = esize(p->dtype), ws_ = esize(p->w_dtype);
    if (!aligned(p->x, 16)) return fail(FLE_ERR_ALIGN, "x must be 16-byte aligned");
    int64_t widest = 0;
    for (int l = 0; l < p->n_layers; ++l) {
        const fle_chain_layer &L = p->layers[l];
        if (L.n < 1 || L.k < 1 || L.n > (int64_t(1) << 24) || L.k > (int64_t(1) << 24)) return fail(FLE_ERR_SHAPE, "layer %d: n and k must be in 1 .. 2^24", l);
        if (l > 0 && L.k != p->layers[l - 1].n) return fail(FLE_ERR_SHAPE, "layer %d takes %lld inputs but layer %d gives %lld", l, (long long)L.k, l - 1, (long long)p->layers[l - 1].n);
        if ((size_t(L.k) * ws_) % 16) return fail(FLE_ERR_ALIGN, "layer %d: a row of W must be a multiple of 16 bytes", l);
        if (!L.w) return fail(FLE_ERR_NULL, "layer %d: w is NULL", l);
        if (!aligned(L.w, 16)) return fail(FLE_ERR_ALIGN, "layer %d: w must be 16-byte aligned", l);
        if (L.act != -1 && L.act != FLE_RELU && L.act != FLE_GELU_ERF && L.act != FLE_GELU_TANH) return fail(FLE_ERR_OP, "layer %d: activation %d is not -1, RELU, GELU_ERF or GELU_TANH", l, L.act);
        if (overlaps(p->out, size_t(p->layers[p->n_layers - 1].n) * es, L.w, size_t(L.n) * size_t(L.k) * ws_)) return fail(FLE_ERR_UNSUPPORTED, "out overlaps the weights of layer %d", l);
        if (l + 1 < p->n_layers && L.n > widest) widest = L.n;
    }
    if (overlaps(p->out, size_t(p->layers[p->n_layers - 1].n) * es, p->x, size_t(p->layers[0].k) * es) && p->n_layers > 1)
        return fail(FLE_ERR_UNSUPPORTED, "out overlaps x");
    *act_bytes = round_up(size_t(widest) * es, 256);
    return FLE_OK;
}

extern "C" {

fle_status fle_validate(const fle_problem *p) {
    Plan plan;
    return make_plan(p, g_forced, g_split, &plan);
}

fle_status fle_workspace_size(const fle_problem *p, size_t *bytes_out) {
    if (!bytes_out) return fail(FLE_ERR_NULL, "bytes_out is NULL");
    Plan plan;
    fle_status s = make_plan(p, g_forced, g_split, &plan);
    if (s != FLE_OK) return s;
    *bytes_out = plan.ws_total;
    remember(plan);
    return FLE_OK;
}

fle_status fle_run(const fle_problem *p) {
    Plan plan;
    fle_status s = plan_for_run(p, g_forced, g_split, &plan);
    if (s != FLE_OK) return s;
    if (p->M == 0) return FLE_OK;
    s = check_workspace(p, plan);
    if (s == FLE_OK) s = launch(p, plan);
    if (s == FLE_OK) remember(plan);
    return s;
}

// A plan choice is valid when it names a variant the force knob knows and a split in 0 .. 64.
static fle_status check_choice(const fle_plan_choice *c) {
    if (!c) return fail(FLE_ERR_NULL, "plan choice is NULL");
    if (c->variant < V_AUTO || c->variant > V_THIN) return fail(FLE_ERR_OP, "plan choice: unknown variant %d", c->variant);
    if (c->split < 0 || c->split > 64) return fail(FLE_ERR_OP, "plan choice: split %d outside 0..64", c->split);
    return FLE_OK;
}

fle_status fle_workspace_size_with(const fle_problem *p, const fle_plan_choice *c, size_t *bytes_out) {
    if (!bytes_out) return fail(FLE_ERR_NULL, "bytes_out is NULL");
    fle_status s = check_choice(c);
    if (s != FLE_OK) return s;
    Plan plan;
    s = make_plan(p, c->variant, c->split, &plan);
    if (s != FLE_OK) return s;
    *bytes_out = plan.ws_total;
    remember(plan);
    return FLE_OK;
}

fle_status fle_run_with(const fle_problem *p, const fle_plan_choice *c) {
    fle_status s = check_choice(c);
    if (s != FLE_OK) return s;
    Plan plan;
    s = plan_for_run(p, c->variant, c->split, &plan);
    if (s != FLE_OK) return s;
    if (p->M == 0) return FLE_OK;
    s = check_workspace(p, plan);
    if (s == FLE_OK) s = launch(p, plan);
    if (s == FLE_OK) remember(plan);
    return s;
}

fle_status fle_run_static(const fle_problem *p) {
    if (!p) return fail(FLE_ERR_NULL, "problem is NULL");
    fle_problem q = *p;
    q.workspace = nullptr;  // the caller's workspace fields are ignored
    q.workspace_bytes = 0;
    Plan plan;
    int allow = PLAN_ALL;  // (unless the array does not hold what that needs)
    fle_status s = make_plan(&q, g_forced, g_split, &plan);
    if (s == FLE_OK && plan.ws_total > size_t(FLE_STATIC_SCRATCH_BYTES)) s = make_plan(&q, g_forced, g_split, &plan, nullptr, allow = PLAN_REFINE);
    if (s == FLE_OK && plan.ws_total > size_t(FLE_STATIC_SCRATCH_BYTES)) s = make_plan(&q, g_forced, g_split, &plan, nullptr, allow = 0);
    if (s == FLE_OK && plan.one_pass && plan.ws_total > size_t(FLE_STATIC_SCRATCH_BYTES)) s = make_plan(&q, g_forced, g_split, &plan, nullptr, allow = PLAN_REFINE | PLAN_SMALL);
    if (s != FLE_OK) return s;
    if (q.M == 0) return FLE_OK;
    if (plan.ws_total > size_t(FLE_STATIC_SCRATCH_BYTES))
        return fail(FLE_ERR_WORKSPACE, "this problem needs %zu bytes of scratch, the static array holds %zu: use fle_run with a workspace", plan.ws_total,
                    size_t(FLE_STATIC_SCRATCH_BYTES));
    if (plan.ws_total > 0) {
        void *ptr = nullptr;
        s = static_scratch(&ptr);
        if (s != FLE_OK) return s;
        q.workspace = ptr;
        q.workspace_bytes = size_t(FLE_STATIC_SCRATCH_BYTES);
        s = make_plan(&q, g_forced, g_split, &plan, nullptr, allow);  // again with the scratch in place: no operand may reach into it
        if (s == FLE_OK) s = check_workspace(&q, plan);
        if (s != FLE_OK) return s;
    }
    s = launch(&q, plan);
    if (s == FLE_OK) remember(plan);
    return s;
}

static fle_status check_groups(const fle_groups *g) { return g ? FLE_OK : fail(FLE_ERR_NULL, "groups is NULL"); }

fle_status fle_validate_grouped(const fle_problem *p, const fle_groups *g) {
    Plan plan;
    fle_status s = check_groups(g);
    return s != FLE_OK ? s : make_plan(p, g_forced, g_split, &plan, g);
}

fle_status fle_workspace_size_grouped(const fle_problem *p, const fle_groups *g, size_t *bytes_out) {
    if (!bytes_out) return fail(FLE_ERR_NULL, "bytes_out is NULL");
    Plan plan;
    fle_status s = check_groups(g);
    if (s == FLE_OK) s = make_plan(p, g_forced, g_split, &plan, g);
    if (s != FLE_OK) return s;
    *bytes_out = plan.ws_total;
    remember(plan);
    return FLE_OK;
}

fle_status fle_run_grouped(const fle_problem *p, const fle_groups *g) {
    Plan plan;
    fle_status s = check_groups(g);
    if (s == FLE_OK) s = make_plan(p, g_forced, g_split, &plan, g);
    if (s != FLE_OK) return s;
    if (p->M == 0) return FLE_OK;
    s = check_workspace(p, plan);
    if (s == FLE_OK) s = launch(p, plan, g);
    if (s == FLE_OK) remember(plan);
    return s;
}

fle_status fle_attention_validate(const fle_attention *p) { return check_attention(p); }

fle_status fle_attention_run(const fle_attention *p) {
    fle_status s = check_attention(p);
    if (s != FLE_OK || p->B == 0) return s;
    const AttnPlan plan = plan_attention(p, 1);
    s = launch_attention(p, plan, nullptr);
    if (s == FLE_OK) remember(plan);
    return s;
}

fle_status fle_attention_workspace_size(const fle_attention *p, size_t *bytes_out) {
    if (!bytes_out) return fail(FLE_ERR_NULL, "bytes_out is NULL");
    fle_status s = check_attention(p);
    if (s != FLE_OK) return s;
    const AttnPlan plan = plan_attention(p, 64);
    *bytes_out = plan.ws_bytes;
    remember(plan);
    return FLE_OK;
}

fle_status fle_attention_run_ws(const fle_attention *p, void *workspace, size_t workspace_bytes) {
    fle_status s = check_attention(p);
    if (s != FLE_OK || p->B == 0) return s;
    const AttnPlan plan = plan_attention(p, 64);
    if (plan.ws_bytes == 0) {
        s = launch_attention(p, plan, nullptr);
        if (s == FLE_OK) remember(plan);
        return s;
    }
    if (!workspace) return fail(FLE_ERR_WORKSPACE, "workspace is NULL but %zu bytes are needed", plan.ws_bytes);
    if (workspace_bytes < plan.ws_bytes) return fail(FLE_ERR_WORKSPACE, "workspace has %zu bytes, %zu needed", workspace_bytes, plan.ws_bytes);
    if (reinterpret_cast<uintptr_t>(workspace) % 256 != 0) return fail(FLE_ERR_ALIGN, "workspace must be 256-byte aligned");
    const int64_t HD = p->H * p->D, Tk = p->Tk > 0 ? p->Tk : p->T;
    const size_t eq = size_t(attention_extent(p->B, p->T, HD, p->ldq, p->sbq > 0 ? p->sbq : p->T * p->ldq)) * 2;
    const size_t ek = size_t(attention_extent(p->B, Tk, HD, p->ldk, p->sbk > 0 ? p->sbk : Tk * p->ldk)) * 2;
    const size_t ev = size_t(attention_extent(p->B, Tk, HD, p->ldv, p->sbv > 0 ? p->sbv : Tk * p->ldv)) * 2;
    const size_t eo = size_t(attention_extent(p->B, p->T, HD, p->ldo, p->sbo > 0 ? p->sbo : p->T * p->ldo)) * 2;
    if (overlaps(workspace, plan.ws_bytes, p->q, eq) || overlaps(workspace, plan.ws_bytes, p->k, ek) || overlaps(workspace, plan.ws_bytes, p->v, ev) ||
        overlaps(workspace, plan.ws_bytes, p->o, eo))
        return fail(FLE_ERR_UNSUPPORTED, "the workspace overlaps q, k, v or o");
    s = launch_attention(p, plan, workspace);
    if (s == FLE_OK) remember(plan);
    return s;
}

fle_status fle_attention_block_validate(const fle_attention_block *p) {
    BlockParts bp;
    if (!p) return fail(FLE_ERR_NULL, "attention block is NULL");
    fle_attention_block t = *p;
    t.workspace = nullptr;  // validation does not look at the workspace
    return plan_block(&t, &bp);
}

fle_status fle_attention_block_workspace_size(const fle_attention_block *p, size_t *bytes_out) {
    if (!bytes_out) return fail(FLE_ERR_NULL, "bytes_out is NULL");
    if (!p) return fail(FLE_ERR_NULL, "attention block is NULL");
    BlockParts bp;
    fle_attention_block t = *p;
    t.workspace = nullptr;
    fle_status s = plan_block(&t, &bp);
    if (s == FLE_OK) *bytes_out = bp.total;
    return s;
}

fle_status fle_attention_block_run(const fle_attention_block *p) {
    BlockParts bp;
    int allow = PLAN_REFINE;  // (unless the workspace is too small for what that needs)
    if (!p) return fail(FLE_ERR_NULL, "attention block is NULL");
    {
        fle_attention_block t = *p;
        t.workspace = nullptr;
        fle_status s = plan_block(&t, &bp);
        if (s == FLE_OK && p->workspace_bytes < bp.total) s = plan_block(&t, &bp, allow = 0);
        if (s != FLE_OK) return s;
    }
    if (p->B == 0) return FLE_OK;
    if (!p->workspace) return fail(FLE_ERR_WORKSPACE, "workspace is NULL but %zu bytes are needed", bp.total);
    if (p->workspace_bytes < bp.total) return fail(FLE_ERR_WORKSPACE, "workspace has %zu bytes, %zu needed", p->workspace_bytes, bp.total);
    if (reinterpret_cast<uintptr_t>(p->workspace) % 256 != 0) return fail(FLE_ERR_ALIGN, "workspace must be 256-byte aligned");
    fle_status s = plan_block(p, &bp, allow);
    if (s != FLE_OK) return s;
    s = check_workspace(&bp.proj, bp.proj_plan);
    if (s == FLE_OK) s = check_workspace(&bp.outp, bp.out_plan);
    if (s == FLE_OK) s = launch(&bp.proj, bp.proj_plan);
    if (s == FLE_OK) s = launch_attention(&bp.att, plan_attention(&bp.att, 1), nullptr);
    if (s == FLE_OK) s = launch(&bp.outp, bp.out_plan);
    if (s == FLE_OK) remember(bp.out_plan);
    return s;
}

fle_status fle_chain_validate(const fle_chain *p) {
    size_t act = 0;
    return check_chain(p, &act);
}

fle_status fle_chain_workspace_size(const fle_chain *p, size_t *bytes_out) {
    if (!bytes_out) return fail(FLE_ERR_NULL, "bytes_out is NULL");
    size_t act = 0;
    fle_status s = check_chain(p, &act);
    if (s == FLE_OK) *bytes_out = kChainSyncBytes + size_t(p->n_layers - 1) * act;
    return s;
}

fle_status fle_chain_run(const fle_chain *p) {
    size_t act = 0;
    fle_status s = check_chain(p, &act);
    if (s != FLE_OK) return s;
    char *ws = reinterpret_cast<char *>(p->workspace);
    const size_t need = kChainSyncBytes + size_t(p->n_layers - 1) * act;
    if (!ws) return fail(FLE_ERR_WORKSPACE, "workspace is NULL but %zu bytes are needed", need);
    if (p->workspace_bytes < need) return fail(FLE_ERR_WORKSPACE, "workspace has %zu bytes, %zu needed", p->workspace_bytes, need);
    if (reinterpret_cast<uintptr_t>(ws) % 256 != 0) return fail(FLE_ERR_ALIGN, "workspace must be 256-byte aligned");
    const size_t es = esize(p->dtype);
    if (overlaps(ws, need, p->x, size_t(p->layers[0].k) * es) || overlaps(ws, need, p->out, size_t(p->layers[p->n_layers - 1].n) * es))
        return fail(FLE_ERR_UNSUPPORTED, "the workspace overlaps x or out");
    ChainPlan plan;
    s = launch_chain(p, ws, ws + kChainSyncBytes, act, &plan);
    if (s == FLE_OK) remember(plan);
    return s;
}

const char *fle_status_string(fle_status s) {
    switch (s) {
    case FLE_OK: return "ok";
    case FLE_ERR_NULL: return "required pointer is NULL";
    case FLE_ERR_SHAPE: return "invalid shape or leading dimension";
    case FLE_ERR_ALIGN: return "misaligned pointer or leading dimension";
    case FLE_ERR_OP: return "invalid epilogue op";
    case FLE_ERR_UNSUPPORTED: return "unsupported combination";
    case FLE_ERR_WORKSPACE: return "workspace missing or too small";
    case FLE_ERR_HIP: return "HIP runtime error";
    }
    return "unknown status";
}

const char *fle_last_error(void) { return g_error; }

fle_status fle_last_plan(char *buf, size_t n) {
    if (!buf || n == 0) return fail(FLE_ERR_NULL, "buf is NULL or empty");
    switch (g_last) {
    case LAST_GEMM: format_plan(g_plan, buf, n); break;
    case LAST_ATTENTION: format_plan(g_attn_plan, buf, n); break;
    case LAST_CHAIN: format_plan(g_chain_plan, buf, n); break;
    case LAST_NONE: buf[0] = 0; break;
    }
    return FLE_OK;
}

void fle_force_variant(int variant) { g_forced = variant; }

void fle_force_split(int split) { g_split = split < 0 ? 0 : split; }

int fle_version(void) { return 1000; }  // 0.10.0: attention with a workspace (0.9.0: fp8 operands, two row reductions, per-call plan choice; 0.8.0: fle_run_static; 0.7.0: store op; 0.6.0: perceptron chain; 0.5.0: attention; 0.4.0: thin kernels; 0.3.0: grouped problems)

}  // extern "C"
