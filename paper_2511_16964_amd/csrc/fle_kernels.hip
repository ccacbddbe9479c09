// Device side of libfle: hand-written gfx950 (CDNA4) kernels and their launcher.
//
//   fle_gemm_tiled.h     gemm_tiled_256 / _128 (+ _grouped_) and gemm_deep_128 (more K steps in LDS): LDS-tiled MFMA GEMM (bf16, fp16, fp32) with the epilogue fused
//   fle_gemm_skinny.h    gemm_bf16_skinny: HBM-bound GEMM for few rows, W staged through LDS in long contiguous runs
//                        (row blocks of 32; bf16 / fp16 also 64 .. 256)
//   fle_gemm_thin.h      gemm_gemv (M <= 4 / 8, row-contiguous loads and dot products), gemm_thin (M <= 32, 16-row W tiles on
//                        the 16x16 MFMA): streams over W without LDS staging, every dtype
//   fle_attention.h      flash_attention: attention forward, 128 queries per workgroup; fle_attention_decode.h: a few queries
//                        per sequence against many keys (decode_attention, decode_combine)
//   fle_gemm_general.h   gemm_general: any shape / alignment / dtype, small tiles, in-block split of K
//   fle_rowops.h         finalize_rows / finalize_lse (second pass of a row reduction + trailing ops),
//                        reduce_slabs (ordered sum of split-K slabs + the ops before the row op)
//   fle_device_common.h  argument structs, dtype-aware loads / stores, elementwise ops, partial statistics
//
// Orientation used by every GEMM kernel: the W tile is MFMA operand A and the x tile is
// operand B, so the accumulator holds a tile of out^T.  In the MFMA result layout a lane owns
// one column and groups of four consecutive rows; with this orientation a lane therefore owns
// one output row m and groups of four consecutive n: stores, bias and residual accesses are
// 8-byte vectors, and a row reduction is in-register work plus one cross-lane exchange.
#include "fle_device_common.h"
#include "fle_gemm_general.h"
#include "fle_gemm_skinny.h"
#include "fle_gemm_thin.h"
#include "fle_attention.h"
#include "fle_attention_decode.h"
#include "fle_chain.h"
#include "fle_gemm_tiled.h"
#include "fle_rowops.h"

#include <atomic>

namespace fle {

// ------------------------------------------------------------------ static scratch (fle_run_static)
// Device memory for callers that cannot allocate: part of the code object, one copy per GPU.  In host code
// the array's name is only a handle for hipGetSymbolAddress; kernels and copies get the looked-up address.
static __device__ __align__(256) unsigned char scratch[FLE_STATIC_SCRATCH_BYTES];
static constexpr int kMaxDevices = 64;
static std::atomic<void *> g_scratch_ptr[kMaxDevices];

fle_status static_scratch(void **ptr) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return fail(FLE_ERR_HIP, "cannot query the current device");
    void *p = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!p) {  // once per device, with that device current (two threads racing here look up the same address)
        const hipError_t err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (err != hipSuccess || !p) return fail(FLE_ERR_HIP, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(err));
        g_scratch_ptr[dev].store(p, std::memory_order_release);
    }
    *ptr = p;
    return FLE_OK;
}

// ------------------------------------------------------------------ launcher
static fle_status check_launch(const char *what) {
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return fail(FLE_ERR_HIP, "%s: %s", what, hipGetErrorString(err));
    return FLE_OK;
}

fle_status launch(const fle_problem *p, const Plan &plan, const fle_groups *grp) {
    hipStream_t stream = reinterpret_cast<hipStream_t>(p->stream);
    const DevEpilogue &e = plan.epi;
    char *ws = reinterpret_cast<char *>(p->workspace);
    const bool bf16 = p->dtype != FLE_F32;  // 2-byte operands (bf16 or fp16)
    const size_t es = bf16 ? 2 : 4;

    GemmArgs g{};
    g.M = p->M; g.N = p->N; g.K = plan.k_run;
    g.x = p->x; g.ldx = p->ldx; g.w = p->w; g.ldw = p->ldw;
    g.np = plan.np;
    g.partials = e.row_kind >= 0 ? reinterpret_cast<float *>(ws + plan.ws_part_off) : nullptr;
    g.tiles_m = int32_t(plan.tiles_m); g.tiles_n = int32_t(plan.tiles_n);
    g.epi = e;
    g.x_scale = plan.x_scale;
    g.w_scale = plan.w_scale;
    if (plan.ln_pre == LN_PRE_FUSED) {
        g.ln_gamma = plan.ln_gamma; g.ln_beta = plan.ln_beta; g.ln_eps = plan.ln_eps;
    } else if (plan.ln_pre == LN_PRE_PASS) {
        // the normalised copy of x, rows contiguous, which the GEMM kernel then reads in place of x
        LnArgs l{};
        l.M = p->M; l.K = p->K; l.x = p->x; l.ldx = p->ldx; l.gamma = plan.ln_gamma; l.beta = plan.ln_beta; l.eps = plan.ln_eps;
        l.dtype = p->dtype; l.dst = ws + plan.ws_xhat_off; l.ldd = plan.k_run;
        if (p->M > 0 && p->K > 0) {
            // One wave per row, four rows per workgroup, where a wave holds the row in 2 vectors per lane (bf16 16384 x 256 with
            // its product 24.4 us) or in 8 and there are four rows for every CU (1273 x 3840: 24.5); else a workgroup per row, up to 16
            // vectors per lane (19 x 2091 18.2 us, 22.1 by one wave; 684 x 15040 fp16 41.7, 58.9 in three sweeps by one wave).
            const int64_t W = 16 / int64_t(es), vecs = (p->K + 64 * W - 1) / (64 * W);  // vectors per lane of a wave
            const bool by_element = p->K < W || vecs > 64, by_wave = !by_element && (vecs <= 2 || (vecs <= 8 && p->M >= 1024));
            auto pick = [&](auto dt_c, auto whole_c) -> void (*)(LnArgs) {
                constexpr int DT = decltype(dt_c)::value;
                constexpr bool WHOLE = decltype(whole_c)::value;
                if (by_element) return ln_prologue<DT>;
                if (by_wave) return vecs <= 2 ? ln_rows<DT, 1, 2, WHOLE> : vecs <= 4 ? ln_rows<DT, 1, 4, WHOLE> : ln_rows<DT, 1, 8, WHOLE>;
                return vecs <= 8 ? ln_rows<DT, 4, 2, WHOLE> : vecs <= 16 ? ln_rows<DT, 4, 4, WHOLE> : vecs <= 32 ? ln_rows<DT, 4, 8, WHOLE> : ln_rows<DT, 4, 16, WHOLE>;
            };
            auto pick_dt = [&](auto dt_c) { return p->K % W == 0 ? pick(dt_c, std::true_type{}) : pick(dt_c, std::false_type{}); };
            void (*lnk)(LnArgs) = p->dtype == FLE_F32 ? pick_dt(std::integral_constant<int, FLE_F32>{})
                                  : p->dtype == FLE_F16 ? pick_dt(std::integral_constant<int, FLE_F16>{}) : pick_dt(std::integral_constant<int, FLE_BF16>{});
            const int64_t wgs_ln = by_wave ? (p->M + 3) / 4 : p->M;
            hipLaunchKernelGGL(lnk, dim3(uint32_t(wgs_ln < 65536 ? wgs_ln : 65536)), dim3(256), 0, stream, l);
            const fle_status ls = check_launch("LayerNorm pass launch");
            if (ls != FLE_OK) return ls;
        }
        g.x = l.dst; g.ldx = plan.k_run;
    }
    if (plan.copy_x || plan.copy_w) {
        CopyArgs c{};
        auto part = [&](CopyArgs::Part &t, const void *src, int64_t rows, int64_t lds, size_t off) {
            t.src = src; t.dst = ws + off; t.rows = rows; t.K = p->K; t.lds = lds; t.ldd = plan.k_run;
            t.blocks = (rows * (plan.k_run * int64_t(es) / 16) + 256 * kCopyVecs - 1) / (256 * kCopyVecs);
        };
        if (plan.copy_x) part(c.part[0], p->x, p->M, p->ldx, plan.ws_xc_off);
        if (plan.copy_w) part(c.part[1], p->w, p->N, p->ldw, plan.ws_wc_off);
        const int64_t blocks = c.part[0].blocks + c.part[1].blocks;
        void (*ck)(CopyArgs) = es == 4 ? copy_rows<4> : copy_rows<2>;
        hipLaunchKernelGGL(ck, dim3(uint32_t(blocks)), dim3(256), 0, stream, c);
        const fle_status cs = check_launch("operand copy launch");
        if (cs != FLE_OK) return cs;
        if (plan.copy_x) { g.x = c.part[0].dst; g.ldx = plan.k_run; }
        if (plan.copy_w) { g.w = c.part[1].dst; g.ldw = plan.k_run; }
    }
    if (e.row_kind < 0 || plan.staging == ST_OUT) { g.dst = p->out; g.ldd = p->ldo; g.dst_f32 = 0; g.dst_rel = plan.stage_rel; }
    else if (plan.staging == ST_WS) { g.dst = ws + plan.ws_y_off; g.ldd = p->N; g.dst_f32 = 1; }
    else { g.dst = nullptr; g.ldd = 0; g.dst_f32 = 0; }

    // Split K: the GEMM writes bare fp32 slabs; reduce_slabs takes over dst, the pre-ops and the partials.
    RedArgs r{};
    const bool split = plan.split_k > 1;
    if (split) {
        r.M = p->M; r.N = p->N;
        r.slabs = reinterpret_cast<const float *>(ws + plan.ws_slab_off);
        r.ld_slab = (p->N + 3) / 4 * 4;
        r.stride = p->M * r.ld_slab;
        r.S = plan.split_k;
        r.dst = g.dst; r.ldd = g.ldd; r.dst_f32 = g.dst_f32; r.dst_rel = g.dst_rel;
        r.np = plan.np; r.partials = g.partials;
        r.epi = e;
        g.dst = ws + plan.ws_slab_off; g.ldd = r.ld_slab; g.dst_f32 = 1; g.dst_rel = 0;
        g.split_stride = r.stride * int64_t(sizeof(float));
        g.partials = nullptr;
        g.epi.n_pre = 0; g.epi.row_kind = -1;
    }
    // skinny kernel: W tiles in groups of 8 (one per XCD), each with all its row blocks
    const int64_t wgs = plan.variant == V_SKINNY ? (plan.tiles_n + 7) / 8 * 8 * plan.tiles_m : plan.tiles_m * plan.tiles_n;
    const dim3 grid{uint32_t(wgs), uint32_t(plan.split_k)};
    if (plan.variant == V_SKINNY) {
        auto pick = [&](auto dt_c) -> void (*)(GemmArgs) {
            constexpr int DT = decltype(dt_c)::value;
            if (plan.bm == 32) return plan.bk == 256 ? gemm_bf16_skinny<1, 256, DT> : plan.bk == 128 ? gemm_bf16_skinny<1, 128, DT> : gemm_bf16_skinny<1, 64, DT>;
            // larger row blocks: 32-row sub-blocks in turn on a 256-wide K step, or (64 rows) both at once on a 128-wide one
            if (plan.bk == 128) return gemm_bf16_skinny<2, 128, DT>;
            return plan.bm == 64 ? gemm_bf16_skinny<2, 256, DT, true> : plan.bm == 128 ? gemm_bf16_skinny<4, 256, DT, true> : gemm_bf16_skinny<8, 256, DT, true>;
        };
        void (*kern)(GemmArgs);
        if (p->dtype == FLE_F32)  // row blocks of 32 only; the K step is half as many elements for the same bytes
            kern = plan.bk == 128 ? gemm_bf16_skinny<1, 128, FLE_F32> : plan.bk == 64 ? gemm_bf16_skinny<1, 64, FLE_F32> : gemm_bf16_skinny<1, 32, FLE_F32>;
        else
            kern = p->dtype == FLE_F16 ? pick(std::integral_constant<int, FLE_F16>{}) : pick(std::integral_constant<int, FLE_BF16>{});
        hipLaunchKernelGGL(kern, grid, dim3(256), 0, stream, g);
    } else if (plan.variant == V_THIN) {
        // dot-product form: 4 rows of W per wave, or (one row of x, many rows of W) one per wave and 16 waves
        const bool wide = plan.bm <= 8 && plan.bk == 1;  // (the plan's K step field carries the rows per wave for this form)
        auto pick = [&](auto dt_c) -> void (*)(GemmArgs) {
            constexpr int DT = decltype(dt_c)::value;
            if (plan.bm <= 8) {  // (the planner gives 5 .. 8 rows to this form for fp32 only)
                if (plan.ln_pre == LN_PRE_FUSED) {  // (the planner fuses up to 4 rows)
                    // up to 2 rows that fit: x normalised once per workgroup (bf16, new operands: 1 x 16384 x 4096 46 -> 35 us, 1 x
                    // 5120 x 13824 58 -> 37, 2 x 2048 x 8192 16.6 -> 15.4; 3 x 2048 x 2048 10.2 -> 11.1, so not more rows)
                    if (p->M <= 2 && p->M * p->K <= kNormDotX && p->K <= (wide ? kNormDotK<DT, 1> : kNormDotK<DT, 4>)) {
                        if (wide) return norm_dot<DT, 1, 1>;
                        return p->M <= 1 ? norm_dot<DT, 1, 4> : norm_dot<DT, 2, 4>;
                    }
                    if (wide) return gemm_gemv<DT, 1, 1, true>;
                    return p->M <= 1 ? gemm_gemv<DT, 1, 4, true> : p->M <= 2 ? gemm_gemv<DT, 2, 4, true> : gemm_gemv<DT, 4, 4, true>;
                }
                if constexpr (DT == FLE_F32)
                    if (p->M > 4) return gemm_gemv<DT, 8, 4>;
                if (wide) return gemm_gemv<DT, 1, 1>;
                return p->M <= 1 ? gemm_gemv<DT, 1, 4> : p->M <= 2 ? gemm_gemv<DT, 2, 4> : gemm_gemv<DT, 4, 4>;
            }
            return plan.bm == 16 ? gemm_thin<DT, 1> : gemm_thin<DT, 2>;
        };
        void (*kern)(GemmArgs) = p->dtype == FLE_F32 ? pick(std::integral_constant<int, FLE_F32>{})
                                 : p->dtype == FLE_F16 ? pick(std::integral_constant<int, FLE_F16>{}) : pick(std::integral_constant<int, FLE_BF16>{});
        const uint32_t threads = wide ? 1024u : 256u;
        hipLaunchKernelGGL(kern, dim3(uint32_t(plan.tiles_n)), dim3(threads), 0, stream, g);
    } else if (plan.variant == V_TILED && grp) {
        const bool edge = plan.edge != 0;
        const int64_t xs = plan.op_dtype == FLE_F8E4M3 ? 1 : int64_t(es);  // bytes per element of W
        GroupArgs ga{grp->row_offsets, grp->n_groups, grp->w_group_stride * xs, grp->b_group_stride * int64_t(es)};
        auto pick = [&](auto dt_c) -> void (*)(GemmArgs, GroupArgs) {
            constexpr int DT = decltype(dt_c)::value;
            if constexpr (DT != FLE_F32) {
                if (plan.deep) return edge ? gemm_deep_grouped_128<DT, true> : gemm_deep_grouped_128<DT, false>;
            }
            if (plan.bm == 256) return edge ? gemm_tiled_grouped_256<DT, true> : gemm_tiled_grouped_256<DT, false>;
            if (plan.w_stream) return edge ? gemm_tiled_grouped_128<DT, true, true> : gemm_tiled_grouped_128<DT, false, true>;
            return edge ? gemm_tiled_grouped_128<DT, true, false> : gemm_tiled_grouped_128<DT, false, false>;
        };
        void (*kern)(GemmArgs, GroupArgs) = p->dtype == FLE_F32 ? pick(std::integral_constant<int, FLE_F32>{})
                                            : p->dtype == FLE_F16 ? pick(std::integral_constant<int, FLE_F16>{})
                                            : p->dtype == FLE_F8E4M3 ? pick(std::integral_constant<int, FLE_F8E4M3>{}) : pick(std::integral_constant<int, FLE_BF16>{});
        hipLaunchKernelGGL(kern, grid, dim3(256), 0, stream, g, ga);
    } else if (plan.variant == V_TILED) {
        // split K writes fp32 slabs with a padded leading dimension: vector stores whatever out looks like
        const bool edge = plan.edge && !split;
        void (*kern)(GemmArgs);
        auto pick = [&](auto dt_c) -> void (*)(GemmArgs) {
            constexpr int DT = decltype(dt_c)::value;
            if constexpr (DT != FLE_F32) {
                if (plan.deep) return edge ? gemm_deep_128<DT, true> : gemm_deep_128<DT, false>;
            }
            if constexpr (DT == FLE_BF16 || DT == FLE_F16) {
                if (plan.bm == 160) return edge ? gemm_rows_256<DT, true, 160> : gemm_rows_256<DT, false, 160>;
                if (plan.bm == 192) return edge ? gemm_rows_256<DT, true, 192> : gemm_rows_256<DT, false, 192>;
                if (plan.bm == 224) return edge ? gemm_rows_256<DT, true, 224> : gemm_rows_256<DT, false, 224>;
            }
            if (plan.bm == 256) return edge ? gemm_tiled_256<DT, true> : gemm_tiled_256<DT, false>;
            return edge ? gemm_tiled_128<DT, true> : gemm_tiled_128<DT, false>;
        };
        if (p->dtype == FLE_F32) kern = pick(std::integral_constant<int, FLE_F32>{});
        else if (p->dtype == FLE_F16) kern = pick(std::integral_constant<int, FLE_F16>{});
        else if (p->dtype == FLE_F8E4M3 && plan.mx && plan.deep)
            kern = edge ? gemm_deep_128<FLE_F8E4M3, true, true> : gemm_deep_128<FLE_F8E4M3, false, true>;
        else if (p->dtype == FLE_F8E4M3 && plan.mx)
            kern = plan.bm == 256 ? (edge ? gemm_tiled_256<FLE_F8E4M3, true, 32, -1, true> : gemm_tiled_256<FLE_F8E4M3, false, 32, -1, true>)
                                  : (edge ? gemm_tiled_128<FLE_F8E4M3, true, 32, -1, true> : gemm_tiled_128<FLE_F8E4M3, false, 32, -1, true>);
        else if (p->dtype == FLE_F8E4M3) kern = pick(std::integral_constant<int, FLE_F8E4M3>{});
        else kern = pick(std::integral_constant<int, FLE_BF16>{});
        hipLaunchKernelGGL(kern, grid, dim3(256), 0, stream, g);
    } else {
        // vector loads need 4-element groups that never straddle K and rows that keep the alignment
        const size_t va = bf16 ? 8 : 16;
        const bool vec = g.K % 4 == 0 && reinterpret_cast<uintptr_t>(g.x) % va == 0 && reinterpret_cast<uintptr_t>(g.w) % va == 0 &&
                         g.ldx % 4 == 0 && g.ldw % 4 == 0;
        auto pick = [&](auto dt_c) -> void (*)(GemmArgs) {
            constexpr int DT = decltype(dt_c)::value;
            if (plan.bm == 32) return vec ? gemm_general<DT, true, 2> : gemm_general<DT, false, 2>;
            return vec ? gemm_general<DT, true, 1> : gemm_general<DT, false, 1>;
        };
        void (*kern)(GemmArgs) = p->dtype == FLE_F32 ? pick(std::integral_constant<int, FLE_F32>{})
                                 : p->dtype == FLE_F16 ? pick(std::integral_constant<int, FLE_F16>{}) : pick(std::integral_constant<int, FLE_BF16>{});
        hipLaunchKernelGGL(kern, grid, dim3(256), 0, stream, g);
    }
    fle_status s = check_launch("GEMM kernel launch");
    if (s == FLE_OK && plan.one_pass) {  // the sum of the slabs, the row reduction and what follows it at once
        auto pick = [&](auto dt_c) -> void (*)(RedArgs, PostEpilogue, void *, int64_t) {
            constexpr int DT = decltype(dt_c)::value;
            return p->N <= 1024 ? reduce_rows<DT, 4, 1> : p->N <= 2048 ? reduce_rows<DT, 4, 2> : reduce_rows<DT, 16, 2>;
        };
        void (*rk)(RedArgs, PostEpilogue, void *, int64_t) = e.dtype == FLE_F32 ? pick(std::integral_constant<int, FLE_F32>{})
                                                             : e.dtype == FLE_F16 ? pick(std::integral_constant<int, FLE_F16>{}) : pick(std::integral_constant<int, FLE_BF16>{});
        const int64_t waves = p->N <= 1024 ? 4 : (p->N + 511) / 512;
        hipLaunchKernelGGL(rk, dim3(uint32_t(p->M)), dim3(uint32_t(waves) * 64), 0, stream, r, PostEpilogue(e, false), p->out, p->ldo);
        return check_launch("split-K and row reduction launch");
    }
    if (s == FLE_OK && split) {
        const int64_t want = (p->M * ((p->N + 255) / 256) + 3) / 4;
        hipLaunchKernelGGL(reduce_slabs, dim3(uint32_t(want < (int64_t(1) << 20) ? want : (int64_t(1) << 20))), dim3(256), 0, stream, r);
        s = check_launch("split-K reduction launch");
    }
    if (s != FLE_OK || e.row_kind < 0) return s;

    FinArgs f{};
    f.M = p->M; f.N = p->N;
    f.np = plan.np; f.part_cols = plan.part_cols;
    f.part_shift = 0;
    while ((1 << f.part_shift) < plan.part_cols) ++f.part_shift;
    if ((1 << f.part_shift) != plan.part_cols) return fail(FLE_ERR_UNSUPPORTED, "internal: partial width %d is not a power of two", plan.part_cols);
    f.partials = split ? r.partials : g.partials;
    f.out = p->out; f.ldo = p->ldo;
    f.epi = PostEpilogue(e, false);
    if (grp && grp->b_group_stride != 0) {  // a bias op after the row op needs the row's group
        for (int o = 0; o < e.n_post; ++o)
            if (e.post[o].kind == FLE_BIAS) {
                f.row_offsets = grp->row_offsets;
                f.n_groups = grp->n_groups;
                f.b_stride_bytes = grp->b_group_stride * int64_t(es);
            }
    }
    if (e.row_kind == FLE_LOGSUMEXP) {
        hipLaunchKernelGGL(finalize_lse, dim3(uint32_t((p->M + 3) / 4)), dim3(256), 0, stream, f);
        return check_launch("logsumexp finalize launch");
    }
    const bool two = e.row2_kind >= 0;  // a second row reduction: this pass hands its values over in fp32
    if (two) { f.out = ws + plan.ws_mid_off; f.ldo = p->N; f.out_f32 = 1; }
    if (split) { f.y = r.dst; f.ldy = r.ldd; f.y_f32 = r.dst_f32; }
    else { f.y = g.dst; f.ldy = g.ldd; f.y_f32 = g.dst_f32; }
    f.y_rel = plan.stage_rel;
    const size_t ysz = f.y_f32 ? 4 : es;
    const bool vec = p->N % 8 == 0 && f.ldy % 8 == 0 && f.ldo % 8 == 0 && reinterpret_cast<uintptr_t>(f.y) % (8 * ysz) == 0 &&
                     reinterpret_cast<uintptr_t>(f.out) % (8 * (two ? 4 : es)) == 0;
    // vector path also needs 16-byte aligned gamma / beta
    const bool gb_ok = reinterpret_cast<uintptr_t>(e.row.p0) % (8 * es) == 0 && reinterpret_cast<uintptr_t>(e.row.p1) % (8 * es) == 0;
    const int64_t items = p->M * ((p->N + 2047) / 2048);
    const int64_t want = (items + 3) / 4;
    const dim3 fgrid(uint32_t(want < (int64_t(1) << 20) ? want : (int64_t(1) << 20)));
    void (*fin)(FinArgs);
    const int fdt = e.dtype;
    auto pick_fin = [&](auto ln_c) -> void (*)(FinArgs) {
        constexpr bool LN = decltype(ln_c)::value;
        auto pick_dt = [&](auto dt_c) -> void (*)(FinArgs) {
            constexpr int DT = decltype(dt_c)::value;
            // (softmax of a few rows: the call is 0.2 us faster on the long form, 100 x 600 x 512 10.6 and 10.8 us; 5000 x 768 x 704 24.2 and 23.4)
            const int64_t n = LN || p->M >= 1024 ? p->N : 2048;
            if (vec && gb_ok) return n <= 512 ? finalize_short<true, LN, DT, 1> : n <= 1024 ? finalize_short<true, LN, DT, 2> : finalize_rows<true, LN, DT>;
            return n <= 512 ? finalize_short<false, LN, DT, 1> : n <= 1024 ? finalize_short<false, LN, DT, 2> : finalize_rows<false, LN, DT>;
        };
        return fdt == FLE_BF16 ? pick_dt(std::integral_constant<int, FLE_BF16>{}) : fdt == FLE_F16 ? pick_dt(std::integral_constant<int, FLE_F16>{}) : pick_dt(std::integral_constant<int, FLE_F32>{});
    };
    fin = e.row_kind == FLE_LAYERNORM ? pick_fin(std::true_type{}) : pick_fin(std::false_type{});
    hipLaunchKernelGGL(fin, fgrid, dim3(256), 0, stream, f);
    s = check_launch("row finalize launch");
    if (s != FLE_OK || !two) return s;
    Row2Args r2{};
    r2.M = p->M; r2.N = p->N;
    r2.v = reinterpret_cast<const float *>(ws + plan.ws_mid_off);
    r2.out = p->out; r2.ldo = p->ldo;
    r2.epi = PostEpilogue(e, true);
    hipLaunchKernelGGL(second_row_op, dim3(uint32_t(p->M < (int64_t(1) << 16) ? p->M : (int64_t(1) << 16))), dim3(256), 0, stream, r2);
    return check_launch("second row reduction launch");
}

template <int DT, int D>
static void launch_attention_dt(const fle_attention *p, const AttnArgs &a, const AttnPlan &plan, void *ws, hipStream_t stream) {
    if (plan.splits > 0) {
        DecodeArgs d;
        d.at = a;
        d.splits = plan.splits;
        d.n_blocks = (a.Tk + kDecodeKeys - 1) / kDecodeKeys;
        const int64_t rows = p->B * p->T * p->H;
        d.part = reinterpret_cast<float *>(ws);
        d.stat = ws ? d.part + int64_t(plan.splits) * rows * D : nullptr;
        hipLaunchKernelGGL((decode_attention<DT, D>), dim3(uint32_t(p->B * p->H * plan.splits)), dim3(64 * decode_waves(D)), 0, stream, d);
        if (plan.splits > 1) hipLaunchKernelGGL((decode_combine<DT, D>), dim3(uint32_t((rows + 3) / 4)), dim3(256), 0, stream, d);
        return;
    }
    // One query tile per wave, 128 queries per workgroup: one (D = 256), two (D = 128) or three (D <= 64) waves per SIMD.
    hipLaunchKernelGGL((flash_attention<DT, D, D == 256 ? 1 : D == 128 ? 2 : 3>), dim3(uint32_t((p->T + 127) / 128 * p->H * p->B)), dim3(256), 0, stream, a);
}

fle_status launch_attention(const fle_attention *p, const AttnPlan &plan, void *ws) {
    hipStream_t stream = reinterpret_cast<hipStream_t>(p->stream);
    AttnArgs a;
    a.q = p->q; a.k = p->k; a.v = p->v; a.o = p->o;
    a.ldq = p->ldq; a.ldk = p->ldk; a.ldv = p->ldv; a.ldo = p->ldo;
    const int64_t Tk = p->Tk > 0 ? p->Tk : p->T;
    a.sbq = p->sbq > 0 ? p->sbq : p->T * p->ldq; a.sbo = p->sbo > 0 ? p->sbo : p->T * p->ldo;
    a.sbk = p->sbk > 0 ? p->sbk : Tk * p->ldk; a.sbv = p->sbv > 0 ? p->sbv : Tk * p->ldv;
    a.T = int32_t(p->T); a.Tk = int32_t(Tk); a.H = int32_t(p->H); a.B = int32_t(p->B); a.causal = p->causal;
    const float scale = p->scale > 0.0f ? p->scale : 1.0f / sqrtf(float(p->D));
    a.scale_log2e = scale * 1.44269504088896340736f;
    const bool f16 = p->dtype == FLE_F16;
    switch (p->D) {
    case 32: f16 ? launch_attention_dt<FLE_F16, 32>(p, a, plan, ws, stream) : launch_attention_dt<FLE_BF16, 32>(p, a, plan, ws, stream); break;
    case 64: f16 ? launch_attention_dt<FLE_F16, 64>(p, a, plan, ws, stream) : launch_attention_dt<FLE_BF16, 64>(p, a, plan, ws, stream); break;
    case 128: f16 ? launch_attention_dt<FLE_F16, 128>(p, a, plan, ws, stream) : launch_attention_dt<FLE_BF16, 128>(p, a, plan, ws, stream); break;
    default: f16 ? launch_attention_dt<FLE_F16, 256>(p, a, plan, ws, stream) : launch_attention_dt<FLE_BF16, 256>(p, a, plan, ws, stream); break;
    }
    return check_launch("attention launch");
}

fle_status launch_chain(const fle_chain *p, void *sync, void *acts, size_t act_stride, ChainPlan *plan) {
    hipStream_t stream = reinterpret_cast<hipStream_t>(p->stream);
    ChainArgs a;
    a.n_layers = p->n_layers;
    a.x = p->x; a.out = p->out; a.sync = reinterpret_cast<uint32_t *>(sync);
    for (int l = 0; l < kChainMaxLayers; ++l) a.act[l] = acts ? reinterpret_cast<char *>(acts) + size_t(l) * act_stride : nullptr;
    int64_t widest = 0, longest = 0, slots8 = 0, slots16 = 0;  // (KB that the weight rows take in rings of 8 and of 16 KB)
    const int64_t ws = p->w_dtype == FLE_F32 ? 4 : 2;
    for (int l = 0; l < p->n_layers; ++l) {
        if (p->layers[l].k > longest) longest = p->layers[l].k;
        slots8 += p->layers[l].n * ((p->layers[l].k * ws + 8191) / 8192 * 8);
        slots16 += p->layers[l].n * ((p->layers[l].k * ws + 16383) / 16384 * 16);
        a.layer[l].w = p->layers[l].w; a.layer[l].bias = p->layers[l].b;
        a.layer[l].n = int32_t(p->layers[l].n); a.layer[l].k = int32_t(p->layers[l].k); a.layer[l].act = p->layers[l].act;
        if (p->layers[l].n > widest) widest = p->layers[l].n;
    }
    // at most one workgroup of 16 waves per CU, so that every workgroup is resident while the others wait at a barrier;
    // fewer when no layer has 16 rows for each
    static thread_local int cu_count[64] = {0};  // per device: CUs (queried once per thread and device)
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return fail(FLE_ERR_HIP, "cannot query the current device");
    if (cu_count[dev] == 0 && (hipDeviceGetAttribute(&cu_count[dev], hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cu_count[dev] < 1)) {
        cu_count[dev] = 0;
        return fail(FLE_ERR_HIP, "cannot query the device's CU count");
    }
    const int cus = cu_count[dev];
    const int64_t want = (widest + 15) / 16;
    const uint32_t grid = uint32_t(want < cus ? want : cus);
    // inputs that fit LDS as fp32: the form with x there and 8 or 16 KB of weights per wave in flight (eight layers of
    // 4096 x 4096 fp32 132 -> 107 us, bf16 weights under fp32 85 -> 68); longer ones: x from the cache, 4 KB.  So do chains of
    // fewer than 16 workgroups, whose few rows gain nothing from more weights in flight: eight layers of 128 33.9 us from the
    // cache and 30.8 from LDS in fp32, 35.4 and 35.7 in bf16; two of 64 7.6 and 8.0, 7.8 and 9.2.  From 16 on a workgroup's
    // activations of a layer fit its kChainLdsGroups rows.
    // Few layers with rows of up to 4 KB have no stream for it to keep up and pay for bringing x into LDS: from the cache and
    // from LDS, one layer of 256 and of 2048 bf16 4.0 and 5.1, 4.8 and 5.8, of 1024 fp32 4.9 and 5.3, but of 1536 6.3 and 5.7; two
    // of 1024 bf16 9.5 and 10.6, three 14.8 and 15.6, six 28.6 each; two of 512 fp32 9.1 and 9.0, two of 3072 bf16 14.3 and 13.4.
    // Nor has a single layer of a 2-byte dtype with at most one row per wave anything to request ahead: from the cache and from LDS, on new
    // weights each time, bf16 3752 x 3752 8.0 and 8.3, 3736 x 7472 12.3 and 13.3, fp16 3024 x 6048 9.7 and 10.3, but 3032 x 3032
    // 7.3 and 7.1; with more rows fp16 4576 x 9152 23.7 and 20.3; fp32 2504 x 2504 8.9 and 8.7, with bf16 weights 3504 x 3504 8.8 and 7.8.
    const bool one_row = p->n_layers == 1 && p->dtype != FLE_F32 && widest <= int64_t(grid) * 16;
    const bool in_lds = longest <= kChainLdsK && kChainLdsK <= int64_t(grid) * 16 * kChainLdsGroups &&  // (every n but the last is a k)
                        !(longest * ws <= 4096 && p->n_layers <= (p->dtype == FLE_F32 ? 1 : 3)) && !one_row;
    *plan = ChainPlan{p->dtype, p->w_dtype, p->n_layers, 0, int32_t(grid)};
    auto pick = [&](auto dt_c, auto dw_c) -> void (*)(ChainArgs) {
        constexpr int DT = decltype(dt_c)::value, DW = decltype(dw_c)::value;
        if (!in_lds) return mlp_chain<DT, DW>;
        // 16 KB per wave where that leaves no more of the ring empty at the ends of rows than 8 KB do.  With 8 and with 16: rows
        // of 16 KB (4096 fp32) 112 and 106 us, of 32 (8192) 382 and 366, of 27 (7000) 132 and 130, but of 19 (4800)
        // 165 and 175, of 4 and 16 KB in turn (2048 and 8192 bf16) 71 and 76, of 2 and 9 (1024 and 4608) 53 and 63
        plan->ahead_kb = slots16 <= slots8 ? 16 : 8;
        return plan->ahead_kb == 16 ? perceptron_lds<DT, DW, 16> : perceptron_lds<DT, DW, 8>;
    };
    using F32 = std::integral_constant<int, FLE_F32>;
    using BF16 = std::integral_constant<int, FLE_BF16>;
    using F16 = std::integral_constant<int, FLE_F16>;
    void (*kern)(ChainArgs) = p->dtype == FLE_F16 ? pick(F16{}, F16{}) : p->dtype == FLE_BF16 ? pick(BF16{}, BF16{})
                              : p->w_dtype == FLE_BF16 ? pick(F32{}, BF16{}) : p->w_dtype == FLE_F16 ? pick(F32{}, F16{}) : pick(F32{}, F32{});
    hipLaunchKernelGGL(kern, dim3(grid), dim3(1024), 0, stream, a);
    return check_launch("mlp_chain");
}

}  // namespace fle
