// Device-side types and helpers shared by every libfle kernel: vector types, kernel argument structs,
// dtype-aware loads and stores, the elementwise ops, and the row-reduction partials.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "fle_plan.h"

namespace fle {


typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(4))) _Float16 f16x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((address_space(3))) void lds_void;

// A vector at an address that is only aligned to ALIGN: global memory takes the access at any element address, the
// compiler has to be told.
template <typename V, int ALIGN>
struct __attribute__((packed, aligned(ALIGN))) AnyAligned {
    V v;
};

// The parts of the op list that each kind of kernel reads.  (A launch copies its arguments: 16 bytes of them take 2.8 us of the
// caller's thread, 256 3.5, 1400 4.3; the whole list in every kernel's arguments made that 1.1 KB.)
struct PreEpilogue {  // up to the (first) row op
    int32_t n_pre, row_kind, dtype;
    const void *bias;
    DevOp pre[FLE_MAX_OPS];
    PreEpilogue() = default;
    PreEpilogue(const DevEpilogue &e) : n_pre(e.n_pre), row_kind(e.row_kind), dtype(e.dtype), bias(e.bias) {
        for (int i = 0; i < FLE_MAX_OPS; ++i) pre[i] = e.pre[i];
    }
};
struct PostEpilogue {  // a row op and what follows it, up to the next
    int32_t n_post, row_kind, dtype;
    const void *bias;
    DevOp row;
    DevOp post[FLE_MAX_OPS];
    PostEpilogue() = default;
    PostEpilogue(const DevEpilogue &e, bool second)
        : n_post(second ? e.n_post2 : e.n_post), row_kind(second ? e.row2_kind : e.row_kind), dtype(e.dtype), bias(e.bias), row(second ? e.row2 : e.row) {
        for (int i = 0; i < FLE_MAX_OPS; ++i) post[i] = second ? e.post2[i] : e.post[i];
    }
};

struct GemmArgs {
    int64_t M, N, K;
    const void *x;
    int64_t ldx;
    const void *w;
    int64_t ldw;
    void *dst;  // where the values after the pre-ops go (nullptr: nowhere, logsumexp)
    int64_t ldd;
    int32_t dst_f32;  // dst holds fp32 regardless of the storage dtype (workspace staging)
    int32_t dst_rel;  // row op staged in a 2-byte dtype: store v - (mean / maximum of v's partial); the finalize pass adds it back in fp32
    int32_t np;       // row-reduction partials per row
    float *partials;  // [M][np][2], or nullptr without a row op
    int32_t tiles_m, tiles_n;
    int64_t split_stride;  // split K (gridDim.y > 1): workgroup row y owns a K range and writes dst + y * split_stride bytes
    const void *x_scale, *w_scale;  // block-scaled fp8 operands: one E8M0 byte per 32 consecutive k, [M][K/32] and [N][K/32]
    const void *ln_gamma, *ln_beta;  // LayerNorm of x over K in front of the multiplication, done by the kernel itself
    float ln_eps;                    // (dot-product kernel for a few rows of x only); gamma / beta [K] or nullptr
    PreEpilogue epi;
};

// LayerNorm of the rows of x over K, written to a contiguous copy (the pass in front of the GEMM kernels).
struct LnArgs {
    int64_t M, K;
    const void *x;
    int64_t ldx;
    const void *gamma, *beta;  // [K] or nullptr
    float eps;
    int32_t dtype;
    void *dst;                 // [M][ldd], the columns from K on zero
    int64_t ldd;
};

// Up to two matrices copied to rows of ldd elements, zeros behind their K (copy_rows).
struct CopyArgs {
    struct Part {
        const void *src;
        void *dst;             // 16-byte aligned, ldd * element size a multiple of 16
        int64_t rows, K, lds, ldd;
        int64_t blocks;        // workgroups of this part
    } part[2];
};

// Sum of the split-K slabs followed by the ops before the row op (reduce_slabs).
struct RedArgs {
    int64_t M, N;
    const float *slabs;  // [S][M][N] fp32
    int64_t stride;      // elements between slabs
    int64_t ld_slab;     // elements between slab rows (N rounded up to a multiple of 4)
    int32_t S;
    int32_t dst_f32;
    int32_t dst_rel;     // as GemmArgs::dst_rel
    void *dst;           // as GemmArgs::dst
    int64_t ldd;
    int32_t np;
    float *partials;     // one partial per (row, 256 columns)
    PreEpilogue epi;
};

struct FinArgs {
    int64_t M, N;
    const void *y;  // staged values: storage dtype (may alias out) or fp32
    int64_t ldy;
    int32_t y_f32;
    int32_t y_rel;  // staged values are relative to the mean / maximum of their partial (2-byte dtypes)
    int32_t np, part_cols;
    int32_t part_shift;  // log2(part_cols): the planner only uses powers of two
    const float *partials;
    void *out;
    int64_t ldo;
    int32_t out_f32;  // out holds fp32 regardless of the storage dtype (the values handed to a second row reduction)
    // grouped problems whose list has a bias op after the row op: the row's group selects the bias
    const int64_t *row_offsets;  // [n_groups + 1] (device), or nullptr
    int32_t n_groups;
    int64_t b_stride_bytes;
    PostEpilogue epi;
};

// Second row reduction of a list (second_row_op): v[M,N] fp32 in, out in the storage dtype.
struct Row2Args {
    int64_t M, N;
    const float *v;  // [M][N] fp32, packed rows
    void *out;       // [M][ldo], or [M] for logsumexp
    int64_t ldo;
    PostEpilogue epi;
};

// ------------------------------------------------------------------ scalar helpers
__device__ __forceinline__ float bf16_bits_to_f32(uint32_t h) { return __uint_as_float(h << 16); }

__device__ __forceinline__ float ld_elem(const void *p, int64_t i, int dtype) {
    if (dtype == FLE_BF16) return bf16_bits_to_f32(reinterpret_cast<const uint16_t *>(p)[i]);
    if (dtype == FLE_F16) return float(reinterpret_cast<const _Float16 *>(p)[i]);
    return reinterpret_cast<const float *>(p)[i];
}

__device__ __forceinline__ void st_elem(void *p, int64_t i, int dtype, float v) {
    if (dtype == FLE_BF16)
        reinterpret_cast<__bf16 *>(p)[i] = static_cast<__bf16>(v);
    else if (dtype == FLE_F16)
        reinterpret_cast<_Float16 *>(p)[i] = static_cast<_Float16>(v);
    else
        reinterpret_cast<float *>(p)[i] = v;
}

__device__ __forceinline__ f32x4 ld4_bf16(const void *p) {  // p is 8-byte aligned
    const uint2 u = *reinterpret_cast<const uint2 *>(p);
    f32x4 r;
    r[0] = __uint_as_float(u.x << 16);
    r[1] = __uint_as_float(u.x & 0xffff0000u);
    r[2] = __uint_as_float(u.y << 16);
    r[3] = __uint_as_float(u.y & 0xffff0000u);
    return r;
}

// 4 consecutive elements at element index i of p as fp32 (p + i aligned to 4 elements).  DT: fle_dtype.
template <int DT>
__device__ __forceinline__ f32x4 ld4(const void *p, int64_t i) {
    if constexpr (DT == FLE_F32) return *reinterpret_cast<const f32x4 *>(reinterpret_cast<const float *>(p) + i);
    else if constexpr (DT == FLE_F16) return __builtin_convertvector(*reinterpret_cast<const f16x4 *>(reinterpret_cast<const _Float16 *>(p) + i), f32x4);
    else return ld4_bf16(reinterpret_cast<const uint16_t *>(p) + i);
}
// ... at any element address.
template <int DT>
__device__ __forceinline__ f32x4 ld4_any(const void *p, int64_t i) {
    if constexpr (DT == FLE_F32) {
        return reinterpret_cast<const AnyAligned<f32x4, 4> *>(reinterpret_cast<const float *>(p) + i)->v;
    } else {
        const u32x2 u = reinterpret_cast<const AnyAligned<u32x2, 2> *>(reinterpret_cast<const uint16_t *>(p) + i)->v;
        if constexpr (DT == FLE_F16) return __builtin_convertvector(__builtin_bit_cast(f16x4, u), f32x4);
        else return f32x4{__uint_as_float(u[0] << 16), __uint_as_float(u[0] & 0xffff0000u), __uint_as_float(u[1] << 16), __uint_as_float(u[1] & 0xffff0000u)};
    }
}
__device__ __forceinline__ f32x4 ld4_any_rt(const void *p, int64_t i, int dtype) {  // dtype known at run time only
    if (dtype == FLE_F32) return ld4_any<FLE_F32>(p, i);
    if (dtype == FLE_F16) return ld4_any<FLE_F16>(p, i);
    return ld4_any<FLE_BF16>(p, i);
}

// 4 fp32 values rounded (to nearest even) to a 2-byte dtype and packed into 8 bytes.
template <int DT>
__device__ __forceinline__ u32x2 pack4(f32x4 v) {
    static_assert(DT == FLE_BF16 || DT == FLE_F16, "2-byte dtypes only");
    if constexpr (DT == FLE_F16) return __builtin_bit_cast(u32x2, __builtin_convertvector(v, f16x4));
    else return __builtin_bit_cast(u32x2, __builtin_convertvector(v, bf16x4));
}
// 4 values rounded to the dtype and stored at element index i, whatever its address.
template <int DT>
__device__ __forceinline__ void st4_any(void *p, int64_t i, f32x4 v) {
    if constexpr (DT == FLE_F32) reinterpret_cast<AnyAligned<f32x4, 4> *>(reinterpret_cast<float *>(p) + i)->v = v;
    else reinterpret_cast<AnyAligned<u32x2, 2> *>(reinterpret_cast<uint16_t *>(p) + i)->v = pack4<DT>(v);
}
__device__ __forceinline__ void st4_any_rt(void *p, int64_t i, int dtype, f32x4 v) {
    if (dtype == FLE_F32) st4_any<FLE_F32>(p, i, v);
    else if (dtype == FLE_F16) st4_any<FLE_F16>(p, i, v);
    else st4_any<FLE_BF16>(p, i, v);
}

__device__ __forceinline__ float relu_f(float v) { return v < 0.0f ? 0.0f : v; }  // NaN stays NaN

// max(v, 0), of the bits as whole numbers: one instruction (fmaxf takes a second one, which quiets signalling NaNs).  NaN: itself or 0.
__device__ __forceinline__ float positive_part(float v) { return __builtin_bit_cast(float, max(__builtin_bit_cast(int, v), 0)); }

// GELU with the exact-erf definition: v (1 + erf(v / sqrt 2)) / 2 = max(v, 0) - |v| h(|v|), h(a) = erfc(a / sqrt 2) / 2.  h is
// 2^P(a) with a polynomial of degree 8 for the smooth log2 h, fitted by linear programming to the least largest error of
// max(a, 0.8) h(a) over 0 .. 6 (P(0) = -1 exactly).  Off float64 by 2.4e-7 at most, by 4.4e-8 of the 2-norm at deviation 1 and 7.5e-8 at
// 0.05 (the rational form before, Abramowitz & Stegun 7.1.26: 3.3e-7, 8.3e-8, 1.8e-7); the left tail to -4 within 4.2e-5 of the value
// (4.7e-4), to -6 within 2e-3 (3.6e-3).  10 or 11 plain and one quarter-rate instruction per value for 13 and two; at 256 values per
// lane that is most of what this epilogue costs a 256 x 256 tile:
// bf16 32768 x 8192 x 2048 972 -> 950 us, 4096 x 4096 x 4096 in fp8 65.8 -> 64.0, fp16 2000 x 4096 x 512 19.5 -> 18.3.
__device__ __forceinline__ float gelu_log2h_near(float a) {
    float p = fmaf(a, -1.190245143e-06f, 1.986793177e-05f);
    p = fmaf(a, p, -9.558258898e-05f);
    p = fmaf(a, p, -3.471522650e-04f);
    p = fmaf(a, p, 7.320655044e-03f);
    p = fmaf(a, p, -5.265637115e-02f);
    p = fmaf(a, p, -4.591638446e-01f);
    p = fmaf(a, p, -1.151108980f);
    return fmaf(a, p, -1.0f);
}
// Behind 6 P falls much faster than log2 h (the value was 7 % off at -7, 42 % at -8, all of it from -9 on); there a polynomial of degree 2
// takes its place, fitted to the least relative error: within 0.22 % of the value to -8, 0.75 % to -12, 1 % to -12.9 (the rational form
// 1 %, 3.1 %, 3.7 %), where h leaves the range of fp32.  (One polynomial for all of it takes a degree of 10 and is then twice as far off near 0.)
constexpr float kGeluFar = 6.0f;
__device__ __forceinline__ float gelu_log2h_far(float a) { return fmaf(a, fmaf(a, -0.712202251f, -0.326766521f), -2.31880403f); }
__device__ __forceinline__ float gelu_of(float v, float log2h) { return fmaf(-fabsf(v), __builtin_amdgcn_exp2f(log2h), positive_part(v)); }
__device__ __forceinline__ float gelu_erf_f(float v) {
    const float a = fabsf(v), near = gelu_log2h_near(a), far = gelu_log2h_far(a);
    return gelu_of(v, a > kGeluFar ? far : near);
}
// The same for a lane's N values, each(f) putting f(value, its number) in every one's place.  The far form runs where the wave has a value
// that needs it, which half an instruction per value finds out; it changes exponents only, so its code, which is seldom run but lies among
// the rest in a 64 KB instruction cache, stays short (with a whole second form there the 160 x 256 tile's kernel grew from 61 to 80 KB).
template <int N, class Each>
__device__ __forceinline__ void gelu_erf_each(Each &&each) {
    float largest = 0.0f, log2h[N];
    each([&](float v, int i) __attribute__((always_inline)) {
        largest = fmaxf(largest, fabsf(v));
        log2h[i] = gelu_log2h_near(fabsf(v));
        return v;
    });
    if (__builtin_expect(__any(largest > kGeluFar), 0))
        each([&](float v, int i) __attribute__((always_inline)) {
            log2h[i] = fabsf(v) > kGeluFar ? gelu_log2h_far(fabsf(v)) : log2h[i];
            return v;
        });
    each([&](float v, int i) __attribute__((always_inline)) { return gelu_of(v, log2h[i]); });
}

// 0.5 v (1 + tanh u) == v / (1 + exp(-2u)),  u = sqrt(2/pi) (v + 0.044715 v^3)
// (exp(-2u) as 2^(v (1 + 0.044715 v^2) k), k = -2 sqrt(2/pi) log2 e: 6 plain and 2 quarter-rate instructions per value)
__device__ __forceinline__ float gelu_tanh_f(float v) {
    const float w = fmaf(0.044715f * v, v, 1.0f);
    const float e = __builtin_amdgcn_exp2f(v * w * (-2.0f * 0.7978845608028654f * 1.4426950408889634f));
    return v * __builtin_amdgcn_rcpf(1.0f + e);
}

// One elementwise op on one value at (m, n).
__device__ __forceinline__ float apply_op(const DevOp &op, float v, int64_t m, int64_t n, const void *bias, int dtype) {
    switch (op.kind) {
    case FLE_BIAS: return v + ld_elem(bias, n, dtype);
    case FLE_SCALE: return v * op.alpha;
    case FLE_RELU: return relu_f(v);
    case FLE_GELU_ERF: return gelu_erf_f(v);
    case FLE_GELU_TANH: return gelu_tanh_f(v);
    case FLE_RESIDUAL: return v + ld_elem(op.p0, m * op.ld + n, dtype);
    case FLE_STORE: st_elem(const_cast<void *>(op.p0), m * op.ld + n, dtype, v); return v;
    default: return v;
    }
}

// ------------------------------------------------------------------ row-reduction partials
// LayerNorm partial over c values: (mean, M2 = sum (v - mean)^2); the count is implied by the
// partial's position.  Softmax / logsumexp partial: (max, sum exp(v - max)).
struct Stat {
    float n, a, b;  // n = count (LayerNorm only); (a, b) = (mean, M2) or (max, sum)
};

__device__ __forceinline__ Stat combine_ln(const Stat &p, const Stat &q) {
    if (q.n == 0.0f) return p;
    if (p.n == 0.0f) return q;
    Stat r;
    r.n = p.n + q.n;
    const float d = q.a - p.a;
    // (one hardware reciprocal, 1 ulp, in place of two IEEE divisions of a dozen instructions each: the combine runs
    // seven times per wave of the finalize pass and was half of its vector-ALU work)
    const float w = q.n * __builtin_amdgcn_rcpf(r.n);
    r.a = fmaf(d, w, p.a);
    r.b = p.b + q.b + d * d * (p.n * w);
    return r;
}

__device__ __forceinline__ Stat combine_sm(const Stat &p, const Stat &q) {
    Stat r;
    r.n = 0.0f;
    r.a = fmaxf(p.a, q.a);
    const float sp = p.b == 0.0f ? 0.0f : p.b * __expf(p.a - r.a);
    const float sq = q.b == 0.0f ? 0.0f : q.b * __expf(q.a - r.a);
    r.b = sp + sq;
    return r;
}

// All lanes of a wave end up with the combination of every partial of `row`, in a fixed order.
// LayerNorm: Chan's update, lane-serial then a butterfly.  Softmax / logsumexp: the row maximum first
// (exact in any order), then every partial sum rescaled to it once and added lane-serially and by
// butterfly: one exp per partial instead of two per pairwise combine.
// first: (LayerNorm) partial first_partial(np, lane) of the row if the caller has already loaded it (with the rest of what it reads), else nullptr.
// Up to 8 partials: every group of 8 lanes takes a copy, and the butterfly ends at the group (what it would go on to combine
// with is empty: the same bits).  (Every power of two so, level by level: 0.2 us more in calls of a few rows with 16 partials and more.)
__device__ __forceinline__ int first_partial(int np, int lane) { return np <= 8 ? lane & 7 : lane; }
template <bool LN>
__device__ __forceinline__ Stat reduce_partials(const float *partials, int64_t row, int np, int part_cols, int64_t N, int lane, const float2 *first = nullptr) {
    Stat s;
    s.n = 0.0f;
    s.a = LN ? 0.0f : -INFINITY;
    s.b = 0.0f;
    const float *pr = partials + row * np * 2;
    if (LN) {  // few partials per row (N / 64 or fewer): one load per lane and round
        const int mine = first_partial(np, lane);
        for (int p = mine; p < np; p += 64) {
            Stat q;
            const int64_t left = N - int64_t(p) * part_cols;
            q.n = float(left < part_cols ? left : part_cols);
            if (first && p == mine) {
                q.a = first->x;
                q.b = first->y;
            } else {
                q.a = pr[2 * p];
                q.b = pr[2 * p + 1];
            }
            s = combine_ln(s, q);
        }
        auto level = [&](int d) {
            Stat o;
            o.n = __shfl_xor(s.n, d);
            o.a = __shfl_xor(s.a, d);
            o.b = __shfl_xor(s.b, d);
            const bool upper = (lane & d) != 0;  // both partners combine (lower lane, upper lane): identical results
            const Stat lo = upper ? o : s, hi = upper ? s : o;
            s = combine_ln(lo, hi);
        };
        if (np <= 8) {
#pragma unroll
            for (int d = 1; d < 8; d <<= 1) level(d);
            return s;
        }
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) level(d);
        return s;
    }
    // softmax / logsumexp: a lane takes partials lane, lane + 64, ...; up to 16 loads go out together so
    // that their latencies overlap (a row of a 32768-column softmax has 1024 partials, 16 per lane)
    constexpr int B = 16;
    if (np <= 64 * B) {  // one batch: keep the partials in registers between the two sweeps
        float2 buf[B];
#pragma unroll
        for (int j = 0; j < B; ++j) {
            const int p = j * 64 + lane;
            buf[j] = make_float2(-INFINITY, 0.0f);
            if (j * 64 < np && p < np) buf[j] = *reinterpret_cast<const float2 *>(pr + 2 * p);  // outer test is wave-uniform
        }
        float mx = -INFINITY;
#pragma unroll
        for (int j = 0; j < B; ++j) mx = fmaxf(mx, buf[j].x);
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) mx = fmaxf(mx, __shfl_xor(mx, d));
        float sum = 0.0f;
#pragma unroll
        for (int j = 0; j < B; ++j)
            if (j * 64 < np && buf[j].y != 0.0f) sum += buf[j].y * __expf(buf[j].x - mx);
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) sum += __shfl_xor(sum, d);  // partners add the same two numbers: identical in every lane
        s.a = mx;
        s.b = sum;
        return s;
    }
    float mx = -INFINITY;
    for (int p = lane; p < np; p += 64) mx = fmaxf(mx, pr[2 * p]);
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) mx = fmaxf(mx, __shfl_xor(mx, d));
    float sum = 0.0f;
    for (int p = lane; p < np; p += 64) {
        const float2 q = *reinterpret_cast<const float2 *>(pr + 2 * p);
        if (q.y != 0.0f) sum += q.y * __expf(q.x - mx);
    }
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) sum += __shfl_xor(sum, d);
    s.a = mx;
    s.b = sum;
    return s;
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {  // s_waitcnt vmcnt(N), other counters untouched
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | 0x0F70);
}

// Sum / max over the 16 lanes of a DPP row by rotations; every lane ends with the result.
template <bool MAX>
__device__ __forceinline__ float row16_allreduce(float v) {
#define FLE_ROR(n)                                                                                              \
    {                                                                                                           \
        const float o = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + (n), 0xF, 0xF, false)); \
        v = MAX ? fmaxf(v, o) : v + o;                                                                          \
    }
    FLE_ROR(8) FLE_ROR(4) FLE_ROR(2) FLE_ROR(1)
#undef FLE_ROR
    return v;
}

}  // namespace fle
