// Second passes: finalize of LayerNorm / softmax / logsumexp, and the split-K reduction.
#pragma once
#include "fle_device_common.h"

namespace fle {

// ------------------------------------------------------------------ finalize passes
// One wave per (row, 2048-column chunk).  The wave combines the row's partials itself (one
// per lane, then a fixed butterfly: identical result in every lane), issues all of its
// 16-byte loads of staged y at once, normalises, applies the trailing elementwise ops, rounds
// and writes 16-byte vectors.
// 8 fp32 values rounded to a 2-byte dtype (stored as one 16-byte vector at element index i).
__device__ __forceinline__ u32x4 pack8_2byte(int dtype, const float (&v)[8]) {
    u32x4 o;
    if (dtype == FLE_F16) {
        f16x8 h;
#pragma unroll
        for (int e = 0; e < 8; ++e) h[e] = static_cast<_Float16>(v[e]);
        o = __builtin_bit_cast(u32x4, h);
    } else {
        bf16x8 h;
#pragma unroll
        for (int e = 0; e < 8; ++e) h[e] = static_cast<__bf16>(v[e]);
        o = __builtin_bit_cast(u32x4, h);
    }
    return o;
}
__device__ __forceinline__ void st8_2byte(void *p, int64_t i, int dtype, const float (&v)[8]) {
    *reinterpret_cast<u32x4 *>(reinterpret_cast<uint16_t *>(p) + i) = pack8_2byte(dtype, v);
}

// 16 bytes of a 2-byte dtype (known at run time) as 8 fp32 values.
__device__ __forceinline__ void unpack8_2byte(const u32x4 r, int dtype, float (&v)[8]) {
    if (dtype == FLE_F16) {
        const f16x8 h = __builtin_bit_cast(f16x8, r);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = float(h[e]);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) { v[2 * e] = __uint_as_float(r[e] << 16); v[2 * e + 1] = __uint_as_float(r[e] & 0xffff0000u); }
    }
}

// LNK: LayerNorm (true) or softmax (false); separate kernels so that each gets its own register budget.
// DT: the storage dtype (the conversions then carry no run-time choice).
// WHOLE: rows are whole vectors of 8 at aligned addresses.  Otherwise the same vectors at whatever address they lie on
// (global memory takes them; the row starts at any element), and the N % 8 columns behind them one per lane.  (With
// element accesses here and in the tiled kernel's epilogue wherever rows were not aligned, a LayerNorm call of
// 1999 x 4099 x 3071 in fp16 took 158 us, now 110; 16384 x 4097 x 1024 in bf16 545 -> 310.)
// IT: vectors per lane and item.
template <bool WHOLE, bool LNK, int DT, int IT>
__device__ __forceinline__ void finalize_items(const FinArgs &a) {
    constexpr int CH = 512 * IT;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr int dtype = DT;
    constexpr bool f32 = DT == FLE_F32;
    constexpr int ES = f32 ? 4 : 2;
    auto ld16 = [](const void *p, int64_t i, auto size_c) __attribute__((always_inline)) -> u32x4 {  // 16 bytes at element i of size_c bytes
        constexpr int SZ = decltype(size_c)::value;
        const char *q = reinterpret_cast<const char *>(p) + i * SZ;
        if constexpr (WHOLE) return *reinterpret_cast<const u32x4 *>(q);
        else return reinterpret_cast<const AnyAligned<u32x4, SZ> *>(q)->v;
    };
    using SZ4 = std::integral_constant<int, 4>;
    using SZE = std::integral_constant<int, ES>;
    constexpr bool ln = LNK;
    const int64_t N = a.N;
    const int64_t chunks = (N + CH - 1) / CH, items = a.M * chunks;
    // item -> (row, first column).  (64-bit divisions cost over a hundred vector instructions each; so does the
    // run-time choice of conversions that a dtype known at compile time avoids: c3's pass 34.4 -> 31.5 us with the
    // cheaper combine of the partials.  Walking several items per wave with the next item's loads ahead: 34.1 us.)
    auto place = [&](int64_t item, int64_t &row, int64_t &c0) {
        if (items <= 0x7fffffff) {
            const uint32_t r32 = uint32_t(item) / uint32_t(chunks);
            row = r32;
            c0 = int64_t(uint32_t(item) - r32 * uint32_t(chunks)) * CH;
        } else {
            row = item / chunks;
            c0 = (item % chunks) * CH;
        }
    };
    for (int64_t item = int64_t(blockIdx.x) * 4 + wave; item < items; item += int64_t(gridDim.x) * 4) {
        int64_t row;
        int64_t c0;
        place(item, row, c0);
        const int64_t nv = WHOLE ? N : N & ~int64_t(7);  // columns that are whole vectors
        const int64_t c1 = c0 + CH < nv ? c0 + CH : nv;
        const bool tail = !WHOLE && nv >= c0 && nv < c0 + CH && lane < N - nv;  // this lane has one of the columns behind them
        // Everything the item reads goes out in one batch in front of the combine of the partials, as loaded
        // (conversions later) and without a branch around any of it: a vector past the end of the row re-reads
        // the row's last one.  (Loads inside per-vector conditions, each converted where it stood, came out as
        // load, wait, convert, load, wait, convert: four round trips to memory per wave instead of one.)
        float y[IT][8];
        u32x4 yr[IT][2];
        [[maybe_unused]] u32x4 gr[LNK ? IT : 1], br[LNK ? IT : 1];
        [[maybe_unused]] float pmean[IT];
        const bool yf = f32 || a.y_f32;                       // staged values are fp32
        constexpr bool early_gb = LNK && !f32;   // gamma / beta of a 2-byte dtype: 4 registers per vector
        [[maybe_unused]] float2 part_first = make_float2(0.0f, 0.0f);
        if constexpr (LNK) {  // this lane's partial of the row, in the same batch
            const int p = first_partial(a.np, lane);
            if (p < a.np) part_first = *reinterpret_cast<const float2 *>(a.partials + (row * a.np + p) * 2);
        }
        if (WHOLE || nv > 0) {
            int64_t nc[IT];
#pragma unroll
            for (int it = 0; it < IT; ++it) {
                const int64_t n = c0 + it * 512 + lane * 8;
                nc[it] = n < c1 ? n : c1 - 8;
            }
            if (yf) {
#pragma unroll
                for (int it = 0; it < IT; ++it) {
                    yr[it][0] = ld16(a.y, row * a.ldy + nc[it], SZ4{});
                    yr[it][1] = ld16(a.y, row * a.ldy + nc[it] + 4, SZ4{});
                }
            } else {
#pragma unroll
                for (int it = 0; it < IT; ++it) yr[it][0] = ld16(a.y, row * a.ldy + nc[it], SZE{});
            }
            if (a.y_rel) {
#pragma unroll
                for (int it = 0; it < IT; ++it) pmean[it] = a.partials[(row * a.np + (nc[it] >> a.part_shift)) * 2];
            }
            if constexpr (early_gb) {
                if (a.epi.row.p0) {
#pragma unroll
                    for (int it = 0; it < IT; ++it) gr[it] = ld16(a.epi.row.p0, nc[it], SZE{});
                }
                if (a.epi.row.p1) {
#pragma unroll
                    for (int it = 0; it < IT; ++it) br[it] = ld16(a.epi.row.p1, nc[it], SZE{});
                }
            }
        }
        float ty = 0.0f, tmean = 0.0f;
        if (tail) {
            ty = ld_elem(a.y, row * a.ldy + nv + lane, a.y_f32 ? FLE_F32 : dtype);
            if (a.y_rel) tmean = a.partials[(row * a.np + ((nv + lane) >> a.part_shift)) * 2];
        }
        float sub, mul;  // out = (y - sub) * mul  (LayerNorm),  exp(y - sub) * mul  (softmax)
        if (ln) {
            const Stat s = reduce_partials<true>(a.partials, row, a.np, a.part_cols, N, lane, &part_first);
            sub = s.a;
            mul = rsqrtf(s.b / float(N) + a.epi.row.alpha);
        } else {
            const Stat s = reduce_partials<false>(a.partials, row, a.np, a.part_cols, N, lane);
            sub = s.a;
            mul = 1.0f / s.b;
        }
        // the bias of this row: of its group for a grouped problem (the last group whose first row is <= row:
        // empty groups share their offset with the next one), else the problem's
        const void *bias = a.epi.bias;
        if (a.row_offsets && bias) {
            int lo = 0, hi = a.n_groups;  // invariant: offsets[lo] <= row (offsets[0] counts as 0), offsets[hi] > row or hi == n_groups
            while (hi - lo > 1) {
                const int mid = (lo + hi) / 2;
                if (a.row_offsets[mid] <= row) lo = mid;
                else hi = mid;
            }
            bias = reinterpret_cast<const char *>(bias) + int64_t(lo) * a.b_stride_bytes;
        }
        auto post = [&](float v, int64_t n) -> float {
            for (int o = 0; o < a.epi.n_post; ++o) v = apply_op(a.epi.post[o], v, row, n, bias, dtype);
            return v;
        };
        {
#pragma unroll
            for (int it = 0; it < IT; ++it) {
                const int64_t n = c0 + it * 512 + lane * 8;
                if (n < c1) {
                    float *v = y[it];
                    if (yf) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) { v[e] = __uint_as_float(yr[it][0][e]); v[4 + e] = __uint_as_float(yr[it][1][e]); }
                    } else {
                        unpack8_2byte(yr[it][0], dtype, y[it]);
                    }
                    // staged relative to the statistic (mean / maximum) of the partial the 8 columns lie in (part_cols is a multiple of 8)
                    const float shift = a.y_rel ? sub - pmean[it] : sub;
                    if (ln) {
                        float g[8], be[8];
#pragma unroll
                        for (int e = 0; e < 8; ++e) { g[e] = 1.0f; be[e] = 0.0f; }
                        if constexpr (early_gb) {
                            if (a.epi.row.p0) unpack8_2byte(gr[it], dtype, g);
                            if (a.epi.row.p1) unpack8_2byte(br[it], dtype, be);
                        } else {
                            auto two = [&](const void *p, float (&d)[8]) {
                                const u32x4 lo = ld16(p, n, SZ4{}), hi = ld16(p, n + 4, SZ4{});
#pragma unroll
                                for (int e = 0; e < 4; ++e) { d[e] = __uint_as_float(lo[e]); d[4 + e] = __uint_as_float(hi[e]); }
                            };
                            if (a.epi.row.p0) two(a.epi.row.p0, g);
                            if (a.epi.row.p1) two(a.epi.row.p1, be);
                        }
#pragma unroll
                        for (int e = 0; e < 8; ++e) v[e] = (v[e] - shift) * mul * g[e] + be[e];
                    } else {
#pragma unroll
                        for (int e = 0; e < 8; ++e) v[e] = __expf(v[e] - shift) * mul;
                    }
                    if (a.epi.n_post > 0) {
#pragma unroll
                        for (int e = 0; e < 8; ++e) v[e] = post(v[e], n + e);
                    }
                    if (f32 || a.out_f32) {
                        float *dstp = reinterpret_cast<float *>(a.out) + row * a.ldo + n;
                        const f32x4 lo = {v[0], v[1], v[2], v[3]}, hi = {v[4], v[5], v[6], v[7]};
                        if constexpr (WHOLE) {
                            *reinterpret_cast<f32x4 *>(dstp) = lo;
                            *reinterpret_cast<f32x4 *>(dstp + 4) = hi;
                        } else {
                            reinterpret_cast<AnyAligned<f32x4, 4> *>(dstp)->v = lo;
                            reinterpret_cast<AnyAligned<f32x4, 4> *>(dstp + 4)->v = hi;
                        }
                    } else if constexpr (WHOLE) {
                        st8_2byte(a.out, row * a.ldo + n, dtype, y[it]);
                    } else {
                        reinterpret_cast<AnyAligned<u32x4, 2> *>(reinterpret_cast<uint16_t *>(a.out) + row * a.ldo + n)->v = pack8_2byte(dtype, y[it]);
                    }
                }
            }
        }
        if (tail) {
            const int64_t n = nv + lane;
            const float shift = a.y_rel ? sub - tmean : sub;
            float v;
            if (ln) {
                v = (ty - shift) * mul;
                if (a.epi.row.p0) v *= ld_elem(a.epi.row.p0, n, dtype);
                if (a.epi.row.p1) v += ld_elem(a.epi.row.p1, n, dtype);
            } else {
                v = __expf(ty - shift) * mul;
            }
            st_elem(a.out, row * a.ldo + n, a.out_f32 ? FLE_F32 : dtype, post(v, n));
        }
    }
}

// (four waves per SIMD where the item's loads go out as one batch: the allocator is two registers over that by itself)
template <bool WHOLE, bool LNK, int DT>
__global__ __launch_bounds__(256, WHOLE && LNK ? 4 : 1) void finalize_rows(const FinArgs a) { finalize_items<WHOLE, LNK, DT, 4>(a); }
// Rows of up to 512 and 1024 columns: one or two vectors a lane and half the registers.  (A row was asked for four, of which the
// end of the row left one or two, and the combine of its partials went through the empty lanes.  The whole call, bf16 with
// LayerNorm: 16384 x 512 x 512 38.5 -> 33.7 us, 7000 x 1001 x 256 38.8 -> 34.1; block-scaled fp8 12554 x 304 x 256 28.7 -> 25.2.)
template <bool WHOLE, bool LNK, int DT, int IT>
__global__ __launch_bounds__(256) void finalize_short(const FinArgs a) { finalize_items<WHOLE, LNK, DT, IT>(a); }

// logsumexp: one wave per row, out[row] = max + log(sum).
__global__ __launch_bounds__(256) void finalize_lse(const FinArgs a) {
    const int lane = threadIdx.x & 63;
    const int64_t row = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (row >= a.M) return;
    const Stat s = reduce_partials<false>(a.partials, row, a.np, a.part_cols, a.N, lane);
    if (lane == 0) st_elem(a.out, row, a.epi.dtype, s.a + __logf(s.b));
}

// ------------------------------------------------------------------ a second row reduction in the list
// One workgroup per row: the values behind the first row reduction (and the ops that follow it) arrive in fp32;
// three sweeps over the row (it stays in the L2): mean or maximum, then sum of squared deviations or of
// exponentials, then normalise, apply the ops behind the reduction, round and store.  Sums are formed per thread
// in index order, across the wave by a fixed butterfly and across the four waves in wave order: reproducible.
__device__ __forceinline__ float block_allreduce(float v, bool max, float *lds) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const float o = __shfl_xor(v, d);
        v = max ? fmaxf(v, o) : v + o;
    }
    const int wave = threadIdx.x >> 6;
    __syncthreads();  // (the previous use of lds is over)
    if ((threadIdx.x & 63) == 0) lds[wave] = v;
    __syncthreads();
    float r = lds[0];
    for (int w = 1; w < 4; ++w) r = max ? fmaxf(r, lds[w]) : r + lds[w];
    return r;
}

__global__ __launch_bounds__(256) void second_row_op(const Row2Args a) {
    __shared__ float lds[4];
    const int64_t N = a.N;
    const int dtype = a.epi.dtype;
    const int kind = a.epi.row_kind;
    for (int64_t row = blockIdx.x; row < a.M; row += gridDim.x) {
        const float *v = a.v + row * N;
        float sub, mul;
        if (kind == FLE_LAYERNORM) {
            float s = 0.0f;
            for (int64_t n = threadIdx.x; n < N; n += 256) s += v[n];
            const float mean = block_allreduce(s, false, lds) / float(N);
            float m2 = 0.0f;
            for (int64_t n = threadIdx.x; n < N; n += 256) m2 += (v[n] - mean) * (v[n] - mean);
            m2 = block_allreduce(m2, false, lds);
            sub = mean;
            mul = rsqrtf(m2 / float(N) + a.epi.row.alpha);
        } else {
            float mx = -INFINITY;
            for (int64_t n = threadIdx.x; n < N; n += 256) mx = fmaxf(mx, v[n]);
            mx = block_allreduce(mx, true, lds);
            float se = 0.0f;
            for (int64_t n = threadIdx.x; n < N; n += 256) se += __expf(v[n] - mx);
            se = block_allreduce(se, false, lds);
            sub = mx;
            mul = 1.0f / se;
            if (kind == FLE_LOGSUMEXP) {
                if (threadIdx.x == 0) st_elem(a.out, row, dtype, mx + __logf(se));
                continue;
            }
        }
        for (int64_t n = threadIdx.x; n < N; n += 256) {
            float o;
            if (kind == FLE_LAYERNORM) {
                o = (v[n] - sub) * mul;
                if (a.epi.row.p0) o *= ld_elem(a.epi.row.p0, n, dtype);
                if (a.epi.row.p1) o += ld_elem(a.epi.row.p1, n, dtype);
            } else {
                o = __expf(v[n] - sub) * mul;
            }
            for (int q = 0; q < a.epi.n_post; ++q) o = apply_op(a.epi.post[q], o, row, n, a.epi.bias, dtype);
            st_elem(a.out, row * a.ldo + n, dtype, o);
        }
    }
}

// ------------------------------------------------------------------ LayerNorm of x in front of the multiplication
// Writes (x - mean) rstd gamma + beta, rounded to the dtype, into a contiguous copy of x that the GEMM kernels read.
// Three phases (mean, squared deviations, result).  Sums per lane in index order, then a fixed butterfly (and the waves in
// wave order): reproducible.
__device__ __forceinline__ float wave_allreduce_sum(float v) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) v += __shfl_xor(v, d);
    return v;
}

// 16 bytes as fp32 values (DT: fle_dtype; 4 values of fp32, else 8).
template <int DT>
__device__ __forceinline__ void unpack_vec(const u32x4 r, float (&v)[8]) {
    if constexpr (DT == FLE_F32) {
#pragma unroll
        for (int e = 0; e < 4; ++e) { v[e] = __uint_as_float(r[e]); v[4 + e] = 0.0f; }
    } else if constexpr (DT == FLE_F16) {
        const f16x8 h = __builtin_bit_cast(f16x8, r);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = float(h[e]);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) { v[2 * e] = __uint_as_float(r[e] << 16); v[2 * e + 1] = __uint_as_float(r[e] & 0xffff0000u); }
    }
}

// A row in the registers of WAVES waves (1: four rows per workgroup), read once whatever its address and length are: all of
// a lane's NV vectors of 16 bytes are requested in one batch, without a branch (one that reaches past the end of the row
// reads the row's last 16 bytes; what lies in front of its own place is left out), and stay in registers for all three phases, 2-byte
// rows mostly as the fp32 values that the compiler keeps: 74 - 133 registers with up to 4 vectors, 186 - 207 with 8 (two waves per SIMD), 316 - 358
// with 16 (one; fp32 137 - 157 and 228 - 270).  gamma and beta come 4 vectors at a time.  Bound by memory: one wave per row as long
// as 8 vectors hold it (more leave a wave with nothing beside it to cover its loads), a workgroup of four above that, where 16 vectors are still far
// ahead of reading the row again: 700 x 24576 in front of 512 columns 214 us element by element, 64.5 so, 4000 x 32768 (128 columns) 1273
// and 215, fp32 700 x 16384 109 in three sweeps and 92.  In front of a product (whole call, three sweeps by one wave or element by element before, now): bf16 3820 x
// 2261 x 13299 681 -> 328 us (the pass itself 425, 100 MB read and written), 9000 x 256 x 1985 142 -> 44, 16384 x 256 x 577 122 -> 37,
// 16384 x 256 x 256 41 -> 24 (a wave held 8 vectors for the one it needs); 4096 x 4096 x 4096 124 either way.
// WHOLE: rows are whole vectors, and a vector is either all in its row or not at all.
template <int DT, int WAVES, int NV, bool WHOLE>
__global__ __launch_bounds__(256) void ln_rows(const LnArgs a) {
    __shared__ float lds[4];
    constexpr int W = DT == FLE_F32 ? 4 : 8, ES = DT == FLE_F32 ? 4 : 2, T = 64 * WAVES;  // elements per vector; lanes per row
    constexpr int NB = NV < 4 ? NV : 4;                                                  // vectors per batch of gamma and beta
    using any_t = AnyAligned<u32x4, ES>;
    const int K = int(a.K), t = int(threadIdx.x) % T;
    const int64_t per_wg = 4 / WAVES;
    auto all = [&](float v) {
        if constexpr (WAVES == 1) return wave_allreduce_sum(v);
        else return block_allreduce(v, false, lds);
    };
    for (int64_t row = int64_t(blockIdx.x) * per_wg + (WAVES == 1 ? threadIdx.x / 64 : 0); row < a.M; row += int64_t(gridDim.x) * per_wg) {
        const char *src = reinterpret_cast<const char *>(a.x) + row * a.ldx * ES;
        u32x4 raw[NV];
        int kc[NV];  // the first element of vector i as loaded
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int k = (i * T + t) * W;
            kc[i] = k + W <= K ? k : K - W;
            raw[i] = reinterpret_cast<const any_t *>(src + int64_t(kc[i]) * ES)->v;
        }
        // the sum of f over vector i's own elements
        auto own = [&](int i, auto &&f) __attribute__((always_inline)) {
            const int k = (i * T + t) * W;
            float v[8], part = 0.0f;
            unpack_vec<DT>(raw[i], v);
            if (WHOLE || (i + 1) * T * W <= K) {  // (uniform)
#pragma unroll
                for (int e = 0; e < W; ++e) part += f(v[e]);
                return k < K ? part : 0.0f;
            }
#pragma unroll
            for (int e = 0; e < W; ++e) part += e >= k - kc[i] ? f(v[e]) : 0.0f;
            return part;
        };
        float s = 0.0f;
#pragma unroll
        for (int i = 0; i < NV; ++i) s += own(i, [](float v) { return v; });
        const float mean = all(s) / float(K);
        float m2 = 0.0f;
#pragma unroll
        for (int i = 0; i < NV; ++i) m2 += own(i, [&](float v) { return (v - mean) * (v - mean); });
        const float rstd = rsqrtf(all(m2) / float(K) + a.eps);
        char *const dst = reinterpret_cast<char *>(a.dst) + row * a.ldd * ES;
#pragma unroll
        for (int h = 0; h < NV; h += NB) {
            u32x4 gr[NB], br[NB];
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                gr[j] = br[j] = u32x4{0u, 0u, 0u, 0u};
                if (a.gamma) gr[j] = reinterpret_cast<const any_t *>(reinterpret_cast<const char *>(a.gamma) + int64_t(kc[h + j]) * ES)->v;
                if (a.beta) br[j] = reinterpret_cast<const any_t *>(reinterpret_cast<const char *>(a.beta) + int64_t(kc[h + j]) * ES)->v;
            }
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const int k = ((h + j) * T + t) * W;
                float v[8], g[8], be[8], o[8];
                unpack_vec<DT>(raw[h + j], v);
#pragma unroll
                for (int e = 0; e < 8; ++e) { g[e] = 1.0f; be[e] = 0.0f; }
                if (a.gamma) unpack_vec<DT>(gr[j], g);
                if (a.beta) unpack_vec<DT>(br[j], be);
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = (v[e] - mean) * rstd * g[e] + be[e];
                if (k + W <= K) {
                    if constexpr (DT == FLE_F32) {
                        st4_any<DT>(dst, k, f32x4{o[0], o[1], o[2], o[3]});
                    } else {
                        const u32x2 lo = pack4<DT>(f32x4{o[0], o[1], o[2], o[3]}), hi = pack4<DT>(f32x4{o[4], o[5], o[6], o[7]});
                        reinterpret_cast<any_t *>(dst + int64_t(k) * ES)->v = u32x4{lo[0], lo[1], hi[0], hi[1]};
                    }
                } else if (!WHOLE && k < K) {
#pragma unroll
                    for (int e = 0; e < W; ++e)
                        if (e >= k - kc[h + j]) st_elem(dst, kc[h + j] + e, DT, o[e]);
                }
            }
        }
        for (int64_t k = K + t; k < a.ldd; k += T) st_elem(dst, k, DT, 0.0f);
    }
}

// Rows of less than one vector, or longer than a workgroup holds: a workgroup per row, element by element, in three sweeps.
template <int DT>
__global__ __launch_bounds__(256) void ln_prologue(const LnArgs a) {
    __shared__ float lds[4];
    const int64_t K = a.K;
    constexpr int dtype = DT;
    for (int64_t row = blockIdx.x; row < a.M; row += gridDim.x) {
        const int64_t base = row * a.ldx;
        auto sweep = [&](auto &&f) {  // f(k, value) for this thread's elements of the row, in index order
            for (int64_t k = threadIdx.x; k < K; k += 256) f(k, ld_elem(a.x, base + k, dtype));
        };
        float s = 0.0f;
        sweep([&](int64_t, float v) { s += v; });
        const float mean = block_allreduce(s, false, lds) / float(K);
        float m2 = 0.0f;
        sweep([&](int64_t, float v) { m2 += (v - mean) * (v - mean); });
        const float rstd = rsqrtf(block_allreduce(m2, false, lds) / float(K) + a.eps);
        sweep([&](int64_t k, float v) {
            float o = (v - mean) * rstd;
            if (a.gamma) o *= ld_elem(a.gamma, k, dtype);
            if (a.beta) o += ld_elem(a.beta, k, dtype);
            st_elem(a.dst, row * a.ldd + k, dtype, o);
        });
        for (int64_t k = K + threadIdx.x; k < a.ldd; k += 256) st_elem(a.dst, row * a.ldd + k, dtype, 0.0f);
    }
}

// ------------------------------------------------------------------ copies of operands the GEMM kernels cannot copy in chunks
// The tiled kernels' loads write LDS directly in 16-byte chunks, so rows of a ragged length or a misaligned address are
// first brought into rows that are whole chunks.  A lane makes one chunk of 16 bytes at a time (one load at whatever
// address, element by element at the end of a row, zeros behind it), CopyVecs of them in flight; consecutive lanes
// write consecutive chunks.  Bound by memory, and mostly by the last-level cache, where the copies still are when the
// GEMM reads them.
constexpr int kCopyVecs = 4;
template <int ES>
__global__ __launch_bounds__(256) void copy_rows(const CopyArgs a) {
    using elem_t = typename std::conditional<ES == 4, uint32_t, uint16_t>::type;
    constexpr int W = 16 / ES;      // elements per chunk
    constexpr int V = kCopyVecs;
    const bool second = int64_t(blockIdx.x) >= a.part[0].blocks;
    const CopyArgs::Part p = a.part[second ? 1 : 0];
    const int64_t block = int64_t(blockIdx.x) - (second ? a.part[0].blocks : 0);
    const uint32_t per_row = uint32_t(p.ldd / W);
    const int64_t first = block * (256 * V), row0 = first / per_row;   // (the same for the workgroup)
    const uint32_t rem = uint32_t(first - row0 * per_row);
    u32x4 v[V];
    int64_t to[V];
#pragma unroll
    for (int i = 0; i < V; ++i) {
        const uint32_t c = rem + uint32_t(i) * 256 + threadIdx.x, down = c / per_row;
        const int64_t row = row0 + down, k = int64_t(c - down * per_row) * W;
        v[i] = u32x4{0u, 0u, 0u, 0u};
        to[i] = row < p.rows ? row * p.ldd + k : -1;
        if (row >= p.rows || k >= p.K) continue;
        const elem_t *src = reinterpret_cast<const elem_t *>(p.src) + row * p.lds + k;
        if (k + W <= p.K) {
            v[i] = reinterpret_cast<const AnyAligned<u32x4, ES> *>(src)->v;
        } else {
#pragma unroll
            for (int e = 0; e < W - 1; ++e)
                if (k + e < p.K) v[i][e * ES / 4] |= uint32_t(src[e]) << (8 * (e * ES % 4));
        }
    }
#pragma unroll
    for (int i = 0; i < V; ++i)
        if (to[i] >= 0) *reinterpret_cast<u32x4 *>(reinterpret_cast<elem_t *>(p.dst) + to[i]) = v[i];
}

// ------------------------------------------------------------------ split-K reduction
// One wave per (row, 256-column chunk), a lane per 4 consecutive columns: sums the S fp32 slabs
// in slab order, applies the ops that precede the row op, writes the value (final, or staged
// for the finalize pass) and, with a row op, the chunk's partial.
template <bool MAX>
__device__ __forceinline__ float wave_allreduce(float v) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const float o = __shfl_xor(v, d);
        v = MAX ? fmaxf(v, o) : v + o;
    }
    return v;
}

__global__ __launch_bounds__(256) void reduce_slabs(const RedArgs a) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t N = a.N;
    const int dtype = a.epi.dtype;
    const bool f32 = dtype == FLE_F32;
    const int64_t chunks = (N + 255) / 256, items = a.M * chunks;
    for (int64_t item = int64_t(blockIdx.x) * 4 + wave; item < items; item += int64_t(gridDim.x) * 4) {
        const int64_t row = item / chunks, c0 = (item % chunks) * 256;
        const int64_t n = c0 + lane * 4;
        const bool ok = n < N;  // at least the first of this lane's four columns exists
        const bool vec = n + 4 <= N;  // all of them: vector accesses, at whatever address the four lie on
        bool okc[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) okc[e] = n + e < N;
        f32x4 v = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        if (ok) {
            const float *src = a.slabs + row * a.ld_slab + n;  // slab rows are padded to whole groups of four
            int s = 0;
            for (; s + 4 <= a.S; s += 4) {
                const f32x4 u0 = *reinterpret_cast<const f32x4 *>(src + (s + 0) * a.stride);
                const f32x4 u1 = *reinterpret_cast<const f32x4 *>(src + (s + 1) * a.stride);
                const f32x4 u2 = *reinterpret_cast<const f32x4 *>(src + (s + 2) * a.stride);
                const f32x4 u3 = *reinterpret_cast<const f32x4 *>(src + (s + 3) * a.stride);
                v = (((v + u0) + u1) + u2) + u3;
            }
            for (; s < a.S; ++s) v += *reinterpret_cast<const f32x4 *>(src + s * a.stride);
            auto add4 = [&](const void *ptr, int64_t idx) {
                if (vec) {
                    v += ld4_any_rt(ptr, idx, dtype);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (okc[e]) v[e] += ld_elem(ptr, idx + e, dtype);
                }
            };
            for (int o = 0; o < a.epi.n_pre; ++o) {
                const DevOp op = a.epi.pre[o];
                switch (op.kind) {
                case FLE_BIAS: add4(a.epi.bias, n); break;
                case FLE_SCALE: v *= op.alpha; break;
                case FLE_RELU:
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = relu_f(v[e]);
                    break;
                case FLE_GELU_ERF:
                    gelu_erf_each<4>([&](auto &&f) __attribute__((always_inline)) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] = f(v[e], e);
                    });
                    break;
                case FLE_GELU_TANH:
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = gelu_tanh_f(v[e]);
                    break;
                case FLE_RESIDUAL: add4(op.p0, row * op.ld + n); break;
                case FLE_STORE: {  // a copy of the values as they stand, rounded to the dtype
                    void *tp = const_cast<void *>(op.p0);
                    if (!vec) {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (okc[e]) st_elem(tp, row * op.ld + n + e, dtype, v[e]);
                    } else {
                        st4_any_rt(tp, row * op.ld + n, dtype, v);
                    }
                    break;
                }
                default: break;
                }
            }
        }
        if (a.epi.row_kind >= 0) {
            float s0, s1;
            if (a.epi.row_kind == FLE_LAYERNORM) {
                const float cnt = float(N - c0 < 256 ? N - c0 : 256);
                float sum = 0.0f;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (okc[e]) sum += v[e];
                const float mean = wave_allreduce<false>(sum) / cnt;
                float m2 = 0.0f;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (okc[e]) m2 += (v[e] - mean) * (v[e] - mean);
                s0 = mean;
                s1 = wave_allreduce<false>(m2);
            } else {
                float mx = -INFINITY;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (okc[e]) mx = fmaxf(mx, v[e]);
                mx = wave_allreduce<true>(mx);
                float se = 0.0f;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (okc[e]) se += __expf(v[e] - mx);
                s0 = mx;
                s1 = wave_allreduce<false>(se);
            }
            if (lane == 0) *reinterpret_cast<float2 *>(a.partials + (row * a.np + c0 / 256) * 2) = make_float2(s0, s1);
            if (a.dst_rel) v -= s0;
        }
        if (a.dst && ok) {
            const bool d32 = a.dst_f32 || f32;
            if (!vec) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (okc[e]) st_elem(a.dst, row * a.ldd + n + e, d32 ? FLE_F32 : dtype, v[e]);
            } else {
                st4_any_rt(a.dst, row * a.ldd + n, d32 ? FLE_F32 : dtype, v);
            }
        }
    }
}

// ------------------------------------------------------------------ split-K reduction and row reduction in one pass
// The same sum for calls whose list goes on with one row reduction: WPR waves hold a whole row in registers (fp32, a lane 4
// columns of every 256 WPR), so the statistic, the normalisation and the ops behind it follow at once, the values are rounded
// once, and the call has a launch less: 16 x 128 x 4096 with LayerNorm in eight ranges 13.5 -> 10.3 us, 2048 x 4096 x 4096 in two 112 -> 107;
// what bounds it is the trips to the slabs, 8 groups of four columns per lane at a time (with two slabs at a time and the loads inside
// conditions 1 x 8192 x 4096 in eight ranges took 45 us, now 22.7, and 24.8 in two passes).
// Over 1024 columns the launch brings as many waves as the row has groups of 256 IT columns; with 16 for every row of over 2048 a CU held one row at a
// time, most of its loads past the row's end: 1556 x 2560 x 10240 in fp16 with LayerNorm, three ranges, 111 -> 101 us, 1200 x 3072 x
// 8192 84.2 -> 76.6, 16 x 2560 x 8192 20.5 -> 19.0.  Up to 1024 columns the number is fixed: reading it stands in front of the first
// load (this kernel on 700 x 1024 in fp16, two ranges: 4.6 us read, 4.3 fixed, 1001 columns 4.7 and 4.55).
template <int DT, int WPR, int IT>  // a workgroup of up to WPR waves holds a row of up to 256 IT columns per wave
__global__ __launch_bounds__(64 * WPR) void reduce_rows(const RedArgs a, const PostEpilogue post, void *out, int64_t ldo) {
    constexpr int U = 8 / IT;  // slabs requested at a time, added in their order
    __shared__ float lds[WPR];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int waves = IT == 1 ? WPR : int(blockDim.x >> 6);
    const int64_t N = a.N, row = blockIdx.x;
    int64_t n[IT], nv[IT], ns[IT];  // this lane's first columns; where it reads 4 of an operand and of a slab (past the end: the row's last)
    f32x4 v[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        n[it] = int64_t(it * waves + wave) * 256 + lane * 4;
        nv[it] = n[it] + 4 <= N ? n[it] : N >= 4 ? N - 4 : 0;
        ns[it] = n[it] < N ? n[it] : a.ld_slab - 4;  // slab rows are padded to whole groups of four
        v[it] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    // (No load stands inside a condition: each would then be waited for before the next one goes out.)
    const float *src = a.slabs + row * a.ld_slab;
    int s = 0;
    for (; s + U <= a.S; s += U) {
        f32x4 u[U][IT];
#pragma unroll
        for (int j = 0; j < U; ++j)
#pragma unroll
            for (int it = 0; it < IT; ++it) u[j][it] = *reinterpret_cast<const f32x4 *>(src + (s + j) * a.stride + ns[it]);
#pragma unroll
        for (int j = 0; j < U; ++j)
#pragma unroll
            for (int it = 0; it < IT; ++it) v[it] += u[j][it];
    }
    if (s < a.S) {  // the last few, clamped and left out past the end
        f32x4 u[U][IT];
#pragma unroll
        for (int j = 0; j < U; ++j)
#pragma unroll
            for (int it = 0; it < IT; ++it) u[j][it] = *reinterpret_cast<const f32x4 *>(src + (s + j < a.S ? s + j : s) * a.stride + ns[it]);
#pragma unroll
        for (int j = 0; j < U; ++j)
#pragma unroll
            for (int it = 0; it < IT; ++it)
                if (s + j < a.S) v[it] += u[j][it];
    }
    // 4 columns of an operand per group, `rest` where they are not there
    auto load4 = [&](f32x4 (&t)[IT], const void *p, int64_t base, float rest) {
        if (N >= 4) {
#pragma unroll
            for (int it = 0; it < IT; ++it) t[it] = ld4_any<DT>(p, base + nv[it]);
        }
#pragma unroll
        for (int it = 0; it < IT; ++it)
            if (n[it] + 4 > N) {  // (the row's last group, or none)
#pragma unroll
                for (int e = 0; e < 4; ++e) t[it][e] = n[it] + e < N ? ld_elem(p, base + n[it] + e, DT) : rest;
            }
    };
    auto add_row = [&](const void *p, int64_t base) {
        f32x4 t[IT];
        load4(t, p, base, 0.0f);
#pragma unroll
        for (int it = 0; it < IT; ++it) v[it] += t[it];
    };
    auto put4 = [&](int it, void *p, int64_t base) {
        if (n[it] + 4 <= N) {
            st4_any<DT>(p, base + n[it], v[it]);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n[it] + e < N) st_elem(p, base + n[it] + e, DT, v[it][e]);
        }
    };
    auto apply = [&](const DevOp &op) {
        switch (op.kind) {
        case FLE_BIAS:
            add_row(a.epi.bias, 0);
            break;
        case FLE_SCALE:
#pragma unroll
            for (int it = 0; it < IT; ++it) v[it] *= op.alpha;
            break;
        case FLE_RELU:
#pragma unroll
            for (int it = 0; it < IT; ++it)
#pragma unroll
                for (int e = 0; e < 4; ++e) v[it][e] = relu_f(v[it][e]);
            break;
        case FLE_GELU_ERF:
            gelu_erf_each<IT * 4>([&](auto &&f) __attribute__((always_inline)) {
#pragma unroll
                for (int it = 0; it < IT; ++it)
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[it][e] = f(v[it][e], it * 4 + e);
            });
            break;
        case FLE_GELU_TANH:
#pragma unroll
            for (int it = 0; it < IT; ++it)
#pragma unroll
                for (int e = 0; e < 4; ++e) v[it][e] = gelu_tanh_f(v[it][e]);
            break;
        case FLE_RESIDUAL:
            add_row(op.p0, row * op.ld);
            break;
        case FLE_STORE:
#pragma unroll
            for (int it = 0; it < IT; ++it)
                if (n[it] < N) put4(it, const_cast<void *>(op.p0), row * op.ld);
            break;
        default: break;
        }
    };
    for (int o = 0; o < a.epi.n_pre; ++o) apply(a.epi.pre[o]);

    auto over_row = [&](float t, auto max_c) -> float {
        constexpr bool MAX = decltype(max_c)::value;
        t = row16_allreduce<MAX>(t);
        const float o1 = __shfl_xor(t, 16);
        t = MAX ? fmaxf(t, o1) : t + o1;
        const float o2 = __shfl_xor(t, 32);
        t = MAX ? fmaxf(t, o2) : t + o2;
        __syncthreads();  // (the previous use of lds is over)
        if (lane == 0) lds[wave] = t;
        __syncthreads();
        t = lds[0];
#pragma unroll
        for (int w = 1; w < WPR; ++w) {
            const float o = lds[w];
            t = w >= waves ? t : MAX ? fmaxf(t, o) : t + o;
        }
        return t;
    };
    if (post.row_kind == FLE_LAYERNORM) {
        float sum = 0.0f;
#pragma unroll
        for (int it = 0; it < IT; ++it)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n[it] + e < N) sum += v[it][e];
        const float mean = over_row(sum, std::false_type{}) / float(N);
        float m2 = 0.0f;
#pragma unroll
        for (int it = 0; it < IT; ++it)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n[it] + e < N) m2 += (v[it][e] - mean) * (v[it][e] - mean);
        const float mul = rsqrtf(over_row(m2, std::false_type{}) / float(N) + post.row.alpha);
        f32x4 g[IT], be[IT];  // (one multiply-add behind the normalisation, as in the finalize pass: a rounding less than two steps)
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            g[it] = f32x4{1.0f, 1.0f, 1.0f, 1.0f};
            be[it] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
        if (post.row.p0) load4(g, post.row.p0, 0, 1.0f);
        if (post.row.p1) load4(be, post.row.p1, 0, 0.0f);
#pragma unroll
        for (int it = 0; it < IT; ++it)
#pragma unroll
            for (int e = 0; e < 4; ++e) v[it][e] = fmaf((v[it][e] - mean) * mul, g[it][e], be[it][e]);
    } else {
        float mx = -INFINITY;
#pragma unroll
        for (int it = 0; it < IT; ++it)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n[it] + e < N) mx = fmaxf(mx, v[it][e]);
        mx = over_row(mx, std::true_type{});
        float sum = 0.0f;
#pragma unroll
        for (int it = 0; it < IT; ++it)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n[it] + e < N) {
                    v[it][e] = __expf(v[it][e] - mx);
                    sum += v[it][e];
                }
        sum = over_row(sum, std::false_type{});
        if (post.row_kind == FLE_LOGSUMEXP) {
            if (threadIdx.x == 0) st_elem(out, row, DT, mx + __logf(sum));
            return;
        }
        const float mul = 1.0f / sum;
#pragma unroll
        for (int it = 0; it < IT; ++it) v[it] *= mul;
    }
    for (int o = 0; o < post.n_post; ++o) apply(post.post[o]);
#pragma unroll
    for (int it = 0; it < IT; ++it)
        if (n[it] < N) put4(it, out, row * ldo);
}

}  // namespace fle
