// Attention of a few new queries (T <= 32 per sequence) against many kept keys: bound by reading K and V once.
#pragma once
#include "fle_attention.h"

namespace fle {

// The 128-query kernel gives such a call one workgroup per sequence and head, of which one wave has queries at all: 4
// sequences x 16 heads of 128 over 8192 keys kept 64 CUs busy with one wave each and streamed at 1.4 TB/s.  Here the
// waves of a workgroup take the key blocks in turn (32 keys each, all for the same single tile of up to 32
// queries), every wave with its own running softmax, and when sequences x heads do not fill the chip the keys are cut
// into `splits` ranges, one workgroup each; the waves' results meet in LDS, the ranges' in the workspace
// (decode_combine).  The waves share nothing until then, so the loop has no barrier: a wave keeps two blocks of K and V in its
// own part of LDS and refills the K half of a stage as soon as the scores are out of it, the V half after the second
// product, so that three quarters of its 2 x 2 buffers are in flight at any time.  Whole calls on new
// operands each time, bf16, against the 128-query kernel: 4 x 16 heads of 128, one query, 8192 keys 190 -> 52 us (5.2
// TB/s); 7 x 16 heads, 2 queries, 15769 keys 378 -> 151; 1 x 16 heads, 16384 keys 187 -> 21; 32 x 12 heads of 256, 512 keys
// 64 -> 39; with enough heads for every CU, 64 x 8 heads of 64 over 2000 keys, 48.3 -> 47.4.
//
// The matrix instructions (laid out as in flash_attention: a lane owns one query) work on mostly empty
// query columns, which costs nothing here: 2 x D / 16 of them per block of 32 keys take a quarter of the time that the
// block's bytes take to arrive.
constexpr int kDecodeQueries = 32;  // queries of one tile
constexpr int kDecodeKeys = 32;     // keys per block of a wave

struct DecodeArgs {
    AttnArgs at;
    int32_t splits;   // key ranges per sequence and head; > 1: partial results go to part, else the result to at.o
    int32_t n_blocks; // blocks of 32 keys
    float *part;      // [splits][B*T*H][D] unnormalised sums over the range's keys
    float *stat;      // [splits][B*T*H][2] reference point (base 2) and sum of the range's exponentials
};

// The copy of 1 KB of one operand into LDS (a member: the builtin is not accepted inside a lambda of a kernel template).
// K and V are read once, so the copies carry the non-temporal hint (4.5 -> 5.2 TB/s at 4 x 16 heads of 128 over 8192
// keys, 4.8 -> 5.3 at 64 x 8 heads of 64 over 2000); at head dimension 32 a row of a head is half a cache line, whose other half
// the next head's workgroup wants, and the hint costs 8 - 14 %.
template <bool ONCE>
struct BufferOne {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ void copy_1k(char *dst, uint32_t off) const { __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void *)dst, 16, off, 0, 0, ONCE ? 2 : 0); }
};

constexpr int decode_waves(int D) { return D == 256 ? 1 : D == 128 ? 2 : 4; }

// Two stages per wave and one, two or four waves make 64 KB of LDS, two workgroups per CU, so that one starts up or ends
// while the other streams (32 KB and four workgroups at D = 32).  Twice the waves at D = 128 and 256, one workgroup per CU:
// 20 x 16 heads of 128 over 1000 keys 51 us against 37, 32 x 12 heads of 256 over 512 keys 52 against 41.
template <int DT, int D>
__global__ __launch_bounds__(D == 256 ? 64 : D == 128 ? 128 : 256) __attribute__((amdgpu_waves_per_eu(D >= 128 ? 1 : D == 64 ? 2 : 4, D >= 128 ? 1 : D == 64 ? 2 : 4))) void decode_attention(const DecodeArgs da) {
    static_assert(DT == FLE_BF16 || DT == FLE_F16, "2-byte dtypes only");
    static_assert(D == 32 || D == 64 || D == 128 || D == 256, "head dimension 32, 64, 128 or 256");
    using frag_t = typename std::conditional<DT == FLE_F16, f16x8, bf16x8>::type;
    constexpr int NW = decode_waves(D), BKV = kDecodeKeys, NST = 2;
    constexpr int NC = D / 16, ND = D / 32, RB = D * 2, CPR = D / 8, HALF = BKV * RB;
    __shared__ __attribute__((aligned(16))) char smem[NW * NST * 2 * HALF];
    __shared__ float stat_m[NW][kDecodeQueries], stat_l[NW][kDecodeQueries];
    const AttnArgs &a = da.at;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l31 = lane & 31, h2 = lane >> 5;
    const int T = a.T, Tk = a.Tk;
    // Items in the order (range, sequence, head), the heads of a sequence next to each other in the rows they read.  They go
    // to the workgroups, and so to the 8 XCDs, in turn; at head dimension 32 an XCD takes a contiguous share, so
    // that the two heads of a cache line find it in one L2 (100 -> 79 us at 40 x 16 heads over 3000 keys; contiguous
    // shares at 64 and more: 1 - 8 % slower).
    const uint32_t n_heads = uint32_t(a.H) * uint32_t(a.B);
    uint32_t item = blockIdx.x;
    if constexpr (D == 32) {
        const uint32_t per = gridDim.x / 8, rem = gridDim.x % 8, xcd = blockIdx.x % 8;
        item = blockIdx.x / 8 + xcd * per + (xcd < rem ? xcd : rem);
    }
    const int split = int(item / n_heads);
    const uint32_t head = item % n_heads;
    const int64_t seq = head / uint32_t(a.H), hcol = head % uint32_t(a.H);
    const int64_t col0 = hcol * D;
    const char *qp = reinterpret_cast<const char *>(a.q) + (seq * a.sbq + col0) * 2;
    const char *kp = reinterpret_cast<const char *>(a.k) + (seq * a.sbk + col0) * 2;
    const char *vp = reinterpret_cast<const char *>(a.v) + (seq * a.sbv + col0) * 2;

    // this range's blocks (ranges differ by at most one block), of which wave w takes the w-th, (w + NW)-th, ...
    const int b0 = int(int64_t(da.n_blocks) * split / da.splits), b1 = int(int64_t(da.n_blocks) * (split + 1) / da.splits);
    const int mine = b1 - b0 > wave ? (b1 - b0 - wave + NW - 1) / NW : 0;

    // keys visible to this lane's query (as in flash_attention)
    const int G = a.causal;
    auto limit_of = [&](int query) {
        const int lim = G ? ((query + Tk - T) / G + 1) * G : Tk;
        return lim < Tk ? lim : Tk;
    };
    const int key_limit = limit_of(l31 < T ? l31 : T - 1), first_limit = limit_of(0);

    frag_t qf[NC];
    {
        const __amdgpu_buffer_rsrc_t rsrc_q = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(qp), 0, uint32_t(int64_t(T - 1) * a.ldq * 2 + RB), 0x00020000);
        const uint32_t off = uint32_t(l31) * uint32_t(a.ldq * 2) + uint32_t(16 * h2);  // rows at or beyond T read as zeros
#pragma unroll
        for (int c = 0; c < NC; ++c) qf[c] = __builtin_bit_cast(frag_t, __builtin_amdgcn_raw_buffer_load_b128(rsrc_q, off + 32 * c, 0, 0));
    }

    f32x16 oacc[ND];
    float m_run = -INFINITY, l_run = 0.0f;
#pragma unroll
    for (int dt = 0; dt < ND; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[dt][r] = 0.0f;

    // Copies as in flash_attention: 1 KB (RPI rows) per instruction, the XOR placement applied on the source side.  A
    // block past the wave's last one is requested at an offset beyond the buffer: zeros, no memory traffic, and the
    // number of copies in flight stays the same to the end.
    constexpr int RPI = 1024 / RB, NI = BKV / RPI;  // rows per instruction; instructions per block and operand
    BufferOne<(D > 32)> rk, rv;
    rk.r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(kp), 0, uint32_t(int64_t(Tk - 1) * a.ldk * 2 + RB), 0x00020000);
    rv.r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(vp), 0, uint32_t(int64_t(Tk - 1) * a.ldv * 2 + RB), 0x00020000);
    uint32_t cp_k[NI], cp_v[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int row = i * RPI + lane / CPR, pos = lane % CPR;
        cp_k[i] = uint32_t(row) * uint32_t(a.ldk * 2) + uint32_t((pos ^ lds_swizzle<D>(row)) * 16);
        cp_v[i] = uint32_t(row) * uint32_t(a.ldv * 2) + uint32_t((pos ^ lds_swizzle<D>(row)) * 16);
    }
    char *const own = smem + wave * (NST * 2 * HALF);
    auto copy_k = [&](int st, int j) {
        const uint32_t k0 = j < mine ? uint32_t((b0 + wave + j * NW) * BKV) * uint32_t(a.ldk * 2) : 0x80000000u;
#pragma unroll
        for (int i = 0; i < NI; ++i) rk.copy_1k(own + st * 2 * HALF + i * 1024, cp_k[i] + k0);
    };
    auto copy_v = [&](int st, int j) {
        const uint32_t v0 = j < mine ? uint32_t((b0 + wave + j * NW) * BKV) * uint32_t(a.ldv * 2) : 0x80000000u;
#pragma unroll
        for (int i = 0; i < NI; ++i) rv.copy_1k(own + st * 2 * HALF + HALF + i * 1024, cp_v[i] + v0);
    };

    int koff[NC];  // K fragment (A operand): row l31, 16-byte chunk 2 c + h2
#pragma unroll
    for (int c = 0; c < NC; ++c) koff[c] = l31 * RB + (((2 * c + h2) ^ lds_swizzle<D>(l31)) * 16);
    const int vj = lane & 15, vg = lane >> 4;
    const int v_key = (vj >> 2) + 4 * (vg >> 1), v_d = 16 * (vg & 1) + 4 * (vj & 3);
    int voff[ND][2];  // V^T fragment, transposing reads
#pragma unroll
    for (int dt = 0; dt < ND; ++dt)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int key = 8 * e + v_key, d = 32 * dt + v_d;
            voff[dt][e] = HALF + key * RB + (((d >> 3) ^ lds_swizzle<D>(key)) * 16) + (d & 7) * 2;
        }

    // LDS accesses stay on their side of a counted wait
    auto hold_order = [] {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    auto block_step = [&](int st, int j) {
        const char *stage = own + st * 2 * HALF;
        const int kb0 = (b0 + wave + j * NW) * BKV;
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.0f;
        wait_vmcnt<3 * NI>();  // this block's K has landed; its V and the next block's K and V may be on their way
        hold_order();
        frag_t kf[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) kf[c] = *reinterpret_cast<const frag_t *>(stage + koff[c]);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if constexpr (DT == FLE_F16) s = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[c], qf[c], s, 0, 0, 0);
            else s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[c], qf[c], s, 0, 0, 0);
        }
        hold_order();
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the stage's K is in registers before it is overwritten
        hold_order();
        copy_k(st, j + NST);
        if (kb0 + BKV > first_limit) {  // diagonal and tail blocks only (uniform over the wave)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (kb0 + 8 * (r / 4) + 4 * h2 + (r % 4) >= key_limit) s[r] = -INFINITY;
        }
        float mx = s[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float cand = mx * a.scale_log2e;
        // the reference point moves when a maximum has grown past it by more than 2^8 (see flash_attention); it stays
        // at -inf while a query has met only masked keys, whose exponentials are then taken against 0
        const bool grow = cand > m_run + 8.0f;
        if (__builtin_amdgcn_ballot_w64(grow) != 0) {
            const float m_new = grow ? cand : m_run;
            const float alpha = grow ? __builtin_amdgcn_exp2f(m_run - m_new) : 1.0f;
            m_run = m_new;
            l_run *= alpha;
#pragma unroll
            for (int dt = 0; dt < ND; ++dt)
#pragma unroll
                for (int r = 0; r < 16; ++r) oacc[dt][r] *= alpha;
        }
        const float m_ref = m_run == -INFINITY ? 0.0f : m_run;
        float ps = 0.0f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            s[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], a.scale_log2e, -m_ref));
            ps += s[r];
        }
        ps += __shfl_xor(ps, 32);
        l_run += ps;
        frag_t pf[2];
#pragma unroll
        for (int c2 = 0; c2 < 2; ++c2) {
            const u32x2 lo = pack4<DT>(f32x4{s[8 * c2 + 0], s[8 * c2 + 1], s[8 * c2 + 2], s[8 * c2 + 3]});
            const u32x2 hi = pack4<DT>(f32x4{s[8 * c2 + 4], s[8 * c2 + 5], s[8 * c2 + 6], s[8 * c2 + 7]});
            pf[c2] = __builtin_bit_cast(frag_t, u32x4{lo[0], lo[1], hi[0], hi[1]});
        }
        hold_order();
        wait_vmcnt<3 * NI>();  // this block's V; behind it the next block's K and V and the refill of this block's K
        hold_order();
#pragma unroll
        for (int c2 = 0; c2 < 2; ++c2)
#pragma unroll
            for (int dt = 0; dt < ND; ++dt) {
                struct { i16x4 e[2]; } part;
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    part.e[e] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4 *)(stage + voff[dt][e] + 16 * c2 * RB));
                const frag_t vf = __builtin_bit_cast(frag_t, part);
                if constexpr (DT == FLE_F16) oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf, pf[c2], oacc[dt], 0, 0, 0);
                else oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[c2], oacc[dt], 0, 0, 0);
            }
        hold_order();
        __builtin_amdgcn_s_waitcnt(0xC07F);
        hold_order();
        copy_v(st, j + NST);
    };
    if (mine > 0) {
        copy_k(0, 0);
        copy_v(0, 0);
        copy_k(1, 1);
        copy_v(1, 1);
#pragma unroll
        for (int c = 0; c < NC; ++c) asm volatile("" : "+v"(qf[c]));  // the wait for Q comes here, counted, and not as a full one in front of the loop
        for (int j = 0; j < mine; j += 2) {
            block_step(0, j);
            if (j + 1 < mine) block_step(1, j + 1);
        }
        wait_vmcnt<0>();  // nothing may still be landing in LDS when it is used for something else
    }

    // The waves' results meet in LDS: sums over keys [wave][query][D] (a row starts 4 floats further than a multiple of
    // 32 banks), reference points and exponential sums [wave][query].
    __syncthreads();
    constexpr int OLD = D + 4;
    static_assert(NW * kDecodeQueries * OLD * 4 <= int(sizeof(smem)), "the waves' sums fit the stages");
    float *const osum = reinterpret_cast<float *>(smem);
    const int rows = T;
    if (l31 < rows) {
#pragma unroll
        for (int dt = 0; dt < ND; ++dt)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *reinterpret_cast<f32x4 *>(osum + (wave * rows + l31) * OLD + 32 * dt + 8 * g + 4 * h2) =
                    f32x4{oacc[dt][4 * g], oacc[dt][4 * g + 1], oacc[dt][4 * g + 2], oacc[dt][4 * g + 3]};
        if (h2 == 0) {
            stat_m[wave][l31] = m_run;
            stat_l[wave][l31] = l_run;
        }
    }
    __syncthreads();
    for (int i = tid; i < rows * (D / 4); i += 64 * NW) {
        const int query = i / (D / 4), d = 4 * (i % (D / 4));
        float m = stat_m[0][query];
#pragma unroll
        for (int w = 1; w < NW; ++w) m = fmaxf(m, stat_m[w][query]);
        f32x4 o = {0.0f, 0.0f, 0.0f, 0.0f};
        float l = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float mw = stat_m[w][query], f = mw == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(mw - m);
            if (mw == -INFINITY && stat_l[w][query] == 0.0f) continue;  // no visible key among this wave's
            l += f * stat_l[w][query];
            o += f * *reinterpret_cast<const f32x4 *>(osum + (w * rows + query) * OLD + d);
        }
        const int64_t row = (seq * T + query) * a.H + hcol;
        if (da.splits > 1) {
            const int64_t slot = int64_t(split) * a.B * T * a.H + row;
            *reinterpret_cast<f32x4 *>(da.part + slot * D + d) = o;
            if (d == 0) *reinterpret_cast<float2 *>(da.stat + slot * 2) = make_float2(m, l);
        } else {
            *reinterpret_cast<u32x2 *>(reinterpret_cast<char *>(a.o) + (seq * a.sbo + int64_t(query) * a.ldo + col0 + d) * 2) = pack4<DT>(o * (1.0f / l));
        }
    }
}

// The ranges of a row put together, in a fixed order: one wave per (token, head), lane s holding range s's reference
// point and sum; D / 4 lanes read one range's sums, the 256 / D groups of lanes take the ranges in turn.
template <int DT, int D>
__global__ __launch_bounds__(256) void decode_combine(const DecodeArgs da) {
    const AttnArgs &a = da.at;
    const int lane = threadIdx.x & 63;
    const int64_t rows = int64_t(a.B) * a.T * a.H, row = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    float2 st = make_float2(-INFINITY, 0.0f);
    if (lane < da.splits) st = *reinterpret_cast<const float2 *>(da.stat + (lane * rows + row) * 2);
    float m = st.x;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) m = fmaxf(m, __shfl_xor(m, d));
    const float f = st.x == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(st.x - m);
    // a range without a visible key has no part; one whose factor underflows has (a NaN or infinity in its sums stays one)
    const bool seen = !(st.x == -INFINITY && st.y == 0.0f);
    const uint64_t ranges = __builtin_amdgcn_ballot_w64(lane < da.splits && seen);
    float l = seen ? f * st.y : 0.0f;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) l += __shfl_xor(l, d);
    constexpr int LPR = D / 4, NG = 64 / LPR;
    const int grp = lane / LPR, d0 = 4 * (lane % LPR);
    f32x4 o = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int s0 = 0; s0 < da.splits; s0 += NG) {  // (uniform: every lane takes part in the exchange of the factors)
        const int s = s0 + grp;
        const float fs = __shfl(f, s < da.splits ? s : 0);
        if (s < da.splits && (ranges >> s & 1)) o += fs * *reinterpret_cast<const f32x4 *>(da.part + (s * rows + row) * D + d0);
    }
#pragma unroll
    for (int d = LPR; d < 64; d <<= 1)
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] += __shfl_xor(o[e], d);
    if (grp == 0) {
        const int64_t h = row % a.H, tok = row / a.H, t = tok % a.T, seq = tok / a.T;
        *reinterpret_cast<u32x2 *>(reinterpret_cast<char *>(a.o) + (seq * a.sbo + t * a.ldo + h * D + d0) * 2) = pack4<DT>(o * (1.0f / l));
    }
}

}  // namespace fle
