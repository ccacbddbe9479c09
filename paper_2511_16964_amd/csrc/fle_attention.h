// Scaled dot-product attention (forward), one pass over the keys with a running softmax.
#pragma once
#include "fle_device_common.h"

namespace fle {

typedef __attribute__((ext_vector_type(4))) short i16x4;
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;

// The transposing LDS read.  __restrict tells the compiler that a copy into LDS that is still on its way does not write
// what is read here; without it every such read waits for all copies (s_waitcnt vmcnt(0) in the middle of a block).
__device__ __forceinline__ i16x4 read_transposed(lds_i16x4 *__restrict p) { return __builtin_amdgcn_ds_read_tr16_b64_v4i16(p); }

#ifndef FLE_ATTN_HEAD_GROUP
#define FLE_ATTN_HEAD_GROUP 8u  // heads an XCD works on at a time (see the workgroup mapping)
#endif

struct AttnArgs {
    const void *q, *k, *v;
    void *o;
    int64_t ldq, ldk, ldv, ldo;  // elements between consecutive tokens
    int64_t sbq, sbk, sbv, sbo;  // elements between consecutive sequences
    int32_t T, Tk, H, B;         // queries and keys per sequence, heads, sequences
    int32_t causal;     // 0: no mask; G >= 1: query t sees the keys below (t / G + 1) * G (G = 1: the plain causal mask)
    float scale_log2e;  // softmax scale times log2(e): the exponentials are taken in base 2
};

// 1 KB from a buffer into LDS: every lane brings 16 bytes from its own offset, the wave writes consecutive addresses.
__device__ __forceinline__ void copy_1k(__amdgpu_buffer_rsrc_t rsrc, char *dst, uint32_t off) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void *)dst, 16, off, 0, 0, 0);
}

// Order of a straight-line stretch of MFMAS matrix instructions, each followed by READS LDS reads for a later one and VALU
// vector instructions, which run while it occupies the matrix pipe.
template <int MFMAS, int READS, int VALU>
__device__ __forceinline__ void interleave() {
#pragma unroll
    for (int i = 0; i < MFMAS; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, READS, 0);
        if (VALU > 0) __builtin_amdgcn_sched_group_barrier(0x402, VALU, 0);
    }
}

// The values of lane & 31 and of (lane & 31) + 32.
struct Halves { float lo, hi; };
__device__ __forceinline__ Halves halves_of(float v) {
    const uint32_t b = __builtin_bit_cast(uint32_t, v);
    const auto r = __builtin_amdgcn_permlane32_swap(b, b, false, false);  // {low half twice, high half twice}
    return {__builtin_bit_cast(float, uint32_t(r[0])), __builtin_bit_cast(float, uint32_t(r[1]))};
}

// acc *= f for accumulators that stay in accumulation registers on both sides (as ordinary values all of them would be read out and
// written back in every block, whether they are scaled or not).  The compiler sees neither what these lines read nor what they
// write, so the waits are part of them: the first waits out the last matrix instruction of every tile (19 states at the most), the last the
// write in front of the next one (2).
template <int N>
__device__ __forceinline__ void scale_in_place(f32x16 (&acc)[N], float f) {
    static_assert(N == 8, "one operand per tile");
    auto wait_for_all = [&]() {
        float e[N];
#pragma unroll
        for (int i = 0; i < N; ++i) e[i] = acc[i][15];
        asm volatile("s_nop 15\n\ts_nop 7" : "+a"(e[0]), "+a"(e[1]), "+a"(e[2]), "+a"(e[3]), "+a"(e[4]), "+a"(e[5]), "+a"(e[6]), "+a"(e[7]));
#pragma unroll
        for (int i = 0; i < N; ++i) acc[i][15] = e[i];
    };
    wait_for_all();
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float x = acc[i][r], t;
            asm volatile("v_accvgpr_read_b32 %1, %0\n\tv_mul_f32 %1, %1, %2\n\tv_accvgpr_write_b32 %0, %1" : "+a"(x), "=&v"(t) : "v"(f));
            acc[i][r] = x;
        }
    wait_for_all();
}

// Placement of the 16-byte chunks of a K / V row in LDS: chunk c of row r sits at position c ^ lds_swizzle(r).
// Two access patterns must spread over all banks (256 bytes per cycle): the K fragment reads (16 consecutive
// rows, the same chunk of each) and the transposing V reads (32 lanes = 4 consecutive rows x 64 contiguous
// bytes).  The first needs 16 consecutive rows to land on 16 different 16-byte positions of a 256-byte bank
// sweep, the second needs rows r .. r + 3 (r a multiple of 4) to move a 64-byte group to 4 different groups.
// D >= 128 (a row is one or two sweeps): the two low row bits go to chunk bits 3 and 2, the next two to the
// low ones.  D = 64 (two rows per sweep, 8 chunks; row parity picks the half sweep): row bit 1 goes to the
// high chunk bit, bits 2 and 3 to the low ones.  D = 32 (four rows per sweep, a row is one 64-byte group, so
// the V reads need nothing): row bits 2 and 3 pick among the four chunks.
template <int D>
__device__ __forceinline__ int lds_swizzle(int row) {
    if constexpr (D >= 128) return ((row & 3) << 2) | ((row >> 2) & 3);
    else if constexpr (D == 64) return (((row >> 1) & 1) << 2) | ((row >> 2) & 3);
    else return (row >> 2) & 3;
}

// Everything is computed transposed, so that a lane owns one query:
//
//     S^T[key, query] = K[key, :] . Q[query, :]          v_mfma_f32_32x32x16 (A = K rows, B = Q rows)
//     O^T[d,   query] += V^T[d, key] * P^T[key, query]   v_mfma_f32_32x32x16 (A = V^T,    B = P^T)
//
// In the 32x32 result layout a lane holds column (lane & 31) -- its query -- and 16 rows, so the
// running maximum, the running sum and the rescaling factor of a query are per-lane scalars (one
// exchange with lane ^ 32 completes a reduction over keys), and the exponentiated S^T registers,
// rounded to the storage dtype, are already laid out as the B operand of the second product: result
// register r of the lane half h = lane >> 5 is key 8 (r / 4) + 4 h + r % 4, so registers 8 c .. 8 c + 7
// are K-slots (h, 0 .. 7) of the 16-key step c, i.e. keys 16 c + 4 h + {0..3} and 16 c + 8 + 4 h + {0..3}.
// The A operand V^T is gathered in the same key order straight from the row-major V block in LDS with
// ds_read_b64_tr_b16: within 16 lanes, source lane j points at 4 consecutive d of key j / 4, and lane i
// receives d = i of those four keys.  A sum over keys does not care about their order, only that both
// operands agree on it.
//
// A workgroup is 4 waves of 32 queries each that walk the same key blocks of 64 through LDS, double buffered (buffer loads
// that write LDS directly), one barrier per block.  Rows of K / V are stored with their 16-byte chunks XOR-ed by
// lds_swizzle(row), which spreads both the row-wise reads of K and the transposing reads of V over all banks.  With the
// causal mask a wave stops computing at its last visible block and only keeps the barriers; the mask itself is applied on
// the diagonal and tail blocks only.
//
// What bounds it: per block and wave the matrix instructions (1024 cycles at D = 128) and about as many cycles of
// exponentials, maxima, sums and conversions.  A wave that does one after the other leaves the overlap to the second wave
// of its SIMD; so it holds the scores of two blocks, and in one straight-line stretch the scores of the next
// block and the second product of this one run on the matrix pipe while the vector instructions of this block are issued
// between them (interleave), and no transposing read waits for the copies (read_transposed).  D = 128, bf16, 16 heads,
// 2 x 8192 tokens, causal: 521 -> 482 us; 5 x 2311 tokens, 8 heads, no mask: 119 -> 111; 16 x 2048, causal: 332 -> 318;
// D = 64, 9 x 1682 tokens, 8 heads, causal: 53.5 -> 49.2.  At D = 256 the sums and the scores of both blocks (192 registers) stay in
// accumulation registers: the sums are scaled there (scale_in_place), the scores read out once.  One block at a time, with all
// sums moved out and back in every block, took 1195 us on 2 x 6607 tokens x 8 heads without a mask where this takes 770, 460 on
// 8 x 2048 x 16 causal (352), 90 on 16 x 400 x 16 causal (72), 173 on 57 x 132 x 25 causal (156); the same bits.
//
// The kernel states the occupancy it is built for (WAVES per SIMD: one at D = 256, two at 128, three below): left to
// itself the register allocator aims one step higher, caps the ordinary VGPRs accordingly and parks the
// output accumulators in AGPRs, copying all of them in and out on every trip of the loop.
template <int DT, int D, int WAVES>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WAVES, WAVES))) void flash_attention(const AttnArgs a) {
    static_assert(DT == FLE_BF16 || DT == FLE_F16, "2-byte dtypes only");
    static_assert(D == 32 || D == 64 || D == 128 || D == 256, "head dimension 32, 64, 128 or 256");
    using frag_t = typename std::conditional<DT == FLE_F16, f16x8, bf16x8>::type;
    constexpr int BKV = 64, WQ = 32, BQ = 4 * WQ;
    constexpr int NC = D / 16, ND = D / 32, RB = D * 2, CPR = D / 8;
    constexpr int STAGE = 2 * BKV * RB;
    __shared__ __attribute__((aligned(16))) char smem[2 * STAGE];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l31 = lane & 31, h2 = lane >> 5;
    const int T = a.T, Tk = a.Tk;
    const int n_qb = (T + BQ - 1) / BQ;
    // Workgroup -> (sequence and head, query block).  Consecutive workgroups go to the 8 XCDs in turn, so
    // workgroup L is the (L / 8)-th one of XCD L % 8.  An XCD takes consecutive heads whole (every query block
    // of a head reads the same K and V, which then stay in that XCD's L2) and, under the causal mask, each
    // head's blocks from the longest to the shortest; handing out query blocks in plain order instead gives
    // XCD j block j of every head, i.e. all the long blocks to one XCD and all the short ones to another.
    const uint32_t n_heads = uint32_t(a.H) * uint32_t(a.B), xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
    int head, qi;
    if (n_heads % 8 == 0) {
        // heads xcd * hpx .. + hpx - 1, in groups of FLE_ATTN_HEAD_GROUP heads that are worked on together
        // (their K and V share the L2), each group block-major: all its longest query blocks first
        const uint32_t hpx = n_heads / 8, gsz = FLE_ATTN_HEAD_GROUP * uint32_t(n_qb);
        const uint32_t g = slot / gsz, u = slot - g * gsz;
        const uint32_t left = hpx - g * FLE_ATTN_HEAD_GROUP, gh = left < FLE_ATTN_HEAD_GROUP ? left : FLE_ATTN_HEAD_GROUP;
        qi = int(u / gh);
        head = int(xcd * hpx + g * FLE_ATTN_HEAD_GROUP + u % gh);
    } else {
        const uint32_t n_items = n_heads * uint32_t(n_qb), per = n_items / 8, rem = n_items % 8;
        const uint32_t item = slot + xcd * per + (xcd < rem ? xcd : rem);  // XCD j owns a contiguous range of items
        head = int(item / uint32_t(n_qb));
        qi = int(item % uint32_t(n_qb));
    }
    const int qb = a.causal ? n_qb - 1 - qi : qi;
    const int q0 = qb * BQ, wq0 = q0 + wave * WQ;
    const int64_t seq = head / a.H;
    const int64_t col0 = int64_t(head % a.H) * D;
    const char *qp = reinterpret_cast<const char *>(a.q) + (seq * a.sbq + col0) * 2;
    const char *kp = reinterpret_cast<const char *>(a.k) + (seq * a.sbk + col0) * 2;
    const char *vp = reinterpret_cast<const char *>(a.v) + (seq * a.sbv + col0) * 2;
    char *op = reinterpret_cast<char *>(a.o) + (seq * a.sbo + col0) * 2;

    // Keys 0 .. limit - 1 are visible to a query; limits grow with the query index, so the last query of a
    // workgroup (of a wave) decides how many key blocks it walks and the first one whether a block needs the mask.
    // Under a mask the T queries stand at the last T of the Tk key positions.
    const int G = a.causal;
    auto limit_of = [&](int query) {
        const int lim = G ? ((query + Tk - T) / G + 1) * G : Tk;
        return lim < Tk ? lim : Tk;
    };
    const int q_last = (q0 + BQ < T ? q0 + BQ : T) - 1, w_last = (wq0 + WQ < T ? wq0 + WQ : T) - 1;
    const int n_blocks = (limit_of(q_last) + BKV - 1) / BKV;
    const int wave_last = wq0 < T && limit_of(w_last) > 0 ? (limit_of(w_last) + BKV - 1) / BKV - 1 : -1;  // a wave of padding rows only keeps the barriers
    const int wave_first_limit = limit_of(wq0), w_limit = limit_of(w_last);
    const int key_limit = limit_of(wq0 + l31);

    // Q fragments stay in registers: B operand, lane = query, 8 consecutive d per 16-wide step
    frag_t qf[NC];
    {
        const __amdgpu_buffer_rsrc_t rsrc_q = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(qp), 0, uint32_t(int64_t(T - 1) * a.ldq * 2 + RB), 0x00020000);
        const uint32_t off = uint32_t(wq0 + l31) * uint32_t(a.ldq * 2) + uint32_t(16 * h2);  // rows at or beyond T read as zeros
#pragma unroll
        for (int c = 0; c < NC; ++c) qf[c] = __builtin_bit_cast(frag_t, __builtin_amdgcn_raw_buffer_load_b128(rsrc_q, off + 32 * c, 0, 0));
    }

    f32x16 oacc[ND];
    float m_run = -INFINITY, l_run = 0.0f;
#pragma unroll
    for (int dt = 0; dt < ND; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[dt][r] = 0.0f;
    auto mma = [](frag_t x, frag_t y, f32x16 c) {
        if constexpr (DT == FLE_F16) return __builtin_amdgcn_mfma_f32_32x32x16_f16(x, y, c, 0, 0, 0);
        else return __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, y, c, 0, 0, 0);
    };

    // Copies of one K / V block, global memory -> LDS without passing registers: one instruction moves
    // 1 KB (RPI rows) to consecutive LDS addresses, so the XOR placement is applied on the source side: the
    // lane that fills chunk position `pos` of a row fetches that row's chunk pos ^ lds_swizzle(row).  Rows at or
    // beyond Tk lie outside the buffer range and arrive as zeros.
    constexpr int RPI = 1024 / RB, NI = BKV / RPI / 4;  // rows per instruction; instructions per wave and operand
    // (a block has a buffer of its own, from its first row to the end of the keys: its start then costs scalar instructions only)
    const uint32_t nrec_k = uint32_t(int64_t(Tk - 1) * a.ldk * 2 + RB), nrec_v = uint32_t(int64_t(Tk - 1) * a.ldv * 2 + RB);
    auto from_row = [](const char *p, uint32_t bytes, uint32_t skip) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(p) + skip, 0, bytes - skip, 0x00020000); };
    uint32_t cp_k[NI], cp_v[NI];  // this lane's source offsets inside a block
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int row = (wave * NI + i) * RPI + lane / CPR, pos = lane % CPR;
        cp_k[i] = uint32_t(row) * uint32_t(a.ldk * 2) + uint32_t((pos ^ lds_swizzle<D>(row)) * 16);
        cp_v[i] = uint32_t(row) * uint32_t(a.ldv * 2) + uint32_t((pos ^ lds_swizzle<D>(row)) * 16);
    }
    auto copy_k = [&](int stage, int kb0) {
        const __amdgpu_buffer_rsrc_t rsrc = from_row(kp, nrec_k, uint32_t(kb0) * uint32_t(a.ldk * 2));
#pragma unroll
        for (int i = 0; i < NI; ++i) copy_1k(rsrc, smem + stage * STAGE + (wave * NI + i) * 1024, cp_k[i]);
    };
    auto copy_v = [&](int stage, int kb0) {
        const __amdgpu_buffer_rsrc_t rsrc = from_row(vp, nrec_v, uint32_t(kb0) * uint32_t(a.ldv * 2));
#pragma unroll
        for (int i = 0; i < NI; ++i) copy_1k(rsrc, smem + stage * STAGE + BKV * RB + (wave * NI + i) * 1024, cp_v[i]);
    };

    // Per-lane LDS byte offsets that do not change over the loop.  The swizzle of a row only depends on the
    // row's low four bits, so the constant parts of a row index (32 kt, 16 c2) are plain address immediates and
    // only the parts that enter the XOR (the chunk, and the key bit 3 of the second half-fragment) need an
    // offset register of their own.
    // K fragment (A operand): row = 32 kt + l31, 16-byte chunk 2 c + h2.
    // (The swizzle is below 16: behind 16 chunks the offsets repeat, 256 bytes further on.)
    constexpr int KC = NC < 8 ? NC : 8, VD = ND < 4 ? ND : 4;
    // (A read's immediate reaches 64 KB: at D = 256 the second stage has offset registers of its own.)
    constexpr int NS = STAGE > 32768 ? 2 : 1;
    int koff[NS][KC];
#pragma unroll
    for (int c = 0; c < KC; ++c) koff[0][c] = l31 * RB + (((2 * c + h2) ^ lds_swizzle<D>(l31)) * 16);
    // V^T fragment: source lane j of a 16-lane group points at key (j >> 2) + 4 h2 (+ 8 e + 16 c2 + 32 kt), d = 16 (group & 1) + 4 (j & 3) (+ 32 dt)
    const int vj = lane & 15, vg = lane >> 4;
    const int v_key = (vj >> 2) + 4 * (vg >> 1), v_d = 16 * (vg & 1) + 4 * (vj & 3);
    int voff[NS][VD][2];
#pragma unroll
    for (int dt = 0; dt < VD; ++dt)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int key = 8 * e + v_key, d = 32 * dt + v_d;
            voff[0][dt][e] = BKV * RB + key * RB + (((d >> 3) ^ lds_swizzle<D>(key)) * 16) + (d & 7) * 2;
        }

    if constexpr (NS == 2) {
        auto second = [](int off) {
            int o = off + STAGE;
            asm("" : "+v"(o));  // (kept, not added up again in front of every read)
            return o;
        };
#pragma unroll
        for (int c = 0; c < KC; ++c) koff[1][c] = second(koff[0][c]);
#pragma unroll
        for (int dt = 0; dt < VD; ++dt)
#pragma unroll
            for (int e = 0; e < 2; ++e) voff[1][dt][e] = second(voff[0][dt][e]);
    }

    // The scores of a block: two independent chains of matrix instructions, one per 32-key tile.
    auto scores = [&](auto stage_c, f32x16 (&s)[2]) {
        constexpr int S = NS == 2 ? decltype(stage_c)::value : 0, SOFF = NS == 2 ? 0 : decltype(stage_c)::value * STAGE;  // compile-time, so that it folds into the address immediates
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int r = 0; r < 16; ++r) s[kt][r] = 0.0f;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) s[kt] = mma(*reinterpret_cast<const frag_t *>(smem + koff[S][c % KC] + (SOFF + 32 * kt * RB + c / KC * 256)), qf[c], s[kt]);
    };
    auto maximum = [&](const f32x16 (&s)[2]) {
        float mx = s[0][0];
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[kt][r]);
        return mx;
    };
    auto mask_scores = [&](f32x16 (&s)[2], int kb0) {
        const int visible = key_limit - kb0 - 4 * h2;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (32 * kt + 8 * (r / 4) + (r % 4) >= visible) s[kt][r] = -INFINITY;
    };
    // A block is summed by itself, over both halves of the lanes, before it joins the running sum: one rounding of the
    // large sum per block of 64 keys (8192 keys: 1.8e-7 off, with the block's groups of four added to it one by one 3.5e-7).  It
    // joins in the next block's stretch, or before that if the reference moves.
    float ps_block = 0.0f;
    auto join_block = [&]() {
        const Halves both = halves_of(ps_block);
        l_run += both.lo + both.hi;
    };
    // The reference point of the exponentials only moves when some row's maximum has grown by more
    // than 2^8 past it (always in the first block): the probabilities of a row then reach at most 256
    // instead of 1, a common factor that the final division by the row sum removes, and in most blocks
    // no lane of the wave has to rescale its accumulators.
    auto move_reference = [&](float mx, auto first_c) {
        const Halves both = halves_of(mx);
        mx = fmaxf(both.lo, both.hi);
        const float cand = mx * a.scale_log2e;
        const bool grow = cand > m_run + 8.0f;
        if (__builtin_amdgcn_ballot_w64(grow) != 0) {
            const float m_new = grow ? cand : m_run;
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
            m_run = m_new;
            if constexpr (decltype(first_c)::value) return;  // (nothing summed yet)
            join_block();
            ps_block = 0.0f;
            l_run *= alpha;
            if constexpr (D == 256) scale_in_place(oacc, alpha);
            else
#pragma unroll
                for (int dt = 0; dt < ND; ++dt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) oacc[dt][r] *= alpha;
        }
    };
    // Probabilities of 16 keys, rounded to the storage dtype as the operand of the second product; ps takes their fp32 sum.
    auto probabilities = [&](const f32x16 &s, int c2, float &ps) {
        float p[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            p[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[8 * c2 + r], a.scale_log2e, -m_run));
            ps += p[r];
        }
        const u32x2 lo = pack4<DT>(f32x4{p[0], p[1], p[2], p[3]}), hi = pack4<DT>(f32x4{p[4], p[5], p[6], p[7]});
        return __builtin_bit_cast(frag_t, u32x4{lo[0], lo[1], hi[0], hi[1]});
    };
    auto weigh_values = [&](auto stage_c, auto kt_c, const frag_t (&pf)[2]) {
        constexpr int S = NS == 2 ? decltype(stage_c)::value : 0, SOFF = NS == 2 ? 0 : decltype(stage_c)::value * STAGE, kt = decltype(kt_c)::value;
#pragma unroll
        for (int c2 = 0; c2 < 2; ++c2)
#pragma unroll
            for (int dt = 0; dt < ND; ++dt) {
                struct { i16x4 e[2]; } part;
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    part.e[e] = read_transposed((lds_i16x4 *)(smem + voff[S][dt % VD][e] + (SOFF + (32 * kt + 16 * c2) * RB + dt / VD * 256)));
                oacc[dt] = mma(__builtin_bit_cast(frag_t, part), pf[c2], oacc[dt]);
            }
    };
    // vector instructions beside each matrix instruction of a step: exponentials of 48 keys under the scores (28 instructions per
    // 16 keys), of the other 16 under the first half of the second product, the maximum under its second half (at D = 256 behind a read of
    // every score from its accumulation register)
    constexpr int VA = (84 + 2 * NC - 1) / (2 * NC), VB = (28 + 2 * ND - 1) / (2 * ND), VC = ((D == 256 ? 64 : 32) + 2 * ND - 1) / (2 * ND);
    // fragments read ahead of the first product: with one wave per SIMD nothing else covers the LDS (3, 6, 9, 12 of them: 789, 777, 770, 769
    // us on 2 x 6607 tokens x 8 heads of 256; at D <= 128 3 and 5: 13.14, 13.06 us on 32 x 197 x 12 of 64, 308.8, 309.2 on 16 x 2048 x 16 of 128 causal)
    // The first product has four instructions at D = 32: the fifth group with its exponentials falls on the second product's first one.  (3, 4, 5: 213.2,
    // 212.7, 212.3 us on 4 x 4096 x 16, 21.44, 21.52, 21.38 on 5 x 1311 x 8.)
    constexpr int LEAD = D == 256 ? 12 : 5;
    using zero_c = std::integral_constant<int, 0>;
    using one_c = std::integral_constant<int, 1>;

    // K of block j + 2 and V of block j + 1 take the places of K of block j and V of block j - 1, which were last read before
    // the barrier that ended step j - 1.
    auto copy_ahead = [&](int j, int stage) {
        if (j + 2 < n_blocks) copy_k(stage, (j + 2) * BKV);
        if (j + 1 < n_blocks) copy_v(stage ^ 1, (j + 1) * BKV);
    };
    auto end_step = [&]() {
        wait_vmcnt<0>();
        __syncthreads();
    };
    // Block j's exponentials and second product, with the scores of block j + 1 ahead of them in one straight-line stretch:
    // the vector instructions of one block run while the matrix pipe works on the other.
    auto step = [&](int j, auto stage_c, const f32x16 (&cur)[2], f32x16 (&next)[2]) {
        constexpr int ST = decltype(stage_c)::value;
        copy_ahead(j, ST);
        const int kb1 = (j + 1) * BKV;
        frag_t pf[2][2];
        float ps = 0.0f;
        __builtin_amdgcn_sched_barrier(0);
        join_block();
        scores(std::integral_constant<int, ST ^ 1>{}, next);
        pf[0][0] = probabilities(cur[0], 0, ps);
        pf[0][1] = probabilities(cur[0], 1, ps);
        pf[1][0] = probabilities(cur[1], 0, ps);
        weigh_values(stage_c, zero_c{}, pf[0]);
        pf[1][1] = probabilities(cur[1], 1, ps);
        weigh_values(stage_c, one_c{}, pf[1]);
        float mx = maximum(next);
        asm volatile("" : "+v"(mx), "+v"(ps), "+v"(l_run));  // (left to itself the compiler moves the sum and the maximum behind the stretch)
        __builtin_amdgcn_sched_group_barrier(0x100, LEAD, 0);
        interleave<(2 * NC > LEAD ? 2 * NC - LEAD : 0), 1, VA>();
        interleave<LEAD, 2, VA>();
        interleave<2 * ND, 2, VB>();
        interleave<2 * ND, 2, VC>();
        __builtin_amdgcn_sched_barrier(0);
        ps_block = ps;
        if (kb1 + BKV > wave_first_limit) {  // diagonal and tail blocks only (uniform over the wave)
            mask_scores(next, kb1);
            mx = maximum(next);
        }
        move_reference(mx, std::false_type{});
        end_step();
    };
    auto last_step = [&](int j, auto stage_c, const f32x16 (&cur)[2]) {
        constexpr int ST = decltype(stage_c)::value;
        copy_ahead(j, ST);
        frag_t pf[2][2];
        float ps = 0.0f;
        join_block();
#pragma unroll
        for (int c2 = 0; c2 < 2; ++c2) pf[0][c2] = probabilities(cur[0], c2, ps);
        __builtin_amdgcn_sched_barrier(0);
        weigh_values(stage_c, zero_c{}, pf[0]);
        if constexpr (D == 64) {
            // The block's second 32 keys may lie behind every query's limit (uniform over the wave): nothing is left to do for them.  32 x
            // 197 tokens x 12 heads, whose last block holds 5 keys, 14.8 -> 14.3 us, 64 x 80 x 16 14.4 -> 13.8.  (A path of its own for
            // it, next to the interleaved one, costs the smallest calls 1 %; at D = 128 there are no registers for it, 1 % everywhere; at
            // 32 the few matrix instructions leave the rest in the open, 8 x 300 x 16 causal 7.7 -> 8.0.)
            if (w_limit > j * BKV + 32) {
#pragma unroll
                for (int c2 = 0; c2 < 2; ++c2) pf[1][c2] = probabilities(cur[1], c2, ps);
                weigh_values(stage_c, one_c{}, pf[1]);
            }
        } else {
#pragma unroll
            for (int c2 = 0; c2 < 2; ++c2) pf[1][c2] = probabilities(cur[1], c2, ps);
            weigh_values(stage_c, one_c{}, pf[1]);
            __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
            interleave<2 * ND, 2, 2 * VB>();
            interleave<2 * ND, 2, 0>();
        }
        __builtin_amdgcn_sched_barrier(0);
        ps_block = ps;
        join_block();
        if (j + 1 < n_blocks) end_step();
    };

    copy_k(0, 0);
    copy_v(0, 0);
    int j = 0;
    f32x16 s_even[2], s_odd[2];
    if (n_blocks > 1) copy_k(1, BKV);
    end_step();
    if (wave_last >= 0) {
        scores(zero_c{}, s_even);
        if (BKV > wave_first_limit) mask_scores(s_even, 0);
        move_reference(maximum(s_even), std::true_type{});
    }
    end_step();
    // two blocks per trip, so that the stage a block sits in is known at compile time
    for (; j + 1 < wave_last; j += 2) {
        step(j, zero_c{}, s_even, s_odd);
        step(j + 1, one_c{}, s_odd, s_even);
    }
    if (j < wave_last) {
        step(j, zero_c{}, s_even, s_odd);
        last_step(j + 1, one_c{}, s_odd);
    } else if (j == wave_last)
        last_step(j, zero_c{}, s_even);
    j = wave_last + 1;
    for (; j < n_blocks; ++j) {  // the barriers of the blocks that this wave does not see
        copy_ahead(j, j & 1);
        if (j + 1 < n_blocks) end_step();
    }
    // O^T registers: lane = query, register r of tile dt is d = 32 dt + 8 (r / 4) + 4 h2 + r % 4
    const int query = wq0 + l31;
    if (query >= T) return;
    const float inv = 1.0f / l_run;
    char *orow = op + int64_t(query) * a.ldo * 2;
#pragma unroll
    for (int dt = 0; dt < ND; ++dt)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f32x4 v = {oacc[dt][4 * g] * inv, oacc[dt][4 * g + 1] * inv, oacc[dt][4 * g + 2] * inv, oacc[dt][4 * g + 3] * inv};
            *reinterpret_cast<u32x2 *>(orow + (32 * dt + 8 * g + 4 * h2) * 2) = pack4<DT>(v);
        }
}

}  // namespace fle
