// A whole perceptron (a chain of Linear + bias + activation layers) at batch 1 in one persistent launch.
#pragma once
#include "fle_gemm_thin.h"

namespace fle {

constexpr int kChainMaxLayers = 16;

struct ChainLayer {
    const void *w;     // [n, k], packed rows
    const void *bias;  // [n] or nullptr
    int32_t n, k;
    int32_t act;       // -1, FLE_RELU, FLE_GELU_ERF or FLE_GELU_TANH
};

struct ChainArgs {
    int32_t n_layers;
    const void *x;     // [k of layer 0]
    void *out;         // [n of the last layer]
    void *act[kChainMaxLayers];  // act[l]: output of layer l < n_layers - 1 (storage dtype), every one a buffer of its own
    uint32_t *sync;    // grid barrier state (20 lines of 128 bytes, see chain_barrier); all zero between calls
    ChainLayer layer[kChainMaxLayers];
};

// Every layer is a matrix-vector product that streams its weight matrix once, exactly as the dot-product thin
// kernel does for a single layer: a wave owns one W row at a time and all of K, keeps two register batches of
// 2 KB of the row in flight, multiplies in fp32 and sums over its 64 lanes; lane 0 adds the bias, applies the
// activation and stores the element in the storage dtype.  What the single launch adds: the workgroups stay
// resident (at most one per CU, under 128 registers per lane and next to no LDS, so all of them fit on the chip at once), a
// grid-wide barrier separates the layers, and the first weight batch of the next layer is requested before a
// workgroup enters that barrier, so the weight stream of layer l + 1 is already under way while the last
// workgroups finish layer l: the cost of draining and refilling the memory pipeline between two dependent
// launches is what bounds a 64 MB layer.
//
// The barrier: a wave of the workgroup counts it in and polls the counts until everybody has arrived.  Nothing here flushes or invalidates a cache.  The activations are the
// only data that cross the barrier.  They are stored with device scope (written through to memory), and every
// storing wave waits for its own stores to be acknowledged (vmcnt(0)) before its workgroup arrives, so the order
// store -> arrive is explicit; relaxed device-scope atomics are then enough (a version with release / acquire
// fences, an L2 write-back and invalidation per workgroup and barrier, cost 30 us per layer).  They are loaded
// with ordinary cached loads: every layer writes a buffer of its own that no workgroup has read earlier in the
// launch, so no XCD's L2 can hold an older copy of a line; across launches the same holds because a kernel
// starts with clean (invalidated) L2s.  Every wait is bounded: a workgroup that gives up raises the error word,
// which ends all later waits at once, fills its share of the output with NaN and leaves, so the kernel always
// terminates, and a call whose workgroups were not all resident cannot be mistaken for a result.  The last
// workgroup to finish the kernel puts the counters back to zero (the error word stays).
constexpr uint32_t kChainSpinLimit = 1u << 21;

// st: 32-bit words, one 128-byte line each: line 1 = finished workgroups, line 2 = error, lines 4 .. 11 = arrivals
// within group g (workgroup index mod 8), counted up over the barriers of a launch; lines 12 .. 19, one for each group
// to watch: word g = the last barrier at which group g was complete, written by the last workgroup of g.  Two levels,
// because device-scope atomics on one address are served one after another (256 arrivals on one counter cost about
// 10 us) and so are loads: up to kChainFlat workgroups watch the eight arrival counts themselves, a trip to memory
// less, which with 256 costs more than it saves (8 layers of 256: 38.2 -> 33.3 us, of 4096: 117 -> 126).
constexpr uint32_t kChainFlat = 64;
constexpr int kChainGroups = 8;
__device__ __forceinline__ uint32_t *chain_word(uint32_t *st, int line) { return st + line * 32; }

// Counts the calling wave's workgroup in for the wait-th time (from 1 on) and waits for the others; false if the wait was given up.
__device__ __forceinline__ bool chain_wait(uint32_t *st, uint32_t n_wg, uint32_t wait) {
    const uint32_t lane = threadIdx.x & 63, group = blockIdx.x % kChainGroups;
    const uint32_t of_lane = (n_wg + kChainGroups - 1 - (lane & 7)) / kChainGroups;  // workgroups of group lane & 7
    const bool flat = n_wg <= kChainFlat;
    uint32_t before = 0;
    if (lane == 0) before = __hip_atomic_fetch_add(chain_word(st, 4 + int(group)), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint32_t *watched = flat ? chain_word(st, 4 + int(lane & 7)) : chain_word(st, 12 + int(group)) + (lane & 7);
    const uint32_t target = flat ? of_lane * wait : of_lane ? wait : 0u;
    if (!flat) {  // the last of the group tells every group
        const uint32_t mine = uint32_t(__builtin_amdgcn_readlane(int(of_lane), int(group))) * wait;
        if (uint32_t(__builtin_amdgcn_readfirstlane(int(before))) + 1 == mine && lane < kChainGroups)
            __hip_atomic_store(chain_word(st, 12 + int(lane)) + group, wait, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    for (uint32_t spins = 0; spins <= kChainSpinLimit; ++spins) {
        // (lanes 8 .. 15 read the error word with the same instruction)
        const uint32_t seen = lane < 16 ? __hip_atomic_load(lane < 8 ? watched : chain_word(st, 2), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
        if (__any(lane >= 8 && seen != 0u)) break;
        if (__all(lane >= 8 || seen >= target)) return true;
        __builtin_amdgcn_s_sleep(1);
    }
    if (lane == 0) __hip_atomic_store(chain_word(st, 2), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return false;
}

// The same for a whole workgroup whose waves have all waited for their activation stores; false to every thread if given up.
__device__ __forceinline__ bool chain_barrier(uint32_t *st, uint32_t n_wg, uint32_t target_gen) {
    __syncthreads();
    const bool ok = threadIdx.x >= 64 || chain_wait(st, n_wg, target_gen);
    return __syncthreads_or(!ok) == 0;
}

// The last workgroup to get here puts the barrier state back to zero (the error word stays if raised).  Called by one wave.
__device__ __forceinline__ void chain_done(uint32_t *st, uint32_t n_wg) {
    const uint32_t lane = threadIdx.x & 63;
    uint32_t before = 0;
    if (lane == 0) before = __hip_atomic_fetch_add(chain_word(st, 1), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (uint32_t(__builtin_amdgcn_readfirstlane(int(before))) != n_wg - 1) return;
    if (lane == 0) __hip_atomic_store(chain_word(st, 1), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (lane < kChainGroups) __hip_atomic_store(chain_word(st, 4 + int(lane)), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(chain_word(st, 12 + int(lane >> 3)) + (lane & 7), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One element of an activation vector, stored with device scope (written through, visible to every XCD).
template <int DT>
__device__ __forceinline__ void store_activation(void *dst, int64_t i, float v) {
    if constexpr (DT == FLE_F32) {
        __hip_atomic_store(reinterpret_cast<uint32_t *>(dst) + i, __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
        uint16_t bits;
        if constexpr (DT == FLE_F16) bits = __builtin_bit_cast(uint16_t, static_cast<_Float16>(v));
        else bits = __builtin_bit_cast(uint16_t, static_cast<__bf16>(v));
        __hip_atomic_store(reinterpret_cast<uint16_t *>(dst) + i, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// DT: dtype of the activations, biases and the output; DW: dtype of the weights (DT, or a 2-byte dtype under
// fp32 activations: reduced-precision weights halve the bytes that bound this kernel).
template <int DT, int DW>
__global__ __launch_bounds__(1024) void mlp_chain(const ChainArgs a) {
    static_assert(DW == DT || (DT == FLE_F32 && DW != FLE_F32), "weights in the activations' dtype, or 2-byte weights under fp32");
    constexpr int ES = DW == FLE_F32 ? 4 : 2;   // bytes per weight
    constexpr int EX = DT == FLE_F32 ? 4 : 2;   // bytes per activation
    constexpr int XW = EX / ES;                 // 16-byte pieces of x that go with 16 bytes of W
    constexpr int D = 2;  // 1 KB blocks of a row per register batch
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    struct Batch {
        u32x4 w[D], x[D][XW];
    };
    // the first row of this wave in a layer, its buffer resource, and the loads of K blocks j D .. j D + D - 1
    auto w_rsrc = [&](const ChainLayer &L, int row) {
        const bool live = row < L.n;
        return __builtin_amdgcn_make_buffer_rsrc(
            const_cast<char *>(reinterpret_cast<const char *>(L.w) + (live ? int64_t(row) * L.k * ES : 0)), 0,
            live ? uint32_t(L.k * ES) : 0u, 0x00020000);
    };
    auto load_w = [&](Batch &b, const __amdgpu_buffer_rsrc_t &rw, uint32_t kbytes, uint32_t j) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const uint32_t col = (j * D + d) * 1024 + uint32_t(lane) * 16;
            b.w[d] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rw, col < kbytes ? col : 0x80000000u, 0, 2));
        }
    };
    // the x elements that go with W bytes col .. col + 15 start at byte col * XW
    auto load_x = [&](Batch &b, const __amdgpu_buffer_rsrc_t &rx, uint32_t kbytes, uint32_t j) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const uint32_t col = (j * D + d) * 1024 + uint32_t(lane) * 16;
#pragma unroll
            for (int h = 0; h < XW; ++h)
                b.x[d][h] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rx, col < kbytes ? col * XW + 16 * h : 0x80000000u, 0, 0));
        }
    };

    Batch b0, b1;
    bool have_w0 = false;  // b0.w and b1.w already hold the first two weight batches of this wave's first row of the layer
    for (int l = 0; l < a.n_layers; ++l) {
        const ChainLayer &L = a.layer[l];
        const void *src = l == 0 ? a.x : a.act[l - 1];
        void *dst = l + 1 == a.n_layers ? a.out : a.act[l];
        const uint32_t kbytes = uint32_t(L.k) * ES;  // of a W row
        const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(src), 0, uint32_t(L.k) * EX, 0x00020000);
        const uint32_t blocks = (kbytes + 1023) / 1024, batches = (blocks + D - 1) / D;
        for (int row = int(blockIdx.x) * 16 + wave; row < L.n; row += int(gridDim.x) * 16) {
            const __amdgpu_buffer_rsrc_t rw = w_rsrc(L, row);
            if (!have_w0) load_w(b0, rw, kbytes, 0);
            const bool have_w1 = have_w0;
            have_w0 = false;
            load_x(b0, rx, kbytes, 0);
            float acc = 0.0f;
            auto multiply = [&](const Batch &b) {
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    const Unpacked<DW> w = unpack16<DW>(b.w[d]);
                    if constexpr (XW == 1) {
                        const Unpacked<DT> x = unpack16<DT>(b.x[d][0]);
#pragma unroll
                        for (int e = 0; e < (DW == FLE_F32 ? 4 : 8); ++e) acc = fmaf(w.v[e], x.v[e], acc);
                    } else {  // 8 two-byte weights against 8 fp32 activations
#pragma unroll
                        for (int e = 0; e < 8; ++e) acc = fmaf(w.v[e], __uint_as_float(b.x[d][e / 4][e % 4]), acc);
                    }
                }
            };
            for (uint32_t j = 0; j < batches; j += 2) {
                if (!(have_w1 && j == 0)) load_w(b1, rw, kbytes, j + 1);
                load_x(b1, rx, kbytes, j + 1);
                __builtin_amdgcn_sched_barrier(0);
                multiply(b0);
                __builtin_amdgcn_sched_barrier(0);
                load_w(b0, rw, kbytes, j + 2);
                load_x(b0, rx, kbytes, j + 2);
                __builtin_amdgcn_sched_barrier(0);
                multiply(b1);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) acc += __shfl_xor(acc, d);
            if (lane == 0) {
                float v = acc;
                if (L.bias) v += ld_elem(L.bias, row, DT);
                if (L.act == FLE_RELU) v = relu_f(v);
                else if (L.act == FLE_GELU_ERF) v = gelu_erf_f(v);
                else if (L.act == FLE_GELU_TANH) v = gelu_tanh_f(v);
                if (l + 1 == a.n_layers) st_elem(dst, row, DT, v);
                else store_activation<DT>(dst, row, v);
            }
        }
        if (l + 1 < a.n_layers) {
            // this wave's activation stores have reached memory before its workgroup arrives at the barrier
            // (and before the loads below, which stay in flight across it, join the same counter)
            wait_vmcnt<0>();
            // request the first two weight batches of the next layer's first row before waiting for the other workgroups
            const ChainLayer &Ln = a.layer[l + 1];
            const int row = int(blockIdx.x) * 16 + wave;
            if (row < Ln.n) {
                const __amdgpu_buffer_rsrc_t rn = w_rsrc(Ln, row);
                load_w(b0, rn, uint32_t(Ln.k) * ES, 0);
                load_w(b1, rn, uint32_t(Ln.k) * ES, 1);
                have_w0 = true;
            }
            if (!chain_barrier(a.sync, gridDim.x, uint32_t(l + 1))) {  // layer l is complete and visible everywhere, or:
                // the wait was given up: this workgroup's share of the result becomes NaN and it computes no further
                const ChainLayer &Le = a.layer[a.n_layers - 1];
                if (lane == 0)
                    for (int row = int(blockIdx.x) * 16 + wave; row < Le.n; row += int(gridDim.x) * 16) st_elem(a.out, row, DT, __builtin_nanf(""));
                break;
            }
        }
    }
    if (threadIdx.x < 64 && a.n_layers > 1) chain_done(a.sync, gridDim.x);
}

// One bias element at a row that the whole wave shares, through the scalar path (it would otherwise wait, as every
// vector load does, for the weights requested in front of it).  A 2-byte element comes with its aligned 4 bytes.
template <int DT>
__device__ __forceinline__ float chain_bias(const void *bias, int row) {
    using word = const __attribute__((address_space(4))) uint32_t;
    if constexpr (DT == FLE_F32) {
        return __uint_as_float(reinterpret_cast<word *>(reinterpret_cast<uintptr_t>(bias))[row]);
    } else {
        const uintptr_t at = reinterpret_cast<uintptr_t>(bias) + uintptr_t(row) * 2;
        const uint32_t both = *reinterpret_cast<word *>(at & ~uintptr_t(3));
        const uint16_t bits = uint16_t(at & 2 ? both >> 16 : both);
        if constexpr (DT == FLE_F16) return float(__builtin_bit_cast(_Float16, bits));
        else return bf16_bits_to_f32(bits);
    }
}

// ------------------------------------------------------------------ layers of up to 16384 inputs
// The same stream with the activations in LDS and P = 8 or 16 KB of weights per wave on their way at any time, across
// rows and across the barriers: 32 or 64 MB on 256 CUs, where the form above has 16 MB, which the memory system
// delivers in less time than a barrier takes.  A wave's P register pieces (1 KB of its row each) form a ring over its
// rows of all layers: a piece is refilled with its place in the next P KB as soon as it is multiplied.  Vector memory
// instructions complete in the order of issue, so nothing may be waited for that stands behind such a request.  That is
// the last wave's work: it requests weights only once x is in LDS, stores the workgroup's 16 activations per group of
// rows (which the others leave in LDS), counts the workgroup in at the grid barrier, polls it, and brings the next
// activations into LDS.  LDS holds x as fp32 (exact for every dtype), zeros up to a whole P KB of weights, so that the
// multiplication masks nothing; for 2-byte weights the two halves of a lane's 8 values lie 1 KB apart: every read is 64
// consecutive 16-byte pieces.
// Eight layers of 4096 x 4096 fp32 (537 MB of weights): 132 -> 107 us, 5.0 TB/s; bf16 76 -> 67 us; eight of 256 (all latency): 40 -> 31.
constexpr int kChainLdsK = 16384;    // inputs of a layer at most
constexpr int kChainLdsGroups = 64;  // rows of a layer but the last: at most 16 times this for each workgroup

// A barrier of the workgroup that waits for LDS only: weights requested ahead stay in flight.  The compiler knows neither
// builtin as an access to memory, so it is told that what LDS holds may change here.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
}

template <int DT, int DW, int P>
__global__ __launch_bounds__(1024) void perceptron_lds(const ChainArgs a) {
    static_assert(DW == DT || (DT == FLE_F32 && DW != FLE_F32), "weights in the activations' dtype, or 2-byte weights under fp32");
    constexpr int ES = DW == FLE_F32 ? 4 : 2;   // bytes per weight
    constexpr int EX = DT == FLE_F32 ? 4 : 2;   // bytes per activation
    constexpr int E = 16 / ES;                  // weights per lane and piece
    __shared__ __attribute__((aligned(16))) float xs[kChainLdsK];
    __shared__ float res[kChainLdsGroups][16];
    __shared__ int alive;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool control = wave == 15;
    const int row0 = int(blockIdx.x) * 16 + wave, row_step = int(gridDim.x) * 16;
    const uint32_t lane16 = uint32_t(lane) * 16;

    u32x4 w[P];
    bool filled = false;  // the ring already holds the start of this wave's first row of the layer
    for (int l = 0; l < a.n_layers; ++l) {
        const ChainLayer &L = a.layer[l];
        const bool last = l + 1 == a.n_layers;
        const uint32_t kbytes = uint32_t(L.k) * ES;  // of a W row
        if (control) {
            // x into LDS, through the (still empty) ring
            const void *src = l == 0 ? a.x : a.act[l - 1];
            const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(src), 0, uint32_t(L.k) * EX, 0x00020000);
            const int pieces = (L.k + 64 * P * E - 1) / (64 * P * E) * (64 * P * E) * EX / 16;  // (a multiple of 64)
#pragma unroll 1
            for (int c0 = 0; c0 < pieces; c0 += 64 * P) {
#pragma unroll
                for (int i = 0; i < P; ++i) w[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rx, uint32_t(c0 + 64 * i) * 16 + lane16, 0, 0));
#pragma unroll
                for (int i = 0; i < P; ++i) {
                    const int c = c0 + 64 * i + lane;  // (LDS holds whole multiples of 64 P pieces)
                    const Unpacked<DT> u = unpack16<DT>(w[i]);
                    // weight piece (1 KB block, lane) and half of it that the 4 values belong to
                    float *to = xs + (E == 4 ? 4 * c : DT != FLE_F32 ? (c >> 6) * 512 + (c & 63) * 4 : (c >> 7) * 512 + (c & 1) * 256 + ((c >> 1) & 63) * 4);
                    *reinterpret_cast<f32x4 *>(to) = f32x4{u.v[0], u.v[1], u.v[2], u.v[3]};
                    if constexpr (DT != FLE_F32) *reinterpret_cast<f32x4 *>(to + 256) = f32x4{u.v[4], u.v[5], u.v[6], u.v[7]};
                }
            }
            if (l == 0 && lane == 0) alive = 1;
        }
        if (!filled && row0 < L.n) {
            const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(reinterpret_cast<const char *>(L.w) + int64_t(row0) * kbytes), 0, kbytes, 0x00020000);
#pragma unroll
            for (int i = 0; i < P; ++i) w[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rw, uint32_t(i) * 1024 + lane16, 0, 2));
        }
        lds_barrier();  // x is in LDS
        if (alive == 0) {  // a barrier wait was given up: this workgroup's share of the result becomes NaN and it computes no further
            const ChainLayer &Le = a.layer[a.n_layers - 1];
            if (lane == 0)
                for (int row = row0; row < Le.n; row += row_step) st_elem(a.out, row, DT, __builtin_nanf(""));
            break;
        }
        // the wave's first row of the next layer, which takes the ring over from the last one of this layer
        const ChainLayer &Ln = a.layer[last ? l : l + 1];
        const bool go_on = !last && !control && row0 < Ln.n;
        for (int row = row0, g = 0; row < L.n; row += row_step, ++g) {
            const float bias = L.bias ? chain_bias<DT>(L.bias, row) : 0.0f;
            float acc = 0.0f;
#pragma unroll 1
            for (uint32_t base = 0; base < kbytes; base += P * 1024) {
                // what takes the pieces' places: the next 8 KB of the row, the next row, the next layer, or nothing
                const bool same = base + P * 1024 < kbytes, more = row + row_step < L.n;
                const char *tw = reinterpret_cast<const char *>(same || more ? L.w : Ln.w);
                const uint32_t tk = same || more ? kbytes : uint32_t(Ln.k) * ES;
                tw += int64_t(same ? row : more ? row + row_step : row0) * tk;
                const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(tw), 0, same || more || go_on ? tk : 0u, 0x00020000);
                const uint32_t to = (same ? base + P * 1024 : 0u) + lane16;
                const float *xp = xs + base / ES + lane * 4;
#pragma unroll
                for (int i = 0; i < P; ++i) {
                    const Unpacked<DW> u = unpack16<DW>(w[i]);
#pragma unroll
                    for (int h = 0; h < E / 4; ++h) {
                        const f32x4 x = *reinterpret_cast<const f32x4 *>(xp + (i * 64 * E + 256 * h));
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc = fmaf(u.v[4 * h + e], x[e], acc);
                    }
                    w[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rw, to + uint32_t(i) * 1024, 0, 2));
                }
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) acc += __shfl_xor(acc, d);
            if (lane == 0) {
                float v = acc;
                if (L.bias) v += bias;
                if (L.act == FLE_RELU) v = relu_f(v);
                else if (L.act == FLE_GELU_ERF) v = gelu_erf_f(v);
                else if (L.act == FLE_GELU_TANH) v = gelu_tanh_f(v);
                if (last) st_elem(a.out, row, DT, v);
                else res[g][wave] = v;
            }
        }
        if (last) break;
        filled = go_on && row0 < L.n;
        lds_barrier();  // every wave's activations are in LDS and its reads of x are over
        if (control) {
            for (int i = lane; ; i += 64) {  // (i / 16: group of rows, i % 16: row of the group)
                const int row = int(blockIdx.x) * 16 + (i >> 4) * row_step + (i & 15);
                if (row < L.n) store_activation<DT>(a.act[l], row, res[i >> 4][i & 15]);
                if (int(blockIdx.x) * 16 + ((i | 63) >> 4) * row_step + row_step >= L.n) break;
            }
            wait_vmcnt<0>();  // they have reached memory before the workgroup counts itself in
            const bool ok = chain_wait(a.sync, gridDim.x, uint32_t(l + 1));
            if (!ok && lane == 0) alive = 0;
        }
    }
    if (control && a.n_layers > 1) chain_done(a.sync, gridDim.x);
}

}  // namespace fle
