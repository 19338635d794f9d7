// Device-side helpers shared by the attention and acceptance kernels.
#pragma once

#include <type_traits>

#include "vs_internal.h"

namespace vs {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

__device__ __forceinline__ float bf16_bits_to_float(uint16_t b) {
    return __uint_as_float((uint32_t)b << 16);
}

// fp32 → bf16 storage, round to nearest even; NaN stays NaN.
__device__ __forceinline__ uint16_t float_to_bf16_bits(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x0040u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    return (uint32_t)float_to_bf16_bits(lo) | ((uint32_t)float_to_bf16_bits(hi) << 16);
}

// Asks for a kernel's arguments in one go. They lie in lines of 64 bytes that the scalar cache does not have yet, a trip to memory
// each (450 - 560 cycles in a stream, 190 in a graph), and the compiler requests every argument where it is used first: the resident attention
// kernel made three such trips in a row before its first key load. 28 layers of one sequence 322.6 -> 309.3 us, four images 10.3 -> 10.0.
// fp32: 2 x 31 nodes, 8 / 2 heads, 600 keys 11.28 -> 10.86. Pipelined kernel: 64 x 400 keys paged 46.2 -> 45.8, 19 x 110 of 64 channels 6.2 -> 6.3.
// Draft tree of four launches 37.0 -> 36.8.
// (Not in attention_mfma_rows.hip: 4 x 60 nodes, 32 / 32 heads, 3100 keys 39.2 without, 39.5 us with it. Nor where it changed nothing: acceptance
// of either kind, 30 sizes, mean 1.000; the straight loop with its combine kernel, bf16 without matrix cores.)
template <typename T>
__device__ __forceinline__ void request_args(const T& p) {
    const uint32_t* w = (const uint32_t*)&p;
    constexpr int N = (sizeof(T) - 4) / 64;
    static_assert(N <= 5, "lines");
    asm volatile("" ::"s"(w[0]), "s"(w[N > 0 ? 16 : 0]), "s"(w[N > 1 ? 32 : 0]), "s"(w[N > 2 ? 48 : 0]), "s"(w[N > 3 ? 64 : 0]), "s"(w[N > 4 ? 80 : 0]), "s"(w[sizeof(T) / 4 - 1]));
}

// ---- Wave-wide reductions on the vector ALU (DPP and lane swaps; a shuffle goes through LDS and takes ten times
// as long, six in a row about 0.3 us). Lanes pair up as in a xor butterfly from 32 down to 1.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, CTRL, 0xf, 0xf, false);
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppXor3 = 0x1B, kDppXor7 = 0x141, kDppXor8 = 0x128;
// op over all 64 lanes, in every lane; T: one or more 32-bit words; op is commutative and associative
template <typename T, typename Op>
__device__ __forceinline__ T wave_all(T x, Op op) {
    constexpr int W = sizeof(T) / 4;
    typedef __attribute__((ext_vector_type(W))) uint32_t words;
    words w = __builtin_bit_cast(words, x), lo, hi;
    auto join = [&]() __attribute__((always_inline)) {
        w = __builtin_bit_cast(words, op(__builtin_bit_cast(T, lo), __builtin_bit_cast(T, hi)));
    };
#pragma unroll
    for (int i = 0; i < W; ++i) {
        const u32x2 r = __builtin_amdgcn_permlane32_swap(w[i], w[i], false, false);
        lo[i] = r[0];
        hi[i] = r[1];
    }
    join();
#pragma unroll
    for (int i = 0; i < W; ++i) {
        const u32x2 r = __builtin_amdgcn_permlane16_swap(w[i], w[i], false, false);
        lo[i] = r[0];
        hi[i] = r[1];
    }
    join();
#pragma unroll
    for (int i = 0; i < W; ++i) {
        lo[i] = w[i];
        hi[i] = dpp<kDppXor8>(w[i]);
    }
    join();
#pragma unroll
    for (int i = 0; i < W; ++i) {
        lo[i] = w[i];
        hi[i] = dpp<kDppXor7>(dpp<kDppXor3>(w[i])); // xor 4
    }
    join();
#pragma unroll
    for (int i = 0; i < W; ++i) {
        lo[i] = w[i];
        hi[i] = dpp<kDppXor2>(w[i]);
    }
    join();
#pragma unroll
    for (int i = 0; i < W; ++i) {
        lo[i] = w[i];
        hi[i] = dpp<kDppXor1>(w[i]);
    }
    join();
    return __builtin_bit_cast(T, w);
}
// For 32-bit words and one operation of the vector ALU a step within rows of sixteen lanes is one instruction that reads its own register from
// other lanes. (The compiler makes five of it: a copy, the wait states, a move between lanes, and for fmaxf one that quiets NaNs.) It
// is written down, so the wait states in front of it are, too; x has not come straight from a matrix instruction. All lanes take part.
#define VS_LANE_STEP(OP, X, LANES) asm("s_nop 1\n\t" OP " %0, %0, %0 " LANES " bank_mask:0xf" : "+v"(X))
#define VS_ROW_ALL(OP, X)                                   \
    VS_LANE_STEP(OP, X, "quad_perm:[1,0,3,2] row_mask:0xf"); \
    VS_LANE_STEP(OP, X, "quad_perm:[2,3,0,1] row_mask:0xf"); \
    VS_LANE_STEP(OP, X, "row_half_mirror row_mask:0xf");     \
    VS_LANE_STEP(OP, X, "row_mirror row_mask:0xf")
// across the four rows, `op` of two registers
template <typename T, typename Op>
__device__ __forceinline__ T rows_all(T x, Op op) {
    u32x2 r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x), false, false);
    x = op(__builtin_bit_cast(T, (uint32_t)r[0]), __builtin_bit_cast(T, (uint32_t)r[1]));
    r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x), false, false);
    return op(__builtin_bit_cast(T, (uint32_t)r[0]), __builtin_bit_cast(T, (uint32_t)r[1]));
}
// fmaxf of operands that are no signaling NaN, as results of arithmetic and of fmaxf never are: no instruction that quiets them stands in front. (Of a
// signaling NaN and a number v_max_f32 makes a quiet NaN, fmaxf the number: not for values as they come from memory. The same below.)
__device__ __forceinline__ float max_of(float a, float b) {
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
// the maximum of the lane's row of sixteen, in all of them; then of the rows
__device__ __forceinline__ float row_max(float x) {
    VS_ROW_ALL("v_max_f32_dpp", x);
    return x;
}
__device__ __forceinline__ float max_of_rows(float x) { return rows_all(x, max_of); }
__device__ __forceinline__ float wave_max(float x) { return max_of_rows(row_max(x)); }
__device__ __forceinline__ float wave_sum(float x) {
    VS_ROW_ALL("v_add_f32_dpp", x);
    return rows_all(x, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ int32_t wave_max(int32_t x) {
    VS_ROW_ALL("v_max_i32_dpp", x);
    return rows_all(x, [](int32_t a, int32_t b) { return max(a, b); });
}
__device__ __forceinline__ int32_t wave_min(int32_t x) {
    VS_ROW_ALL("v_min_i32_dpp", x);
    return rows_all(x, [](int32_t a, int32_t b) { return min(a, b); });
}
__device__ __forceinline__ uint32_t wave_max(uint32_t x) {
    VS_ROW_ALL("v_max_u32_dpp", x);
    return rows_all(x, [](uint32_t a, uint32_t b) { return max(a, b); });
}

// Sum of the lanes up to and including one's own: within rows of sixteen (lanes without a lane to read from keep theirs), then across them.
#define VS_SCAN(OP, X)                                 \
    VS_LANE_STEP(OP, X, "row_shr:1 row_mask:0xf");      \
    VS_LANE_STEP(OP, X, "row_shr:2 row_mask:0xf");      \
    VS_LANE_STEP(OP, X, "row_shr:4 row_mask:0xf");      \
    VS_LANE_STEP(OP, X, "row_shr:8 row_mask:0xf");      \
    VS_LANE_STEP(OP, X, "row_bcast:15 row_mask:0xa");   \
    VS_LANE_STEP(OP, X, "row_bcast:31 row_mask:0xc")
__device__ __forceinline__ float wave_scan(float x) {
    VS_SCAN("v_add_f32_dpp", x);
    return x;
}
__device__ __forceinline__ int32_t wave_scan(int32_t x) {
    VS_SCAN("v_add_u32_dpp", x);
    return x;
}

// Sixteen bytes at any address that is a multiple of four (a row of logits need not start at a multiple of sixteen).
typedef f32x4 __attribute__((aligned(4))) f32x4_any;
__device__ __forceinline__ f32x4 load4_stream(const float* p) { return __builtin_nontemporal_load((const f32x4_any*)p); }

// ---- Results that workgroups hand to each other inside a kernel: device scope, past this XCD's L2.
template <typename T>
__device__ __forceinline__ void store_device(T* p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T load_device(const T* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Who of n workgroups comes last. The word may hold anything before its first use (a value without the tag counts as
// zero and is replaced before the first arrival) and is back at zero when the last one has come.
constexpr uint64_t kArrivalZero = 0xffc3a57bull << 32; // a NaN: no partial result looks like this
__device__ __forceinline__ void arrival_open(uint64_t* w, uint64_t seen) { // one thread of each, any time before it arrives; seen: *w
    if ((seen >> 32) != (kArrivalZero >> 32))
        __hip_atomic_compare_exchange_strong(w, &seen, kArrivalZero, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool arrival_last(uint64_t* w, uint32_t n) { // that thread, when its workgroup's results are in memory
    const bool last = (uint32_t)__hip_atomic_fetch_add(w, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n - 1;
    if (last) store_device(w, kArrivalZero);
    return last;
}

// Loads one tree's parent row into LDS and checks it (parent[0] == -1, 0 <= parent[i] < i).
// Every thread of the workgroup must call it; blockDim.x >= T. Returns the vs_status.
__device__ __forceinline__ int32_t load_tree(const int32_t* __restrict__ parent_row, int T,
                                             int32_t* sp, int32_t* sflag) {
    const int tid = threadIdx.x;
    if (tid == 0) *sflag = 0;
    __syncthreads();
    if (tid < T) {
        const int32_t pv = parent_row[tid];
        sp[tid] = pv;
        if (tid == 0) {
            if (pv != -1) atomicOr(sflag, 1);
        } else if (pv < 0 || pv >= tid) {
            atomicOr(sflag, 2);
        }
    }
    __syncthreads();
    const int32_t f = *sflag;
    return (f & 1) ? VS_STATUS_BAD_ROOT : ((f & 2) ? VS_STATUS_BAD_PARENT : VS_STATUS_OK);
}

// Ancestor-or-self bit mask of `node` for a tree already validated by load_tree.
__device__ __forceinline__ uint64_t ancestor_mask(const int32_t* sp, int node) {
    uint64_t m = 1ull << node;
    int j = node;
    while (j > 0) {
        j = sp[j];
        m |= 1ull << j;
    }
    return m;
}

// Is this sequence's prefix length usable? (inside the host's bound and inside the cache)
__device__ __forceinline__ bool prefix_ok(const AttnParams& p, int32_t S) {
    if (S < 0 || S > p.max_prefix_len) return false;
    if (p.tree_keys == 0 && S < 1) return false; // nothing to attend to
    const int64_t need = (int64_t)S + p.tree_keys;
    const int64_t have = p.paged ? (int64_t)p.max_blocks * p.block_size : p.capacity;
    return need <= have;
}

// Element offset of logical token `tok` of KV head `kvh` in sequence `b`'s cache.
// Paged mode clamps a block id outside the pool to block 0 so that no access can leave
// the pool (the status array reports the bad entry separately).
__device__ __forceinline__ int64_t token_offset(const AttnParams& p, int b, int kvh, int tok) {
    if (p.paged) {
        int32_t blk = p.block_table[(int64_t)b * p.max_blocks + (tok >> p.block_shift)];
        if ((uint32_t)blk >= (uint32_t)p.num_blocks) blk = 0;
        return (int64_t)blk * p.stride_block + (int64_t)kvh * p.stride_head +
               (int64_t)(tok & (p.block_size - 1)) * p.stride_tok;
    }
    return (int64_t)b * p.stride_seq + (int64_t)kvh * p.stride_head + (int64_t)tok * p.stride_tok;
}

// The workgroup that owns a sequence's status entry calls this (all of its threads):
// writes tree / prefix problems, otherwise scans the block-table entries in use.
// PAGED false: a kernel for contiguous caches, without the code for a block table.
template <bool PAGED = true>
__device__ __forceinline__ void report_status(const AttnParams& p, int b, int32_t tree_code,
                                              bool s_ok, int32_t S, int32_t* sflag) {
    if (!p.status) return;
    int32_t code = tree_code;
    if (code == VS_STATUS_OK && !s_ok) code = VS_STATUS_BAD_PREFIX;
    if (PAGED && code == VS_STATUS_OK && p.paged) {
        // *sflag is 0 here (load_tree leaves it 0 for a valid tree)
        const int nblk = (S + p.tree_keys + p.block_size - 1) >> p.block_shift;
        for (int i = threadIdx.x; i < nblk; i += blockDim.x) {
            const int32_t blk = p.block_table[(int64_t)b * p.max_blocks + i];
            if ((uint32_t)blk >= (uint32_t)p.num_blocks) atomicOr(sflag, 4);
        }
        __syncthreads();
        if (*sflag & 4) code = VS_STATUS_BAD_BLOCK;
    }
    if (threadIdx.x == 0) p.status[b] = code;
}

} // namespace vs
