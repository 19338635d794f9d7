// Pieces shared by the matrix-core attention kernels: vector types, cross-half reductions
// and the workspace layout of split partial results.
#pragma once

#include "vs_device.h"

namespace vs {

typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

typedef __attribute__((address_space(3))) void lds_void;

// s_waitcnt immediate that waits until at most n vector-memory loads are outstanding and
// for nothing else (expcnt = 7, lgkmcnt = 15 are their maxima). Loads return in order.
constexpr int wait_vm(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }

constexpr float kLazy = 8.f; // log2 slack of the running softmax reference

// max(a, b, c); chains of these become v_max3_f32. (Not inline assembly: the compiler pads
// the wait states an MFMA result needs before a vector instruction may read it only for
// instructions it can see, and an asm statement reading a fresh MFMA result returned stale
// registers now and then - run-to-run differences in the softmax reference.)
__device__ __forceinline__ float max3(float a, float b, float c) { return __builtin_fmaxf(__builtin_fmaxf(a, b), c); }

// The same with NaN coming through: v_maximum3_f32, without the two v_max x, x in which fmaxf turns signalling NaNs into quiet ones.
__device__ __forceinline__ float maximum3(float a, float b, float c) { return __builtin_elementwise_maximum(__builtin_elementwise_maximum(a, b), c); }

// max / sum over the two 32-lane halves, result in every lane (v_permlane32_swap)
__device__ __forceinline__ float half_max(float x) {
    const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_maximum(float x) {
    const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __builtin_elementwise_maximum(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_sum(float x) {
    const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Which keys of a 32-key tile a row may see, one bit per key. rel: tree slot of the tile's first key (negative:
// prefix), keys: keys of the tile that exist (both uniform). One word per tile and a bit-field extract and
// insert per score; tests on the 64-bit mask cost four times as many instructions, and in a launch
// that waits for its slowest wave the waves with tree slots are that wave.
__device__ __forceinline__ uint32_t tile_visible(uint64_t mask, int rel, int keys) {
    uint32_t w;
    if (rel >= 0) w = rel < 64 ? (uint32_t)(mask >> rel) : 0u;
    else if (rel > -32) w = (uint32_t)(mask << -rel) | ((1u << -rel) - 1u);
    else w = ~0u;
    return keys >= 32 ? w : (keys <= 0 ? 0u : w & ((1u << keys) - 1u));
}
// s where bit `bit` (a constant) of w is set, else -inf
__device__ __forceinline__ float visible_or_inf(float s, uint32_t w, int bit) {
    const uint32_t m = (uint32_t)((int32_t)(w << (31 - bit)) >> 31);
    return __uint_as_float((__float_as_uint(s) & m) | (0xff800000u & ~m));
}

// 1 KB from memory into LDS at byte `lds` (lane l's sixteen bytes at lds + 16 l), without a stop in registers. Not the
// builtin: the compiler would make every later LDS read wait for all of these loads, not for the tile it reads. Earlier
// LDS reads have returned before the load is issued; it has arrived after a wait for the vector-memory counter.
// Five wait states lie between a vector instruction that writes a scalar register - v_readlane, the reload of a spilled one
// too - and a load that reads it, and the compiler minds them only for instructions that it can see. So the load goes by a copy
// made on the scalar side, which has no such rule (an s_nop 4 instead: short calls of own tiles 6.0 -> 6.1 us).
// m0 is an operand, so the compiler knows what it holds: its own loads into LDS go by it, too. The copy is the wait state
// that a load needs behind a write of it.
// ONCE: data that nobody reads a second time (nt: it need not stay in a cache), here and below.
template <bool ONCE = false>
__device__ __forceinline__ void load_to_lds(uint32_t lds, const void* base, uint32_t lane_off) {
    const void* at;
    if constexpr (ONCE) asm volatile("s_mov_b64 %0, %3\n\tglobal_load_lds_dwordx4 %2, %0 nt" : "=&s"(at) : "{m0}"(lds), "v"(lane_off), "s"(base) : "memory");
    else asm volatile("s_mov_b64 %0, %3\n\tglobal_load_lds_dwordx4 %2, %0" : "=&s"(at) : "{m0}"(lds), "v"(lane_off), "s"(base) : "memory");
}
// the same from a bounded range: what lies outside reads as zeros (four registers, two moves that nothing here can write down: five wait
// states. 20 x 60 nodes, 16 / 16 heads of 64, 1500 keys 32.0 us with two of them, 32.3 with five)
template <bool ONCE = false>
__device__ __forceinline__ void load_to_lds(uint32_t lds, __amdgpu_buffer_rsrc_t range, uint32_t off) {
    if constexpr (ONCE) asm volatile("s_nop 4\n\tbuffer_load_dwordx4 %1, %2, 0 offen nt lds" ::"{m0}"(lds), "v"(off), "s"(range) : "memory");
    else asm volatile("s_nop 4\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"{m0}"(lds), "v"(off), "s"(range) : "memory");
}
// the same from every lane's own address (in vector registers; one wait state for m0)
__device__ __forceinline__ void load_to_lds(uint32_t lds, const void* lane_at) {
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"{m0}"(lds), "v"(lane_at) : "memory");
}
__device__ __forceinline__ void load_to_lds4(uint32_t lds, const void* base, uint32_t lane_off) { // 256 bytes, four of each lane
    const void* at;
    asm volatile("s_mov_b64 %0, %3\n\tglobal_load_lds_dword %2, %0" : "=&s"(at) : "{m0}"(lds), "v"(lane_off), "s"(base) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_loads() { // at most N of this wave's loads outstanding (they return in order)
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void wait_lds_reads() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// What a workgroup of a launch with equal splits works on. Consecutive ids go round-robin over the XCDs; the remap gives
// every XCD a contiguous range, splits fastest: row groups and neighbouring splits of a (sequence, KV head) share its L2.
struct WorkItem {
    int b, kvh, rg, split;
    bool none; // the last workgroups of a launch that is no multiple of eight
};
__device__ __forceinline__ WorkItem work_item(const AttnParams& p) {
    const uint32_t v = (blockIdx.x & 7) * (uint32_t)((p.total_wgs + 7) >> 3) + (blockIdx.x >> 3);
    uint32_t split, rg, kvh;
    const uint32_t b = fast_div(fast_div(fast_div(v, p.by_splits, split), p.by_groups, rg), p.by_heads, kvh);
    return {(int)b, (int)kvh, (int)rg, (int)split, v >= (uint32_t)p.total_wgs};
}

__device__ __forceinline__ int row_node(const AttnParams& p, int r) { return node_of_row(r, p.group, p.inv_group); }
// the nodes of N rows, behind one branch
template <int N>
__device__ __forceinline__ void row_nodes(const AttnParams& p, const int (&r)[N], int (&node)[N]) {
    if (p.group <= kShortGroup) {
#pragma unroll
        for (int i = 0; i < N; ++i) node[i] = node_of_row_short(r[i], p.inv_group);
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) node[i] = node_of_row(r[i], p.group, p.inv_group);
    }
}
// Element offset of (sequence b, KV head kvh)'s first query row in q and out, uniform
template <int D>
__device__ __forceinline__ int64_t row_start(const AttnParams& p, int b, int kvh) {
    return ((int64_t)b * p.T * p.Hq + (int64_t)kvh * p.group) * D;
}
// row r from there on
template <int D>
__device__ __forceinline__ const char* row_at(const AttnParams& p, const char* first, int r, int node) {
    return first + (uint64_t)row_number(r, node, p.row_skip) * (uint32_t)(D * 2);
}
// the same as one offset
__device__ __forceinline__ int64_t row_offset(const AttnParams& p, int b, int kvh, int r, int node) {
    return (((int64_t)b * p.T) * p.Hq + (int64_t)kvh * p.group) * p.d + row_elements(r, node, p.node_stride, p.d);
}

// The sequence of rank `rank` when the longest come first (at most 64 sequences, a lane each; out-of-range lengths sort
// like any other). The whole wave calls it.
__device__ __forceinline__ int sequence_by_rank(const AttnParams& p, int rank, int lane) {
    int len = lane < p.B ? p.prefix_len[lane] : INT32_MIN;
    asm volatile("" : "+v"(len)); // waited for here, not where its register is used again, with other loads on their way
    int above = 0; // sequences that come before this lane's
    for (int i = 0; i < p.B; ++i) {
        const int li = __builtin_amdgcn_readlane(len, i);
        above += (li > len || (li == len && i < lane)) ? 1 : 0;
    }
    return __builtin_ctzll(__ballot(lane < p.B && above == rank));
}

// ---- Queries through LDS. As MFMA operands neighbouring lanes hold different rows; read like that from
// memory every four lanes touch four cache lines, and the eight loads of a 32-row block keep the CU's address
// units busy for 0.2 us - with eight waves that is 1.7 us in which no key can be requested. So a row
// block is fetched in whole rows (one load instruction = 1 KB of consecutive rows), stored with chunk c of
// row r at position c ^ r % (chunks per row) - conflict-free both ways - and read back as operands.
// N of D / 16 pieces: number piece(i) of the row block that starts at row base(i) (rows past the end repeat the last one).
template <int D, int N, typename Base, typename Piece>
__device__ __forceinline__ void load_q_pieces(const AttnParams& p, int b, int kvh, Base base, Piece piece, int lane, u32x4 (&q)[N]) {
    constexpr int LPR = D / 8, RPI = 64 / LPR;
    const char* first = (const char*)((const uint16_t*)p.q + row_start<D>(p, b, kvh) + lane % LPR * 8);
    int r[N], node[N];
#pragma unroll
    for (int i = 0; i < N; ++i) r[i] = min(base(i) + RPI * piece(i) + lane / LPR, p.rows - 1);
    row_nodes(p, r, node);
#pragma unroll
    for (int i = 0; i < N; ++i) q[i] = *(const u32x4*)row_at<D>(p, first, r[i], node[i]);
}
template <int D>
__device__ __forceinline__ void store_q_piece(uint16_t* sq, u32x4 v, int i, int lane) {
    constexpr int LPR = D / 8, RPI = 64 / LPR;
    const int r = RPI * i + lane / LPR;
    *(u32x4*)(sq + r * D + ((lane % LPR) ^ (r % LPR)) * 8) = v;
}
// All pieces of a row block without a stop in registers: the fetching lanes take the chunks in the order they are stored in.
// `sq` is uniform; the pieces have arrived after a wait for the vector-memory counter.
// COUNTED: loads that the compiler does not know of, for whoever waits for them by counting.
template <int D, bool COUNTED = false>
__device__ __forceinline__ void copy_q_block(const AttnParams& p, int b, int kvh, int row_base, uint16_t* sq, int lane) {
    constexpr int LPR = D / 8, RPI = 64 / LPR, N = D / 16;
    const char* first = (const char*)((const uint16_t*)p.q + row_start<D>(p, b, kvh));
    int r[N], node[N];
#pragma unroll
    for (int i = 0; i < N; ++i) r[i] = min(row_base + RPI * i + lane / LPR, p.rows - 1);
    row_nodes(p, r, node);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const char* at = row_at<D>(p, first + ((lane % LPR) ^ ((RPI * i + lane / LPR) % LPR)) * 16, r[i], node[i]);
        if constexpr (COUNTED) load_to_lds((uint32_t)(uintptr_t)(lds_void*)(sq + i * 512), at);
        else __builtin_amdgcn_global_load_lds((const uint16_t*)at, (lds_void*)(sq + i * 512), 16, 0, 0);
    }
}
template <int D>
__device__ __forceinline__ bf16x8 read_q_frag(const uint16_t* sq, int ks, int col, int half) {
    constexpr int LPR = D / 8;
    return __builtin_bit_cast(bf16x8, *(const u32x4*)(sq + col * D + ((2 * ks + half) ^ (col % LPR)) * 8));
}

// Partial results of one (sequence, KV head, split, 32-row block): D/32 accumulator blocks,
// each stored as 2 pieces of [64 lanes x 8 values] (register r = 4*q4 + e of lane l in piece
// db*2 + q4/2 at l*8 + (q4%2)*4 + e: a wave's store or load of a piece is 1 KB of consecutive memory),
// and 32 x (max, sum) in fp32. The splits of a piece lie next to each other - [unit][row block][piece]
// [split] - as do a row block's (max, sum) pairs: what a wave gathers when it merges a piece is one run of
// memory, in one page instead of one page per split. A partial output
// row is divided by its own sum before it is rounded: a convex combination of V rows, as large
// as the largest visible |V| and no larger. It is stored as bf16, which has V's own exponent
// range (fp16 would turn any |v| > 65504 into infinity) and costs half the bytes of fp32: what a
// split costs is mostly the write-back of these bytes at the end of the kernel. The 2^-9
// rounding of each partial enters the merged row once (the merge weights sum to one), next to
// the 2^-9 rounding of the final bf16 result.
__device__ __forceinline__ u32x2 pack_partial(float a, float b, float c, float d, float inv) {
    const f32x2 lo = {a * inv, b * inv}, hi = {c * inv, d * inv};
    u32x2 w;
    w[0] = __builtin_bit_cast(uint32_t, __builtin_convertvector(lo, bf16x2));
    w[1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(hi, bf16x2));
    return w;
}
__device__ __forceinline__ f32x4 unpack_partial(u32x2 w) {
    const f32x4 r = {__uint_as_float(w[0] << 16), __uint_as_float(w[0] & 0xffff0000u), __uint_as_float(w[1] << 16),
                     __uint_as_float(w[1] & 0xffff0000u)};
    return r;
}
// elements: piece 0 of (unit, split, row block), and from there to another piece
template <int D>
__device__ __forceinline__ int64_t part_block(const AttnParams& p, int64_t unit, int split, int rbk) {
    return ((unit * (p.rows_pad / kRowBlock) + rbk) * (D / 16) * p.num_splits + split) * 512;
}
__device__ __forceinline__ int64_t piece_at(const AttnParams& p, int piece) { return piece_elements(piece, p.num_splits); }

// Partial results travel between workgroups on different XCDs: stores that write through to memory and loads
// that do not stop at this XCD's L2 (cache policy bit sc1 = device scope).
constexpr int kDeviceScope = 16;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t span_of(const void* base) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, 0x7fffffff, 0x00027000);
}

// Keys of the longest sequence that the host allows: inside the cache, and token offsets up to there fit 32 bits (those of a
// cache's further slots need not).
__device__ __forceinline__ int64_t most_keys(const AttnParams& p) { return (int64_t)p.max_prefix_len + p.tree_keys; }
// The rows of a contiguous cache's slice (one sequence's KV head) from k0 on, at most a split and no further than the longest
// sequence; what lies past them reads as zeros. (Where offsets of rows behind those wrap, they read live rows: their keys are
// masked and their values replaced by zeros all the same.) stride: bytes from row to row.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t slice_of(const uint16_t* slice, int k0, const AttnParams& p, uint32_t stride) {
    const uint32_t bytes = slice_bytes(most_keys(p), k0, p.keys_per_split, stride, (uint32_t)p.d * 2);
    return __builtin_amdgcn_make_buffer_rsrc((char*)const_cast<uint16_t*>(slice) + (int64_t)k0 * stride, 0, (int)bytes, 0x00027000);
}

// A lane's 16 bytes of piece `piece`, a constant, of a partial result that begins at `blk`. MERGE: at most 128 splits (balanced slots), so one
// base and offsets of 32 bits do. (Never a scalar offset instead: for such stores the compiler leaves out the wait
// state that a 16-byte store needs before its data registers are written again, and later values were stored in their place.)
// For the combine kernel a caller may have the keys in any number of splits: 64 bits.
template <bool MERGE>
__device__ __forceinline__ void store_piece(const AttnParams& p, uint16_t* blk, int piece, int lane, u32x4 w) {
    if constexpr (MERGE) __builtin_amdgcn_raw_buffer_store_b128(w, span_of(blk), lane * 16 + piece * p.num_splits * 1024, 0, kDeviceScope);
    else *(u32x4*)(blk + piece_at(p, piece) + lane * 8) = w;
}
// One 32-channel accumulator block of a row block, divided by the rows' sums: two 16-byte pieces per
// lane. `blk` = piece 0 of the (unit, split, row block), db = channel block.
template <bool MERGE = false>
__device__ __forceinline__ void store_partial(const AttnParams& p, uint16_t* blk, int db, int lane, const f32x16& a, float inv) {
#pragma unroll
    for (int hp = 0; hp < 2; ++hp) {
        const u32x2 lo = pack_partial(a[8 * hp], a[8 * hp + 1], a[8 * hp + 2], a[8 * hp + 3], inv);
        const u32x2 hi = pack_partial(a[8 * hp + 4], a[8 * hp + 5], a[8 * hp + 6], a[8 * hp + 7], inv);
        const u32x4 w = {lo[0], lo[1], hi[0], hi[1]};
        store_piece<MERGE>(p, blk, db * 2 + hp, lane, w);
    }
}
// (max, sum) pairs are grouped per row block with the splits adjacent: index of the
// first of the 32 rows of (unit, rbk, split), in pairs.
__device__ __forceinline__ int64_t ml_block(const AttnParams& p, int64_t unit, int split, int rbk) {
    return ((unit * (p.rows_pad / kRowBlock) + rbk) * p.num_splits + split) * (int64_t)kRowBlock;
}

// ---- Merging key splits inside the kernel that computes them.
// The workgroups of a row group (same sequence, KV head and rows, n live splits of the keys) meet at a
// barrier in the workspace and then merge the row group together, every one a share of the row blocks' pieces: one
// trip to memory for the partials of n splits, spread over n CUs, in place of a second kernel (launch,
// arguments, lengths, the same trip, drain: 5 us). A barrier between workgroups only ends when all of
// them get to run, which nobody promises while other streams hold CUs. So the wait is bounded: who waits
// longer than p.merge_wait hands its share over to the workgroup that arrives last and leaves.
// The gate's word is kMergeTag << 40 | abandoned shares << 8 | arrivals. Anything else (first use of the workspace) counts as zero
// and is replaced before the first arrival; the last arrival puts it back to zero. So who has arrived and finds n arrivals, or
// none, knows that all have. (They waited for a second word that the last one changed once its own arrival had returned: us per
// call, before / so, 28 / 4 heads, 60 nodes, 1696 keys, 28 layers 291.0 / 284.5; 32 / 8 heads of 64, 8 x 31 nodes, up to 2047 keys
// 12.41 / 12.27; 4757 drawn calls with two and more splits, geometric mean 0.976. Fewer looks while many are still missing, or pauses between
// them, were slower in the mean.)
// Where many wait on nearly all CUs, their looks hold up those who arrive. So 28 splits and more on 224 workgroups (CROWD) have a second word to look
// at, in another cache line, which the last one changes, from any value; it is read ahead of the wait for the partial results. Drawn calls, time
// relative to two words from the start, one word / two so: rounds of four row blocks, 16 .. 19 splits 0.989 / 0.992, 24 .. 27 1.004 / 1.002, 28 .. 31
// 1.023 (up to 1.15) / 1.002, 32 1.047 / 1.001; own tiles 16 .. 19 0.991 / 1.020, 28 .. 31 1.029 (1.11) / 1.000. The resident kernel's merges wait
// less and gain by one word to the end (28 .. 31 splits 0.986). One sequence, 58 nodes, 16 / 1 heads, 7960 keys 17.2 / 15.2 us.
// The call before on the same workspace has ended (calls that share one are ordered), so the word is at rest.
// Word kGateHanded of the gate counts the shares handed over (from any value, not read here: for tests and whoever looks for slow merges).
static_assert(kMergeMaxSplits == 32, "bits of the abandoned set");
constexpr uint64_t kMergeTag = 0xffc3a9ull;           // no partial result or (max, sum) pair looks like this (a NaN)
static_assert(kMergeTag != kArrivalZero >> 40, "an arrival word that vs_draft_expand left in a shared workspace is no gate");
constexpr uint64_t kMergeZero = kMergeTag << 40;

__device__ __forceinline__ uint64_t gate_load(const uint64_t* w) {
    return __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Thread 0 of every workgroup of the row group, any time before it arrives; `seen`: the word, asked for earlier (loads return in
// order: asked for behind the tiles, it comes behind the tiles). null: the splits are merged by the combine kernel.
__device__ __forceinline__ void merge_open(uint64_t* gate, uint64_t seen) {
    if ((seen >> 40) != kMergeTag) // lost to another workgroup: then it did the same
        __hip_atomic_compare_exchange_strong(gate, &seen, kMergeZero, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Thread 0, after every wave's partial results are in memory. Returns the splits whose shares this workgroup
// has to merge besides its own; `go` false: its own share was handed over.
// CROWD: who waits looks at word kGateFlag, which was `flag` before this workgroup arrived and which the last one changes, see above.
template <bool CROWD>
__device__ __forceinline__ uint32_t merge_meet(uint64_t* gate, uint64_t flag, uint32_t wait, int split, int n, bool& go) {
    go = true;
    const uint64_t old = __hip_atomic_fetch_add(gate, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((int)(old & 0xff) == n - 1) {
        __hip_atomic_store(gate, kMergeZero, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if constexpr (CROWD) __hip_atomic_store(gate + kGateFlag, flag + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return (uint32_t)(old >> 8);
    }
    const auto all = [&](uint64_t w) { return (int)(w & 0xff) == 0 || (int)(w & 0xff) == n; };
    const uint64_t t0 = wall_clock64();
    uint64_t w = old + 1;
    for (uint32_t looks = 0; wait != 0;) { // (a wait of zero: without a look)
        if (CROWD ? gate_load(gate + kGateFlag) != flag : all(w = gate_load(gate))) return 0;
        if ((++looks & 7) == 0 && wall_clock64() - t0 > wait) break; // (the clock takes as long as a look)
    }
    if (CROWD && wait != 0 && all(w = gate_load(gate))) return 0;
    do {
        if (__hip_atomic_compare_exchange_strong(gate, &w, w | (256ull << split), __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
            __hip_atomic_fetch_add(gate + kGateHanded, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            go = false;
            return 0;
        }
    } while (!all(w)); // else the last one has come in the meantime
    return 0;
}
// Half a piece (eight channels of the 32 rows of a row block, see store_partial: the 32 lanes of one half of the
// accumulators): where it is read and written. The addresses are worked out before the wait, the rest after it.
constexpr int kMergeGroup = 4; // items a wave merges at once, at most
struct MergeItem {
    uint32_t ml, po; // byte offsets in the row group's (max, sum) pairs and partial rows, uniform
    uint16_t* out;   // null: a row past the last one
};
template <int D>
__device__ __forceinline__ MergeItem merge_item(const AttnParams& p, int b, int kvh, int rb0, int i, int lane) {
    constexpr int NP = D / 8; // half pieces per row block
    const int rb = i / NP, piece = (i % NP) >> 1, hl = i & 1;
    MergeItem it;
    it.ml = (uint32_t)(rb * p.num_splits) * (kRowBlock * 8);
    it.po = (uint32_t)((rb * (D / 16) + piece) * p.num_splits) * 1024 + hl * 512;
    const int r = (rb0 + rb) * kRowBlock + (lane & 31);
    const char* first = (const char*)((uint16_t*)p.out + row_start<D>(p, b, kvh) + piece * 16 + 4 * hl + 8 * (lane >> 5));
    it.out = r < p.rows ? (uint16_t*)row_at<D>(p, first, r, row_node(p, r)) : nullptr;
    return it;
}
// Where a lane finds its splits of any item: lanes r and r + 32 share row r and take every other split (past the last
// one the last is read again, with weight 0). Worked out before the wait, like the items.
constexpr int kMergePairs = 8; // pairs of splits in flight, at most
struct MergeLane {
    uint32_t ml[kMergePairs], po[kMergePairs]; // byte offsets
};
__device__ __forceinline__ MergeLane merge_lane(int s0, int n) {
    const int row = threadIdx.x & 31, odd = (threadIdx.x >> 5) & 1;
    MergeLane at;
#pragma unroll
    for (int u = 0; u < kMergePairs; ++u) {
        const uint32_t s = (uint32_t)min(s0 + 2 * u + odd, n - 1);
        at.ml[u] = s * (kRowBlock * 8) + row * 8;
        at.po[u] = s * 1024 + row * 16;
        asm("" : "+v"(at.ml[u]), "+v"(at.po[u]));
    }
    return at;
}
// log-sum-exp of G items over n splits, then the final rows' channels. One wave. BATCH pairs of splits of every item are
// in flight together; there is no branch around a load.
template <int BATCH, int G>
__device__ __forceinline__ void merge_run_by(const MergeItem (&it)[kMergeGroup], const float* ml, const uint16_t* po, MergeLane at, int n) {
    const int odd = (threadIdx.x >> 5) & 1;
    float M[G], den[G], num[G][8];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        M[g] = -INFINITY;
        den[g] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) num[g][e] = 0.f;
    }
    for (int s0 = 0;;) {
        u32x2 w[G][BATCH];
        u32x4 o[G][BATCH];
#pragma unroll
        for (int g = 0; g < G; ++g) {
#pragma unroll
            for (int u = 0; u < BATCH; ++u) w[g][u] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(span_of(ml), at.ml[u], it[g].ml, kDeviceScope));
#pragma unroll
            for (int u = 0; u < BATCH; ++u) o[g][u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(span_of(po), at.po[u], it[g].po, kDeviceScope));
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            float Mb = M[g];
#pragma unroll
            for (int u = 0; u < BATCH; ++u) Mb = fmaxf(Mb, __uint_as_float(w[g][u][0]));
            Mb = half_max(Mb);
            const float Ms = Mb == -INFINITY ? 0.f : Mb; // no visible key so far: all weights are 2^-inf = 0
            if (s0 > 0) {
                const float resc = __builtin_amdgcn_exp2f(M[g] - Ms);
                den[g] *= resc;
#pragma unroll
                for (int e = 0; e < 8; ++e) num[g][e] *= resc;
            }
            M[g] = Mb;
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const float f = __builtin_amdgcn_exp2f(__uint_as_float(w[g][u][0]) - Ms) * (s0 + 2 * u + odd < n ? __uint_as_float(w[g][u][1]) : 0.f);
                den[g] += f;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    num[g][2 * e] += f * __uint_as_float(o[g][u][e] << 16);
                    num[g][2 * e + 1] += f * __uint_as_float(o[g][u][e] & 0xffff0000u);
                }
            }
        }
        s0 += 2 * BATCH;
        if (BATCH < kMergePairs || s0 >= n) break;
        at = merge_lane(s0, n);
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const float sum = half_sum(den[g]);
        float r[4]; // lower half: channels 0 .. 3 of both halves added up, upper half: channels 4 .. 7
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const u32x2 x = __builtin_amdgcn_permlane32_swap(__float_as_uint(num[g][e]), __float_as_uint(num[g][4 + e]), false, false);
            r[e] = __uint_as_float(x[0]) + __uint_as_float(x[1]);
        }
        if (it[g].out) *(u32x2*)it[g].out = pack_partial(r[0], r[1], r[2], r[3], 1.f / sum);
    }
}
template <int BATCH>
__device__ __forceinline__ void merge_run_few(const MergeItem (&it)[kMergeGroup], int got, const float* ml, const uint16_t* po, MergeLane at, int n) {
    if (got == 1) merge_run_by<BATCH, 1>(it, ml, po, at, n);
    else if (got == 2) merge_run_by<BATCH, 2>(it, ml, po, at, n);
    else if (got == 3) merge_run_by<BATCH, 3>(it, ml, po, at, n);
    else merge_run_by<BATCH, 4>(it, ml, po, at, n);
}
// The end of a split's workgroup: all waves, after their last partial store. Row blocks rb0 .. rb1 - 1 belong to
// the row group, n >= 2; `s_word` is two words of LDS that nobody else uses any more. What an item costs is the trip
// to memory (0.7 us), so a wave that has several - few splits, many rows - takes up to four at once: 192 rows in two
// splits 23.6 -> 19.2 us (23 sequences of up to 290 keys); one sequence of five row blocks and splits 12.3 -> 11.4.
template <int D, bool CROWD = false>
__device__ __forceinline__ void merge_splits(const AttnParams& p, uint64_t* gate, int b, int kvh, int rb0, int rb1, int split, int n,
                                             int waves, uint32_t* s_word) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int NP = D / 8; // half pieces per row block
    const int items = (rb1 - rb0) * NP;
    int step = n * waves;
    const int most = n <= 4 ? kMergeGroup : n <= 8 ? 2 : 1; // items at once
    MergeItem it[kMergeGroup] = {};
    int got = 0;
    auto gather = [&](int i) __attribute__((always_inline)) { // items i, i + step, ... as far as there are
        it[0] = merge_item<D>(p, b, kvh, rb0, i, lane);
        got = 1;
#pragma unroll
        for (int k = 1; k < kMergeGroup; ++k) {
            const int at = i + k * step;
            if (k >= most || at >= items) return;
            it[k] = merge_item<D>(p, b, kvh, rb0, at, lane);
            got = k + 1;
        }
    };
    const MergeLane at = merge_lane(0, n);
    const int64_t unit = (int64_t)b * p.Hkv + kvh;
    const float* ml = p.part_ml + ml_block(p, unit, 0, rb0) * 2;
    const uint16_t* po = p.part_o + part_block<D>(p, unit, 0, rb0);
    int i = split + n * wave;
    if (i < items) gather(i);
    uint64_t flag = 0;
    if (CROWD && wave == 0) flag = gate_load(gate + kGateFlag); // arrives with what the partial results are waited for
    __builtin_amdgcn_s_waitcnt(wait_vm(0)); // this wave's partial results are in memory
    __syncthreads();
    if (tid == 0) {
        bool go;
        s_word[0] = merge_meet<CROWD>(gate, flag, p.merge_wait, split, n, go);
        s_word[1] = go;
    }
    __syncthreads();
    if (s_word[1] == 0) return;
    uint32_t shares = s_word[0]; // handed over by workgroups that left
    if (shares && shares == ((uint32_t)((1ull << n) - 1) & ~(1u << split))) { // by all of them: one share
        shares = 0;
        step = waves;
        i = wave;
        if (i < items) gather(i);
    }
    for (;;) {
        while (i < items) {
            if (n > 8) merge_run_by<8, 1>(it, ml, po, at, n);
            else if (n > 4) got == 1 ? merge_run_by<4, 1>(it, ml, po, at, n) : merge_run_by<4, 2>(it, ml, po, at, n);
            else if (n > 2) merge_run_few<2>(it, got, ml, po, at, n);
            else merge_run_few<1>(it, got, ml, po, at, n);
            i += most * step;
            if (i < items) gather(i);
        }
        if (shares == 0) break;
        i = __builtin_ctz(shares) + n * wave;
        shares &= shares - 1;
        if (i < items) gather(i);
    }
}

// ---- Balanced schedule: the key ranges of a whole ragged batch, cut into shares of equal cost.
// The keys of all sequences, counted in 64-key steps, are laid end to end (sequence 0 first); share c
// of W covers steps [bound(c), bound(c + 1)) of that line, and the part of a sequence that falls
// into a share is a piece of work: a share that crosses from one sequence into the next is worked
// off piece by piece. A piece costs its steps plus kBalPieceCost (queries, first tiles, the
// pipeline's fill and drain: what happens before a piece's first and after its last step takes about
// as long as six steps). Lane i of a wave holds sequence i (at most 64 sequences). Every workgroup
// derives the shares from the prefix lengths, so all agree on where a piece's partial result lies:
// slot (share + sequence) of its KV head. The last slot is never a piece's; its first KB in a row group's first
// row block holds the arrival words of the row group's pieces, one per sequence.
// (By stamps a piece costs 4.2 steps. Six and three: with a smaller cost or stubs the shares end more evenly, 92 against 99 us on cold clocks, but
// more sequences are cut and merged; 4 / 1, 5 / 1, 5 / 2, 8 / 3, 6 / 5 were 0 - 3 % slower over twelve batches.)
constexpr int kBalPieceCost = 6;
constexpr int kBalSnap = 3; // no piece this short (in steps) is left behind at a sequence's end

// this lane's sequence (of prefix length S; -1: none): its first step on the line and its number of steps (0: not usable)
__device__ __forceinline__ int bal_steps(const AttnParams& p, int32_t S) { return (S + p.tree_keys + kIterKeys - 1) / kIterKeys; } // of a usable one
__device__ __forceinline__ void bal_scan(const AttnParams& p, int32_t S, int& start, int& steps, int& total) {
    steps = prefix_ok(p, S) ? bal_steps(p, S) : 0;
    const int inc = wave_scan(steps);
    start = inc - steps;
    total = __builtin_amdgcn_readlane(inc, 63);
}

// the steps [a, b) of a sequence (first step s0, t steps) that fall into [lo, hi) of the line; false: none
__device__ __forceinline__ bool bal_piece(int lo, int hi, int s0, int t, int& a, int& b) {
    a = max(lo, s0) - s0;
    b = min(hi, s0 + t) - s0;
    return b > a;
}

// lane c (c < W): first step of share c; the other lanes: the end of the line.
// Two cuts are priced (most expensive share, a piece costing its steps plus kBalPieceCost) and the
// cheaper one is taken:
//  * even: the line with kBalPieceCost units inserted in front of every sequence is divided into W
//    equal parts; a boundary that falls into such a start-up stretch, or within kBalSnap steps of
//    either end of a sequence, moves onto the sequence's boundary (no stubs);
//  * regular, when W is a multiple of the number of sequences: every sequence gets W / B shares of
//    ceil(longest sequence / (W / B)) steps - what equal splits per sequence would be. Batches of
//    (nearly) equal lengths keep their equal splits this way.
// All lanes work side by side, a lane per share. Nothing is requested before this is known, so it is kept short: where a
// share's ends lie among the sequences is counted (their starts and ends ascend), and nothing is divided.
__device__ __forceinline__ int bal_bounds(const AttnParams& p, int lane, int start, int steps, int total) {
    const int W = p.bal_chunks;
    const uint64_t usable = __ballot(steps > 0);
    const int nseq = __popcll(usable);
    // start-up stretches in front of this lane's sequence: the usable sequences before it
    const int before = __popcll(usable & ((1ull << lane) - 1ull));
    const int lstart = start + kBalPieceCost * before; // this lane's sequence on the stretched line
    const int ltotal = total + kBalPieceCost * nseq;
    uint32_t part, over; // ltotal / W and what is left: lane * ltotal / W without a long division
    part = fast_div((uint32_t)ltotal, p.by_shares, over);
    uint32_t rem;
    const int raw = lane < W ? (int)(lane * part + fast_div(lane * over, p.by_shares, rem)) : ltotal;
    const int snap = min(kBalSnap, (int)part / 4);
    int at = -1; // the last sequence that starts at or before `raw` (a usable one: no other stands alone at its place)
    for (int i = 0; i < p.B; ++i) at += __builtin_amdgcn_readlane(lstart, i) <= raw ? 1 : 0;
    const int l0 = __shfl(lstart, at), s0 = __shfl(start, at), t = __shfl(steps, at);
    const int lend = l0 + kBalPieceCost + t;
    const int even = lane >= W ? total : raw - l0 <= kBalPieceCost + snap ? s0 : lend - raw <= snap ? s0 + t : s0 + (raw - l0 - kBalPieceCost);
    if (p.bal_per_seq.d == 0) return even;
    uint32_t j;
    const int b = min((int)fast_div((uint32_t)lane, p.bal_per_seq, j), p.B - 1);
    const int k = (int)fast_div((uint32_t)wave_max(steps) + p.bal_per_seq.d - 1, p.bal_per_seq, rem);
    const int sb = __shfl(start, b), tb = __shfl(steps, b);
    const int regular = lane < W ? sb + (int)min(j * (uint32_t)k, (uint32_t)tb) : total;
    // a share's pieces: the usable sequences that start before its end, without those that end at or before its start
    const int even_hi = lane + 1 < W ? __shfl_down(even, 1) : total, regular_hi = lane + 1 < W ? __shfl_down(regular, 1) : total;
    const int from = steps > 0 ? start : INT32_MAX, to = steps > 0 ? start + steps : INT32_MAX;
    int even_n = 0, regular_n = 0;
    for (int i = 0; i < p.B; ++i) {
        const int f = __builtin_amdgcn_readlane(from, i), e = __builtin_amdgcn_readlane(to, i);
        even_n += (f < even_hi ? 1 : 0) - (e <= even ? 1 : 0);
        regular_n += (f < regular_hi ? 1 : 0) - (e <= regular ? 1 : 0);
    }
    auto cost = [&](int lo, int hi, int n) __attribute__((always_inline)) { return lane < W && hi > lo ? hi - lo + kBalPieceCost * n : 0; };
    return wave_max(cost(regular, regular_hi, regular_n)) <= wave_max(cost(even, even_hi, even_n)) ? regular : even;
}

} // namespace vs
