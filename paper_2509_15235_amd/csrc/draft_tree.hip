// Draft-tree construction (paper Section 3.1 adopts EAGLE-2's context-aware dynamic draft
// tree; Appendix A: 30 draft tokens, depth 3, 8 nodes kept per expansion). A node's score
// is the sum of the draft model's log-probabilities along its path. An expansion step gives
// every frontier node its K most likely tokens as children and keeps the K best-scored
// children as the next frontier; at the end the N best-scored candidates of all levels are
// the tree. The draft model's forward pass is not part of this: its logits are inputs.
//
// Two kernels. (1) An expansion: every workgroup reduces a chunk of a logits row (8192 floats, or 10240 or 12288) to (maximum, sum of
// exp, the chunk's K largest entries); the workgroup of a sequence that finishes last merges the chunks into each
// row's top K and log-sum-exp, scores the F*K candidates and picks the next frontier. (That second part used to
// be a kernel of its own: 7.8 us for one trip to memory and half a microsecond of work, three times per tree.)
// (2) One workgroup per sequence for the final selection, which emits parent[] / tokens[] in candidate order.
//
// Selection without bookkeeping: entries are taken in the strict total order (value descending, index
// ascending), as integers of 64 bits, also between the workgroups. In a chunk a bound that at least K entries reach is found
// from the largest of every group of lanes, the few entries at or above it are compacted and ranked by
// counting; the chunks' lists, and a frontier's rows, stand in order already and are merged in registers. Nothing has to be marked as taken.
#include <type_traits>

#include "vs_device.h"

namespace vs {

namespace {

constexpr int kSelThreads = 256;
constexpr int kExpandThreads = 512;
constexpr int kExpandWaves = kExpandThreads / kWave;
static_assert(kDraftVec == kExpandThreads * 4, "a load of every thread");

// a comes strictly before b in (value descending, index ascending)
__device__ __forceinline__ bool before(float av, int32_t ai, float bv, int32_t bi) {
    return av > bv || (av == bv && ai < bi);
}

constexpr int kGroups = kExpandThreads / 16; // rows of lanes of a workgroup
static_assert(kMaxDraftK <= kGroups && kGroups == 32, "K groups, a lane each");
constexpr int kCandCap = 128;        // entries of a wave's candidate list in LDS
constexpr int kListPad = 16, kListLen = kCandCap + kListPad;

// Larger float -> larger key (no NaN), -0 below +0; every real key is > 0, which stands for "no entry".
__device__ __forceinline__ uint32_t order_key(float v) {
    const uint32_t u = __float_as_uint(v);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_value(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// The same with signed zeros equal (-0 + 0 = +0), as `before` has them: for keys that are compared with each other.
__device__ __forceinline__ uint32_t rank_key(float v) { return order_key(v + 0.f); }
// An entry as one integer: larger = earlier in (value descending, index ascending); 0 is no entry.
__device__ __forceinline__ uint64_t entry_key(float v, int32_t i) { return ((uint64_t)rank_key(v) << 32) | (uint32_t)~i; }
// The same in an expansion, where NaN is never taken.
__device__ __forceinline__ uint64_t child_key(float v, int32_t i) { return v == v ? entry_key(v, i) : 0; }
__device__ __forceinline__ float entry_value(uint64_t k) { return key_value((uint32_t)(k >> 32)); }
__device__ __forceinline__ int32_t entry_index(uint64_t k) { return (int32_t)~(uint32_t)k; }

// A key that at least K of the lanes' keys reach and that few more do; 0 if fewer than K lanes have one (keys are > 0). From
// the largest key down in growing steps, then by halves until at most K + 8 reach it: 4 or 5 ballots for a row of logits,
// where the bits of the bound one by one took 16. (Down to 2^16, the last seven bits of the mantissa's upper half.)
__device__ __forceinline__ uint32_t kth_bound(uint32_t key, int K) {
    auto reach = [&](uint32_t k) __attribute__((always_inline)) { return (int)__popcll(__ballot(key >= k)); };
    if (reach(1) < K) return 0;
    uint32_t hi = wave_max(key), lo = 0;
    int n = kWave; // lanes that reach lo
    for (uint32_t step = 1u << 23; hi > step; step <<= 2) {
        const int c = reach(hi - step);
        if (c >= K) {
            lo = hi - step;
            n = c;
            break;
        }
        hi -= step;
        if (step >= 1u << 29) break;
    }
    while (n > K + 8 && hi - lo > 0xffffu) {
        const uint32_t mid = lo + ((hi - lo) >> 1);
        const int c = reach(mid);
        if (c >= K) {
            lo = mid;
            n = c;
        } else {
            hi = mid;
        }
    }
    return lo;
}
// Ranks the n <= kCandCap keys of a wave's list by counting, sixteen at a time (read by all lanes at once; behind the list is
// room for as many zeros). emit(rank, key) once per rank 0..K-1 by some lane, key 0 past the last entry.
typedef __attribute__((ext_vector_type(2))) uint64_t u64x2;
template <typename Emit>
__device__ __forceinline__ void rank_list(uint64_t* list, int n, int K, Emit emit) {
    const int lane = threadIdx.x & 63;
    if (lane < kListPad) list[n + lane] = 0;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup"); // the list is read by other lanes of this wave
    for (int t = lane; t < ((n + kWave - 1) & ~(kWave - 1)); t += kWave) {
        const uint64_t k = list[t < n ? t : n];
        int rank = 0;
        for (int o = 0; o < n; o += kListPad) {
#pragma unroll
            for (int e = 0; e < kListPad; e += 2) {
                const u64x2 x = *(const u64x2*)&list[o + e];
                rank += (x[0] > k ? 1 : 0) + (x[1] > k ? 1 : 0);
            }
        }
        if (t < n && rank < K) emit(rank, k);
    }
    if (n < K && lane >= n && lane < K) emit(lane, 0);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup"); // reads done before the list is reused
}

// The K largest of a wave's keys (every lane passes NE, 0: none): emit(rank, key) as rank_list does.
// How: a bound that K of the lanes' own largest reach is a lower bound of the K-th largest, so the keys that reach it are a
// small superset of the answer; they are compacted into the wave's LDS list and ranked by counting. A plateau of equal
// values or a nearly empty wave can overflow the list: then the keys are extracted one by one instead. No workgroup barrier
// inside; the list is private to the wave.
template <int NE, typename Emit>
__device__ __forceinline__ void wave_topk(const uint64_t (&key)[NE], int K, uint64_t* list, Emit emit) {
    const int lane = threadIdx.x & 63;
    uint32_t best = 0;
#pragma unroll
    for (int e = 0; e < NE; ++e) best = max(best, (uint32_t)(key[e] >> 32));
    const uint32_t bound = max(kth_bound(best, K), 1u);
    int n = 0;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        const bool in = (uint32_t)(key[e] >> 32) >= bound;
        const uint64_t mask = __ballot(in);
        const int pos = n + __popcll(mask & ((1ull << lane) - 1ull));
        if (in && pos < kCandCap) list[pos] = key[e];
        n += __popcll(mask);
    }
    if (n <= kCandCap) {
        rank_list(list, n, K, emit);
    } else {
        uint64_t last = ~0ull;
        for (int r = 0; r < K; ++r) {
            uint64_t mine = 0;
#pragma unroll
            for (int e = 0; e < NE; ++e)
                if (key[e] < last && key[e] > mine) mine = key[e];
            last = wave_all(mine, [](uint64_t a, uint64_t b) { return a > b ? a : b; });
            if (lane == 0) emit(r, last);
        }
    }
}

// ---- Sorted lists side by side: every P lanes (8 or 16) of a register hold a list of P keys, largest first, zeros behind the last one. The P
// largest of two such lists are the larger ones of a[i] and b[P - 1 - i], which rise and fall once and so are sorted by log2 P steps of
// comparing with the lane at distance P / 2 .. 1. A step is six to eight instructions without a branch, so 16 lists of 8 become one
// in 0.4 us; bound, list in LDS and ranks (wave_topk) took 1.3.
template <int CTRL>
__device__ __forceinline__ uint64_t lanes_of(uint64_t x) { // every lane has a lane to read from
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)x, CTRL, 0xf, 0xf, true), hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(x >> 32), CTRL, 0xf, 0xf, true);
    return ((uint64_t)hi << 32) | lo;
}
template <int D>
__device__ __forceinline__ uint64_t lane_xor(uint64_t x) {
    if constexpr (D == 1) return lanes_of<kDppXor1>(x);
    else if constexpr (D == 2) return lanes_of<kDppXor2>(x);
    else if constexpr (D == 8) return lanes_of<kDppXor8>(x);
    else { // 4: the lower quads of each eight from the upper ones and back
        auto word = [](uint32_t w) __attribute__((always_inline)) {
            const int up = __builtin_amdgcn_update_dpp((int)w, (int)w, 0x104, 0xf, 0x5, false); // row_shl:4
            return (uint32_t)__builtin_amdgcn_update_dpp(up, (int)w, 0x114, 0xf, 0xa, false);   // row_shr:4
        };
        return ((uint64_t)word((uint32_t)(x >> 32)) << 32) | word((uint32_t)x);
    }
}
template <int D>
__device__ __forceinline__ uint64_t sort_step(uint64_t x) {
    const uint64_t y = lane_xor<D>(x);
    return (y > x) != ((threadIdx.x & D) != 0) ? y : x;
}
template <int P>
__device__ __forceinline__ uint64_t sort_list(uint64_t x) { // of keys that rise and fall once, or fall and rise
    if constexpr (P == 16) x = sort_step<8>(x);
    x = sort_step<4>(x);
    x = sort_step<2>(x);
    return sort_step<1>(x);
}
template <int P>
__device__ __forceinline__ uint64_t merge_lists(uint64_t a, uint64_t b) {
    b = lanes_of<P == 8 ? 0x141 : 0x140>(b); // the list backwards: row_half_mirror, row_mirror
    return sort_list<P>(a > b ? a : b);
}
// all lists of a register into one, in each of them
template <int P>
__device__ __forceinline__ uint64_t merge_register(uint64_t x) {
    if constexpr (P == 8) {
        const uint64_t y = lanes_of<0x140>(x); // the neighbouring list backwards
        x = sort_list<8>(x > y ? x : y);
    }
    u32x2 lo = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)x, false, false), hi = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(x >> 32), false, false);
    x = merge_lists<P>(((uint64_t)hi[0] << 32) | lo[0], ((uint64_t)hi[1] << 32) | lo[1]);
    lo = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)x, false, false);
    hi = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(x >> 32), false, false);
    return merge_lists<P>(((uint64_t)hi[0] << 32) | lo[0], ((uint64_t)hi[1] << 32) | lo[1]);
}

// What the last workgroup of a sequence asks for and makes of one frontier row, P >= K lanes to a chunk's list.
constexpr int kRowRegs = 4; // registers of lists on their way
struct RowInput {
    uint64_t ms, key[kRowRegs];
    float cum;
};
template <int P>
__device__ __forceinline__ void fetch_lists(const DraftExpandParams& p, int64_t row, int c0, uint64_t (&key)[kRowRegs]) {
    constexpr int G = kWave / P;
    const int lane = threadIdx.x & 63, list = lane / P, r = lane % P;
    const uint64_t* top = p.part_top + row * p.chunks * p.K;
#pragma unroll
    for (int q = 0; q < kRowRegs; ++q) {
        key[q] = 0;
        if (c0 + q * G < p.chunks) { // uniform
            const int c = c0 + q * G + list;
            const uint64_t k = load_device(top + min(c, p.chunks - 1) * p.K + min(r, p.K - 1));
            key[q] = c < p.chunks && r < p.K ? k : 0;
        }
    }
}
template <int P>
__device__ __forceinline__ RowInput row_request(const DraftExpandParams& p, int64_t row) {
    RowInput in;
    in.ms = load_device(p.part_ms + row * p.chunks + min((int)(threadIdx.x & 63), p.chunks - 1)); // (no branch around a load)
    fetch_lists<P>(p, row, 0, in.key);
    in.cum = p.cum_in ? p.cum_in[row] : 0.f;
    return in;
}
// lanes 0 .. K - 1: the row's first K entries; lse: its log-sum-exp
template <int P>
__device__ __forceinline__ uint64_t row_top(const DraftExpandParams& p, int64_t row, RowInput in, float& lse) {
    constexpr int G = kWave / P;
    const int lane = threadIdx.x & 63;
    const uint64_t* pms = p.part_ms + row * p.chunks;
    auto max_part = [](uint64_t ms) { return __uint_as_float((uint32_t)ms); };
    auto sum_part = [](uint64_t ms) { return __uint_as_float((uint32_t)(ms >> 32)); };
    const float m0 = lane < p.chunks ? max_part(in.ms) : -INFINITY;
    float m = m0;
    for (int c = lane + kWave; c < p.chunks; c += kWave) m = fmaxf(m, max_part(load_device(pms + c)));
    m = wave_max(m);
    float z = (m0 > -INFINITY) ? sum_part(in.ms) * __builtin_amdgcn_exp2f((m0 - m) * 1.4426950408889634f) : 0.f;
    for (int c = lane + kWave; c < p.chunks; c += kWave) {
        const uint64_t ms = load_device(pms + c);
        if (max_part(ms) > -INFINITY) z += sum_part(ms) * __builtin_amdgcn_exp2f((max_part(ms) - m) * 1.4426950408889634f);
    }
    lse = m + __logf(wave_sum(z));
    uint64_t top = in.key[0];
    for (int c0 = 0;;) {
#pragma unroll
        for (int q = 1; q < kRowRegs; ++q)
            if (c0 + q * G < p.chunks) top = merge_lists<P>(top, in.key[q]);
        c0 += kRowRegs * G;
        if (c0 >= p.chunks) break;
        fetch_lists<P>(p, row, c0, in.key);
        top = merge_lists<P>(top, in.key[0]);
    }
    return merge_register<P>(top);
}
// The `keep` first of the rows' candidates in (score descending, index ascending) order, in lanes 0 .. keep - 1: their keys, 0 past the last. One
// wave. A row's candidates stand in that order already: cum + (entry - lse) falls with the entry, equal ones come in the order of their
// index, and NaN is the score of all of them or of the last (an infinite sum plus an entry of -inf).
template <int P>
__device__ __forceinline__ uint64_t frontier_top(const float* score, int F, int K) {
    constexpr int G = kWave / P;
    const int lane = threadIdx.x & 63, r = lane % P;
    uint64_t top = 0;
    for (int f0 = 0; f0 < F; f0 += G) {
        const int f = f0 + lane / P, c = min(f, F - 1) * K + min(r, K - 1);
        const uint64_t key = f < F && r < K ? child_key(score[c], c) : 0;
        top = f0 == 0 ? key : merge_lists<P>(top, key);
    }
    return merge_register<P>(top);
}

// grid = B * F * chunks, block = 512. Bound by its serial chain. Stamps of a level of 2 x 8 x 152064 logits (us after the first wave's entry,
// median and last): logits 0.9 / 1.3, statistics 1.7 / 2.1, bound and list 3.1 / 3.6, ranks in memory 4.0 / 4.6, last arrival known 5.7,
// the chunks' results read 6.9, rows merged 7.7, frontier written 8.3; 1.4 between two levels. What that took before:
//   a workgroup on every CU and two on some instead (chunks of 8192 logits): all ranks in memory at 5.8
//   the chunks' lists and the frontier by bound, list and ranks (wave_topk) instead of merges of sorted lists: 2.0 and 1.0 instead of 0.8
//   and 0.6, every eight rows
// Three levels and the selection, us: 2 x 8 x 152064 35.0 -> 31.8, K = 16 64.7 -> 47.4 (1 x 16 x 152064), 8 x 10 x 32000 39.9 -> 33.7.
// (Earlier: one list for the whole workgroup with the K-th largest of 32 groups as its bound, sixteen keys ranked a step and chunk lists
// of 64-bit keys 43.2 -> 37.8; the chunk's statistics on a second wave beside the ranking 35.9 -> 35.1.)
template <int VEC>
__global__ __launch_bounds__(kExpandThreads) void draft_expand_kernel(const DraftExpandParams p) {
    request_args(p);
    constexpr int CHUNK = VEC * kDraftVec;
    __shared__ float s_m[kExpandWaves], s_s[kExpandWaves];
    __shared__ __attribute__((aligned(16))) uint64_t s_list[kExpandWaves * kListLen];
    __shared__ uint64_t s_wave[kExpandWaves * kMaxDraftK];
    __shared__ float s_score[kMaxDraftCand];
    __shared__ int32_t s_token[kMaxDraftCand];
    __shared__ __attribute__((aligned(16))) uint32_t s_group[kGroups];
    __shared__ int32_t s_last, s_n;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int F = p.F, K = p.K;
    int b;
    {
        // workgroup id = row * chunks + chunk (the host keeps the product below 2^31)
        uint32_t chunk_u, f_u;
        const int64_t row = fast_div(blockIdx.x, p.by_chunks, chunk_u);
        const int chunk = (int)chunk_u;
        b = (int)fast_div((uint32_t)row, p.by_F, f_u);
        uint64_t* const arrivals = p.arrivals + (int64_t)b * kArrivalWords;
        uint64_t seen = 0;
        if (wave == 0) seen = load_device(arrivals); // ahead of the logits: loads return in order
        const float* __restrict__ lg = p.logits + row * p.ld;
        const int begin = chunk * CHUNK;
        const int end = min(p.V, begin + CHUNK);
        // every thread holds 4 * VEC entries and perhaps one of the up to three behind the last four; a chunk of at most 256 * VEC
        // entries (the last of a row) lies in the first wave alone
        const int nvec = (end - begin) >> 2;
        const bool one_wave = nvec <= kWave * VEC;
        const int stride = one_wave ? kWave : kExpandThreads, nmine = one_wave && wave != 0 ? 0 : nvec;
        float ev[4 * VEC + 1];
#pragma unroll
        for (int j = 0; j < VEC; ++j) {
            const int k = tid + j * stride;
            const f32x4 x = (k < nmine) ? load4_stream(lg + begin + 4 * k) : f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
            for (int e = 0; e < 4; ++e) ev[4 * j + e] = x[e];
        }
        const int tail = begin + 4 * nvec + tid;
        ev[4 * VEC] = tail < end ? lg[tail] : -INFINITY;
        auto key_of = [&](int e) __attribute__((always_inline)) { // of ev[e]
            const int k = tid + (e >> 2) * stride;
            const bool has = e == 4 * VEC ? tail < end : k < nmine;
            return has ? child_key(ev[e], e == 4 * VEC ? tail : begin + 4 * k + (e & 3)) : 0;
        };
        if (tid == 0) {
            arrival_open(arrivals, seen);
            s_n = 0;
        }

        // ---- the chunk's maximum and sum of exp (per wave, then of the waves), and its K first entries: the K-th largest of
        // the maxima of 32 groups of 64 * VEC entries is a bound that K entries reach and few others do
        float own = ev[0];
#pragma unroll
        for (int q = 1; q <= 4 * VEC; ++q) own = fmaxf(own, ev[q]);
        float m = row_max(own); // of the group
        if ((lane & 15) == 0) s_group[tid >> 4] = ((m == m ? order_key(m) : 0) & ~(kGroups - 1u)) | (tid >> 4); // all different
        if (!one_wave) {
            m = max_of_rows(m);
            float s = 0.f;
            if (m > -INFINITY) {
#pragma unroll
                for (int q = 0; q <= 4 * VEC; ++q) s += __builtin_amdgcn_exp2f((ev[q] - m) * 1.4426950408889634f); // exp2(-inf) = 0
            }
            s = wave_sum(s);
            if (lane == 0) {
                s_m[wave] = m;
                s_s[wave] = s;
            }
        } else if (wave == 0 || wave >= VEC) { // the same sums as of a long chunk: those of VEC waves
#pragma unroll
            for (int j = 0; j < VEC; ++j) {
                const float last = j == 0 ? ev[4 * VEC] : -INFINITY;
                const float mj = wave_max(fmaxf(fmaxf(fmaxf(ev[4 * j], ev[4 * j + 1]), fmaxf(ev[4 * j + 2], ev[4 * j + 3])), last));
                float s = 0.f;
                if (mj > -INFINITY) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) s += __builtin_amdgcn_exp2f((ev[4 * j + q] - mj) * 1.4426950408889634f);
                    s += __builtin_amdgcn_exp2f((last - mj) * 1.4426950408889634f);
                }
                s = wave_sum(s);
                if (lane == 0 && (wave == 0 || j == 0)) {
                    s_m[wave + j] = mj;
                    s_s[wave + j] = s;
                }
            }
        }
        __syncthreads();
        if (!one_wave) {
            const uint32_t g = s_group[lane & (kGroups - 1)];
            int above = 0;
#pragma unroll
            for (int q = 0; q < kGroups; q += 4) {
                const u32x4 x = *(const u32x4*)&s_group[q];
#pragma unroll
                for (int e = 0; e < 4; ++e) above += x[e] > g ? 1 : 0;
            }
            const uint32_t bound = (uint32_t)__builtin_amdgcn_readlane(g, __builtin_ctzll(__ballot(above == K - 1))) & ~(kGroups - 1u);
            const float tau = key_value(bound);
            if (bound <= 0x007fffffu) { // -inf among the K
                if (tid == 0) s_n = kCandCap + 1;
            } else if (own >= tau) { // few lanes
#pragma unroll
                for (int e = 0; e <= 4 * VEC; ++e)
                    if (ev[e] >= tau) {
                        const int at = atomicAdd(&s_n, 1); // the order of the list does not matter
                        if (at < kCandCap) s_list[at] = key_of(e);
                    }
            }
            __syncthreads();
        }
        const int n = s_n;
        auto topk_own = [&](uint64_t* list, auto emit) __attribute__((always_inline)) {
            uint64_t key[4 * VEC + 1];
#pragma unroll
            for (int e = 0; e <= 4 * VEC; ++e) key[e] = key_of(e);
            wave_topk(key, K, list, emit);
        };
        if (n > kCandCap) { // a plateau of equal values: every wave's first K, then those of all
            __syncthreads();
            topk_own(s_list + wave * kListLen, [&](int r, uint64_t k) { s_wave[wave * kMaxDraftK + r] = k; });
            __syncthreads();
        }
        if (wave == 1) { // the chunk's statistics, while the first wave ranks its list: one after the other took a tree from 35.1 to 35.9 us
            const float wm = lane < kExpandWaves ? s_m[lane] : -INFINITY;
            const float cm = wave_max(wm);
            const float cs = wave_sum(wm > -INFINITY ? s_s[lane & (kExpandWaves - 1)] * __builtin_amdgcn_exp2f((wm - cm) * 1.4426950408889634f) : 0.f);
            if (lane == 0) store_device(p.part_ms + row * p.chunks + chunk, ((uint64_t)__float_as_uint(cs) << 32) | __float_as_uint(cm));
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // in memory
        }
        if (wave == 0) {
            uint64_t* const top = p.part_top + (row * p.chunks + chunk) * K;
            auto out = [&](int r, uint64_t k) { store_device(top + r, k); }; // 0 when the chunk has fewer than r + 1 entries
            if (one_wave) {
                topk_own(s_list, out);
            } else if (n <= kCandCap) {
                rank_list(s_list, n, K, out);
            } else {
                constexpr int NE = kExpandWaves * kMaxDraftK / kWave;
                uint64_t key[NE];
#pragma unroll
                for (int q = 0; q < NE; ++q) { // rank r of wave w
                    const int e = lane + q * kWave;
                    key[q] = (e & (kMaxDraftK - 1)) < K ? s_wave[e] : 0;
                }
                wave_topk(key, K, s_list, out);
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
        __syncthreads(); // this chunk's results are in memory
        if (tid == 0) s_last = arrival_last(arrivals, (uint32_t)(F * p.chunks)) ? 1 : 0;
        __syncthreads();
        if (s_last == 0) return;
    }

    // ---- the sequence's last workgroup: one wave per frontier row (rows beyond eight take turns)
    const int C = F * K;
    const int keep = min(K, C);
    constexpr int CPT = kMaxDraftCand / kExpandThreads; // candidates per thread, at most
    int32_t par_own[CPT]; // the candidates' parents (the frontier rows they extend): requested now, written out at the end
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
        const int c = tid + i * kExpandThreads;
        uint32_t r;
        par_own[i] = (c < C && p.frontier_cand) ? p.frontier_cand[(int64_t)b * F + fast_div(c, p.by_K, r)] : -1;
    }

    // ---- per row: log-sum-exp and the K first entries of the merged chunk lists. The next row's are asked for before the row's are used.
    auto rows = [&](auto width) __attribute__((always_inline)) {
        constexpr int P = decltype(width)::value;
        RowInput in = {};
        if (wave < F) in = row_request<P>(p, (int64_t)b * F + wave);
        for (int f = wave; f < F; f += kExpandWaves) {
            RowInput next = {};
            if (f + kExpandWaves < F) next = row_request<P>(p, (int64_t)b * F + f + kExpandWaves);
            float lse;
            const uint64_t k = row_top<P>(p, (int64_t)b * F + f, in, lse);
            if (lane < K) {
                s_token[f * K + lane] = k != 0 ? entry_index(k) : INT32_MAX;
                s_score[f * K + lane] = in.cum + ((k != 0 ? entry_value(k) : -INFINITY) - lse);
            }
            in = next;
        }
    };
    if (K <= 8) rows(std::integral_constant<int, 8>{});
    else rows(std::integral_constant<int, 16>{});
    __syncthreads();

    // ---- the candidates, and the next frontier: the `keep` first of them in (score descending, index ascending),
    // listed in ascending index
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
        const int c = tid + i * kExpandThreads;
        if (c < C) {
            const int64_t g = (int64_t)b * p.cand_capacity + p.cand_base + c;
            p.cand_token[g] = s_token[c];
            p.cand_score[g] = s_score[c];
            p.cand_parent[g] = par_own[i];
        }
    }
    if (keep == C) { // one row, or one child per row: all of them
        if (tid < C) {
            p.next_frontier_cand[(int64_t)b * keep + tid] = p.cand_base + tid;
            p.next_cum[(int64_t)b * keep + tid] = s_score[tid];
        }
        return;
    }
    if (wave != 0) return;
    const uint64_t first = K <= 8 ? frontier_top<8>(s_score, F, K) : frontier_top<16>(s_score, F, K);
    const uint64_t k = lane < keep ? first : 0;
    const int32_t c = k != 0 ? entry_index(k) : INT32_MAX;
    int pos = 0;
    for (int o = 0; o < keep; ++o) pos += __builtin_amdgcn_readlane(c, o) < c ? 1 : 0;
    if (k != 0) {
        p.next_frontier_cand[(int64_t)b * keep + pos] = p.cand_base + c;
        p.next_cum[(int64_t)b * keep + pos] = s_score[c];
    }
}

// grid = B, block = 256.
__global__ __launch_bounds__(kSelThreads) void draft_tree_build_kernel(const DraftBuildParams p) {
    request_args(p);
    constexpr int kWords = kMaxDraftTotal / 64;
    constexpr int kRounds = kMaxDraftTotal / kSelThreads; // candidates per thread, at most
    constexpr int kSelWaves = kSelThreads / kWave;
    constexpr int kList = 256;                            // candidates that can be ranked among themselves
    __shared__ __attribute__((aligned(16))) float s_score[kMaxDraftTotal + 4];
    __shared__ int32_t s_parent[kMaxDraftTotal];
    __shared__ uint64_t s_mask[kWords];   // picked candidates, one bit each
    __shared__ int32_t s_before[kWords];  // picked candidates below word w
    __shared__ int32_t s_bad;
    __shared__ uint32_t s_top[kSelThreads];               // every thread's largest key
    __shared__ __attribute__((aligned(16))) uint64_t s_list[kList];
    __shared__ int32_t s_n;
    const int b = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int M = p.M, N = p.N;
    const int take = min(N, M);
    const int32_t* tok = p.cand_token + (int64_t)b * p.cand_capacity;
    const float* score = p.cand_score + (int64_t)b * p.cand_capacity;
    const int32_t* par = p.cand_parent + (int64_t)b * p.cand_capacity;
    float v[kRounds];
    int32_t pc_own[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) { // candidate r * 256 + tid
        const int c = r * kSelThreads + tid;
        v[r] = c < M ? score[c] : -INFINITY;
        pc_own[r] = c < M ? par[c] : -1;
    }
    if (tid == 0) {
        s_bad = 0;
        s_n = 0;
    }
    if (tid < kWords) s_mask[tid] = 0;
    uint32_t top = 0;
    bool bad_own = false;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int c = r * kSelThreads + tid;
        if (c < M) {
            s_score[c] = v[r];
            s_parent[c] = pc_own[r];
            bad_own |= pc_own[r] < -1 || pc_own[r] >= c;
            top = max(top, rank_key(v[r]));
        }
    }
    s_top[tid] = top;
    if (tid < ((M + 3) & ~3) - M) s_score[M + tid] = -INFINITY; // padding of the last group of four
    __syncthreads();
    if (__ballot(bad_own) && lane == 0) atomicOr(&s_bad, 1);
    // The `take`-th largest of the threads' own largest scores is a bound that at least `take` candidates reach
    // (none if fewer threads hold a candidate); those that reach it are few. Every wave finds it for itself.
    // (Ranking all candidates among all took 85 us at 800 candidates.)
    uint32_t tops[kSelWaves];
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) tops[w] = s_top[w * kWave + lane];
    uint32_t bound = 0;
#pragma unroll
    for (int bit = 31; bit >= 16; --bit) {
        const uint32_t trial = bound | (1u << bit);
        int n = 0;
#pragma unroll
        for (int w = 0; w < kSelWaves; ++w) n += __popcll(__ballot(tops[w] >= trial));
        if (n >= take) bound = trial;
    }
    int base = 0;
    bool in[kRounds];
    {
        int mine = 0;
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const int c = r * kSelThreads + tid;
            in[r] = c < M && rank_key(v[r]) >= bound;
            mine += __popcll(__ballot(in[r]));
        }
        if (lane == 0) base = atomicAdd(&s_n, mine); // the order of the list does not matter
        base = __builtin_amdgcn_readfirstlane(base);
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const uint64_t m = __ballot(in[r]);
            const int pos = base + __popcll(m & ((1ull << lane) - 1ull));
            if (in[r] && pos < kList) s_list[pos] = entry_key(v[r], r * kSelThreads + tid);
            base += __popcll(m);
        }
    }
    __syncthreads();
    const int n = s_n;
    if (n <= kList) {
        // rank by counting among the list, picked = rank < take, one bit per candidate
        if (tid < (n & 1)) s_list[n + tid] = 0; // comes before nothing (n is even at kList)
        __syncthreads();
        if (tid < n) {
            const uint64_t k = s_list[tid];
            const int c = entry_index(k);
            typedef __attribute__((ext_vector_type(2))) uint64_t u64x2;
            int rank = 0;
#pragma unroll 4
            for (int o = 0; o < n; o += 2) {
                const u64x2 ko = *(const u64x2*)&s_list[o];
                rank += (ko[0] > k ? 1 : 0) + (ko[1] > k ? 1 : 0);
            }
            if (rank < take) atomicOr((unsigned long long*)&s_mask[c >> 6], 1ull << (c & 63));
        }
    } else {
        // a plateau of equal scores: rank every candidate among all (four scores per LDS read; a padding entry
        // is -inf at an index >= M > c, which comes before nothing)
        const int M4 = (M + 3) & ~3;
        for (int r = 0; r < kRounds && r * kSelThreads < M; ++r) { // every thread runs all rounds: the ballots need whole waves
            const int c = r * kSelThreads + tid;
            bool pick = false;
            if (c < M) {
                const float sc = s_score[c];
                int rank = 0;
                for (int o = 0; o < M4; o += 4) {
                    const f32x4 so = *(const f32x4*)&s_score[o];
#pragma unroll
                    for (int e = 0; e < 4; ++e) rank += before(so[e], o + e, sc, c) ? 1 : 0;
                }
                pick = rank < take;
            }
            const uint64_t m = __ballot(pick);
            if (lane == 0) s_mask[c >> 6] = m;
        }
    }
    __syncthreads();
    const int words = (M + 63) >> 6;
    if (tid == 0) {
        int acc = 0;
        for (int w = 0; w < words; ++w) {
            s_before[w] = acc;
            acc += __builtin_popcountll(s_mask[w]);
        }
    }
    auto picked = [&](int c) { return (s_mask[c >> 6] >> (c & 63)) & 1ull; };
    if (!s_bad) {
        for (int c = tid; c < M; c += kSelThreads)
            if (picked(c) && s_parent[c] >= 0 && !picked(s_parent[c])) atomicOr(&s_bad, 1);
    }
    __syncthreads();
    const bool bad = s_bad != 0;
    int32_t* o_parent = p.parent + (int64_t)b * (N + 1);
    int32_t* o_tokens = p.tokens + (int64_t)b * (N + 1);
    int32_t* o_cand = p.node_cand + (int64_t)b * (N + 1);
    for (int t = tid; t <= N; t += kSelThreads) { // the root, and -1 wherever no node is written below
        if (!bad && t >= 1 && t <= take) continue;
        o_parent[t] = -1;
        o_tokens[t] = (t == 0 && p.root_token) ? p.root_token[b] : -1;
        o_cand[t] = -1;
    }
    if (tid == 0) {
        p.num_nodes[b] = bad ? 0 : take + 1;
        if (p.status) p.status[b] = bad ? VS_STATUS_BAD_CANDIDATE : VS_STATUS_OK;
    }
    if (bad) return;
    // node id = 1 + number of picked candidates with a smaller index
    auto node_of = [&](int c) { return 1 + s_before[c >> 6] + __builtin_popcountll(s_mask[c >> 6] & ((1ull << (c & 63)) - 1ull)); };
    for (int c = tid; c < M; c += kSelThreads) {
        if (!picked(c)) continue;
        const int node = node_of(c);
        if (node > take) continue; // only NaN scores can rank more than `take` candidates first
        const int32_t pc = s_parent[c];
        o_parent[node] = pc >= 0 ? node_of(pc) : 0;
        o_tokens[node] = tok[c];
        o_cand[node] = c;
    }
}

} // namespace

hipError_t launch_draft_expand(const DraftExpandParams& p, hipStream_t s) {
    const dim3 grid((unsigned)((int64_t)p.chunks * p.B * p.F)), block(kExpandThreads);
    if (p.vec == 4) hipLaunchKernelGGL(draft_expand_kernel<4>, grid, block, 0, s, p);
    else if (p.vec == 5) hipLaunchKernelGGL(draft_expand_kernel<5>, grid, block, 0, s, p);
    else if (p.vec == 6) hipLaunchKernelGGL(draft_expand_kernel<6>, grid, block, 0, s, p);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_draft_tree_build(const DraftBuildParams& p, hipStream_t s) {
    hipLaunchKernelGGL(draft_tree_build_kernel, dim3(p.B), dim3(kSelThreads), 0, s, p);
    return hipGetLastError();
}

} // namespace vs
