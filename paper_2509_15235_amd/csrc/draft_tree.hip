// Draft-tree construction (paper Section 3.1 adopts EAGLE-2's context-aware dynamic draft
// tree; Appendix A: 30 draft tokens, depth 3, 8 nodes kept per expansion). A node's score
// is the sum of the draft model's log-probabilities along its path. An expansion step gives
// every frontier node its K most likely tokens as children and keeps the K best-scored
// children as the next frontier; at the end the N best-scored candidates of all levels are
// the tree. The draft model's forward pass is not part of this: its logits are inputs.
//
// Two kernels. (1) An expansion: every workgroup reduces an 8192-float chunk of a logits row to (maximum, sum of
// exp, the chunk's K largest entries); the workgroup of a sequence that finishes last merges the chunks into each
// row's top K and log-sum-exp, scores the F*K candidates and picks the next frontier. (That second part used to
// be a kernel of its own: 7.8 us for one trip to memory and half a microsecond of work, three times per tree.)
// (2) One workgroup per sequence for the final selection, which emits parent[] / tokens[] in candidate order.
//
// Selection without bookkeeping: entries are taken in the strict total order (value descending, index
// ascending). A bound that at least K entries reach is found bit by bit with ballots, the few entries at or
// above it are compacted and ranked by counting; nothing has to be marked as taken.
#include <type_traits>

#include "vs_device.h"

namespace vs {

namespace {

constexpr int kVec = 4;          // 16-byte loads per thread and chunk
constexpr int kSelThreads = 256;
constexpr int kExpandThreads = 512;
constexpr int kExpandWaves = kExpandThreads / kWave;
static_assert(kDraftChunk == kExpandThreads * kVec * 4, "a chunk is one set of loads");

struct Ent {
    float v;
    int32_t i;
};

// a comes strictly before b in (value descending, index ascending)
__device__ __forceinline__ bool before(float av, int32_t ai, float bv, int32_t bi) {
    return av > bv || (av == bv && ai < bi);
}

__device__ __forceinline__ Ent wave_first(Ent e) {
    return wave_all(e, [](Ent x, Ent y) { return before(y.v, y.i, x.v, x.i) ? y : x; });
}

constexpr int32_t kNone = INT32_MAX; // index of "no entry": loses every comparison at value -inf
constexpr int kCandCap = 128;        // entries of a wave's candidate list in LDS

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
// An entry as one integer: larger = earlier in (value descending, index ascending).
__device__ __forceinline__ uint64_t entry_key(float v, int32_t i) { return ((uint64_t)rank_key(v) << 32) | (uint32_t)~i; }
__device__ __forceinline__ float entry_value(uint64_t k) { return key_value((uint32_t)(k >> 32)); }
__device__ __forceinline__ int32_t entry_index(uint64_t k) { return (int32_t)~(uint32_t)k; }

// The first K of a wave's entries in (value descending, index ascending); every lane passes NE
// entries v[e] with index idx(e) (kNone = none). emit(rank, value, index) is called once per rank 0..K-1 by
// some lane; ranks past the number of entries get (-inf, kNone).
// How: the K-th largest of the lanes' own maxima (found bit by bit with ballots) is a lower
// bound of the K-th largest entry, so the entries at or above it are a small superset of the
// answer; they are compacted into the wave's LDS list and ranked by counting. A plateau of
// equal values or a nearly empty wave can overflow the list: then the entries are extracted
// one by one instead. No workgroup barrier inside; the list is private to the wave.
template <int NE, typename Idx, typename Emit>
__device__ __forceinline__ void wave_topk(const float (&v)[NE], Idx idx, int K, uint64_t* list, Emit emit) {
    const int lane = threadIdx.x & 63;
    uint32_t best = 0;
#pragma unroll
    for (int e = 0; e < NE; ++e)
        if (idx(e) != kNone) best = max(best, order_key(v[e]));
    // (the upper sixteen bits of the bound are enough: it only has to be one that K lanes reach and few entries do)
    uint32_t res = 0;
#pragma unroll
    for (int bit = 31; bit >= 16; --bit) {
        const uint32_t trial = res | (1u << bit);
        if (__popcll(__ballot(best >= trial)) >= K) res = trial;
    }
    // res below the key of -inf: fewer than K lanes hold entries, or nothing above -inf bounds them
    const float tau = res > 0x007fffffu ? key_value(res) : -INFINITY;
    int n = 0;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        const bool pred = v[e] >= tau && idx(e) != kNone;
        const uint64_t mask = __ballot(pred);
        if (mask == 0) continue; // most of the time
        const int pos = n + __popcll(mask & ((1ull << lane) - 1ull));
        if (pred && pos < kCandCap) list[pos] = entry_key(v[e], idx(e));
        n += __popcll(mask);
    }
    if (n <= kCandCap) {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup"); // the list is read by other lanes of this wave
        if (n <= kWave) { // one entry per lane, the others' by v_readlane
            const uint64_t k = lane < n ? list[lane] : 0;
            int rank = 0;
            for (int o = 0; o < n; ++o) {
                const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)k, o), hi = __builtin_amdgcn_readlane((uint32_t)(k >> 32), o);
                rank += (((uint64_t)hi << 32) | lo) > k ? 1 : 0;
            }
            if (lane < n && rank < K) emit(rank, entry_value(k), entry_index(k));
        } else {
            for (int t = lane; t < n; t += kWave) {
                const uint64_t k = list[t];
                int rank = 0;
                for (int o = 0; o < n; ++o) rank += list[o] > k ? 1 : 0;
                if (rank < K) emit(rank, entry_value(k), entry_index(k));
            }
        }
        for (int r = n + lane; r < K; r += kWave) emit(r, -INFINITY, kNone);
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup"); // reads done before the list is reused
    } else {
        float last_v = INFINITY;
        int32_t last_i = -1;
        for (int r = 0; r < K; ++r) {
            Ent mine = {-INFINITY, kNone};
#pragma unroll
            for (int e = 0; e < NE; ++e)
                if (idx(e) != kNone && before(last_v, last_i, v[e], idx(e)) && before(v[e], idx(e), mine.v, mine.i))
                    mine = {v[e], idx(e)};
            const Ent w = wave_first(mine);
            if (lane == 0) emit(r, w.v, w.i);
            last_v = w.v;
            last_i = w.i;
        }
    }
}

// grid = B * F * chunks, block = 512.
__global__ __launch_bounds__(kExpandThreads) void draft_expand_kernel(const DraftExpandParams p) {
    __shared__ float s_m[kExpandWaves], s_s[kExpandWaves];
    __shared__ uint64_t s_list[kExpandWaves * kCandCap];
    __shared__ float s_wv[kExpandWaves * kMaxDraftK];
    __shared__ int32_t s_wi[kExpandWaves * kMaxDraftK];
    __shared__ float s_score[kMaxDraftCand];
    __shared__ int32_t s_token[kMaxDraftCand];
    __shared__ int32_t s_last;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int F = p.F, K = p.K;
    int b;
    {
        // workgroup id = row * chunks + chunk (the host keeps the product below 2^31)
        const int64_t row = blockIdx.x / (uint32_t)p.chunks;
        const int chunk = (int)(blockIdx.x - (uint32_t)row * (uint32_t)p.chunks);
        b = (int)(row / F);
        const float* __restrict__ lg = p.logits + row * p.ld;
        const int begin = chunk * kDraftChunk;
        const int end = min(p.V, begin + kDraftChunk);
        // every thread holds 16 entries and perhaps one of the up to three behind the last four
        const int nvec = (end - begin) >> 2;
        float ev[4 * kVec + 1];
#pragma unroll
        for (int j = 0; j < kVec; ++j) {
            const int k = tid + j * kExpandThreads;
            const f32x4 x = (k < nvec) ? load4_stream(lg + begin + 4 * k) : f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
            for (int e = 0; e < 4; ++e) ev[4 * j + e] = x[e];
        }
        const int tail = begin + 4 * nvec + tid;
        ev[4 * kVec] = tail < end ? lg[tail] : -INFINITY;
        auto index = [&](int e) { // of ev[e]
            if (e == 4 * kVec) return tail < end ? tail : kNone;
            const int k = tid + (e >> 2) * kExpandThreads;
            return k < nvec ? begin + 4 * k + (e & 3) : kNone;
        };
        if (tid == 0) arrival_open(p.arrivals + (int64_t)b * kArrivalWords);

        // ---- per wave: maximum, sum of exp, the K first entries; one barrier, then wave 0 merges the waves
        float m = ev[0];
#pragma unroll
        for (int q = 1; q <= 4 * kVec; ++q) m = fmaxf(m, ev[q]);
        m = wave_max(m);
        float s = 0.f;
        if (m > -INFINITY) {
#pragma unroll
            for (int q = 0; q <= 4 * kVec; ++q) s += __builtin_amdgcn_exp2f((ev[q] - m) * 1.4426950408889634f); // exp2(-inf) = 0
        }
        s = wave_sum(s);
        if (lane == 0) {
            s_m[wave] = m;
            s_s[wave] = s;
        }
        wave_topk(ev, index, K, s_list + wave * kCandCap, [&](int r, float v, int32_t i) {
            s_wv[wave * kMaxDraftK + r] = v;
            s_wi[wave * kMaxDraftK + r] = i;
        });
        __syncthreads();
        if (wave == 0) {
            const float wm = lane < kExpandWaves ? s_m[lane] : -INFINITY;
            const float cm = wave_max(wm);
            const float cs = wave_sum(wm > -INFINITY ? s_s[lane & (kExpandWaves - 1)] * __builtin_amdgcn_exp2f((wm - cm) * 1.4426950408889634f) : 0.f);
            if (lane == 0) {
                store_device(p.part_m + row * p.chunks + chunk, cm);
                store_device(p.part_s + row * p.chunks + chunk, cs);
            }
            constexpr int NE = kExpandWaves * kMaxDraftK / kWave;
            float mv[NE];
            int32_t mi[NE];
#pragma unroll
            for (int q = 0; q < NE; ++q) { // entry (wave w, rank r) = w * K + r
                const int e = lane + q * kWave, w = e / K, r = e - w * K;
                const bool has = w < kExpandWaves;
                mv[q] = has ? s_wv[w * kMaxDraftK + r] : -INFINITY;
                mi[q] = has ? s_wi[w * kMaxDraftK + r] : kNone;
            }
            float* out_v = p.part_tv + (row * p.chunks + chunk) * K;
            int32_t* out_i = p.part_ti + (row * p.chunks + chunk) * K;
            wave_topk(mv, [&](int e) { return mi[e]; }, K, s_list, [&](int rr, float v, int32_t i) {
                store_device(out_v + rr, v);
                store_device(out_i + rr, i); // kNone when the chunk has fewer than rr+1 entries
            });
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // this chunk's results are in memory
            if (lane == 0) s_last = arrival_last(p.arrivals + (int64_t)b * kArrivalWords, (uint32_t)(F * p.chunks)) ? 1 : 0;
        }
        __syncthreads();
        if (s_last == 0) return;
    }

    // ---- the sequence's last workgroup: one wave per frontier row (rows beyond eight take turns)
    const int C = F * K;
    const int keep = min(K, C);
    // candidates' parents (the frontier rows they extend): requested now, written out at the end
    constexpr int CPT = kMaxDraftCand / kExpandThreads; // candidates per thread, at most
    int32_t par_own[CPT];
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
        const int c = tid + i * kExpandThreads;
        par_own[i] = (c < C && p.frontier_cand) ? p.frontier_cand[(int64_t)b * F + c / K] : -1;
    }

    // ---- per row: log-sum-exp and the K first entries of the merged chunk lists
    // (chunk statistics, score and the first 256 list entries are requested before anything is used; longer
    // lists come in further batches, the K best so far among them)
    const int n = p.chunks * K;
    for (int f = wave; f < F; f += kExpandWaves) {
        const int64_t row = (int64_t)b * F + f;
        const float* pm = p.part_m + row * p.chunks;
        const float* ps = p.part_s + row * p.chunks;
        const float* tv = p.part_tv + row * n;
        const int32_t* ti = p.part_ti + row * n;
        constexpr int NE = 4;
        float v[NE + 1];
        int32_t idx[NE + 1];
        auto fetch = [&](int e0) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < NE; ++q) {
                const int e = e0 + lane + q * kWave;
                v[q] = -INFINITY;
                idx[q] = kNone;
                if (e0 + q * kWave < n) { // uniform
                    const float x = load_device(tv + min(e, n - 1));
                    const int32_t i = load_device(ti + min(e, n - 1));
                    v[q] = e < n ? x : -INFINITY;
                    idx[q] = e < n ? i : kNone;
                }
            }
        };
        float m0 = load_device(pm + min(lane, p.chunks - 1)); // (no branch around a load)
        const float s0 = load_device(ps + min(lane, p.chunks - 1));
        fetch(0);
        const float cum = p.cum_in ? p.cum_in[row] : 0.f;
        if (lane >= p.chunks) m0 = -INFINITY;
        float m = m0;
        for (int c = lane + kWave; c < p.chunks; c += kWave) m = fmaxf(m, load_device(pm + c));
        m = wave_max(m);
        float z = (m0 > -INFINITY) ? s0 * __builtin_amdgcn_exp2f((m0 - m) * 1.4426950408889634f) : 0.f;
        for (int c = lane + kWave; c < p.chunks; c += kWave) {
            const float mc = load_device(pm + c);
            if (mc > -INFINITY) z += load_device(ps + c) * __builtin_amdgcn_exp2f((mc - m) * 1.4426950408889634f);
        }
        z = wave_sum(z);
        const float lse = m + __logf(z);
        float* best_v = s_wv + wave * kMaxDraftK;
        int32_t* best_i = s_wi + wave * kMaxDraftK;
        for (int e0 = 0; e0 < n; e0 += NE * kWave) {
            if (e0 > 0) fetch(e0);
            const bool more = e0 > 0 && lane < K;
            v[NE] = more ? best_v[lane] : -INFINITY;
            idx[NE] = more ? best_i[lane] : kNone;
            wave_topk(v, [&](int e) { return idx[e]; }, K, s_list + wave * kCandCap, [&](int r, float x, int32_t i) {
                best_v[r] = x;
                best_i[r] = i;
            });
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup"); // read by other lanes of this wave
        }
        if (lane < K) {
            s_token[f * K + lane] = best_i[lane];
            s_score[f * K + lane] = cum + (best_v[lane] - lse);
        }
    }
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
    uint64_t* const list = s_list + wave * kCandCap;
    if (C > kWave) { // every wave's share first
        constexpr int NE = kMaxDraftCand / kExpandThreads;
        float fv[NE];
        int32_t fi[NE];
#pragma unroll
        for (int q = 0; q < NE; ++q) {
            const int c = tid + q * kExpandThreads;
            fv[q] = c < C ? s_score[c] : -INFINITY;
            fi[q] = c < C ? c : kNone;
        }
        wave_topk(fv, [&](int e) { return fi[e]; }, keep, list, [&](int r, float v, int32_t i) {
            s_wv[wave * kMaxDraftK + r] = v;
            s_wi[wave * kMaxDraftK + r] = i;
        });
        __syncthreads();
    }
    if (wave != 0) return;
    {
        constexpr int NE = kExpandWaves * kMaxDraftK / kWave;
        float fv[NE];
        int32_t fi[NE];
#pragma unroll
        for (int q = 0; q < NE; ++q) {
            const int e = lane + q * kWave;
            if (C > kWave) {
                const bool has = (e & (kMaxDraftK - 1)) < keep;
                fv[q] = has ? s_wv[e] : -INFINITY;
                fi[q] = has ? s_wi[e] : kNone;
            } else {
                fv[q] = e < C ? s_score[e] : -INFINITY;
                fi[q] = e < C ? e : kNone;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup"); // the lists have been read
        wave_topk(fv, [&](int e) { return fi[e]; }, keep, list, [&](int r, float v, int32_t i) {
            s_wv[r] = v;
            s_wi[r] = i;
        });
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    const int32_t c = lane < keep ? s_wi[lane] : kNone;
    const float sc = lane < keep ? s_wv[lane] : 0.f;
    int pos = 0;
    for (int o = 0; o < keep; ++o) pos += __builtin_amdgcn_readlane(c, o) < c ? 1 : 0;
    if (c != kNone) {
        p.next_frontier_cand[(int64_t)b * keep + pos] = p.cand_base + c;
        p.next_cum[(int64_t)b * keep + pos] = sc;
    }
}

// grid = B, block = 256.
__global__ __launch_bounds__(kSelThreads) void draft_tree_build_kernel(const DraftBuildParams p) {
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
    hipLaunchKernelGGL(draft_expand_kernel, dim3((unsigned)((int64_t)p.chunks * p.B * p.F)), dim3(kExpandThreads), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_draft_tree_build(const DraftBuildParams& p, hipStream_t s) {
    hipLaunchKernelGGL(draft_tree_build_kernel, dim3(p.B), dim3(kSelThreads), 0, s, p);
    return hipGetLastError();
}

} // namespace vs
