// Stochastic acceptance over a draft tree (paper Section 3.1: accept a draft token with
// probability min(1, p / p_hat), otherwise continue with norm(max(0, p - p_hat)) and, when
// no candidate is left, draw the next token from it). The tree's candidates come from a
// deterministic top-k expansion, so the proposal for a candidate is a point mass: child c
// with token x is accepted iff u_accept[c] < r(x), r being the target softmax at the
// current node with the tokens rejected so far removed and the rest renormalised.
//
// Two kernels: (1) a bandwidth-bound scan that reduces every chunk of a logits row to (maximum, sum of exp); (2) one
// workgroup per sequence that walks the tree on those pairs alone - removing a token subtracts its weight from its
// chunk - and draws the bonus token by inverting the residual's cumulative sum in index order: chunk sums first,
// then one scan inside the chunk that holds the target. The second kernel touches the logits only for the
// candidates' own entries, for that one chunk, and for a chunk whose sum a removal cancelled (re-summed
// without the removed tokens).
#include "logits_scan.h"

namespace vs {

namespace {

constexpr int kScanWaves = kScanThreads / kWave;
constexpr int kRowThreads = kScanThreads / VS_MAX_TREE; // threads of the walk that share a row's chunks
static_assert(kRowThreads == 8, "three steps of a butterfly");
// Pairs of a sequence that the walk keeps in LDS (17 KB): 64 rows of up to 262144 logits, and everything of up to 4096 pairs
// of half as many logits (T * ceil(V / 4096) <= 4096 means T * ceil(V / 8192) <= 2048 + T / 2).
// Beyond, the walk reads them again from memory, which costs little where nothing has to be removed from a chunk (2 x 60 x 262144, us,
// 1536 / 2080 kept: 29.1 / 29.1; 1 x 64 x 256000 20.35 / 20.28; smaller calls the same).
constexpr int kKeepStats = 2048 + VS_MAX_TREE / 2;
constexpr int kPerThread = 16;            // chunk elements per thread of the walk
static_assert(kScanThreads * kPerThread == kScanChunk && kScanChunk == 1 << 13, "the walk takes one chunk at a time, half of its threads a short one");

// grid = B*T*chunks, block = THREADS: (max of the raw logits, sum of 2^((l - max) * k)) of a chunk, k = log2(e) / temperature.
template <int THREADS>
__global__ __launch_bounds__(THREADS, 8) void softmax_stats_partial_kernel(const SampleParams p) {
    constexpr int kWaves = THREADS / kWave;
    __shared__ float sred[2][kWaves];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const ScanItem it = scan_item(p.by_chunks);
    const ScanChunk c = scan_load<THREADS>(p.logits + (int64_t)it.row * p.ld, it.chunk, p.V);
    float m = c.tail;
#pragma unroll
    for (int j = 0; j < kScanVec; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) m = fmaxf(m, c.a[j][e]);
    m = wave_max(m);
    float s = 0.f; // relative to the wave's maximum: one barrier for both
    if (m > -INFINITY) {
#pragma unroll
        for (int j = 0; j < kScanVec; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) s += __builtin_amdgcn_exp2f((c.a[j][e] - m) * p.k_log2); // exp2(-inf) = 0
        s += __builtin_amdgcn_exp2f((c.tail - m) * p.k_log2);
    }
    s = wave_sum(s);
    if (lane == 0) {
        sred[0][wave] = m;
        sred[1][wave] = s;
    }
    __syncthreads();
    if (wave == 0) {
        const float wm = lane < kWaves ? sred[0][lane] : -INFINITY;
        m = wave_max(wm);
        s = wave_sum(wm > -INFINITY ? sred[1][lane & (kWaves - 1)] * __builtin_amdgcn_exp2f((wm - m) * p.k_log2) : 0.f);
        if (lane == 0) p.pairs[(int64_t)it.row * p.chunks + it.chunk] = ((uint64_t)__float_as_uint(s) << 32) | __float_as_uint(m);
    }
}

// grid = B, block = 512. Every wave runs the (short, sequential) walk on the same registers, so its branches are uniform and
// the whole workgroup can turn to a chunk-wide pass when one is needed. Everything the walk compares is fetched up front
// (row maxima and masses, the uniforms, every candidate's weight in its parent's row), so a step of the walk costs no
// memory round trip: removing a rejected token just lowers the row's mass. Only when that subtraction would cancel (the
// rejected token held > 95 % of the mass), and once at the end for the bonus draw, the row's per-chunk masses are
// needed - from the copy of all rows' chunk statistics in LDS when those fit, else from memory. A chunk is 2^SHIFT logits.
template <int SHIFT>
__global__ __launch_bounds__(kScanThreads) void accept_sample_walk_kernel(const SampleParams p) {
    __shared__ float sred[kScanWaves];
    __shared__ float sM[VS_MAX_TREE];      // row maxima
    __shared__ float sZ[VS_MAX_TREE];      // row masses relative to the maxima
    __shared__ float slogit[VS_MAX_TREE];  // logit of node c's token in its parent's row
    __shared__ float su[VS_MAX_TREE];
    __shared__ int32_t sparent[VS_MAX_TREE], stoken[VS_MAX_TREE];
    __shared__ float sch[kMaxSampleChunks]; // residual weight per chunk of the current row
    __shared__ uint64_t skeep[kKeepStats];  // every row's chunk statistics, when they fit
    __shared__ int32_t spick[kScanWaves], slast[kScanWaves];
    const int b = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T = p.T;
    // the tree and its draws, a lane per node, asked for ahead of the statistics (by all waves, and the parents used behind those: at the end of
    // a branch or where they are compared the compiler waits for them, before the statistics are asked for)
    const int64_t at = (int64_t)b * T + min(lane, T - 1);
    int32_t own_parent = p.parent[at];
    const int32_t own_token = p.draft[at];
    const float own_u = p.u_accept[at], u_bonus = p.u_bonus[b];
    const int ri = tid / kRowThreads, sub = tid % kRowThreads;
    const uint64_t* pairs = p.pairs + (int64_t)b * T * p.chunks;
    constexpr int kPre = 4;
    uint64_t w[kPre];
    auto fetch = [&](int c0) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < kPre; ++q) w[q] = pairs[min(ri, T - 1) * p.chunks + min(c0 + kRowThreads * q, p.chunks - 1)];
    };
    fetch(sub);
    asm volatile("" : "+v"(own_parent)::"memory"); // used from here on
    if (wave == 0) {
        own_parent = lane < T ? own_parent : -2;
        // the candidates' logits (parent index clamped: a malformed tree is reported below and must not steer a load out of bounds)
        const bool has = lane >= 1 && lane < T && own_token >= 0 && own_token < p.V;
        float l = -INFINITY;
        if (has) l = p.logits[((int64_t)b * T + min(max(own_parent, 0), T - 1)) * p.ld + own_token];
        sparent[lane] = own_parent;
        stoken[lane] = has ? own_token : -1; // no candidate: weight 0, nothing to remove
        su[lane] = own_u;
        slogit[lane] = l;
    }

    // ---- row maxima and masses, merged online. When all rows' chunk statistics fit they also stay in LDS, so that the
    // per-chunk masses a rejection or the bonus draw needs later cost no second trip to memory.
    const bool keep = T * (int64_t)p.chunks <= kKeepStats;
    {
        float m = -INFINITY, z = 0.f;
        for (int c0 = sub; c0 < p.chunks; c0 += kRowThreads * kPre) {
            if (c0 != sub) fetch(c0);
            float pm[kPre], bm = m;
#pragma unroll
            for (int q = 0; q < kPre; ++q) {
                const int c = c0 + kRowThreads * q;
                const bool ok = ri < T && c < p.chunks;
                if (ok && keep) skeep[ri * p.chunks + c] = w[q];
                pm[q] = ok ? __uint_as_float((uint32_t)w[q]) : -INFINITY;
                bm = fmaxf(bm, pm[q]);
            }
            if (bm > -INFINITY) {
                z *= __builtin_amdgcn_exp2f((m - bm) * p.k_log2); // m = -inf: z is 0 and stays 0
#pragma unroll
                for (int q = 0; q < kPre; ++q)
                    if (pm[q] > -INFINITY) z += __uint_as_float((uint32_t)(w[q] >> 32)) * __builtin_amdgcn_exp2f((pm[q] - bm) * p.k_log2);
                m = bm;
            }
        }
        auto from = [](float x, auto step) __attribute__((always_inline)) { return __uint_as_float(step(__float_as_uint(x))); };
        auto x1 = [](uint32_t x) __attribute__((always_inline)) { return dpp<kDppXor1>(x); };
        auto x2 = [](uint32_t x) __attribute__((always_inline)) { return dpp<kDppXor2>(x); };
        auto x4 = [](uint32_t x) __attribute__((always_inline)) { return dpp<kDppXor7>(dpp<kDppXor3>(x)); };
        float mm = fmaxf(m, from(m, x1));
        mm = fmaxf(mm, from(mm, x2));
        mm = fmaxf(mm, from(mm, x4));
        if (m > -INFINITY) z *= __builtin_amdgcn_exp2f((m - mm) * p.k_log2);
        z += from(z, x1);
        z += from(z, x2);
        z += from(z, x4);
        if (ri < T && sub == 0) {
            sM[ri] = mm;
            sZ[ri] = z;
        }
    }
    __syncthreads();
    const int32_t parent = sparent[lane], token = stoken[lane];
    const int32_t tree_code = tree_check(parent, T);
    if (tree_code != VS_STATUS_OK) { // uniform
        if (wave != 0) return;
        if (lane < T) p.path[(int64_t)b * T + lane] = -1;
        if (lane == 0) {
            if (p.status) p.status[b] = tree_code;
            p.accepted_len[b] = 0;
            p.bonus[b] = -1;
        }
        return;
    }
    // every candidate's weight in its parent's row
    const float Mp = sM[max(parent, 0)], u_acc = su[lane];
    const float ex_own = (token >= 0 && Mp > -INFINITY) ? __builtin_amdgcn_exp2f((slogit[lane] - Mp) * p.k_log2) : 0.f;
    const float Z_own = sZ[min(lane, T - 1)];
    auto lane_of = [](float x, int c) __attribute__((always_inline)) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int32_t, x), c)); };

    // This thread's first element of chunk c; behind the row where the chunk has none for it
    auto place = [&](int c) __attribute__((always_inline)) { return kScanChunk == 1 << SHIFT || tid * kPerThread < 1 << SHIFT ? c * (1 << SHIFT) + tid * kPerThread : p.V; };
    // This thread's 16 consecutive weights of chunk c of row `node`; the tokens of the nodes in `removed` weigh nothing.
    auto load_weights = [&](int node, int c, uint64_t removed, float (&w)[kPerThread]) {
        const float* lg = p.logits + ((int64_t)b * T + node) * p.ld;
        const float M = sM[node];
        const int j0 = place(c);
        if (p.V >= 4) {
            // four at a time, the row's last four at its end: there the wanted ones are moved to the front
            f32x4 a[kPerThread / 4];
#pragma unroll
            for (int q = 0; q < kPerThread / 4; ++q) a[q] = *(const f32x4_any*)(lg + min(j0 + 4 * q, p.V - 4));
            if (__any(j0 + kPerThread > p.V)) {
#pragma unroll
                for (int q = 0; q < kPerThread / 4; ++q) {
                    const int by = j0 + 4 * q - (p.V - 4); // so many of the four lie before the wanted ones
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        float x = by <= 0 ? a[q][e] : -INFINITY;
#pragma unroll
                        for (int d = 1; d < 4 - e; ++d) x = by == d ? a[q][e + d] : x;
                        a[q][e] = x;
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < kPerThread / 4; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) w[4 * q + e] = __builtin_amdgcn_exp2f((a[q][e] - M) * p.k_log2); // exp2(-inf) = 0
        } else {
#pragma unroll
            for (int e = 0; e < kPerThread; ++e)
                w[e] = (j0 + e < p.V) ? __builtin_amdgcn_exp2f((lg[j0 + e] - M) * p.k_log2) : 0.f;
        }
        for (; removed != 0; removed &= removed - 1) {
            const int off = __builtin_amdgcn_readlane(token, __builtin_ctzll(removed)) - j0;
            if ((unsigned)off < (unsigned)kPerThread) {
#pragma unroll
                for (int e = 0; e < kPerThread; ++e)
                    if (e == off) w[e] = 0.f;
            }
        }
    };
    // Mass of chunk c of row `node`, nothing removed.
    auto chunk_mass = [&](int node, int c) -> float {
        const uint64_t ms = keep ? skeep[node * p.chunks + c] : pairs[(int64_t)node * p.chunks + c];
        const float mc = __uint_as_float((uint32_t)ms);
        return (mc > -INFINITY) ? __uint_as_float((uint32_t)(ms >> 32)) * __builtin_amdgcn_exp2f((mc - sM[node]) * p.k_log2) : 0.f;
    };
    // Sum of sch[0..chunks), the same value in every wave.
    auto chunk_total = [&]() -> float {
        float s = 0.f;
        for (int c = lane; c < p.chunks; c += kWave) s += sch[c];
        return wave_sum(s);
    };
    // Takes node c's token out of its chunk's mass in sch; `removed`: the nodes whose tokens are gone by then, c among them.
    auto remove_from_chunks = [&](int node, int c, uint64_t removed) {
        const int xc = __builtin_amdgcn_readlane(token, c) / (1 << SHIFT);
        const float old = sch[xc];
        float fresh = old - lane_of(ex_own, c);
        if (!(fresh >= 0.25f * old)) {
            // the subtraction cancelled most of the chunk: sum it again without the removed tokens
            float w[kPerThread];
            load_weights(node, xc, removed, w);
            float s = 0.f;
#pragma unroll
            for (int e = 0; e < kPerThread; ++e) s += w[e];
            s = wave_sum(s);
            __syncthreads();
            if (lane == 0) sred[wave] = s;
            __syncthreads();
            fresh = 0.f;
#pragma unroll
            for (int q = 0; q < kScanWaves; ++q) fresh += sred[q];
        }
        __syncthreads(); // every thread has read the old value
        if (tid == 0) sch[xc] = fresh;
        __syncthreads();
    };
    // Per-chunk masses of row `node` in sch with the tokens of `removed` taken out in order; returns their sum.
    auto materialize = [&](int node, uint64_t removed) -> float {
        __syncthreads(); // sch may still be read
        for (int c = tid; c < p.chunks; c += kScanThreads) sch[c] = chunk_mass(node, c);
        __syncthreads();
        uint64_t gone = 0;
        for (uint64_t r = removed; r != 0; r &= r - 1) {
            gone |= r & -r;
            remove_from_chunks(node, __builtin_ctzll(r), gone);
        }
        return chunk_total();
    };

    // ---- the walk: a lane per node. The children of the current node are considered in order, and all that come before
    // the first accepted one are rejected: so the mass that each of them sees is the row's less a prefix sum over its
    // earlier siblings, and the first that its uniform accepts is a ballot.
    int cur = 0, alen = 0;
    uint64_t removed = 0; // the rejected children of the current node whose tokens are out of its mass
    float Z = 0.f;
    bool have_chunks = false; // sch holds the current node's masses
    for (;;) {
        Z = lane_of(Z_own, cur);
        have_chunks = false;
        const bool kid = parent == cur;
        const uint64_t kids = __ballot(kid);
        if (kids == 0) {
            removed = 0;
            break;
        }
        bool live = kid && token >= 0; // a token that an earlier sibling has is gone already
        for (uint64_t k = kids & (kids - 1); k != 0; k &= k - 1) {
            const int c = __builtin_ctzll(k);
            if (__ballot(kid && lane < c && token == __builtin_amdgcn_readlane(token, c)) && lane == c) live = false;
        }
        const float ex = live ? ex_own : 0.f;
        const float before = Z - (wave_scan(ex) - ex);
        const float prob = before > 0.f ? ex / before : 0.f;
        const uint64_t accepted = __ballot(kid && u_acc < prob);
        const int first = accepted ? __builtin_ctzll(accepted) : kWave;
        const uint64_t rejected = __ballot(live) & (accepted ? (1ull << first) - 1 : ~0ull);
        int next = accepted ? first : -1;
        if (rejected & __ballot(!(before - ex >= 0.05f * before))) {
            // a rejected token holds almost all of what was left: one child after the other, the masses by chunk from there on
            next = -1;
            removed = 0;
            for (uint64_t k = kids; k != 0 && next < 0; k &= k - 1) {
                const int c = __builtin_ctzll(k);
                const float e = lane_of(ex, c), pr = (Z > 0.f) ? e / Z : 0.f;
                if (lane_of(u_acc, c) < pr) {
                    next = c;
                } else if ((__ballot(live) >> c) & 1) {
                    removed |= 1ull << c;
                    if (have_chunks) {
                        remove_from_chunks(cur, c, removed);
                        Z = chunk_total();
                    } else if (Z - e >= 0.05f * Z) {
                        Z -= e;
                    } else {
                        Z = materialize(cur, removed);
                        have_chunks = true;
                    }
                }
            }
        } else {
            removed = rejected;
        }
        if (next < 0) break;
        cur = next;
        ++alen;
    }

    // ---- bonus token: inverse of the residual's cumulative sum, index order. First the chunk; every wave finds it for itself,
    // up to 64 chunks in registers unless a removal cancels one of them.
    int kb = -1, last_pos = -1;
    float target = 0.f, before = 0.f;
    auto find_chunk = [&](float cs, int c0, float carry) __attribute__((always_inline)) { // returns the carry behind these chunks
        const float inc = carry + wave_scan(cs);
        const uint64_t pos = __ballot(cs > 0.f), over = __ballot(cs > 0.f && inc > target);
        if (pos) last_pos = c0 + 63 - __builtin_clzll(pos);
        if (over) {
            const int l = __builtin_ctzll(over);
            kb = c0 + l;
            before = l == 0 ? carry : lane_of(inc, l - 1);
        }
        return lane_of(inc, 63);
    };
    bool in_lanes = p.chunks <= kWave && !have_chunks;
    if (in_lanes) {
        float cs = lane < p.chunks ? chunk_mass(cur, lane) : 0.f;
        bool cancelled = false;
        for (uint64_t r = removed; r != 0; r &= r - 1) {
            const int c = __builtin_ctzll(r);
            if (lane == __builtin_amdgcn_readlane(token, c) / (1 << SHIFT)) {
                const float fresh = cs - lane_of(ex_own, c);
                cancelled = cancelled || !(fresh >= 0.25f * cs);
                cs = fresh;
            }
        }
        in_lanes = !__any(cancelled);
        if (in_lanes) {
            target = u_bonus * wave_sum(cs);
            find_chunk(cs, 0, 0.f);
        }
    }
    if (!in_lanes) {
        if (!have_chunks) Z = materialize(cur, removed);
        target = u_bonus * Z;
        float carry = 0.f;
        for (int c0 = 0; c0 < p.chunks && kb < 0; c0 += kWave) carry = find_chunk(c0 + lane < p.chunks ? sch[c0 + lane] : 0.f, c0, carry);
    }
    if (kb < 0) { // u * total rounded up to the whole mass: last token with weight
        kb = last_pos;
        before = -INFINITY;
    }
    int32_t pick = -1;
    if (kb >= 0) {
        float w[kPerThread];
        load_weights(cur, kb, removed, w);
        float s = 0.f;
        int last = -1;
        const int j0 = place(kb);
#pragma unroll
        for (int e = 0; e < kPerThread; ++e) {
            s += w[e];
            if (w[e] > 0.f) last = j0 + e;
        }
        // inclusive scan of the threads' sums: inside the wave, then across the waves
        float inc = wave_scan(s);
        __syncthreads(); // sred is free
        if (lane == 63) sred[wave] = inc;
        __syncthreads();
#pragma unroll
        for (int wv = 0; wv < kScanWaves; ++wv)
            if (wv < wave) inc += sred[wv];
        const float local = target - before; // +inf when the whole mass is below the target
        int cand = INT32_MAX;
        if (inc > local && last >= 0) {
            // first element of this thread whose running sum passes the target; the scan's and
            // the running sum's roundings may disagree by an ulp, then the last weighted one
            float acc = inc - s;
            cand = -1;
#pragma unroll
            for (int e = 0; e < kPerThread; ++e) {
                acc += w[e];
                if (cand < 0 && acc > local && w[e] > 0.f) cand = j0 + e;
            }
            if (cand < 0) cand = last;
        }
        const int wcand = wave_min(cand), wlast = wave_max(last);
        if (lane == 0) {
            spick[wave] = wcand;
            slast[wave] = wlast;
        }
        __syncthreads();
        if (wave == 0) {
            pick = wave_min(lane < kScanWaves ? spick[lane] : INT32_MAX);
            if (pick == INT32_MAX) pick = wave_max(lane < kScanWaves ? slast[lane] : -1); // -1: no token carries weight (inputs must be finite)
        }
    }
    // ---- results
    if (wave != 0) return;
    const int32_t path = tree_path(parent, cur, alen);
    if (lane < T) p.path[(int64_t)b * T + lane] = path;
    if (lane == 0) {
        if (p.status) p.status[b] = VS_STATUS_OK;
        p.accepted_len[b] = alen;
        p.bonus[b] = pick;
    }
}

} // namespace

// workspace: 8 bytes per (row, chunk); sized by chunks half as long, it holds them with room to spare
hipError_t launch_accept_sample(SampleParams p, void* workspace, hipStream_t s) {
    const bool short_chunks = scan_short_chunks(p.V, (int64_t)p.B * p.T);
    const int chunk = short_chunks ? kScanChunk / 2 : kScanChunk;
    p.chunks = (int32_t)(((int64_t)p.V + chunk - 1) / chunk);
    p.by_chunks = fast_div_by(p.chunks);
    p.pairs = (uint64_t*)workspace;
    const dim3 grid((unsigned)((int64_t)p.chunks * p.B * p.T));
    if (short_chunks) hipLaunchKernelGGL(softmax_stats_partial_kernel<kScanThreads / 2>, grid, dim3(kScanThreads / 2), 0, s, p);
    else hipLaunchKernelGGL(softmax_stats_partial_kernel<kScanThreads>, grid, dim3(kScanThreads), 0, s, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (short_chunks && p.chunks > 1) hipLaunchKernelGGL(accept_sample_walk_kernel<12>, dim3(p.B), dim3(kScanThreads), 0, s, p);
    else hipLaunchKernelGGL(accept_sample_walk_kernel<13>, dim3(p.B), dim3(kScanThreads), 0, s, p);
    return hipGetLastError();
}

} // namespace vs
