// Tree-masked attention for few row blocks per KV head: splits of any length in rounds of 128 keys.
//
// Math and MFMA layouts are those of attention_mfma.hip (paper Eq. 1 with a softmax scale over
// the prefix plus the ancestor-or-self tree slots, Section 3.1): S^T = K . Q^T with
// v_mfma_f32_32x32x16_bf16, a lane holds 16 keys of ONE query row, the probabilities are the
// B operand of O^T += V^T . P^T, V is transposed by ds_read_b64_tr_b16 on its way out of LDS.
//
// A workgroup of eight waves owns NRB row blocks x KQ = 8 / NRB key parts of a split. A round is NT = 4 tiles of 32 keys
// in LDS; two sets of tiles make one barrier a round enough. The next two rounds are on their way in two sets of
// staging registers (one set, us: 8 x 31 nodes, 32 / 8 heads of 64, 257 .. 2047 keys 14.9, so 14.1; 4 x 60, 32 / 32 heads, 1500 keys 27.5 /
// 26.2; 2 x 1500 18.9 / 18.1; 60 nodes, 28 / 4 heads, 6684 keys 19.7 / 19.4). The first round's loads are issued
// before anything is waited for, ordered by stage (stage j holds the j-th tile of every key part), and a stage is worked on while the
// later ones are still on their way.
// Two waves per SIMD cover each other's stalls; at the end the key parts are merged through LDS (log-sum-exp).
// Splits that fit the resident kernel run there: its parts need no merge.
#include <type_traits>

#include "attn_mfma_common.h"

namespace vs {

namespace {

constexpr int kRndWaves = 8;

// CROWD: many splits on nearly all CUs, whose workgroups wait for each other at another word (merge_meet).
template <int D, int NRB, bool PAGED, bool CROWD>
__global__ __launch_bounds__(kRndWaves * 64, 2) void attn_mfma_rounds_kernel(const AttnParams p) {
    request_args(p);
    constexpr int NT = kRoundKeys / kTileKeys; // tiles of a round
    constexpr int KS = D / 16;          // k-steps of the S^T product
    constexpr int DB = D / 32;          // 32-channel blocks of the output
    constexpr int KQ = kRndWaves / NRB; // key parts inside the workgroup
    constexpr int PPM = (NT + KQ - 1) / KQ; // tiles per key part = stages
    constexpr int SUB = kTileKeys * D;  // elements per 32-key tile of K (or V)
    constexpr int LPR = D / 8;          // lanes (16-byte chunks) per row
    constexpr int RPI = 64 / LPR;       // rows per load instruction
    constexpr int RPB = kRndWaves * RPI;  // rows that one load of every wave fetches: one tile (128 channels) or two
    constexpr int NB = kRoundKeys / RPB;  // loads per wave and tensor in a round
    static_assert(RPB % kTileKeys == 0 && KQ * kTileKeys % RPB == 0, "loads lie in a stage");
    constexpr int TILE_BYTES = 2 * NT * SUB * 2;
    constexpr int MERGE_BYTES = kRndWaves * (DB * 1024 + 128) * 4; // every wave's exchange area: accumulators, max, sum
    constexpr int Q_BYTES = NRB * kRowBlock * D * 2;
    // the queries lie behind the tiles: where a second round's tiles go when they have been read (stages of round 0
    // end in barriers, so with two of them nobody can still be reading)
    constexpr int KEEP_BYTES = PPM >= 2 && Q_BYTES <= TILE_BYTES ? 2 * TILE_BYTES : 2 * TILE_BYTES + Q_BYTES;
    constexpr int Q_AT = PPM == 1 ? 2 * TILE_BYTES : TILE_BYTES;
    constexpr int SMEM_ELEMS = (KEEP_BYTES > MERGE_BYTES ? KEEP_BYTES : MERGE_BYTES) / 2;
    static_assert(SMEM_ELEMS * 2 + 512 <= kLdsBytesPerCU, "LDS");

    // tiles of a round: K[t] at smem + t*SUB, V[t] at smem + (NT + t)*SUB, odd rounds TILE_BYTES further; after the
    // last tile has been consumed the same memory carries the key parts' results to the merging waves
    __shared__ __attribute__((aligned(1024))) uint16_t smem[SMEM_ELEMS];
    __shared__ int32_t sp[VS_MAX_TREE];
    __shared__ int32_t sflag;
    uint16_t* sK = smem;
    uint16_t* sV = smem + NT * SUB;
    uint16_t* sQ = smem + Q_AT / 2; // queries: row blocks of D-channel rows (see load_q_pieces)

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5;
    const int col = lane & 31;
    const int rbw = wave % NRB; // row block inside the group
    const int kq = wave / NRB;  // key part

    const WorkItem at0 = work_item(p);
    if (at0.none) return;
    const int b = at0.b, kvh = at0.kvh, rg = at0.rg, split = at0.split;

    const int32_t S = p.prefix_len[b]; // requested first, needed last: everything below is issued before it arrives

    // ---- request the first round's keys and values. Load u of wave w fetches rows u * RPB + w * RPI .. + RPI - 1 of the round, 1 KB
    // of consecutive memory. The loads do not wait for the prefix length: they are bounded by the longest sequence that the
    // host allows, and values past the sequence's last key are zeroed on their way into LDS (whatever the
    // cache holds there - NaN included - must not meet a zero probability). A block-table entry outside the pool reads
    // block 0 (reported through status).
    const uint16_t* kbase = (const uint16_t*)p.k;
    const uint16_t* vbase = (const uint16_t*)p.v;
    const int64_t head_base = (PAGED ? 0 : (int64_t)b * p.stride_seq) + (int64_t)kvh * p.stride_head;
    const uint32_t stride = (uint32_t)p.stride_tok * 2u; // bytes; the host keeps a slice's offsets below 2^31 bytes
    const int lrow = lane / LPR, lchunk = lane % LPR;
    const int k0 = split * p.keys_per_split; // the host keeps k0 below max_prefix_len + tree_keys, hence inside the cache
    const int srow = wave * RPI + lrow;      // this lane's row of load 0
    u32x4 kreg[2][NB], vreg[2][NB];          // two rounds
    // Paged caches: the offsets of the next 64 blocks sit one per lane (see attention_mfma_pipe.hip).
    const int32_t* bt_row = PAGED ? p.block_table + (int64_t)b * p.max_blocks : nullptr;
    int bt_base = k0 >> p.block_shift;
    uint32_t bt_lo = 0, bt_hi = 0;
    int32_t bt_next = 0; // block id of lane 0 + 32 + lane, on its way
    auto bt_fetch = [&](int first) __attribute__((always_inline)) { return bt_row[min(first + lane, p.max_blocks - 1)]; };
    auto bt_set = [&](int32_t blk) __attribute__((always_inline)) {
        if ((uint32_t)blk >= (uint32_t)p.num_blocks) blk = 0; // reported through status
        const int64_t off = (int64_t)blk * p.stride_block;
        bt_lo = (uint32_t)off;
        bt_hi = (uint32_t)(off >> 32);
    };
    // byte offset of this lane's 16 bytes of the rows from r0 on, in one cache block; rows past `last` repeat it
    auto paged_at = [&](int r0, int last) __attribute__((always_inline)) {
        const int rel = (min(r0, last) >> p.block_shift) - bt_base; // 0 .. 63
        const int64_t block = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)bt_hi, rel) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)bt_lo, rel));
        return (head_base + block) * 2 + (uint32_t)(min(r0 + lrow, last) & (p.block_size - 1)) * stride + lchunk * 16;
    };
    if constexpr (PAGED) {
        const int32_t now = bt_fetch(bt_base);
        bt_next = bt_fetch(bt_base + 32);
        bt_set(now);
    }
    const uint32_t lane_off = (uint32_t)srow * stride + lchunk * 16; // contiguous caches
    const __amdgpu_buffer_rsrc_t krs0 = slice_of(kbase + head_base, k0, p, stride), vrs0 = slice_of(vbase + head_base, k0, p, stride);
    const int kend = early_end(most_keys(p), k0, p.keys_per_split);
    constexpr int LPS = KQ * kTileKeys / RPB; // loads per stage
    auto issue_stage = [&](auto is_v, int j) __attribute__((always_inline)) {
        constexpr bool ISV = decltype(is_v)::value;
#pragma unroll
        for (int u = j * LPS; u < (j + 1) * LPS; ++u) {
            u32x4& to = ISV ? vreg[0][u] : kreg[0][u];
            if constexpr (PAGED) to = *(const u32x4*)((const char*)(ISV ? vbase : kbase) + paged_at(k0 + u * RPB + wave * RPI, kend - 1));
            else to = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(ISV ? vrs0 : krs0, lane_off + (uint32_t)(u * RPB) * stride, 0, 0));
        }
    };
    issue_stage(std::false_type{}, 0); // the first keys lead: the first scores need them and the queries

    // ---- this wave's rows, mask and queries (in flight together with the tiles)
    const int row_base = rg * (NRB * kRowBlock) + rbw * kRowBlock;
    const bool wave_active = row_base < p.rows;
    const int r = min(row_base + col, p.rows - 1); // rows past the end repeat the last row (results discarded)
    const int node = row_node(p, r);
    // the waves of a row block share the fetch of its queries
    constexpr int QPW = (KS + KQ - 1) / KQ; // pieces per wave
    u32x4 qreg[QPW];
    load_q_pieces<D>(p, b, kvh, [&](int) { return row_base; }, [&](int i) { return min(kq * QPW + i, KS - 1); }, lane, qreg);
    // the gate of the row group (thread 0 opens it below)
    uint64_t* const gate = p.gates ? p.gates + kGateWords * (int64_t)((b * p.Hkv + kvh) * p.row_groups + rg) : nullptr;
    uint64_t seen = 0;
    if (p.gates && wave == 0) seen = gate_load(gate);
    // the row's ancestor mask, when the caller supplies the masks: requested ahead of the later stages
    uint64_t mask_given = 0;
    if (p.tree_mask && p.tree_keys != 0) mask_given = p.tree_mask[(int64_t)b * p.T + node];
    issue_stage(std::true_type{}, 0);
#pragma unroll
    for (int j = 1; j < PPM; ++j) {
        issue_stage(std::false_type{}, j);
        issue_stage(std::true_type{}, j);
    }

    int32_t tree_code = VS_STATUS_OK;
    if (p.tree_mask || p.tree_keys == 0) {
        if (tid == 0) sflag = 0;
        __syncthreads();
    } else {
        tree_code = load_tree(p.parent + (int64_t)b * p.T, p.T, sp, &sflag);
    }
    const uint64_t mask = p.tree_keys == 0 ? 0ull : (p.tree_mask ? mask_given : (tree_code == VS_STATUS_OK ? ancestor_mask(sp, node) : 0ull));
    const bool s_ok = prefix_ok(p, S);
    if (kvh == 0 && split == 0 && rg == 0) report_status(p, b, tree_code, s_ok, S, &sflag);
    if (tree_code != VS_STATUS_OK || !s_ok) return;

    const int nk = S + p.tree_keys;
    if (k0 >= nk) return;
    const bool final_rows = p.num_splits == 1 || (p.gates && nk <= p.keys_per_split); // a sequence of one split has nothing to merge
    const bool merge = p.gates && !final_rows;
    if (merge && tid == 0) merge_open(gate, seen);
    const int k1 = min(nk, k0 + p.keys_per_split);

    // ---- later rounds: the sequence's length is known. Rows past the split's last key read as zeros (paged caches: repeat it). Round 1
    // is requested whether it exists or not: behind a branch the compiler could not count these loads and would wait for them
    // with the first round's (8 x 31 nodes, 32 / 8 heads of 64, 257 .. 2047 keys: 13.9 us, so 14.8). For the rounds behind it what
    // such a request takes at the end of a split costs more than the wait (16 x 16 nodes, 28 / 4 heads, 1500 keys 19.2, always 21.0).
    const uint32_t live_bytes = (uint32_t)(k1 - k0 - 1) * stride + D * 2;
    const __amdgpu_buffer_rsrc_t krs = __builtin_amdgcn_make_buffer_rsrc((char*)const_cast<uint16_t*>(kbase + head_base) + (int64_t)k0 * stride, 0, (int)live_bytes, 0x00027000);
    const __amdgpu_buffer_rsrc_t vrs = __builtin_amdgcn_make_buffer_rsrc((char*)const_cast<uint16_t*>(vbase + head_base) + (int64_t)k0 * stride, 0, (int)live_bytes, 0x00027000);
    auto issue_round = [&](auto set_tag, int kr) __attribute__((always_inline)) {
        constexpr int SET = decltype(set_tag)::value;
        if constexpr (PAGED) {
            if ((min(kr, k1 - 1) >> p.block_shift) >= bt_base + 32) { // uniform
                bt_base += 32;
                bt_set(bt_next);
                bt_next = bt_fetch(bt_base + 32);
            }
            int64_t at[NB];
#pragma unroll
            for (int u = 0; u < NB; ++u) at[u] = paged_at(kr + u * RPB + wave * RPI, k1 - 1);
#pragma unroll
            for (int u = 0; u < NB; ++u) kreg[SET][u] = *(const u32x4*)((const char*)kbase + at[u]);
#pragma unroll
            for (int u = 0; u < NB; ++u) vreg[SET][u] = *(const u32x4*)((const char*)vbase + at[u]);
        } else {
            const uint32_t off = lane_off + (uint32_t)(kr - k0) * stride;
#pragma unroll
            for (int u = 0; u < NB; ++u) kreg[SET][u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(krs, off + (uint32_t)(u * RPB) * stride, 0, 0));
#pragma unroll
            for (int u = 0; u < NB; ++u) vreg[SET][u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(vrs, off + (uint32_t)(u * RPB) * stride, 0, 0));
        }
    };
    constexpr int ROUND = NT * kTileKeys;
    using Set0 = std::integral_constant<int, 0>;
    using Set1 = std::integral_constant<int, 1>;
    issue_round(Set1{}, k0 + ROUND);

    // per-lane LDS offsets (elements); everything else is a compile-time immediate
    const int k_lane[2] = {(col >> 4) * (DB * 512) + half * 128 + ((col & 15) ^ (4 * half)) * 8,
                           (col >> 4) * (DB * 512) + half * 128 + ((col & 15) ^ (8 + 4 * half)) * 8};
    const int t16 = lane & 15;
    const int v_lane = half * 128 + (t16 >> 2) * 32 + ((lane >> 4) & 1) * 16 + ((t16 >> 1) & 1) * 8 + (t16 & 1) * 4;
    // loads [u0, u1) of a staged round -> LDS. Chunk c of tile row r lands where the fragment reads expect it (same placement as
    // the streaming kernels):
    //   K: ((r/16)*DB + c/4) * 1024 + (c%4) * 256 + ((r%16) ^ 4*(c%4)) * 16
    //   V: ((r/16)*DB + c/4) * 1024 + (4*(r%16) + c%4) * 16
    const int rr = srow & (kTileKeys - 1); // (RPB is a multiple of a tile)
    const uint32_t in_tiles = (uint32_t)((srow / kTileKeys) * (SUB * 2) + ((rr >> 4) * DB + (lchunk >> 2)) * 1024);
    const uint32_t ko = in_tiles + (lchunk & 3) * 256 + (((rr & 15) ^ (4 * (lchunk & 3))) * 16), vo = in_tiles + (4 * (rr & 15) + (lchunk & 3)) * 16;
    auto stash = [&](auto set_tag, auto first_tag, int u0, int u1, int at) __attribute__((always_inline)) {
        constexpr int SET = decltype(set_tag)::value;
#pragma unroll
        for (int u = u0; u < u1; ++u) {
            *(u32x4*)((char*)(sK + at) + ko + u * (RPB / kTileKeys * SUB * 2)) = kreg[SET][u];
            u32x4 v = vreg[SET][u];
            if (decltype(first_tag)::value && k0 + u * RPB + srow >= k1) v = u32x4{0u, 0u, 0u, 0u};
            *(u32x4*)((char*)(sV + at) + vo + u * (RPB / kTileKeys * SUB * 2)) = v;
        }
    };

    // ---- this wave's key part: tiles j * KQ + kq of every round. The softmax comes once per round, over all of
    // the part's tiles of it (its independent halves hide each other's latency), and then the output.
    bf16x8 qf[KS];
    f32x16 s[PPM];
    // S^T = K . Q^T: lane (col, half) gets keys 8*(q/4) + 4*half + q%4 of row `col`
    auto scores = [&](int j, int at) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 16; ++q) s[j][q] = 0.f;
        const uint16_t* kt_ = sK + at + min(j * KQ + kq, NT - 1) * SUB;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const bf16x8 a = __builtin_bit_cast(bf16x8, *(const u32x4*)(kt_ + k_lane[ks & 1] + ks * 256));
            s[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[ks], s[j], 0, 0, 0);
        }
    };
    float m2 = -INFINITY, lsum = 0.f; // reference (log2 domain, scaled; -inf: no visible key yet), this lane's share of the sum
    f32x16 acc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[db][q] = 0.f;
    auto output = [&](auto first_tag, int kr, int at) __attribute__((always_inline)) {
        constexpr bool FIRST = decltype(first_tag)::value;
        // uniform: tree slots, the end of the range, or a last stage without a tile for this key part
        if (kr + NT * kTileKeys > min(S, k1) || (PPM - 1) * KQ + kq >= NT) {
#pragma unroll
            for (int j = 0; j < PPM; ++j) {
                const int first = kr + (j * KQ + kq) * kTileKeys;
                const uint32_t w = tile_visible(mask, first - S, j * KQ + kq < NT ? k1 - first : 0) >> (4 * half);
#pragma unroll
                for (int q = 0; q < 16; ++q) s[j][q] = visible_or_inf(s[j][q], w, 8 * (q >> 2) + (q & 3));
            }
        }
        float mx = -INFINITY;
#pragma unroll
        for (int j = 0; j < PPM; ++j)
#pragma unroll
            for (int q = 0; q < 16; q += 2) mx = max3(mx, s[j][q], s[j][q + 1]);
        const float mt = half_max(mx) * p.scale_log2;
        const float m_new = FIRST ? mt : (mt > m2 + kLazy ? mt : m2); // lazy: moves in steps of more than 2^8
        const float m_use = m_new == -INFINITY ? 0.f : m_new;
        float ps0 = 0.f, ps1 = 0.f;
#pragma unroll
        for (int j = 0; j < PPM; ++j)
#pragma unroll
            for (int q = 0; q < 16; q += 2) {
                s[j][q] = __builtin_amdgcn_exp2f(fmaf(s[j][q], p.scale_log2, -m_use)); // exp2(-inf) = 0
                s[j][q + 1] = __builtin_amdgcn_exp2f(fmaf(s[j][q + 1], p.scale_log2, -m_use));
                ps0 += s[j][q];
                ps1 += s[j][q + 1];
            }
        if constexpr (!FIRST) {
            const float alpha = __builtin_amdgcn_exp2f(m2 - m_use);
            lsum *= alpha;
            if (__any(alpha != 1.f)) {
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int q = 0; q < 16; ++q) acc[db][q] *= alpha;
            }
        }
        lsum += ps0 + ps1;
        m2 = m_new;
        // O^T += V^T . P^T: the A operand comes from two transposing reads of 4 keys x 16 channels
#pragma unroll
        for (int j = 0; j < PPM; ++j) {
            const uint16_t* vt_ = sV + at + min(j * KQ + kq, NT - 1) * SUB + v_lane;
            bf16x8 pf[2];
#pragma unroll
            for (int sl = 0; sl < 2; ++sl) {
                u32x4 w;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const f32x2 pr = {s[j][8 * sl + 2 * e], s[j][8 * sl + 2 * e + 1]};
                    w[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pr, bf16x2));
                }
                pf[sl] = __builtin_bit_cast(bf16x8, w);
            }
#pragma unroll
            for (int sl = 0; sl < 2; ++sl)
#pragma unroll
                for (int db = 0; db < DB; ++db) {
                    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vt_ + sl * (DB * 512) + db * 512));
                    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vt_ + sl * (DB * 512) + db * 512 + 256));
                    const bf16x8 a = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                    acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pf[sl], acc[db], 0, 0, 0);
                }
        }
    };

    // ---- round 0, stage by stage as the loads arrive (they return in order; the compiler counts them and waits
    // for exactly the stage's before their first use)
#pragma unroll
    for (int j = 0; j < PPM; ++j) {
        stash(Set0{}, std::true_type{}, j * LPS, (j + 1) * LPS, 0);
        if (j == 0) {
#pragma unroll
            for (int i = 0; i < QPW; ++i) store_q_piece<D>(sQ + rbw * (kRowBlock * D), qreg[i], min(kq * QPW + i, KS - 1), lane);
        }
        __syncthreads();
        if (j == 0) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) qf[ks] = read_q_frag<D>(sQ + rbw * (kRowBlock * D), ks, col, half);
        }
        scores(j, 0);
    }
    if (k0 + 2 * ROUND < k1) issue_round(Set0{}, k0 + 2 * ROUND);
    output(std::true_type{}, k0, 0);
    // ---- the other rounds: two sets of tiles in LDS, one barrier per round
    auto round = [&](auto set_tag, int kr) __attribute__((always_inline)) {
        constexpr int at = decltype(set_tag)::value * (TILE_BYTES / 2);
        stash(set_tag, std::false_type{}, 0, NB, at);
        __syncthreads();
        if (kr + 2 * ROUND < k1) issue_round(set_tag, kr + 2 * ROUND);
#pragma unroll
        for (int j = 0; j < PPM; ++j) scores(j, at);
        output(std::false_type{}, kr, at);
    };
    for (int kr = k0 + ROUND; kr < k1; kr += 2 * ROUND) {
        round(Set1{}, kr);
        if (kr + ROUND >= k1) break;
        round(Set0{}, kr + ROUND);
    }

    // ---- merge the key parts through LDS (log-sum-exp) and write the rows. The work is shared: a row
    // block's accumulators are 2 * DB pieces of eight registers (piece = channel block * 2 + half of
    // its registers, the 16-byte unit of the partial-result layout); key part k owns pieces
    // k * PPK .. (k + 1) * PPK - 1, receives the other parts' versions of those, merges them in ascending
    // part order (so every wave of a row block computes the same sum) and stores them. Every wave
    // hands (8 - PPK pieces, max, sum) over and takes as much back, instead of part 0 doing all of it.
    __syncthreads(); // every wave is done with the tiles
    float* sm = (float*)smem;
    constexpr int NP = 2 * DB;                    // pieces per row block
    constexpr int PPK = NP / KQ > 0 ? NP / KQ : 1; // pieces owned by a key part
    constexpr int OWNERS = NP / PPK;              // key parts that own pieces (all of them unless KQ > NP)
    constexpr int XCH = NP * 512 + 128;           // floats a wave's exchange area holds: pieces [piece][2][64 lanes][4], max[64], sum[64]
    static_assert(kRndWaves * XCH * 4 <= SMEM_ELEMS * 2, "exchange area fits");
    float* mine = sm + (rbw * KQ + kq) * XCH;
    auto piece_owner = [](int pc) { return pc / PPK; };
    if (wave_active) {
#pragma unroll
        for (int pc = 0; pc < NP; ++pc) {
            // written by everybody but the owner; which pieces those are depends on kq, the registers
            // they come from do not
            if (piece_owner(pc) != kq) {
                const int db = pc >> 1, hp = pc & 1;
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) {
                    const f32x4 w = {acc[db][8 * hp + 4 * hh], acc[db][8 * hp + 4 * hh + 1], acc[db][8 * hp + 4 * hh + 2],
                                     acc[db][8 * hp + 4 * hh + 3]};
                    *(f32x4*)(mine + pc * 512 + hh * 256 + lane * 4) = w;
                }
            }
        }
        mine[NP * 512 + lane] = m2;
        mine[NP * 512 + 64 + lane] = lsum;
    }
    __syncthreads();
    if (wave_active && kq < OWNERS) {

    // reference and sum over all key parts, the same arithmetic in every wave of the row block
    float mo[KQ], lo[KQ];
#pragma unroll
    for (int o = 0; o < KQ; ++o) {
        const float* src = sm + (rbw * KQ + o) * XCH;
        mo[o] = src[NP * 512 + lane];
        lo[o] = src[NP * 512 + 64 + lane];
    }
    float M = mo[0];
#pragma unroll
    for (int o = 1; o < KQ; ++o) M = fmaxf(M, mo[o]);
    const float Ms = (M == -INFINITY) ? 0.f : M; // no part has seen a visible key: every factor below is 2^-inf = 0
    float fo[KQ], lall = 0.f;
#pragma unroll
    for (int o = 0; o < KQ; ++o) {
        fo[o] = __builtin_amdgcn_exp2f(mo[o] - Ms);
        lall += lo[o] * fo[o];
    }
    const float l = half_sum(lall);
    const int r_local = row_base + col;
    const float inv = l > 0.f ? 1.f / l : 0.f; // no visible key in this split (partials only): zeros, weight 0
    uint16_t* orow = (uint16_t*)p.out + row_offset(p, b, kvh, r, node);
    uint16_t* po = p.part_o + part_block<D>(p, (int64_t)b * p.Hkv + kvh, split, row_base >> 5);

    // this wave's pieces: lane (col, half) holds, for row `col`, channels db*32 + 8*(q/4) + 4*half + q%4. All of
    // them are read and added up before the first store (one trip through LDS, not one per piece).
    auto finish = [&](auto kq_tag) __attribute__((always_inline)) {
        constexpr int MY = decltype(kq_tag)::value;
        float r[PPK][8];
#pragma unroll
        for (int i = 0; i < PPK; ++i) {
            const int pc = MY * PPK + i, db = pc >> 1, hp = pc & 1;
#pragma unroll
            for (int e = 0; e < 8; ++e) r[i][e] = 0.f;
#pragma unroll
            for (int o = 0; o < KQ; ++o) {
                if (o == MY) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) r[i][e] += fo[o] * acc[db][8 * hp + e];
                } else {
                    const float* src = sm + (rbw * KQ + o) * XCH + pc * 512 + lane * 4;
                    const f32x4 a0 = *(const f32x4*)src, a1 = *(const f32x4*)(src + 256);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        r[i][e] += fo[o] * a0[e];
                        r[i][4 + e] += fo[o] * a1[e];
                    }
                }
            }
        }
        if (final_rows) {
            if (r_local < p.rows) {
#pragma unroll
                for (int i = 0; i < PPK; ++i)
#pragma unroll
                    for (int hh = 0; hh < 2; ++hh)
                        *(u32x2*)(orow + (MY * PPK + i) * 16 + 8 * hh + 4 * half) =
                            pack_partial(r[i][4 * hh], r[i][4 * hh + 1], r[i][4 * hh + 2], r[i][4 * hh + 3], inv);
            }
        } else {
#pragma unroll
            for (int i = 0; i < PPK; ++i) {
                const u32x2 w0 = pack_partial(r[i][0], r[i][1], r[i][2], r[i][3], inv), w1 = pack_partial(r[i][4], r[i][5], r[i][6], r[i][7], inv);
                const u32x4 w = {w0[0], w0[1], w1[0], w1[1]};
                if (merge) store_piece<true>(p, po, MY * PPK + i, lane, w);
                else store_piece<false>(p, po, MY * PPK + i, lane, w);
            }
        }
    };
    switch (kq) { // uniform per wave; the case fixes which registers are this wave's
    case 0: finish(std::integral_constant<int, 0>{}); break;
    case 1: finish(std::integral_constant<int, 1 % OWNERS>{}); break;
    case 2: finish(std::integral_constant<int, 2 % OWNERS>{}); break;
    case 3: finish(std::integral_constant<int, 3 % OWNERS>{}); break;
    case 4: finish(std::integral_constant<int, 4 % OWNERS>{}); break;
    case 5: finish(std::integral_constant<int, 5 % OWNERS>{}); break;
    case 6: finish(std::integral_constant<int, 6 % OWNERS>{}); break;
    default: finish(std::integral_constant<int, 7 % OWNERS>{}); break;
    }
    if (!final_rows && kq == 0 && half == 0) {
        const f32x2 ml = {M, l};
        const int64_t mlb = ml_block(p, (int64_t)b * p.Hkv + kvh, split, row_base >> 5);
        float* dst = p.part_ml + mlb * 2;
        if (merge) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, ml), span_of(dst), col * 8, 0, kDeviceScope);
        else *(f32x2*)(dst + col * 2) = ml;
    }
    }
    if (merge) {
        const int nrb = p.rows_pad / kRowBlock, rb0 = rg * NRB;
        merge_splits<D, CROWD>(p, gate, b, kvh, rb0, min(rb0 + NRB, nrb), split, (nk + p.keys_per_split - 1) / p.keys_per_split, kRndWaves,
                        (uint32_t*)sp);
    }
}

template <int D, int NRB>
hipError_t launch_rnd(const AttnParams& p, hipStream_t s) {
    const dim3 grid(((p.total_wgs + 7) / 8) * 8);
    const dim3 block(kRndWaves * kWave);
    if (p.paged && p.crowd) hipLaunchKernelGGL((attn_mfma_rounds_kernel<D, NRB, true, true>), grid, block, 0, s, p);
    else if (p.paged) hipLaunchKernelGGL((attn_mfma_rounds_kernel<D, NRB, true, false>), grid, block, 0, s, p);
    else if (p.crowd) hipLaunchKernelGGL((attn_mfma_rounds_kernel<D, NRB, false, true>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((attn_mfma_rounds_kernel<D, NRB, false, false>), grid, block, 0, s, p);
    return hipGetLastError();
}

} // namespace

// Four or two row blocks per workgroup.
hipError_t launch_attention_mfma_rounds(const AttnParams& p, int row_blocks, hipStream_t s) {
    if (p.keys_per_split <= resident_max_keys(row_blocks)) return launch_attention_mfma_resident(p, row_blocks, s);
    if ((row_blocks != 4 && row_blocks != 2) || p.keys_per_split % kIterKeys) return hipErrorInvalidValue;
    if (p.d == 128) return row_blocks == 4 ? launch_rnd<128, 4>(p, s) : launch_rnd<128, 2>(p, s);
    if (p.d == 64) return row_blocks == 4 ? launch_rnd<64, 4>(p, s) : launch_rnd<64, 2>(p, s);
    return hipErrorInvalidValue;
}

} // namespace vs
