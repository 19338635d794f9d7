// Tree-masked attention for launches of few query rows per KV head (one or two row blocks): every wave has key tiles of
// its own.
//
// Math and MFMA layouts are those of attention_mfma.hip (paper Eq. 1 with a softmax scale over the prefix plus the
// ancestor-or-self tree slots, Section 3.1): S^T = K . Q^T with v_mfma_f32_32x32x16_bf16, a lane holds 16 keys of ONE
// query row, the probabilities are the B operand of O^T += V^T . P^T, V is transposed by ds_read_b64_tr_b16 on its way
// out of LDS.
//
// What bounds it: with 32 or 64 rows a 16 KB tile of K and V keeps a SIMD busy for a tenth to a quarter of the time
// in which it comes from memory, so the bytes in flight decide (a CU's share of 6 TB/s times 1.5 us of latency is 35 KB).
// The kernels that share tiles among their waves pay a barrier per tile and leave waves without rows idle. Here the
// waves of a workgroup take the 32-key tiles of a split in turn, each for all rows: a tile goes from memory straight into
// LDS of the wave's own, keys and values by turns (64 to 128 KB in flight per CU), with no barrier anywhere in the
// loop. Through registers the same took 5 % longer at the start of a launch and left no room for a second row
// block. The waves' results are merged through LDS (log-sum-exp), the splits as in merge_splits.
// us per call, before / this kernel (28 / 4 or 32 / 32 heads of 128 channels unless stated):
//   1 x 4 nodes, 484 keys 14.2 / 7.6; 16 x 4 nodes, 1024 .. 8191 keys paged 62.6 / 35.2; 64 x 4 nodes, 8000 keys 304 / 180
//   (5.8 TB/s); 4 x 4 nodes, 32 KV heads, 3100 keys 47.4 / 41.1; 16 x 20 nodes, 16 / 16 heads of 64, up to 3000 keys 46.4 / 31.4;
//   two row blocks: 64 x 9 nodes, 1024 .. 8191 keys 178 / 129; 8 x 60 nodes, 32 / 32 heads, up to 8000 keys 164 / 132.
// (Three and four row blocks, one wave per SIMD with 512 registers, lost: 16 x 13 nodes, up to 8191 keys 57 / 79.)
#include <type_traits>

#include "attn_mfma_common.h"

namespace vs {

namespace {

// NW waves, RB row blocks. (PAGED is part of the kernel for the scalar registers: with a branch 14 of them were spilled, in the loop over the
// tiles too: 4 x 60 nodes, 32 / 32 heads, 3100 keys 39.7 -> 39.2 us, one sequence of 484 keys and four nodes 7.4 -> 7.2.)
// ONCE: tiles as data that is read once (the host's rule says when). Part of the kernel as well: a branch at every load 5 % of two row blocks'
// time, a loop of its own for either kind 3 % of a short call's.
// CROWD: many splits on nearly all CUs, whose workgroups wait for each other at another word (merge_meet).
template <int D, int NW, int RB, bool PAGED, bool ONCE, bool CROWD = false>
__global__ __launch_bounds__(NW * 64, 2) void attn_mfma_rows_kernel(const AttnParams p) {
    constexpr int KS = D / 16;          // k-steps of the S^T product
    constexpr int DB = D / 32;          // 32-channel blocks of the output
    constexpr int SUB = kTileKeys * D;  // elements per 32-key tile of K (or V)
    constexpr int BPS = SUB * 2 / 1024; // loads (1 KB) per tile
    constexpr int LPR = D / 8;          // lanes (16-byte chunks) per row
    constexpr int RPI = 64 / LPR;       // rows per load
    constexpr int ROUND = NW * kTileKeys;
    constexpr bool QREG = RB == 1;      // the queries stay in registers
    constexpr int TILE_ELEMS = NW * 2 * SUB;
    constexpr int NP = 2 * DB;                                 // pieces of a row block's accumulators, see below
    constexpr int KEEP_ELEMS = TILE_ELEMS + RB * kRowBlock * D; // tiles, queries
    constexpr int SMEM_ELEMS = KEEP_ELEMS + NW * 256;          // ... a reference and a sum per lane
    static_assert(NP * 512 * 4 <= 2 * SUB * 2, "a row block's accumulators take the wave's tiles' place");
    static_assert(SMEM_ELEMS * 2 + 512 <= kLdsBytesPerCU, "LDS");

    // wave w: its K tile at smem + w * 2 * SUB, its V tile behind it, and behind all tiles the queries
    __shared__ __attribute__((aligned(1024))) uint16_t smem[SMEM_ELEMS];
    __shared__ int32_t sp[VS_MAX_TREE];
    __shared__ int32_t sflag;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5;
    const int col = lane & 31;
    uint16_t* sK = smem + wave * 2 * SUB;
    uint16_t* sV = sK + SUB;
    uint16_t* sQ = smem + TILE_ELEMS;

    // workgroup id -> (sequence, KV head, split), splits fastest; same XCD-aware remap as the other kernels. More whole
    // sequences than run at once: the longest first, dealt over the XCDs (see attention_mfma_pipe.hip).
    int b, kvh, split = 0, rg = 0; // (longest first: one row group)
    if (p.by_length) { // one split each
        if (blockIdx.x >= (uint32_t)p.total_wgs) return;
        uint32_t head;
        b = sequence_by_rank(p, (int)fast_div(blockIdx.x, p.by_heads, head), lane);
        kvh = (int)head;
    } else {
        const WorkItem at = work_item(p);
        if (at.none) return;
        b = at.b;
        kvh = at.kvh;
        split = at.split;
        rg = at.rg;
    }
    const int block0 = rg * RB, row0 = block0 * kRowBlock; // first row block and row of the workgroup
    const int unit = b * p.Hkv + kvh;

    const int32_t S = p.prefix_len[b]; // requested first, needed last: the first tiles are requested before it arrives

    // ---- this wave's tiles: keys first, first + ROUND, ... The first one is clamped to the longest allowed sequence instead
    // of this one; rows that turn out to lie past the sequence's last key become zeros on their way into LDS (whatever the
    // cache holds there, NaN included, must not meet a zero probability). Later ones repeat the last key.
    const int k0 = split * p.keys_per_split; // the host keeps k0 below max_prefix_len + tree_keys, hence inside the cache
    const int first = k0 + wave * kTileKeys;
    const int kend = early_end(most_keys(p), k0, p.keys_per_split);
    const uint16_t* kbase = (const uint16_t*)p.k;
    const uint16_t* vbase = (const uint16_t*)p.v;
    const int64_t head_base = (PAGED ? 0 : (int64_t)b * p.stride_seq) + (int64_t)kvh * p.stride_head;
    const int stride_tok = (int)p.stride_tok; // host guarantees 32-bit lane offsets
    const int lrow = lane / LPR, lchunk = lane % LPR;
    // Paged caches: a tile is two half tiles of 16 keys, each in one cache block. Lane 2 * i + h holds the id of half
    // h of the wave's tile i, from tile `bt_from` on: one load for 32 tiles.
    int bt_from = first;
    int32_t bt_win = 0;
    auto bt_fetch = [&]() __attribute__((always_inline)) {
        const int lb = (bt_from + (lane >> 1) * ROUND + (lane & 1) * 16) >> p.block_shift;
        const int32_t blk = p.block_table[(int64_t)b * p.max_blocks + min(lb, p.max_blocks - 1)];
        bt_win = (uint32_t)blk < (uint32_t)p.num_blocks ? blk : 0; // a bad entry is reported through status
    };
    if (PAGED) bt_fetch();
    // Tiles lie in LDS as whole rows, chunk c (16 bytes) of row r at position c ^ kx(r) (keys) or c ^ vx(r) (values) of
    // its row: a load's lanes fetch the chunks of a row in that order. kx(r) = r % (chunks per row): the rows' chunks that
    // an operand read takes lie in different banks. vx(r): the transposing reads take 4 rows x 2 (4) chunks per 16
    // (32) lanes, which then lie in different banks too.
    auto vx = [](int r) __attribute__((always_inline)) { return D == 128 ? 4 * (r & 3) ^ 2 * ((r ^ (r >> 1)) & 1) : 2 * (r & 3); };
    // This lane's bytes from a load's first row on, per load: the keys' chunk depends on the row (KV of them differ).
    constexpr int KV = LPR / RPI > 0 ? LPR / RPI : 1;
    const uint32_t stride = (uint32_t)stride_tok * 2u;
    uint32_t k_off[KV], v_off = (uint32_t)lrow * stride + (uint32_t)(lchunk ^ vx(lrow)) * 16u;
#pragma unroll
    for (int j = 0; j < KV; ++j) k_off[j] = (uint32_t)lrow * stride + (uint32_t)(lchunk ^ ((RPI * j + lrow) % LPR)) * 16u;
    // tile at key kt into LDS, keys past `last` repeat it; kt <= last
    auto issue = [&](auto is_v, uint16_t* to, int kt, int last) __attribute__((always_inline)) {
        constexpr bool ISV = decltype(is_v)::value;
        const uint16_t* g = (ISV ? vbase : kbase) + head_base;
        const uint16_t* base[2] = {g, g};
        int row0[2] = {kt, kt + kTileKeys / 2}; // of the tile's halves
        if (PAGED) {
            const int at = (kt - bt_from) / ROUND * 2;
            base[0] += (int64_t)__builtin_amdgcn_readlane(bt_win, at) * p.stride_block;
            base[1] += (int64_t)__builtin_amdgcn_readlane(bt_win, at + (kt + 16 <= last)) * p.stride_block;
            row0[0] &= p.block_size - 1;
            row0[1] &= p.block_size - 1;
        }
        const uint32_t lds = (uint32_t)(uintptr_t)(lds_void*)to;
        if (kt + kTileKeys - 1 <= last) { // uniform: every row is there, so a load's address is uniform but for the lane's bytes
#pragma unroll
            for (int i = 0; i < BPS; ++i) {
                const int h = 2 * i / BPS;
                const char* from = (const char*)base[h] + (uint32_t)(row0[h] + RPI * (i % (BPS / 2))) * stride;
                load_to_lds<ONCE>(lds + 1024 * i, from, ISV ? v_off : k_off[i % KV]);
            }
        } else {
#pragma unroll
            for (int i = 0; i < BPS; ++i) {
                int tok = min(kt + RPI * i + lrow, last);
                if (PAGED) tok &= p.block_size - 1;
                load_to_lds(lds + 1024 * i, base[2 * i / BPS], (uint32_t)(tok - lrow) * stride + (ISV ? v_off : k_off[i % KV]));
            }
        }
    };
    // ---- queries (every wave fetches its share of the pieces), rows, masks: requested ahead of
    // the tiles (loads return in order, and whoever waits for the queries would wait for a tile in front of them)
    constexpr int PIECES = RB * KS, QPW = (PIECES + NW - 1) / NW;
    u32x4 qreg[QPW];
    load_q_pieces<D>(p, b, kvh, [&](int i) { return row0 + min(wave + NW * i, PIECES - 1) / KS * kRowBlock; },
                     [&](int i) { return min(wave + NW * i, PIECES - 1) % KS; }, lane, qreg);
    int node[RB];
    uint64_t mask[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        node[rb] = row_node(p, min(row0 + rb * kRowBlock + col, p.rows - 1)); // rows past the end repeat the last row
        mask[rb] = p.tree_mask && p.tree_keys != 0 ? p.tree_mask[(int64_t)b * p.T + node[rb]] : 0ull;
    }
    // the gate of the (sequence, KV head), opened below
    uint64_t* const gate = p.gates ? p.gates + kGateWords * ((int64_t)unit * p.row_groups + rg) : nullptr;
    uint64_t seen = 0;
    if (p.gates && wave == 0) seen = gate_load(gate);
    if (first < kend) { // uniform per wave
        issue(std::false_type{}, sK, first, kend - 1);
        issue(std::true_type{}, sV, first, kend - 1);
    }

    int32_t tree_code = VS_STATUS_OK;
    if (p.tree_mask || p.tree_keys == 0) {
        if (tid == 0) sflag = 0;
        __syncthreads();
    } else {
        tree_code = load_tree(p.parent + (int64_t)b * p.T, p.T, sp, &sflag);
        if (tree_code == VS_STATUS_OK) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) mask[rb] = ancestor_mask(sp, node[rb]);
        }
    }
    const bool s_ok = prefix_ok(p, S);
    if (kvh == 0 && split == 0 && rg == 0) report_status<PAGED>(p, b, tree_code, s_ok, S, &sflag);
    if (tree_code != VS_STATUS_OK || !s_ok) return;
    const int nk = S + p.tree_keys;
    if (k0 >= nk) return;
    const bool final_rows = p.num_splits == 1 || (p.gates && nk <= p.keys_per_split); // a sequence of one split has nothing to merge
    const bool merge = p.gates && !final_rows;
    if (merge && tid == 0) [[unlikely]] merge_open(gate, seen); // (most waves only jump over it)
    const int k1 = min(nk, k0 + p.keys_per_split);

#pragma unroll
    for (int i = 0; i < QPW; ++i) {
        const int pc = min(wave + NW * i, PIECES - 1);
        store_q_piece<D>(sQ + pc / KS * (kRowBlock * D), qreg[i], pc % KS, lane);
    }
    __syncthreads();

    // operand reads: row `col`, chunk 2 * ks + half of the keys; four keys x 16 channels of the values per lane group
    const int k_lane = col * D, k_x = half ^ (col % LPR);
    const int v_row = 4 * half + ((lane & 15) >> 2);
    int v_lane[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
        v_lane[db] = v_row * D + ((4 * db + 2 * ((lane >> 4) & 1) + ((lane >> 1) & 1)) ^ vx(v_row)) * 8 + (lane & 1) * 4;
    float m2[RB], lsum[RB]; // reference (log2 domain, scaled; -inf: no visible key yet), this lane's share of the sum
    f32x16 acc[RB][DB];
    bf16x8 qf[QREG ? RB : 1][KS];
    if constexpr (QREG) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) qf[rb][ks] = read_q_frag<D>(sQ + rb * (kRowBlock * D), ks, col, half);
    }
    // FIRST: the wave's first tile
    auto tile = [&](auto first_tag, int kt) __attribute__((always_inline)) {
        constexpr bool FIRST = decltype(first_tag)::value;
        const int next = kt + ROUND;
        wait_loads<BPS>(); // outstanding: K(kt), V(kt)
        const bool plain = kt + kTileKeys <= min(S, k1); // prefix keys only
        bf16x8 pf[RB][2];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            // S^T = K . Q^T: lane (col, half) gets keys 8*(q/4) + 4*half + q%4 of row `col`
            f32x16 s;
#pragma unroll
            for (int q = 0; q < 16; ++q) s[q] = 0.f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const bf16x8 a = __builtin_bit_cast(bf16x8, *(const u32x4*)(sK + k_lane + ((2 * ks) ^ k_x) * 8));
                s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, QREG ? qf[rb][ks] : read_q_frag<D>(sQ + rb * (kRowBlock * D), ks, col, half), s, 0, 0, 0);
            }
            if (rb == RB - 1 && next < k1) {
                if (PAGED && next - bt_from >= 32 * ROUND) { // uniform
                    bt_from = next;
                    bt_fetch();
                }
                wait_lds_reads();
                issue(std::false_type{}, sK, next, k1 - 1);
            }
            if (!plain) { // uniform: tree slots or the end of the range
                const uint32_t w = tile_visible(mask[rb], kt - S, k1 - kt) >> (4 * half);
#pragma unroll
                for (int q = 0; q < 16; ++q) s[q] = visible_or_inf(s[q], w, 8 * (q >> 2) + (q & 3));
            }
            float mx = -INFINITY;
#pragma unroll
            for (int q = 0; q < 16; q += 2) mx = max3(mx, s[q], s[q + 1]);
            const float mt = half_max(mx) * p.scale_log2;
            const float m_new = FIRST ? mt : (mt > m2[rb] + kLazy ? mt : m2[rb]); // lazy: moves in steps of more than 2^8
            const float m_use = m_new == -INFINITY ? 0.f : m_new;
            float ps0 = 0.f, ps1 = 0.f;
#pragma unroll
            for (int q = 0; q < 16; q += 2) {
                s[q] = __builtin_amdgcn_exp2f(fmaf(s[q], p.scale_log2, -m_use)); // exp2(-inf) = 0
                s[q + 1] = __builtin_amdgcn_exp2f(fmaf(s[q + 1], p.scale_log2, -m_use));
                ps0 += s[q];
                ps1 += s[q + 1];
            }
            if constexpr (!FIRST) {
                const float alpha = __builtin_amdgcn_exp2f(m2[rb] - m_use);
                lsum[rb] *= alpha;
                if (__any(alpha != 1.f)) {
#pragma unroll
                    for (int db = 0; db < DB; ++db)
#pragma unroll
                        for (int q = 0; q < 16; ++q) acc[rb][db][q] *= alpha;
                }
            }
            lsum[rb] = FIRST ? ps0 + ps1 : lsum[rb] + (ps0 + ps1);
            m2[rb] = m_new;
#pragma unroll
            for (int sl = 0; sl < 2; ++sl) {
                u32x4 w;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const f32x2 pr = {s[8 * sl + 2 * e], s[8 * sl + 2 * e + 1]};
                    w[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pr, bf16x2));
                }
                pf[rb][sl] = __builtin_bit_cast(bf16x8, w);
            }
        }
        if (next < k1) wait_loads<BPS>(); // outstanding: V(kt), K(next)
        else wait_loads<0>();
        if (FIRST && kt + kTileKeys > k1) {
#pragma unroll
            for (int i = 0; i < BPS; ++i)
                if (kt + RPI * i + lrow >= k1) *(u32x4*)(sV + 512 * i + lane * 8) = u32x4{0u, 0u, 0u, 0u};
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); // other lanes of this wave read them
        }
        // O^T += V^T . P^T: the A operand comes from two transposing reads of 4 keys x 16 channels
#pragma unroll
        for (int sl = 0; sl < 2; ++sl)
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(sV + v_lane[db] + sl * (16 * D)));
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(sV + v_lane[db] + sl * (16 * D) + 8 * D));
                const bf16x8 a = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
                    acc[rb][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pf[rb][sl], FIRST && sl == 0 ? f32x16{} : acc[rb][db], 0, 0, 0);
            }
        if (next < k1) {
            wait_lds_reads();
            issue(std::true_type{}, sV, next, k1 - 1);
        }
    };
    if (first < k1) {
        tile(std::true_type{}, first);
        for (int kt = first + ROUND; kt < k1; kt += ROUND) tile(std::false_type{}, kt);
    } else {
        // A wave without a tile adds nothing. Written here and from a register that the compiler knows nothing about: constants it wrote in front
        // of the branch, where every wave with a tile waited for 64 of them (128 for two row blocks). Those and the code that rarely runs,
        // in the way to the first tile, took 0.1 - 0.2 us of the shortest calls: us per call with both / without, 28 / 4 heads, 2 x 3 nodes, 201
        // keys 6.06 / 5.89; 7 x 3, 378 keys 6.47 / 6.36; 1 x 4, 484 keys 7.28 / 7.12; 40 x 2, 32 / 32 heads, 250 keys 26.5 / 26.3.
        float zero = 0.f;
        asm volatile("" : "+v"(zero));
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            m2[rb] = -INFINITY;
            lsum[rb] = 0.f;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int q = 0; q < 16; ++q) acc[rb][db][q] = zero;
        }
    }
    wait_loads<0>(); // (a wave without a live tile may have requested one)

    // ---- merge the waves' results through LDS (log-sum-exp) and write the rows. The accumulators are NP pieces of eight
    // registers (piece = channel block * 2 + half of its registers, the 16-byte unit of the partial-result layout):
    // wave w owns pieces w * PPW .., takes the other waves' versions of them and merges in ascending order.
    constexpr int PPW = NP / NW > 0 ? NP / NW : 1;
    // A wave hands its first row block over in the place of its own tiles, as soon as it is done with them: the last one then
    // writes alone, and one barrier less (us: 3 x 2 nodes, 8 / 2 heads, 330 keys 6.9, so 6.5; 18 x 1, 28 / 4 heads, 1600 keys 16.5 / 16.1; 4 x 60,
    // 32 / 32 heads, ~3100 keys 47.9 / 47.5).
    auto area = [&](int w) __attribute__((always_inline)) { return (float*)(smem + w * 2 * SUB); };
    float* const ml = (float*)(smem + KEEP_ELEMS); // [wave][reference, sum][lane]
    float* const mine = area(wave);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        if (rb > 0) __syncthreads(); // every wave is done with the row block before
#pragma unroll
        for (int pc = 0; pc < NP; ++pc) {
            const int db = pc >> 1, hp = pc & 1;
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                const f32x4 w = {acc[rb][db][8 * hp + 4 * hh], acc[rb][db][8 * hp + 4 * hh + 1], acc[rb][db][8 * hp + 4 * hh + 2], acc[rb][db][8 * hp + 4 * hh + 3]};
                *(f32x4*)(mine + pc * 512 + hh * 256 + lane * 4) = w;
            }
        }
        ml[wave * 128 + lane] = m2[rb];
        ml[wave * 128 + 64 + lane] = lsum[rb];
        __syncthreads();
        if (wave * PPW < NP) {
            float mo[NW], lo[NW];
#pragma unroll
            for (int o = 0; o < NW; ++o) {
                mo[o] = ml[o * 128 + lane];
                lo[o] = ml[o * 128 + 64 + lane];
            }
            float M = mo[0];
#pragma unroll
            for (int o = 1; o < NW; ++o) M = fmaxf(M, mo[o]);
            const float Ms = (M == -INFINITY) ? 0.f : M; // no wave has seen a visible key: every factor below is 2^-inf = 0
            float lall = 0.f, r[PPW][8];
#pragma unroll
            for (int i = 0; i < PPW; ++i)
#pragma unroll
                for (int e = 0; e < 8; ++e) r[i][e] = 0.f;
#pragma unroll
            for (int o = 0; o < NW; ++o) {
                const float f = __builtin_amdgcn_exp2f(mo[o] - Ms);
                lall += lo[o] * f;
#pragma unroll
                for (int i = 0; i < PPW; ++i) {
                    const float* src = area(o) + (wave * PPW + i) * 512 + lane * 4;
                    const f32x4 a0 = *(const f32x4*)src, a1 = *(const f32x4*)(src + 256);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        r[i][e] += f * a0[e];
                        r[i][4 + e] += f * a1[e];
                    }
                }
            }
            const float l = half_sum(lall);
            const float inv = l > 0.f ? 1.f / l : 0.f; // no visible key in this split (partials only): zeros, weight 0
#pragma unroll
            for (int i = 0; i < PPW; ++i) {
                const int pc = wave * PPW + i;
                const u32x2 w0 = pack_partial(r[i][0], r[i][1], r[i][2], r[i][3], inv), w1 = pack_partial(r[i][4], r[i][5], r[i][6], r[i][7], inv);
                // lane (col, half) holds, for row `col`, channels pc * 16 + 8 * {0, 1} + 4 * half + 0..3
                if (final_rows) {
                    if (row0 + rb * kRowBlock + col < p.rows) {
                        uint16_t* o = (uint16_t*)p.out + row_offset(p, b, kvh, row0 + rb * kRowBlock + col, node[rb]) + pc * 16 + 4 * half;
                        *(u32x2*)o = w0;
                        *(u32x2*)(o + 8) = w1;
                    }
                } else {
                    const u32x4 w = {w0[0], w0[1], w1[0], w1[1]};
                    uint16_t* to = p.part_o + part_block<D>(p, unit, split, block0 + rb);
                    if (merge) store_piece<true>(p, to, pc, lane, w);
                    else store_piece<false>(p, to, pc, lane, w);
                }
            }
            if (!final_rows && wave == 0 && half == 0) {
                const f32x2 ml = {M, l};
                float* to = p.part_ml + ml_block(p, unit, split, block0 + rb) * 2;
                if (merge) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, ml), span_of(to), col * 8, 0, kDeviceScope);
                else *(f32x2*)(to + col * 2) = ml;
            }
        }
    }
    if (merge) merge_splits<D, CROWD>(p, gate, b, kvh, block0, block0 + RB, split, (nk + p.keys_per_split - 1) / p.keys_per_split, NW, (uint32_t*)sp);
}

template <int D, int NW, int RB>
hipError_t launch_rows(const AttnParams& p, hipStream_t s) {
    const dim3 grid(((p.total_wgs + 7) / 8) * 8);
    if (p.once && p.paged) return hipErrorInvalidValue;
    if constexpr (NW == 8 && RB == 1)
        if (p.crowd) {
            if (p.paged) hipLaunchKernelGGL((attn_mfma_rows_kernel<D, NW, RB, true, false, true>), grid, dim3(NW * kWave), 0, s, p);
            else hipLaunchKernelGGL((attn_mfma_rows_kernel<D, NW, RB, false, false, true>), grid, dim3(NW * kWave), 0, s, p);
            return hipGetLastError();
        }
    if (p.once) hipLaunchKernelGGL((attn_mfma_rows_kernel<D, NW, RB, false, true>), grid, dim3(NW * kWave), 0, s, p);
    else if (p.paged) hipLaunchKernelGGL((attn_mfma_rows_kernel<D, NW, RB, true, false>), grid, dim3(NW * kWave), 0, s, p);
    else hipLaunchKernelGGL((attn_mfma_rows_kernel<D, NW, RB, false, false>), grid, dim3(NW * kWave), 0, s, p);
    return hipGetLastError();
}

} // namespace

// One row block and four or eight waves; with 128 channels also two row blocks and eight waves.
bool attention_rows_supported(int d, int row_blocks, int waves) {
    return (row_blocks == 1 && (waves == 4 || waves == 8)) || (d == 128 && row_blocks == 2 && waves == 8);
}

hipError_t launch_attention_mfma_rows(const AttnParams& p, int waves, hipStream_t s) {
    const int blocks = p.rows_per_group / kRowBlock;
    if (p.row_groups * p.rows_per_group != p.rows_pad || (p.by_length && p.row_groups != 1)) return hipErrorInvalidValue;
    if (p.keys_per_split % kIterKeys || !attention_rows_supported(p.d, blocks, waves)) return hipErrorInvalidValue;
    if (p.d == 128) return blocks == 2 ? launch_rows<128, 8, 2>(p, s) : waves == 8 ? launch_rows<128, 8, 1>(p, s) : launch_rows<128, 4, 1>(p, s);
    if (p.d == 64) return waves == 8 ? launch_rows<64, 8, 1>(p, s) : launch_rows<64, 4, 1>(p, s);
    return hipErrorInvalidValue;
}

} // namespace vs
