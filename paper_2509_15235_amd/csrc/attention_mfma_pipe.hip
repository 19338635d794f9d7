// Tree-masked attention on the matrix cores, software-pipelined across key tiles.
//
// Same math, work decomposition, LDS chunk placement and partial-result layout as the
// kernel in attention_mfma.hip (paper Eq. 1 restricted by tree ancestry, Section 3.1).
// The difference is the schedule. Per 32-key tile t a wave has three pieces of work:
//   S(t)  = K(t) . Q^T            8 MFMAs per row block
//   P(t)  = online softmax of S(t) on the vector ALU (exp2, running max and sum, bf16)
//   O    += V(t)^T . P(t)^T       8 MFMAs per row block
// S -> P -> O of one tile depend on each other, so a straight loop leaves the matrix
// core idle during P and the vector ALU idle during S and O. Here the step for tile t
// issues S(t+1) and O(t-1) together with P(t): the sixteen MFMAs have no operand in
// common with the softmax of the same step and the hardware runs them side by side.
// One loop iteration covers two tiles (so the roles of the two score / probability
// register sets are fixed at compile time) and ends in the only barrier. Inside a step
// the instruction stream is written slot by slot - one MFMA, the LDS read of a fragment
// two slots ahead, one sixteenth of the softmax - and K and V^T fragments alternate so
// that consecutive MFMAs never share an accumulator.
//
// K/V tiles travel global -> registers -> LDS, 1 KB of consecutive memory per load
// instruction. Copies are grouped per iteration (two K tiles, two V tiles); a group is
// requested two iterations before the one that writes it to LDS in its middle, so two
// groups are in flight in two register sets. K tiles reach LDS three to four tiles ahead
// of their S step, V tiles one to two ahead of their O step, in two four-slot rings
// (tile t lives in slot t % 4).
//
// Measured on MI355X with N(0,1) inputs the loop sustains about 0.6 PFLOP/s; a loop of
// nothing but these MFMAs on random operands reaches 1.76 PFLOP/s on this machine (2.27
// on constant operands: the clock is power-managed), so the remaining gap is barrier skew,
// copy issue and the two general iterations at either end of the key range.
#include <type_traits>

#include "attn_mfma_common.h"

namespace vs {

namespace {

// WPS: waves of a SIMD that have registers at the same time. Three workgroups of four waves and 64 channels on a CU
// instead of two where that makes one round of a launch that is one and a half: us per call in two / three, 16 / 16 heads,
// 33 x 43 nodes (528 workgroups), 450 keys 27.4 / 21.2, 1500 paged 71.1 / 55.1; 46 x 60 (736), 200 .. 450 paged 33.1 / 25.6; outside
// those 256 workgroups two have the faster loop (below): 20 x 60 (320), 1500 paged 42.1 / 47.2, 50 x 60 (800), 450 34.9 / 38.5.
template <int D, int RPW, int NW, bool PAGED, bool BAL, int WPS = 2>
__global__ __launch_bounds__(NW * 64, WPS) void attn_mfma_pipe_kernel(const AttnParams p) {
    constexpr int KS = D / 16;                 // k-steps of the S^T product
    constexpr int DB = D / 32;                 // 32-channel blocks of the output
    constexpr int SUB = kTileKeys * D;         // elements per 32-key tile of K (or V)
    constexpr int BPS = SUB * 2 / 1024;        // 1 KB blocks (16 keys x 32 channels) per tile
    constexpr int BPW = (BPS + NW - 1) / NW;   // ... copied by each wave
    constexpr int NSLOT = 4;
    // Eight waves of 64 channels are twice as many as a tile has blocks: the lower half copies K, the upper half V, one block
    // of every tile each. (With all copies on the lower half, behind a branch per copy, the compiler cannot count the
    // loads in flight and waits for all of them in front of every LDS write, the one just requested included: us per call,
    // so / now, 60 nodes, 32 / 8 heads, 18 x 1000 keys 38.1 / 28.2, 48 x 250 .. 2000 101 / 77, 24 x 1000 .. 8000 paged 155 / 112.)
    constexpr bool HALVES = NW == 2 * BPS;
    static_assert(HALVES || NW * BPW == BPS, "the waves' blocks make up a tile");

    __shared__ __attribute__((aligned(1024))) uint16_t sK[NSLOT][SUB];
    __shared__ __attribute__((aligned(1024))) uint16_t sV[NSLOT][SUB];
    __shared__ int32_t sp[VS_MAX_TREE];
    __shared__ int32_t sflag;
    __shared__ uint64_t sgen;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // Final rows of row block rb out of the accumulators' lanes (quad(e): this lane's channels 8 * e + 4 * half .. + 3 of its row), half of the
    // channels at a time through this wave's eighth (quarter) of the K ring, which nobody reads behind the last tile:
    // a store of 16 bytes a lane then touches 8 lines of 128 bytes, not 32 lines in 8-byte pieces, sixteen times over.
    auto store_rows = [&](int b, int kvh, int rb, auto quad) __attribute__((always_inline)) {
        int t = threadIdx.x;
        asm volatile("" : "+v"(t));
        const int lane = t & 63, half = lane >> 5, col = lane & 31;
        constexpr int CH = D / 16, RPS = 64 / CH, NST = kRowBlock / RPS; // 16-byte chunks of a row, rows per store, stores
        char* const mine = (char*)&sK[0][0] + wave * (kRowBlock * D);
        uint16_t* o[NST];
#pragma unroll
        for (int i = 0; i < NST; ++i) {
            const int r = rb * kRowBlock + i * RPS + lane / CH;
            o[i] = r < p.rows ? (uint16_t*)p.out + row_offset(p, b, kvh, r, row_node(p, r)) + (lane % CH) * 8 : nullptr;
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int e = 0; e < CH; ++e) *(u32x2*)(mine + col * D + ((e ^ (col & (CH - 1))) * 16) + half * 8) = quad(h * CH + e);
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup"); // read by other lanes of this wave
#pragma unroll
            for (int i = 0; i < NST; ++i) {
                const int r = i * RPS + lane / CH;
                const u32x4 w = *(const u32x4*)(mine + r * D + (((lane % CH) ^ (r & (CH - 1))) * 16));
                if (o[i]) *(u32x4*)(o[i] + h * (D / 2)) = w;
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup"); // the reads are done before it is written again
        }
    };

    // One piece of work: the rows of row group `rg` of (sequence b, KV head kvh) against the keys
    // [k0, k0 + klen) of that sequence (k0 lies inside the cache). `whole`: no other piece shares these
    // rows, they leave as final output; else as the partial result of slot `slot`.
    auto run_piece = [&](const int b, const int kvh, const int rg, const int k0, const int klen, const int slot,
                         bool whole) __attribute__((always_inline)) {
    int tid = threadIdx.x;
    // What depends on the lane alone is worked out for every piece: kept from one piece to the next it takes registers that the loop
    // needs. Four waves of 128 channels had 41 of them in scratch memory, and the wait for a spilled value in the
    // loop waits for all tile copies in flight: 20 x 60 nodes, 32 / 32 heads, 250 .. 2000 keys 131 us, so 117
    // (8 of 1024 .. 8191 keys 159 / 147, paged 163 / 154; eight waves: no spills either, 1 %).
    if (BAL) asm volatile("" : "+v"(tid));
    const int lane = tid & 63, half = lane >> 5, col = lane & 31;
    const int32_t S = p.prefix_len[b]; // requested first, needed last: the first tiles and the queries are requested before it arrives

    // ---- tile copies. One load instruction of a wave fetches 1 KB of consecutive memory:
    // RPI whole rows (tokens) of D channels, lane q -> row q / LPR, 16-byte chunk q % LPR, so
    // every touched cache line is used completely. The 16-byte chunks are then scattered into
    // LDS so that the fragment reads are conflict-free; chunk c of tile row r lives at byte
    //   K: ((r/16)*DB + c/4) * 1024 + (c%4) * 256 + ((r%16) ^ 4*(c%4)) * 16
    //   V: ((r/16)*DB + c/4) * 1024 + (4*(r%16) + c%4) * 16
    // (the XOR spreads the chunks of one K row over the banks: 4-way instead of 16-way write
    // conflicts; reads of 16 rows at one chunk stay a permutation of 16 consecutive slots).
    // Tokens past the last valid one re-read that token (finite values that get zero weight).
    constexpr int LPR = D / 8;        // lanes (16-byte chunks) per row
    constexpr int RPI = 64 / LPR;     // rows per load instruction
    static_assert(BPS * RPI == kTileKeys, "a tile is BPS blocks of RPI rows");
    const uint16_t* kbase = (const uint16_t*)p.k;
    const uint16_t* vbase = (const uint16_t*)p.v;
    const int64_t head_base = (PAGED ? 0 : (int64_t)b * p.stride_seq) + (int64_t)kvh * p.stride_head;
    const int stride_tok = (int)p.stride_tok; // host guarantees 32-bit lane offsets
    const int lrow = lane / LPR, lchunk = lane % LPR;
    const uint32_t lane_off = (uint32_t)(lrow * stride_tok + lchunk * 8) * 2u; // bytes
    const int block0 = HALVES ? wave % BPS : wave * BPW; // this wave's first block of a tile
    const bool upper = HALVES && wave >= BPS;
    uint32_t k_st[BPW], v_st[BPW]; // this lane's LDS byte offsets inside a tile slot, per block
#pragma unroll
    for (int j = 0; j < BPW; ++j) {
        const int r = (block0 + j) * RPI + lrow, c = lchunk;
        k_st[j] = (uint32_t)(((r >> 4) * DB + (c >> 2)) * 1024 + (c & 3) * 256 + (((r & 15) ^ (4 * (c & 3))) * 16));
        v_st[j] = (uint32_t)(((r >> 4) * DB + (c >> 2)) * 1024 + (4 * (r & 15) + (c & 3)) * 16);
    }
    // Paged caches: where the blocks of the tiles to come lie sits one per lane - a window of 64 consecutive table
    // entries, fetched with one coalesced load and moved along by 32 as the tiles advance - so a tile copy gets
    // it with v_readlane instead of a scalar load per copy (whose result the copy would have to wait for, together with
    // every LDS read in flight: scalar loads and LDS share one wait counter). The clamp and the product are done once
    // per window, by all lanes at once, and the loaded register is only touched where the window moves: with ids in
    // a window of 128 read twice per lookup 28 x 60 nodes of 28 / 4 heads over 1696 keys took 62.1 us, so 59.3 (54.8 unpaged).
    const int32_t* bt_row = PAGED ? p.block_table + (int64_t)b * p.max_blocks : nullptr;
    int bt_base = k0 >> p.block_shift; // logical block of lane 0
    uint32_t bt_lo = 0, bt_hi = 0;     // element offset of the lane's block
    int32_t bt_next = 0;               // block id of lane 0 + 32 + lane, on its way
    auto bt_fetch = [&](int first) __attribute__((always_inline)) { return bt_row[min(first + lane, p.max_blocks - 1)]; };
    auto bt_set = [&](int32_t blk) __attribute__((always_inline)) {
        if ((uint32_t)blk >= (uint32_t)p.num_blocks) blk = 0; // reported through status
        const int64_t off = (int64_t)blk * p.stride_block;
        bt_lo = (uint32_t)off;
        bt_hi = (uint32_t)(off >> 32);
    };
    int32_t bt_first = 0;
    if (PAGED) { // (with the prefix length: one trip)
        bt_first = bt_fetch(bt_base);
        bt_next = bt_fetch(bt_base + 32);
    }
    auto bt_lookup = [&](int lb) __attribute__((always_inline)) {
        const int rel = lb - bt_base; // 0 .. 63 by construction
        return (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)bt_hi, rel) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)bt_lo, rel));
    };
    u32x4 stage[2][4][BPW];
    // ---- this wave's rows and queries (in flight together with the first tiles)
    const int row_base = rg * p.rows_per_group + wave * (RPW * kRowBlock);
    const bool wave_active = row_base < p.rows;
    bf16x8 qf[RPW][KS];
    int node_of[RPW];
#pragma unroll
    for (int rb = 0; rb < RPW; ++rb) {
        // rows past the end repeat the last row (finite data, results discarded)
        const int r = min(row_base + rb * kRowBlock + col, p.rows - 1);
        node_of[rb] = row_node(p, r);
    }
    static_assert(RPW == 1 && NW <= 2 * NSLOT, "a row block's queries take a tile slot");
    // through the tile slot of this wave's number (nothing is in the rings yet)
    uint16_t* sq = wave < NSLOT ? sK[wave & (NSLOT - 1)] : sV[wave & (NSLOT - 1)];
    auto copy_queries = [&]() __attribute__((always_inline)) {
        if (!wave_active) return;
#pragma unroll
        for (int i = 0; i < KS; ++i) copy_q_piece<D>(p, b, kvh, row_base, sq, i, lane);
    };
    if (PAGED) { // the queries while the block ids are on their way
        copy_queries();
        bt_set(bt_first);
    }
    constexpr bool EARLY = !(BAL && PAGED && NW == 4); // registers: 4 waves of 128 channels 188 us, so 171 (8 x 60 nodes, 32 / 32 heads, 1024 .. 8191 keys)
    // The first four tiles - K(0), K(1), K(2), V(0), through register set 1 - are requested before
    // the prefix length is known: clamped to the longest allowed sequence instead of this one, and rows that
    // turn out to lie past the sequence's last key are zeroed when the tiles go into LDS
    // (whatever the cache holds there, NaN included, must not meet a zero probability).
    if constexpr (EARLY) {
        const int kend = early_end(most_keys(p), k0, klen);
        auto load_tile_early = [&](auto is_v, int t, u32x4(&r)[BPW]) __attribute__((always_inline)) {
            const uint16_t* gbase = decltype(is_v)::value ? vbase : kbase;
#pragma unroll
            for (int j = 0; j < BPW; ++j) {
                const int r0 = min(k0 + t * kTileKeys + RPI * (block0 + j), kend - 1); // RPI divides 16: one cache block in paged mode
                int tok = min(r0 + lrow, kend - 1);
                int64_t base = head_base;
                if (PAGED) {
                    base += bt_lookup(r0 >> p.block_shift);
                    tok &= p.block_size - 1;
                }
                r[j] = *(const u32x4*)(gbase + base + (uint32_t)(tok * stride_tok + lchunk * 8));
            }
        };
        if (!upper) {
            load_tile_early(std::false_type{}, 0, stage[1][0]);
            load_tile_early(std::false_type{}, 1, stage[1][1]);
            load_tile_early(std::false_type{}, 2, stage[1][2]);
        }
        if (!HALVES || upper) load_tile_early(std::true_type{}, 0, stage[1][3]);
    }

    if (!PAGED) copy_queries();

    int32_t tree_code = VS_STATUS_OK;
    if (p.tree_mask || p.tree_keys == 0) {
        if (tid == 0) sflag = 0;
        __syncthreads();
    } else {
        tree_code = load_tree(p.parent + (int64_t)b * p.T, p.T, sp, &sflag);
    }
    const bool s_ok = prefix_ok(p, S);
    if (kvh == 0 && k0 == 0 && rg == 0) report_status(p, b, tree_code, s_ok, S, &sflag);
    if (tree_code != VS_STATUS_OK || !s_ok) return;

    const int nk = S + p.tree_keys;
    if (k0 >= nk) return;
    if (!BAL && p.gates && nk <= klen) whole = true; // a sequence of one split has nothing to merge
    const bool merge = !BAL && p.gates && !whole;
    const MergeGate gate{merge ? p.gates + kGateWords * (((int64_t)b * p.Hkv + kvh) * p.row_groups + rg) : nullptr, &sgen};
    if (merge && tid == 0) merge_open(gate);
    const int k1 = min(nk, k0 + klen);
    const int n = (k1 - k0 + kTileKeys - 1) / kTileKeys; // tiles of this split

    const int n_full = (k1 - k0) / kTileKeys; // tiles without a ragged end
    // first key of the split in this (sequence, KV head) slice; only used when not paged
    const char* kfast = (const char*)(kbase + head_base + (int64_t)k0 * stride_tok);
    const char* vfast = (const char*)(vbase + head_base + (int64_t)k0 * stride_tok);
    // moves the window so that it starts less than 32 blocks before logical block `lb_min` (called once per iteration)
    auto bt_advance = [&](int lb_min) __attribute__((always_inline)) {
        if (PAGED && lb_min >= bt_base + 32) { // uniform
            bt_base += 32;
            bt_set(bt_next);
            bt_next = bt_fetch(bt_base + 32);
        }
    };
    // this lane's 16 bytes of the block at a uniform address: a scalar address plus lane_off (left to itself the compiler adds
    // them up first, and the copies' addresses take two registers each)
    auto load_at = [&](const void* block) __attribute__((always_inline)) {
        const __attribute__((address_space(1))) char* base = (const __attribute__((address_space(1))) char*)block;
        asm("" : "+s"(base));
        return *(const __attribute__((address_space(1))) u32x4*)(base + lane_off);
    };
    // is_v: a constant or, with HALVES, `upper`
    // LFAST: a full tile, so the address is a wave-uniform base plus a per-lane constant and nothing
    // needs clamping.
    auto load_tile = [&](auto lfast_tag, auto is_v, int t, u32x4(&r)[BPW]) __attribute__((always_inline)) {
        constexpr bool LFAST = decltype(lfast_tag)::value;
        const bool ISV = is_v;
        if constexpr (LFAST && PAGED) {
            // a full tile of a paged cache: the RPI rows of a copy block lie in one cache block, so the
            // address is a wave-uniform base (block id from the window, KV head, first row inside the
            // block - all scalar arithmetic) plus the same per-lane constant as for a contiguous cache
#pragma unroll
            for (int j = 0; j < BPW; ++j) {
                const int r0 = k0 + t * kTileKeys + RPI * (block0 + j); // uniform per wave
                const int64_t sbase = head_base + bt_lookup(r0 >> p.block_shift) + (int64_t)((r0 & (p.block_size - 1)) * stride_tok);
                r[j] = load_at((ISV ? vbase : kbase) + sbase);
            }
        } else if constexpr (LFAST) {
#pragma unroll
            for (int j = 0; j < BPW; ++j) {
                const uint32_t off = (uint32_t)((t * kTileKeys + RPI * (block0 + j)) * stride_tok) * 2u; // uniform per wave
                r[j] = load_at((ISV ? vfast : kfast) + off);
            }
        } else {
            const uint16_t* gbase = ISV ? vbase : kbase;
            if (k0 + t * kTileKeys >= k1) return; // no such tile: its LDS image is never used
#pragma unroll
            for (int j = 0; j < BPW; ++j) {
                const int r0 = k0 + t * kTileKeys + RPI * (block0 + j); // RPI divides 16: one cache block in paged mode
                int tok = min(r0 + lrow, k1 - 1);
                int64_t base = head_base;
                if (PAGED) {
                    base += bt_lookup(min(r0, k1 - 1) >> p.block_shift);
                    tok &= p.block_size - 1;
                }
                const uint32_t off = (uint32_t)(tok * stride_tok + lchunk * 8);
                r[j] = *(const u32x4*)(gbase + base + off);
            }
        }
    };
    auto stash_tile = [&](auto is_v, int t, const u32x4(&r)[BPW]) __attribute__((always_inline)) {
        const bool ISV = is_v;
        char* slot = (char*)(ISV ? sV[t & 3] : sK[t & 3]);
#pragma unroll
        for (int j = 0; j < BPW; ++j) *(u32x4*)(slot + (ISV ? v_st[j] : k_st[j])) = r[j];
    };
    // Copies are grouped per iteration: group g = K(2g+3), K(2g+4), V(2g+1), V(2g+2) is what
    // iteration g writes to LDS. Its loads are issued in iteration g - 2, so two groups are
    // in flight and alternate between two register sets.
    // Part 0 .. 3 of a group (HALVES: 0 and 2, this wave's first and second tile): what do(is_v, tile, registers) gets.
    auto part_of = [&](auto part_tag, auto set_tag, int g, auto what) __attribute__((always_inline)) {
        constexpr int PART = decltype(part_tag)::value, SET = decltype(set_tag)::value;
        if constexpr (HALVES) {
            if constexpr (PART % 2 == 0) what(upper, 2 * g + (upper ? 1 : 3) + PART / 2, stage[SET][PART / 2]);
        } else if constexpr (PART < 2) {
            what(std::false_type{}, 2 * g + 3 + PART, stage[SET][PART]);
        } else {
            what(std::true_type{}, 2 * g - 1 + PART, stage[SET][PART]);
        }
    };
    using P0 = std::integral_constant<int, 0>;
    using P1 = std::integral_constant<int, 1>;
    using P2 = std::integral_constant<int, 2>;
    using P3 = std::integral_constant<int, 3>;
    auto each_part = [&](auto set_tag, int g, auto what) __attribute__((always_inline)) {
        part_of(P0{}, set_tag, g, what);
        part_of(P1{}, set_tag, g, what);
        part_of(P2{}, set_tag, g, what);
        part_of(P3{}, set_tag, g, what);
    };
    auto load_group = [&](auto lfast_tag, auto set_tag, int g) __attribute__((always_inline)) {
        each_part(set_tag, g, [&](auto is_v, int t, u32x4(&r)[BPW]) __attribute__((always_inline)) { load_tile(lfast_tag, is_v, t, r); });
    };
    auto stash_group = [&](auto set_tag, int g) __attribute__((always_inline)) { each_part(set_tag, g, stash_tile); };

    if constexpr (!EARLY) {
        if (!upper) {
            load_tile(std::false_type{}, std::false_type{}, 0, stage[1][0]);
            load_tile(std::false_type{}, std::false_type{}, 1, stage[1][1]);
            load_tile(std::false_type{}, std::false_type{}, 2, stage[1][2]);
        }
        if (!HALVES || upper) load_tile(std::false_type{}, std::true_type{}, 0, stage[1][3]);
    }
    // the rest of the prologue copies: group 0 (set 0)
    load_group(std::false_type{}, std::integral_constant<int, 0>{}, 0);

    uint64_t mask[RPW];
#pragma unroll
    for (int rb = 0; rb < RPW; ++rb)
        mask[rb] = p.tree_keys == 0 ? 0ull : (p.tree_mask ? p.tree_mask[(int64_t)b * p.T + node_of[rb]] : ancestor_mask(sp, node_of[rb]));

    float m2[RPW], lsum[RPW]; // running reference (log2 domain, scaled) and this lane's share of the sum
    f32x16 acc[RPW][DB];
#pragma unroll
    for (int rb = 0; rb < RPW; ++rb) {
        m2[rb] = -INFINITY;
        lsum[rb] = 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[rb][db][r] = 0.f;
    }

    // per-lane LDS offsets (elements); everything else is a compile-time immediate
    // K fragment of k-step ks (chunk 2*ks + half of row `col`): k_lane[ks & 1] + ks * 256
    const int k_lane[2] = {(col >> 4) * (DB * 512) + half * 128 + ((col & 15) ^ (4 * half)) * 8,
                           (col >> 4) * (DB * 512) + half * 128 + ((col & 15) ^ (8 + 4 * half)) * 8};
    const int t16 = lane & 15;
    const int v_lane = half * 128 + (t16 >> 2) * 32 + ((lane >> 4) & 1) * 16 + ((t16 >> 1) & 1) * 8 + (t16 & 1) * 4;

    // S^T = K . Q^T for one tile: lane (col, half) gets keys 8*(r/4) + 4*half + r%4 of row `col`
    auto qk = [&](f32x16(&s)[RPW], const uint16_t* kslot) __attribute__((always_inline)) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const bf16x8 a = __builtin_bit_cast(bf16x8, *(const u32x4*)(kslot + k_lane[ks & 1] + ks * 256));
#pragma unroll
            for (int rb = 0; rb < RPW; ++rb) {
                if (ks == 0) {
                    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                    s[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[rb][ks], zero, 0, 0, 0);
                } else {
                    s[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[rb][ks], s[rb], 0, 0, 0);
                }
            }
        }
    };
    // O^T += V^T . P^T: the A operand comes from two transposing reads of 4 keys x 16 channels
    auto pv = [&](const uint16_t* vslot, const bf16x8(&pf)[RPW][2]) __attribute__((always_inline)) {
        const uint16_t* tV = vslot + v_lane;
#pragma unroll
        for (int sl = 0; sl < 2; ++sl)
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(tV + sl * (DB * 512) + db * 512));
                const s16x4 hi =
                    __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(tV + sl * (DB * 512) + db * 512 + 256));
                const bf16x8 a = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
                for (int rb = 0; rb < RPW; ++rb)
                    acc[rb][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pf[rb][sl], acc[rb][db], 0, 0, 0);
            }
    };
    // Online softmax of one tile's scores (vector ALU only): masks, running reference and sum,
    // probabilities as bf16 B operands. Returns the factors the accumulators must be scaled
    // by before this tile's probabilities are applied (1 almost always, see kLazy).
    auto softmax = [&](auto masked_tag, int kt, f32x16(&sc)[RPW], bf16x8(&pf)[RPW][2], float(&alpha)[RPW])
                       __attribute__((always_inline)) {
        constexpr bool MASKED = decltype(masked_tag)::value;
#pragma unroll
        for (int rb = 0; rb < RPW; ++rb) {
            f32x16& s = sc[rb];
            if constexpr (MASKED) {
                const uint32_t w = tile_visible(mask[rb], kt - S, k1 - kt) >> (4 * half);
#pragma unroll
                for (int r = 0; r < 16; ++r) s[r] = visible_or_inf(s[r], w, 8 * (r >> 2) + (r & 3));
            }
            float mx = fmaxf(fmaxf(s[0], s[1]), s[2]);
#pragma unroll
            for (int r = 3; r < 15; r += 2) mx = fmaxf(fmaxf(mx, s[r]), s[r + 1]);
            mx = fmaxf(mx, s[15]);
            mx = half_max(mx);
            // lazy reference: moves only when the tile's maximum exceeds it by more than kLazy
            const float mt = mx * p.scale_log2;
            const float m_new = (mt > m2[rb] + kLazy) ? mt : m2[rb];
            const float m_use = (MASKED && m_new == -INFINITY) ? 0.f : m_new; // no visible key yet
            alpha[rb] = __builtin_amdgcn_exp2f(m2[rb] - m_use);
            m2[rb] = m_new;
            float psum = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], p.scale_log2, -m_use)); // exp2(-inf) = 0
                psum += s[r];
            }
            lsum[rb] = lsum[rb] * alpha[rb] + psum;
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
    };
    auto rescale = [&](const float(&alpha)[RPW]) __attribute__((always_inline)) {
        bool need = false;
#pragma unroll
        for (int rb = 0; rb < RPW; ++rb) need |= alpha[rb] != 1.f;
        if (__any(need)) {
#pragma unroll
            for (int rb = 0; rb < RPW; ++rb)
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[rb][db][r] *= alpha[rb];
        }
    };

    // One pipeline step for prefix-only tiles with every neighbour present, written slot
    // by slot so that the instruction stream alternates between the two units: slot (f, rb)
    // holds one MFMA (fragment f: the KS fragments of K for S(next), then the 2*DB
    // fragments of V^T for O += V(prev)^T . P(prev)^T), the LDS read of the fragment two
    // slots ahead, and one share of the softmax of S(cur) -> P(cur) for row block rb. The
    // softmax is cut into 16 groups per row block: 4 of running-maximum work (the last one
    // fixes the reference), 8 of two exponentials each, 4 of bf16 packing.
    // copy_tag >= 0 (a register set): the step also carries the iteration's tile copies, one
    // tile per four slots - the staged tile goes to LDS and its registers are refilled with the
    // tile two groups ahead - so that the LDS writes trickle in between the fragment reads
    // instead of arriving as one 32 KB burst that stalls every wave's reads behind it.
    auto fast_step = [&](auto copy_tag, auto lfast_tag, int g, f32x16(&s_next)[RPW], const uint16_t* kslot,
                         const uint16_t* vslot, const bf16x8(&p_prev)[RPW][2], f32x16(&s_cur)[RPW],
                         bf16x8(&p_cur)[RPW][2], float(&alpha)[RPW]) __attribute__((always_inline)) {
        constexpr int CSET = decltype(copy_tag)::value;
        constexpr int NF = KS + 2 * DB; // fragments = MFMA slots per row block
        constexpr int GPS = 16 / NF;    // softmax groups per slot
        static_assert(16 % NF == 0, "softmax groups must divide evenly over the slots");
        constexpr int PF = 2;
        const uint16_t* tK[2] = {kslot + k_lane[0], kslot + k_lane[1]};
        const uint16_t* tV = vslot + v_lane;
        u32x4 frag[PF + 1];
        // slot order: K and V^T fragments alternate, so that consecutive MFMAs never use the
        // same accumulator (a dependent MFMA issued right behind its predecessor stalls the
        // wave's whole instruction stream until the result is back)
        static_assert(KS == 2 * DB, "as many K fragments as V^T fragments");
        auto load_frag = [&](int f) __attribute__((always_inline)) {
            const int h = f >> 1;
            if ((f & 1) == 0) {
                frag[f % (PF + 1)] = *(const u32x4*)(tK[h & 1] + h * 256);
            } else {
                const int sl = h / DB, db = h % DB;
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(tV + sl * (DB * 512) + db * 512));
                const s16x4 hi =
                    __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(tV + sl * (DB * 512) + db * 512 + 256));
                frag[f % (PF + 1)] = __builtin_bit_cast(u32x4, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            }
        };
        float mx[RPW], nm[RPW], psum[RPW], psum2[RPW];
        u32x4 pw[RPW][2];
        auto softmax_group = [&](int rb, int g) __attribute__((always_inline)) {
            f32x16& sc = s_cur[rb];
            if (g < 4) {
                mx[rb] = g == 0 ? max3(max3(sc[0], sc[1], sc[2]), sc[3], sc[3])
                                : max3(max3(mx[rb], sc[4 * g], sc[4 * g + 1]), sc[4 * g + 2], sc[4 * g + 3]);
                if (g == 3) {
                    const float mt = half_max(mx[rb]) * p.scale_log2;
                    const float m_new = (mt > m2[rb] + kLazy) ? mt : m2[rb]; // finite: prefix keys are always visible
                    alpha[rb] = __builtin_amdgcn_exp2f(m2[rb] - m_new);
                    m2[rb] = m_new;
                    nm[rb] = -m_new;
                    psum[rb] = 0.f;
                    psum2[rb] = 0.f;
                }
            } else if (g < 12) {
#pragma unroll
                for (int e = 2 * (g - 4); e < 2 * (g - 4) + 2; ++e)
                    sc[e] = __builtin_amdgcn_exp2f(fmaf(sc[e], p.scale_log2, nm[rb]));
                // the previous group's pair joins the sum here, one group late, so that the add
                // never waits for an exponential; two running sums keep the adds independent. The
                // empty asm keeps each add in its slot (otherwise all sixteen are sunk behind the
                // step as one dependent chain, out of the MFMAs' shadow).
                if (g > 4) {
                    psum[rb] += sc[2 * (g - 5)];
                    psum2[rb] += sc[2 * (g - 5) + 1];
                    asm volatile("" : "+v"(psum[rb]), "+v"(psum2[rb]));
                }
            } else {
                const int q = g - 12, sl = q >> 1;
                if (g == 12) {
                    psum[rb] += sc[14];
                    psum2[rb] += sc[15];
                }
#pragma unroll
                for (int e = 2 * (q & 1); e < 2 * (q & 1) + 2; ++e) {
                    const f32x2 pr = {sc[8 * sl + 2 * e], sc[8 * sl + 2 * e + 1]};
                    pw[rb][sl][e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pr, bf16x2));
                    asm volatile("" : "+v"(pw[rb][sl][e]));
                }
                if (g == 15) lsum[rb] = lsum[rb] * alpha[rb] + (psum[rb] + psum2[rb]);
            }
        };
#pragma unroll
        for (int f = 0; f < PF; ++f) load_frag(f);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            if (f + PF < NF) load_frag(f + PF);
            const bf16x8 a = __builtin_bit_cast(bf16x8, frag[f % (PF + 1)]);
#pragma unroll
            for (int rb = 0; rb < RPW; ++rb) {
                const int h = f >> 1;
                if (f == 0) {
                    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                    s_next[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[rb][0], zero, 0, 0, 0);
                } else if ((f & 1) == 0) {
                    s_next[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[rb][h], s_next[rb], 0, 0, 0);
                } else {
                    const int sl = h / DB, db = h % DB;
                    acc[rb][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, p_prev[rb][sl], acc[rb][db], 0, 0, 0);
                }
#pragma unroll
                for (int sg = f * GPS; sg < (f + 1) * GPS; ++sg) softmax_group(rb, sg);
                if constexpr (CSET >= 0) {
                    if (rb == 0 && f % (NF / 4) == 1) {
                        auto renew = [&](auto part_tag) __attribute__((always_inline)) {
                            part_of(part_tag, copy_tag, g, stash_tile);
                            part_of(part_tag, copy_tag, g + 2, [&](auto is_v, int t, u32x4(&r)[BPW]) __attribute__((always_inline)) {
                                load_tile(lfast_tag, is_v, t, r);
                            });
                        };
                        const int part = f / (NF / 4); // known after unrolling
                        if (part == 0) renew(P0{});
                        else if (part == 1) renew(P1{});
                        else if (part == 2) renew(P2{});
                        else renew(P3{});
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int rb = 0; rb < RPW; ++rb)
#pragma unroll
            for (int sl = 0; sl < 2; ++sl) {
                // the empty asm pins the softmax results to this step: without it the compiler
                // sinks the exponentials past the (rare) rescale branch that follows, out of
                // the shadow of the MFMAs
                asm volatile("" : "+v"(pw[rb][sl]));
                p_cur[rb][sl] = __builtin_bit_cast(bf16x8, pw[rb][sl]);
            }
    };

    // Every load so far (tiles, queries, masks) has landed after this wait. Stating it here,
    // outside any branch, also keeps the compiler from re-waiting for the query registers
    // inside the loop, where such a wait would drain the tile copies in flight.
    __builtin_amdgcn_s_waitcnt(wait_vm(0));
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[0][ks] = read_q_frag<D>(sq, ks, col, half);
    __syncthreads(); // every wave has its queries: the rings may be filled
    {
        // the early tiles: rows at or past k1 become zeros
        auto stash_tile_live = [&](auto is_v, uint16_t* slot, const u32x4(&r)[BPW], int t) __attribute__((always_inline)) {
            constexpr bool ISV = decltype(is_v)::value;
#pragma unroll
            for (int j = 0; j < BPW; ++j) {
                const bool live = k0 + t * kTileKeys + RPI * (block0 + j) + lrow < k1;
                const u32x4 zero = {0u, 0u, 0u, 0u};
                *(u32x4*)((char*)slot + (ISV ? v_st[j] : k_st[j])) = live ? r[j] : zero;
            }
        };
        if (!upper) {
            stash_tile_live(std::false_type{}, sK[0], stage[1][0], 0);
            stash_tile_live(std::false_type{}, sK[1], stage[1][1], 1);
            stash_tile_live(std::false_type{}, sK[2], stage[1][2], 2);
        }
        if (!HALVES || upper) stash_tile_live(std::true_type{}, sV[0], stage[1][3], 0);
    }
    load_group(std::false_type{}, std::integral_constant<int, 1>{}, 1);
    __syncthreads();

    f32x16 sa[RPW], sb[RPW];  // scores of the iteration's first / second tile
    bf16x8 pa[RPW][2], pb[RPW][2];
#pragma unroll
    for (int rb = 0; rb < RPW; ++rb)
#pragma unroll
        for (int sl = 0; sl < 2; ++sl) pb[rb][sl] = __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u});
    if (wave_active) qk(sa, sK[0]);
    __syncthreads(); // slot 0 of the K ring is rewritten at the end of the first iteration

    // Iteration g handles tiles ta = 2g and tb = 2g + 1. CFAST iterations have every
    // neighbour tile present and only prefix keys; the general form checks and masks.
    auto iteration = [&](auto active, auto cfast_tag, auto lfast_tag, auto set_tag, int ta) __attribute__((always_inline)) {
        constexpr bool FAST = decltype(cfast_tag)::value;
        // set_tag: the register set of the copy group that this iteration stashes
        using masked_t = std::integral_constant<bool, !FAST>;
        const int tb = ta + 1;
        const int g = ta >> 1;
        // this iteration requests group g + 2 = tiles 2g + 5 .. 2g + 8
        bt_advance(min(k0 + (2 * g + 5) * kTileKeys, k1 - 1) >> p.block_shift);
        // first tile: S(tb), O(ta - 1) | P(ta)
        if (active) {
            float alpha[RPW];
            if constexpr (FAST) {
                // the very first step applies all-zero probabilities to V(0)
                fast_step(std::integral_constant<int, -1>{}, lfast_tag, g, sb, sK[tb & 3], sV[ta ? (ta - 1) & 3 : 0], pb, sa,
                          pa, alpha);
            } else {
                if (tb < n) qk(sb, sK[tb & 3]);
                if (ta > 0) pv(sV[(ta - 1) & 3], pb);
                softmax(masked_t{}, k0 + ta * kTileKeys, sa, pa, alpha);
            }
            rescale(alpha);
        }
        // In the middle of the iteration: group g (requested one and a half iterations ago) goes
        // to LDS and its registers are refilled with group g + 2. The LDS writes complete under
        // the second tile's work; the barrier at the end publishes them for iteration g + 1.
        // (the fast form spreads the same copies over the slots of its second step, see fast_step;
        // waves without rows have no such step and copy here)
        // (with four waves a tile is two blocks per wave and the interleaved form runs out of registers)
        constexpr bool SPREAD = FAST && BPW == 1;
        if (!SPREAD || !active) {
            stash_group(set_tag, g);
            load_group(lfast_tag, set_tag, g + 2);
        }
        // second tile: S(ta + 2), O(ta) | P(tb)
        if (active) {
            float alpha[RPW];
            if constexpr (FAST) {
                using copy_t = std::conditional_t<SPREAD, decltype(set_tag), std::integral_constant<int, -1>>;
                fast_step(copy_t{}, lfast_tag, g, sa, sK[(ta + 2) & 3], sV[ta & 3], pa, sb, pb, alpha);
                rescale(alpha);
            } else {
                if (ta + 2 < n) qk(sa, sK[(ta + 2) & 3]);
                pv(sV[ta & 3], pa);
                if (tb < n) {
                    softmax(masked_t{}, k0 + tb * kTileKeys, sb, pb, alpha);
                    rescale(alpha);
                }
            }
        }
        __syncthreads();
    };
    using T = std::true_type;
    using F = std::false_type;
    using S0 = std::integral_constant<int, 0>;
    using S1 = std::integral_constant<int, 1>;
    // tiles that end at or before min(S, k1) hold prefix keys only
    const int n_plain = max(0, min(S, k1) - k0) / kTileKeys;
    const int fast_end = min(n_plain, n - 1) & ~1; // CFAST iterations need tiles ta + 1 (plain) and ta + 2 (present)
    // Iterations come in pairs so that the two register sets alternate at compile time. The
    // forms only ever get more general as ta grows (prefix tiles first, copies near the end
    // of the range last), so three loops in a row cover every case. Iteration ta loads
    // group ta/2 + 2 = tiles up to ta + 8.
    auto all_tiles = [&](auto active) __attribute__((always_inline)) {
        int ta = 0;
        for (; ta + 2 < fast_end && ta + 10 < n_full; ta += 4) {
            iteration(active, T{}, T{}, S0{}, ta);
            iteration(active, T{}, T{}, S1{}, ta + 2);
        }
        for (; ta + 2 < fast_end; ta += 4) {
            iteration(active, T{}, F{}, S0{}, ta);
            iteration(active, T{}, F{}, S1{}, ta + 2);
        }
        for (; ta < n; ta += 4) {
            iteration(active, F{}, F{}, S0{}, ta);
            if (ta + 2 < n) iteration(active, F{}, F{}, S1{}, ta + 2);
        }
    };
    // Waves without rows only copy, in loops of their own: where both kinds pass through the same code, the compiler
    // cannot tell which copies are still on their way and waits for all of them in every iteration, the ones just
    // requested included (12 x 60 nodes, 16 / 16 heads of 64 channels, up to 8000 keys 68 -> 57 us; eight waves
    // of 128 channels 1 %). Four waves of 128 channels run out of registers that way (32 x 60 nodes of 32 / 32
    // heads, 3136 keys 304 -> 377 us) and are bound by memory, not by its latency; so do three waves per SIMD.
    if constexpr ((D == 128 && NW == 4) || WPS == 3) all_tiles(wave_active);
    else if (wave_active) all_tiles(T{});
    else all_tiles(F{});
    if (wave_active) {
    if ((n & 1) == 0) pv(sV[(n - 1) & 3], pb);

    // ---- epilogue: lane (col, half) holds, for row `col`, channels db*32 + 8*(r/4) + 4*half + r%4
    // (what depends on the lane alone is worked out again: kept over the loop it takes registers)
    int tid_end = threadIdx.x;
    asm volatile("" : "+v"(tid_end));
    const int lane = tid_end & 63, half = lane >> 5, col = lane & 31;
#pragma unroll
    for (int rb = 0; rb < RPW; ++rb) {
        const float l = half_sum(lsum[rb]);
        if (whole) {
            // Lines pay for eight waves of 128 channels: us per call, 8-byte pieces / lines, 60 nodes, 28 / 4 heads, 64 x 400 keys 53.4 / 48.7,
            // 28 x 1696 59.9 / 58.6. With four waves or 64 channels the trip through LDS costs more: 12 x 35 nodes, 32 / 32
            // heads, 90 keys 12.9 / 13.4; 56 x 9 nodes, 32 / 8 heads of 64, 152 .. 305 keys 13.2 / 13.7.
            if constexpr (D == 128 && NW == 8) {
                const float inv = 1.f / l;
                store_rows(b, kvh, (row_base >> 5) + rb, [&](int e) __attribute__((always_inline)) {
                    const f32x16& a = acc[rb][e >> 2];
                    return pack_partial(a[4 * (e & 3)], a[4 * (e & 3) + 1], a[4 * (e & 3) + 2], a[4 * (e & 3) + 3], inv);
                });
            } else {
                const int r_local = row_base + rb * kRowBlock + col;
                if (r_local >= p.rows) continue;
                uint16_t* o = (uint16_t*)p.out + row_offset(p, b, kvh, r_local, row_node(p, r_local));
                const float inv = 1.f / l;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4) {
                        *(u32x2*)(o + db * 32 + 8 * q4 + 4 * half) =
                            pack_partial(acc[rb][db][4 * q4], acc[rb][db][4 * q4 + 1], acc[rb][db][4 * q4 + 2], acc[rb][db][4 * q4 + 3], inv);
                    }
            }
        } else {
            if (row_base + rb * kRowBlock >= p.rows) continue; // whole block is padding
            const int64_t unit = BAL ? kvh : (int64_t)b * p.Hkv + kvh;
            uint16_t* po = p.part_o + part_block<D>(p, unit, slot, (row_base >> 5) + rb);
            const float inv = l > 0.f ? 1.f / l : 0.f; // no visible key in this split: zeros, weight 0
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                if (BAL || merge) store_partial<true>(p, po, db, lane, acc[rb][db], inv);
                else store_partial(p, po, db, lane, acc[rb][db], inv);
            }
            if (half == 0) {
                const f32x2 ml = {m2[rb], l};
                float* dst = p.part_ml + ml_block(p, unit, slot, (row_base >> 5) + rb) * 2;
                if (BAL || merge) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, ml), span_of(dst), col * 8, 0, kDeviceScope);
                else *(f32x2*)(dst + col * 2) = ml;
            }
        }
    }
    }
    if (merge) {
        const int rb0 = rg * (p.rows_per_group / kRowBlock);
        merge_splits<D>(p, gate, b, kvh, rb0, min(rb0 + NW * RPW, p.rows_pad / kRowBlock), slot, (nk + p.keys_per_split - 1) / p.keys_per_split,
                        NW, (uint32_t*)sp);
    }
    }; // run_piece

    if constexpr (!BAL) {
        int b, kvh, rg, split = 0;
        if (p.by_length) {
            // More workgroups than run at once, one per (sequence, KV head, row group): the longest
            // sequences first. Workgroup slot j of an XCD is handed out when the ones before it run or are
            // done, so the second round's work goes to the CUs in the order in which they fall free - the
            // shortest of the first round takes the longest of the rest. In sequence order the launch lasted
            // as long as its unluckiest CU (64 paged sequences of 1024 .. 8191 keys, 28 / 4 heads: 421 us
            // against 354 us). The cost is the wait for the lengths before the first tile can be requested.
            const int j = blockIdx.x >> 3;
            rg = j % p.row_groups;
            const int k = (j / p.row_groups) * 8 + (blockIdx.x & 7); // units by rank of their sequence, dealt over the XCDs
            if (k >= p.B * p.Hkv) return;
            b = sequence_by_rank(p, k / p.Hkv, lane);
            kvh = k % p.Hkv;
        } else {
            const WorkItem at = work_item(p);
            if (at.none) return;
            b = at.b;
            kvh = at.kvh;
            rg = at.rg;
            split = at.split;
        }
        // the host keeps every split's first key below max_prefix_len + tree_keys, hence inside the cache
        run_piece(b, kvh, rg, split * p.keys_per_split, p.keys_per_split, split, p.num_splits == 1);
    } else {
        // workgroup id -> (share, KV head, row group): the row groups of a (share, KV head) sit next to each
        // other on one XCD (they read the same keys), consecutive (share, KV head) pairs on different ones
        uint32_t rg_u, kvh_u;
        const int u = (int)fast_div(blockIdx.x >> 3, p.by_groups, rg_u) * 8 + (blockIdx.x & 7);
        const int c = (int)fast_div((uint32_t)u, p.by_heads, kvh_u);
        const int rg = (int)rg_u, kvh = (int)kvh_u;
        if (c >= p.bal_chunks) return;
        const int rb = rg * (p.rows_per_group / kRowBlock) + wave; // this wave's row block
        const bool has_rows = rb * kRowBlock < p.rows;
        const int32_t S = lane < p.B ? p.prefix_len[lane] : -1;
        uint64_t* const words = (uint64_t*)(p.part_o + part_block<D>(p, kvh, p.num_splits - 1, rb)); // a word per sequence
        uint64_t seen = 0;
        if (has_rows) seen = load_device(words + lane);
        int start, steps, total;
        bal_scan(p, S, start, steps, total);
        // sequences that no piece will ever visit report their bad prefix length here
        if (c == 0 && kvh == 0 && rg == 0 && wave == 0 && lane < p.B && steps == 0 && !prefix_ok(p, S) && p.status) p.status[lane] = VS_STATUS_BAD_PREFIX;
        const int bounds = bal_bounds(p, lane, start, steps, total);
        const int lo = __builtin_amdgcn_readlane(bounds, c);
        const int hi = c + 1 < p.bal_chunks ? __builtin_amdgcn_readlane(bounds, c + 1) : total;
        // (in LDS, every wave its own copy: registers that the loop over the tiles needs)
        __shared__ int32_t s_start[NW][kBalMaxSeqs], s_steps[NW][kBalMaxSeqs], s_bounds[NW][kBalMaxChunks + 1];
        s_start[wave][lane] = start;
        s_steps[wave][lane] = steps;
        s_bounds[wave][lane] = lane < p.bal_chunks ? bounds : total;
        if (lane == 0) s_bounds[wave][kBalMaxChunks] = total;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup"); // read by all lanes of this wave
        int p0, p1;
        const uint64_t pieces = __ballot(bal_piece(lo, hi, start, steps, p0, p1));
        const uint64_t shared = __ballot(bal_piece(lo, hi, start, steps, p0, p1) && !(p0 == 0 && p1 == steps)); // others have the rest
        if (has_rows && ((shared >> lane) & 1)) arrival_open(words + lane, seen);
        for (uint64_t left = pieces; left != 0; left &= left - 1) { // in the order of the line
            const int i = __builtin_ctzll(left);
            const int s0 = __builtin_amdgcn_readfirstlane(s_start[wave][i]), t = __builtin_amdgcn_readfirstlane(s_steps[wave][i]);
            int t0, t1;
            bal_piece(lo, hi, s0, t, t0, t1);
            __syncthreads(); // the previous piece's last reads of the tile rings, the tree and the flag
            run_piece(i, kvh, rg, t0 * kIterKeys, (t1 - t0) * kIterKeys, c + i, ((shared >> i) & 1) == 0);
        }
        if (shared == 0 || !has_rows) return;

        // ---- The wave that comes last to a sequence's pieces of its row block merges them; nobody waits. All of a share's
        // pieces arrive at its end (the shares end together anyway, and a piece in the middle would hold up the next one
        // for the trip of its stores). A combine kernel behind the launch took 8.5 us of 98 (16 x 60 nodes, 28 / 4 heads, 1024 ..
        // 8191 keys); one arrival per workgroup instead of one per wave leaves a whole row group to one CU.
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int ln = tid & 63;
        auto shares_of = [&](int i) __attribute__((always_inline)) { // the shares that hold pieces of sequence i
            const int s0 = __builtin_amdgcn_readfirstlane(s_start[wave][i]), t = __builtin_amdgcn_readfirstlane(s_steps[wave][i]);
            int t0, t1;
            return __ballot(ln < p.bal_chunks && bal_piece(s_bounds[wave][ln], s_bounds[wave][ln + 1], s0, t, t0, t1));
        };
        int pieces_of = 0;
        for (uint64_t left = shared; left != 0; left &= left - 1) {
            const int i = __builtin_ctzll(left), k = __popcll(shares_of(i));
            pieces_of = ln == i ? k : pieces_of;
        }
        const int col = ln & 31;
        __builtin_amdgcn_s_waitcnt(wait_vm(0)); // this wave's partial results are in memory
        uint64_t left = __ballot(((shared >> ln) & 1) && arrival_last((uint64_t*)(p.part_o + part_block<D>(p, kvh, p.num_splits - 1, rb)) + ln, (uint32_t)pieces_of));
        const float* ml_row = p.part_ml + ml_block(p, kvh, 0, rb) * 2;
        const uint16_t* po_row = p.part_o + part_block<D>(p, kvh, 0, rb);
        for (; left != 0; left &= left - 1) {
            const int i = __builtin_ctzll(left);
            const uint64_t all = shares_of(i);
            // pieces in batches of three (most sequences have two or three); the next batch's maximum joins the running one
            float den = 0.f, M = -INFINITY;
            f32x4 num[4 * DB];
#pragma unroll
            for (int e = 0; e < 4 * DB; ++e) num[e] = f32x4{0.f, 0.f, 0.f, 0.f};
            bool first = true;
            for (uint64_t rest = all; rest != 0;) {
                constexpr int BATCH = 3;
                u32x2 ml[BATCH];
                u32x4 x[BATCH][2 * DB];
                const int n = min(__popcll(rest), BATCH);
#pragma unroll
                for (int q = 0; q < BATCH; ++q)
                    if (q < n) { // uniform
                        const int slot = (int)__builtin_ctzll(rest) + i;
                        rest &= rest - 1;
                        ml[q] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(span_of(ml_row), col * 8, slot * (kRowBlock * 8), kDeviceScope));
#pragma unroll
                        for (int e = 0; e < 2 * DB; ++e)
                            x[q][e] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(span_of(po_row), ln * 16, (e * p.num_splits + slot) * 1024, kDeviceScope));
                    }
                float Mb = M;
#pragma unroll
                for (int q = 0; q < BATCH; ++q)
                    if (q < n) Mb = fmaxf(Mb, __uint_as_float(ml[q][0]));
                if (!first) { // what was summed so far is rescaled
                    const float resc = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(M - Mb);
                    den *= resc;
#pragma unroll
                    for (int e = 0; e < 4 * DB; ++e) num[e] *= resc;
                }
                first = false;
                M = Mb;
#pragma unroll
                for (int q = 0; q < BATCH; ++q)
                    if (q < n) {
                        // a piece that saw no visible key for the row has max -inf, sum 0 and zero partials
                        const float m = __uint_as_float(ml[q][0]);
                        const float w = m != -INFINITY ? __builtin_amdgcn_exp2f(m - M) * __uint_as_float(ml[q][1]) : 0.f;
                        den += w;
#pragma unroll
                        for (int e = 0; e < 2 * DB; ++e) {
                            num[2 * e] += w * unpack_partial(u32x2{x[q][e][0], x[q][e][1]});
                            num[2 * e + 1] += w * unpack_partial(u32x2{x[q][e][2], x[q][e][3]});
                        }
                    }
            }
            const float inv = 1.f / den;
            store_rows(i, kvh, rb, [&](int e) __attribute__((always_inline)) { return pack_partial(num[e][0], num[e][1], num[e][2], num[e][3], inv); });
        }
    }
}

template <int D, int RPW, int NW>
hipError_t launch_pipe(const AttnParams& p, hipStream_t s) {
    if (p.bal_chunks > 0) {
        const dim3 grid(((p.bal_chunks * p.Hkv + 7) / 8) * 8 * p.row_groups);
        if (p.paged) hipLaunchKernelGGL((attn_mfma_pipe_kernel<D, RPW, NW, true, true>), grid, dim3(NW * kWave), 0, s, p);
        else hipLaunchKernelGGL((attn_mfma_pipe_kernel<D, RPW, NW, false, true>), grid, dim3(NW * kWave), 0, s, p);
        return hipGetLastError();
    }
    const dim3 grid(p.by_length ? (p.B * p.Hkv + 7) / 8 * 8 * p.row_groups : (p.total_wgs + 7) / 8 * 8);
    if constexpr (D == 64 && NW == 4) {
        if (pipe_three_per_cu(D, NW, p.total_wgs)) {
            if (p.paged) hipLaunchKernelGGL((attn_mfma_pipe_kernel<D, RPW, NW, true, false, 3>), grid, dim3(NW * kWave), 0, s, p);
            else hipLaunchKernelGGL((attn_mfma_pipe_kernel<D, RPW, NW, false, false, 3>), grid, dim3(NW * kWave), 0, s, p);
            return hipGetLastError();
        }
    }
    if (p.paged) hipLaunchKernelGGL((attn_mfma_pipe_kernel<D, RPW, NW, true, false>), grid, dim3(NW * kWave), 0, s, p);
    else hipLaunchKernelGGL((attn_mfma_pipe_kernel<D, RPW, NW, false, false>), grid, dim3(NW * kWave), 0, s, p);
    return hipGetLastError();
}

} // namespace

// One row block per wave; four waves (two workgroups per CU) or eight.
bool attention_pipe_supported(int rpw, int waves) { return rpw == 1 && (waves == 4 || waves == 8); }

hipError_t launch_attention_mfma_pipe(const AttnParams& p, int rpw, int waves, hipStream_t s) {
    if (!attention_pipe_supported(rpw, waves) || (p.d != 128 && p.d != 64)) return hipErrorInvalidValue;
    if (p.d == 128) return waves == 8 ? launch_pipe<128, 1, 8>(p, s) : launch_pipe<128, 1, 4>(p, s);
    return waves == 8 ? launch_pipe<64, 1, 8>(p, s) : launch_pipe<64, 1, 4>(p, s);
}

} // namespace vs
