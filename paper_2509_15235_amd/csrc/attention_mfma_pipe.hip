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
// K/V tiles go from memory straight into LDS (1 KB of consecutive memory per load instruction), two or three iterations ahead of
// the one that reads them, into rings of eight (six) tiles each; the wait for them counts loads, so the copies take
// nothing but their issue. Four waves of 128 channels, two workgroups on a CU, have no room for such rings: their tiles travel
// through registers, requested two iterations before the one that writes them to rings of four tiles in its middle.
// (Before, all kernels copied like that. 64 x 60 nodes, 28 / 4 heads, 1024 .. 8192 keys paged, cycles for a tile of the two waves of a SIMD:
// 1893 with every copy's address worked out by 17 scalar instructions and the softmax's rare parts in line, 1622 with
// addresses kept in lanes and the rare parts behind a branch, 1536 with the tiles going straight into LDS; 1250 are left with
// nothing but the matrix instructions and the barriers. The clock gives way to the power that busier matrix cores take - 2.1, 1.9, 1.87 and
// 2.35 GHz - so 898, 842, 815 and 534 ns a tile, and the call 322 -> 292 us. Sharing the exponentials out evenly over a step's slots, or
// fragments read three or four slots ahead: nothing.)
#include <type_traits>

#include "attn_mfma_common.h"

namespace vs {

namespace {

// Waves of a SIMD that have registers at the same time: two, and three (workgroups of four waves on a CU) with 64 channels.
template <int D, int RPW, int NW, bool PAGED, bool BAL, bool ONCE>
__global__ __launch_bounds__(NW * 64, D == 64 && NW == 4 ? 3 : 2) void attn_mfma_pipe_kernel(const AttnParams p) {
    request_args(p);
    constexpr int KS = D / 16;                 // k-steps of the S^T product
    constexpr int DB = D / 32;                 // 32-channel blocks of the output
    constexpr int SUB = kTileKeys * D;         // elements per 32-key tile of K (or V)
    constexpr int BPS = SUB * 2 / 1024;        // 1 KB blocks (16 keys x 32 channels) per tile
    constexpr int BPW = (BPS + NW - 1) / NW;   // ... copied by each wave
    // Tiles go straight from memory into LDS where a workgroup has room for rings that reach far enough ahead: eight tiles each of K and V for eight
    // waves (one workgroup on a CU), six for four waves of 64 channels (three workgroups). Two workgroups of four waves of 128
    // channels have not, and take their tiles through registers.
    constexpr bool DIRECT = NW == 8 || D == 64;
    constexpr int NSLOT = NW == 8 ? 8 : DIRECT ? 6 : 4;
    // Eight waves of 64 channels are twice as many as a tile has blocks: the lower half copies K, the upper half V, one block
    // of every tile each.
    constexpr bool HALVES = NW == 2 * BPS;
    static_assert(HALVES || NW * BPW == BPS, "the waves' blocks make up a tile");

    __shared__ __attribute__((aligned(1024))) uint16_t sK[NSLOT][SUB];
    __shared__ __attribute__((aligned(1024))) uint16_t sV[NSLOT][SUB];
    __shared__ int32_t sBt[DIRECT && PAGED ? NW : 1][kWave]; // block ids, see bt_advance
    __shared__ int32_t sLen[DIRECT && !BAL ? NW : 1][kWave]; // the sequence's length, a copy for every wave
    __shared__ int32_t sp[VS_MAX_TREE];
    __shared__ int32_t sflag;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // Final rows of row block rb out of the accumulators' lanes (quad(e): this lane's channels 8 * e + 4 * half .. + 3 of its row), half of the
    // channels at a time through 4 KB (2 of 64 channels) of the K ring for this wave, which nobody reads behind the last tile:
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
    // S_known: the sequence's prefix length, where the caller has read it (BAL).
    auto run_piece = [&](const int b, const int kvh, const int rg, const int k0, const int klen, const int slot,
                         bool whole, const int32_t S_known) __attribute__((always_inline)) {
    int tid = threadIdx.x;
    // What depends on the lane alone is worked out for every piece: kept from one piece to the next it takes registers that the loop
    // needs. Four waves of 128 channels had 41 of them in scratch memory, and the wait for a spilled value in the
    // loop waits for all tile copies in flight: 20 x 60 nodes, 32 / 32 heads, 250 .. 2000 keys 131 us, so 117
    // (8 of 1024 .. 8191 keys 159 / 147, paged 163 / 154; eight waves: no spills either, 1 %).
    if (BAL) asm volatile("" : "+v"(tid));
    const int lane = tid & 63, half = lane >> 5, col = lane & 31;
    // The prefix length is requested first and needed last: the first tiles and the queries are requested before it arrives. DIRECT: it and the
    // first block ids come through LDS like the tiles and are waited for by counting loads, since the compiler, which does not know of loads
    // straight into LDS - or takes those that it knows for flat ones - would wait for all of them with any of its own.
    // (Before, the wave waited for the length, and paged for the queries, before it asked for the tiles: us per layer, 28 / 4 heads, before /
    // so: 6 x 60 nodes, 2044 .. 4089 keys paged 33.2 / 32.3; 6 x 23, 903 .. 1806 keys 17.9 / 17.4; longer launches 0 - 1 %.)
    int32_t S = S_known;
    if constexpr (DIRECT && !BAL) load_to_lds4((uint32_t)(uintptr_t)(lds_void*)&sLen[wave][0], p.prefix_len + b, 0u);
    else if constexpr (!BAL) S = p.prefix_len[b];

    // ---- tile copies. One load instruction of a wave fetches 1 KB of consecutive memory:
    // RPI whole rows (tokens) of D channels, lane q -> row q / LPR, 16-byte chunk q % LPR, so
    // every touched cache line is used completely. DIRECT: the rows lie in LDS as they are, their chunks in another order (kx,
    // vx below), and what lies past the last valid token reads as zeros or is another row. Through registers: the chunks are scattered into
    // LDS so that the fragment reads are conflict-free; chunk c of tile row r lives at byte
    //   K: ((r/16)*DB + c/4) * 1024 + (c%4) * 256 + ((r%16) ^ 4*(c%4)) * 16
    //   V: ((r/16)*DB + c/4) * 1024 + (4*(r%16) + c%4) * 16
    // (the XOR spreads the chunks of one K row over the banks: 4-way instead of 16-way write
    // conflicts; reads of 16 rows at one chunk stay a permutation of 16 consecutive slots).
    // Tokens past the last valid one re-read that token (finite values that get zero weight; paged: whatever the pool holds there, V's rows become zeros).
    constexpr int LPR = D / 8;        // lanes (16-byte chunks) per row
    constexpr int RPI = 64 / LPR;     // rows per load instruction
    static_assert(BPS * RPI == kTileKeys, "a tile is BPS blocks of RPI rows");
    const uint16_t* kbase = (const uint16_t*)p.k;
    const uint16_t* vbase = (const uint16_t*)p.v;
    const int64_t head_base = (PAGED ? 0 : (int64_t)b * p.stride_seq) + (int64_t)kvh * p.stride_head;
    const int stride_tok = (int)p.stride_tok; // host guarantees 32-bit lane offsets
    const int lrow = lane / LPR, lchunk = lane % LPR;
    const uint32_t stride = (uint32_t)stride_tok * 2u; // bytes
    uint32_t lane_off = (uint32_t)lrow * stride + (uint32_t)lchunk * 16u; // bytes
    const int block0 = HALVES ? wave % BPS : wave * BPW; // this wave's first block of a tile
    const bool upper = HALVES && wave >= BPS;
    // DIRECT: a load leaves lane l's sixteen bytes at 16 l of a block, so the lanes fetch the chunks of a row in the order in
    // which they are to lie: chunk c of tile row r at position c ^ kx(r) (keys) or c ^ vx(r) (values), which spreads
    // what an operand read takes over all banks (16 rows of one chunk; 4 rows x 2 or 4 chunks).
    auto kx = [](int r) __attribute__((always_inline)) { return r % LPR; };
    auto vx = [](int r) __attribute__((always_inline)) { return D == 128 ? 4 * (r & 3) ^ 2 * ((r ^ (r >> 1)) & 1) : 2 * (r & 3); };
    uint32_t direct_off[2] = {(uint32_t)lrow * stride + (uint32_t)(lchunk ^ kx(block0 * RPI + lrow)) * 16u,
                              (uint32_t)lrow * stride + (uint32_t)(lchunk ^ vx(lrow)) * 16u};
    if (HALVES && upper) direct_off[0] = direct_off[1]; // one tensor only
    uint32_t k_st[BPW], v_st[BPW]; // this lane's LDS byte offsets inside a tile slot, per block
#pragma unroll
    for (int j = 0; j < BPW; ++j) {
        const int r = (block0 + j) * RPI + lrow, c = lchunk;
        k_st[j] = (uint32_t)(((r >> 4) * DB + (c >> 2)) * 1024 + (c & 3) * 256 + (((r & 15) ^ (4 * (c & 3))) * 16));
        v_st[j] = (uint32_t)(((r >> 4) * DB + (c >> 2)) * 1024 + (4 * (r & 15) + (c & 3)) * 16);
    }
    // Paged caches: where this wave's rows of the tiles to come lie sits one tile per lane - a window of 64 tiles, moved along
    // by 32 as they advance, with the next one's block ids on their way - as addresses ready to load from: a tile copy is two
    // v_readlane and the load. (Block offsets in the lanes, the rest of the address by scalar instructions in front
    // of every copy: 17 of them, a sixth of all instructions of the loop, and a wave issues one every 9 cycles at best.)
    const int32_t* bt_row = PAGED ? p.block_table + (int64_t)b * p.max_blocks : nullptr;
    constexpr int WINS = HALVES || !DIRECT ? 1 : 2; // K and V, or this wave's one of them (four waves, short of registers: K)
    int bt_base = 0;                     // tile of lane 0
    uint32_t bt_lo[WINS], bt_hi[WINS];   // address of this wave's first row of the lane's tile
    int32_t bt_next = 0;                 // block id of the tile 32 further on
    // (unsigned: rows past the last allowed one may pass 2^31; past the table its last entry is read)
    auto bt_token = [&](int first) __attribute__((always_inline)) { return (uint32_t)k0 + (uint32_t)(first + lane) * kTileKeys + (uint32_t)(block0 * RPI); };
    auto bt_index = [&](int first) __attribute__((always_inline)) { return min(bt_token(first) >> p.block_shift, (uint32_t)p.max_blocks - 1u); };
    auto bt_fetch = [&](int first) __attribute__((always_inline)) { return bt_row[bt_index(first)]; };
    auto bt_set = [&](int32_t blk) __attribute__((always_inline)) {
        if ((uint32_t)blk >= (uint32_t)p.num_blocks) blk = 0; // reported through status
        const uint32_t in_block = (bt_token(bt_base) & (uint32_t)(p.block_size - 1)) * (uint32_t)stride_tok;
        const uint64_t off = (uint64_t)((int64_t)blk * p.stride_block + head_base + in_block) * 2;
#pragma unroll
        for (int w = 0; w < WINS; ++w) {
            const uint64_t at = (uint64_t)((HALVES ? upper : w == 1) ? vbase : kbase) + off;
            bt_lo[w] = (uint32_t)at;
            bt_hi[w] = (uint32_t)(at >> 32);
        }
    };
    int32_t bt_first = 0;
    if constexpr (PAGED && DIRECT) { // (with the prefix length: one trip)
        load_to_lds4((uint32_t)(uintptr_t)(lds_void*)&sBt[wave][0], bt_row, bt_index(0) * 4u);
    } else if constexpr (PAGED) {
        bt_first = bt_fetch(0);
        bt_next = bt_fetch(32);
    }
    auto bt_lookup = [&](bool is_v, int t) __attribute__((always_inline)) {
        const int rel = t - bt_base, w = WINS == 1 || !is_v ? 0 : 1; // rel: 0 .. 63
        const char* at = (const char*)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)bt_hi[w], rel) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)bt_lo[w], rel));
        return !DIRECT && is_v ? at + ((const char*)vbase - (const char*)kbase) : at;
    };
    // (DIRECT) this wave's 1 KB of tile t into slot `slot` of its ring, t any tile (FULL: one with all its keys). Contiguous caches: `rows` ends at the last key that
    // may be asked for, what lies past it reads as zeros (or, where offsets that far wrap, as other rows). Paged: tiles past
    // `last` repeat that one, rows past the end are whatever the pool holds there.
    __amdgpu_buffer_rsrc_t rows[2];
    int last = 0;
    auto rows_up_to = [&](int end) __attribute__((always_inline)) {
        if constexpr (PAGED) {
            last = (end - 1 - k0) / kTileKeys;
        } else {
            const uint32_t bytes = slice_bytes(end, k0, klen, stride, D * 2);
#pragma unroll
            for (int w = 0; w < WINS; ++w)
                rows[w] = __builtin_amdgcn_make_buffer_rsrc((char*)const_cast<uint16_t*>(((HALVES ? upper : w == 1) ? vbase : kbase) + head_base) + (int64_t)k0 * stride, 0,
                                                            (int)bytes, 0x00027000);
        }
    };
    auto fetch = [&](auto full_tag, bool is_v, int t, int slot) __attribute__((always_inline)) {
        const int w = HALVES ? 0 : is_v;
        const bool v = HALVES ? upper : is_v;
        const uint32_t lds = (uint32_t)(uintptr_t)(lds_void*)(v ? &sV[0][0] : &sK[0][0]) + (uint32_t)(slot * SUB * 2 + block0 * 1024);
        if constexpr (PAGED) load_to_lds<ONCE>(lds, bt_lookup(v, decltype(full_tag)::value ? t : min(t, last)), direct_off[w]);
        else load_to_lds<ONCE>(lds, rows[w], direct_off[w] + (uint32_t)(t * kTileKeys + RPI * block0) * stride);
    };
    // rows of V tile t (this wave's, arrived) that no key has become zeros: whatever the cache holds there, NaN included,
    // must not meet a zero probability
    auto zero_tail = [&](int t, int slot, int end) __attribute__((always_inline)) {
        if ((HALVES && !upper) || k0 + (t + 1) * kTileKeys <= end) return; // uniform
        if (k0 + t * kTileKeys + RPI * block0 + lrow >= end) *(u32x4*)(sV[slot] + block0 * 512 + lane * 8) = u32x4{0u, 0u, 0u, 0u};
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
    static_assert(RPW == 1 && (DIRECT || NW <= NSLOT), "a row block's queries take a tile slot");
    // through a tile slot that nothing is on its way to yet. DIRECT: the last K slots from Q_K on and the last V slots from Q_V on
    constexpr int Q_K = NW == 8 ? 5 : NSLOT, Q_V = NSLOT - (NW - (NSLOT - Q_K));
    uint16_t* sq = !DIRECT ? sK[wave & (NSLOT - 1)] : wave < NSLOT - Q_K ? sK[min(Q_K + wave, NSLOT - 1)] : sV[min(Q_V + wave - (NSLOT - Q_K), NSLOT - 1)];
    // (DIRECT: all waves, so that the loads can be counted; one without rows fetches the last one.)
    auto copy_queries = [&]() __attribute__((always_inline)) {
        if constexpr (DIRECT) copy_q_block<D, true>(p, b, kvh, row_base, sq, lane);
        else if (wave_active) copy_q_block<D>(p, b, kvh, row_base, sq, lane);
    };
    if constexpr (PAGED) { // the queries while the block ids are on their way
        copy_queries();
        if constexpr (DIRECT) {
            wait_loads<KS>(); // all but the queries
            bt_first = sBt[wave][lane];
            wait_lds_reads();
            load_to_lds4((uint32_t)(uintptr_t)(lds_void*)&sBt[wave][0], bt_row, bt_index(32) * 4u);
        }
        bt_set(bt_first);
    }
    constexpr bool EARLY = DIRECT || !(BAL && PAGED); // registers: 4 waves of 128 channels 188 us, so 171 (8 x 60 nodes, 32 / 32 heads, 1024 .. 8191 keys)
    // this lane's 16 bytes of the block at a uniform address: a scalar address plus lane_off. (The second statement keeps the
    // lane's part in one register: extended to 64 bits in front of the loop it takes two and an addition per copy.)
    auto load_at = [&](const void* block) __attribute__((always_inline)) {
        const __attribute__((address_space(1))) char* base = (const __attribute__((address_space(1))) char*)block;
        asm("" : "+s"(base));
        asm volatile("" : "+v"(lane_off));
        const auto* at = (const __attribute__((address_space(1))) u32x4*)(base + lane_off);
        return ONCE ? __builtin_nontemporal_load(at) : *at;
    };
    const int64_t block_bytes = (int64_t)RPI * stride_tok * 2; // from one of this wave's blocks of a tile to the next
    // The first four tiles - K(0), K(1), K(2), V(0) - and, DIRECT, all others that the queries leave room for are requested before
    // the prefix length is known (BAL knows it): up to the longest allowed sequence's end instead of this one's (paged: the block
    // table's). Values of rows that turn out to lie past the sequence's last key become zeros in LDS (DIRECT: zero_tail) or on their way there from register set 1: whatever the cache holds there, NaN included,
    // must not meet a zero probability.
    if constexpr (EARLY) {
        const int kend = early_end(BAL ? S_known + p.tree_keys : most_keys(p), k0, klen);
        if constexpr (DIRECT) rows_up_to(kend);
        auto load_tile_early = [&](auto is_v, int t, u32x4(&r)[BPW]) __attribute__((always_inline)) {
            const uint16_t* gbase = decltype(is_v)::value ? vbase : kbase;
#pragma unroll
            for (int j = 0; j < BPW; ++j) {
                if constexpr (PAGED) {
                    r[j] = load_at(bt_lookup(decltype(is_v)::value, t) + j * block_bytes);
                } else {
                    const int tok = min(k0 + t * kTileKeys + RPI * (block0 + j) + lrow, kend - 1);
                    r[j] = *(const u32x4*)(gbase + head_base + (uint32_t)(tok * stride_tok + lchunk * 8));
                }
            }
        };
        if constexpr (DIRECT) {
            if (!upper) {
                for (int t = 0; t < Q_K && t <= NSLOT - 2; ++t) fetch(std::false_type{}, false, t, t);
            }
            if (!HALVES || upper) {
                for (int t = 0; t < Q_V; ++t) fetch(std::false_type{}, true, t, t);
            }
        } else {
            load_tile_early(std::false_type{}, 0, stage[1][0]);
            load_tile_early(std::false_type{}, 1, stage[1][1]);
            load_tile_early(std::false_type{}, 2, stage[1][2]);
            load_tile_early(std::true_type{}, 0, stage[1][3]);
        }
    }

    if constexpr (!PAGED) copy_queries();

    int32_t tree_code = VS_STATUS_OK;
    const bool reports = kvh == 0 && k0 == 0 && rg == 0;
    if (p.tree_mask || p.tree_keys == 0) {
        if (reports) {
            if (tid == 0) sflag = 0;
            __syncthreads();
        }
    } else {
        tree_code = load_tree(p.parent + (int64_t)b * p.T, p.T, sp, &sflag);
    }
    if constexpr (DIRECT && !BAL) {
        // loads behind it: those above, the fewest of any wave
        constexpr int TILES_K = Q_K < NSLOT - 1 ? Q_K : NSLOT - 1;
        wait_loads<(PAGED ? 2 : 0) + KS + (HALVES ? (TILES_K < Q_V ? TILES_K : Q_V) : TILES_K + Q_V)>();
        S = __builtin_amdgcn_readfirstlane(sLen[wave][0]);
    }
    const bool s_ok = prefix_ok(p, S);
    if (reports) report_status(p, b, tree_code, s_ok, S, &sflag);
    const int nk = S + p.tree_keys;
    if (tree_code != VS_STATUS_OK || !s_ok || k0 >= nk) { // uniform
        wait_loads<0>(); // tiles (DIRECT) and queries on their way to LDS
        if (BAL) __syncthreads(); // other pieces follow, or merges that take the rings' place
        return;
    }
    if (!BAL && p.gates && nk <= klen) whole = true; // a sequence of one split has nothing to merge
    const bool merge = !BAL && p.gates && !whole;
    uint64_t* const gate = merge ? p.gates + kGateWords * (((int64_t)b * p.Hkv + kvh) * p.row_groups + rg) : nullptr;
    if (merge && tid == 0) merge_open(gate, gate_load(gate));
    const int k1 = min(nk, k0 + klen);
    const int n = (k1 - k0 + kTileKeys - 1) / kTileKeys; // tiles of this split

    const int n_full = (k1 - k0) / kTileKeys; // tiles without a ragged end
    // first key of the split in this (sequence, KV head) slice; only used when not paged
    const char* kfast = (const char*)(kbase + head_base + (int64_t)k0 * stride_tok);
    const char* vfast = (const char*)(vbase + head_base + (int64_t)k0 * stride_tok);
    // moves the window so that it starts less than 32 tiles before tile `t_min` (called once per iteration)
    auto bt_advance = [&](int t_min) __attribute__((always_inline)) {
        if (PAGED && t_min >= bt_base + 32) { // uniform
            bt_base += 32;
            if constexpr (DIRECT) {
                // The next ids come through LDS like the tiles: a load that the compiler knows of would have it wait for all copies in
                // flight. These have been there since long: requested 16 iterations ago.
                bt_set(sBt[wave][lane]);
                wait_lds_reads();
                load_to_lds4((uint32_t)(uintptr_t)(lds_void*)&sBt[wave][0], bt_row, bt_index(bt_base + 32) * 4u);
            } else {
                bt_set(bt_next);
                bt_next = bt_fetch(bt_base + 32);
            }
        }
    };
    // LFAST: a full tile, so the address is a wave-uniform base plus a per-lane constant and nothing
    // needs clamping.
    auto load_tile = [&](auto lfast_tag, auto is_v, int t, u32x4(&r)[BPW]) __attribute__((always_inline)) {
        constexpr bool LFAST = decltype(lfast_tag)::value;
        const bool ISV = is_v;
        if constexpr (PAGED) {
            // the same for every tile: rows past k1 lie in the pool, too (V's are zeroed on their way into LDS)
            if (!LFAST && k0 + t * kTileKeys >= k1) return; // no such tile: its LDS image is never used
            const char* at = bt_lookup(ISV, t);
#pragma unroll
            for (int j = 0; j < BPW; ++j) r[j] = load_at(at + j * block_bytes);
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
                const int tok = min(k0 + t * kTileKeys + RPI * (block0 + j) + lrow, k1 - 1);
                const uint32_t off = (uint32_t)(tok * stride_tok + lchunk * 8);
                r[j] = *(const u32x4*)(gbase + head_base + off);
            }
        }
    };
    auto stash_tile = [&](auto lfast_tag, auto is_v, int t, const u32x4(&r)[BPW]) __attribute__((always_inline)) {
        const bool ISV = is_v;
        char* slot = (char*)(ISV ? sV[t & (NSLOT - 1)] : sK[t & (NSLOT - 1)]);
#pragma unroll
        for (int j = 0; j < BPW; ++j) {
            u32x4 w = r[j];
            if constexpr (PAGED && !decltype(lfast_tag)::value) {
                const u32x4 zero = {0u, 0u, 0u, 0u};
                if (ISV) w = k0 + t * kTileKeys + RPI * (block0 + j) + lrow < k1 ? w : zero;
            }
            *(u32x4*)(slot + (ISV ? v_st[j] : k_st[j])) = w;
        }
    };
    // Copies through registers are grouped per iteration: group g = K(2g+3), K(2g+4), V(2g+1), V(2g+2) is what
    // iteration g writes to LDS. Its loads are issued in iteration g - 2, so two groups are
    // in flight and alternate between two register sets.
    auto load_group = [&](auto lfast_tag, auto set_tag, int g) __attribute__((always_inline)) {
        constexpr int SET = decltype(set_tag)::value;
        load_tile(lfast_tag, std::false_type{}, 2 * g + 3, stage[SET][0]);
        load_tile(lfast_tag, std::false_type{}, 2 * g + 4, stage[SET][1]);
        load_tile(lfast_tag, std::true_type{}, 2 * g + 1, stage[SET][2]);
        load_tile(lfast_tag, std::true_type{}, 2 * g + 2, stage[SET][3]);
    };
    auto stash_group = [&](auto lfast_tag, auto set_tag, int g) __attribute__((always_inline)) {
        constexpr int SET = decltype(set_tag)::value;
        stash_tile(lfast_tag, std::false_type{}, 2 * g + 3, stage[SET][0]);
        stash_tile(lfast_tag, std::false_type{}, 2 * g + 4, stage[SET][1]);
        stash_tile(lfast_tag, std::true_type{}, 2 * g + 1, stage[SET][2]);
        stash_tile(lfast_tag, std::true_type{}, 2 * g + 2, stage[SET][3]);
    };

    if constexpr (!EARLY) {
        load_tile(std::false_type{}, std::false_type{}, 0, stage[1][0]);
        load_tile(std::false_type{}, std::false_type{}, 1, stage[1][1]);
        load_tile(std::false_type{}, std::false_type{}, 2, stage[1][2]);
        load_tile(std::false_type{}, std::true_type{}, 0, stage[1][3]);
    }
    // through registers: the rest of the prologue copies, group 0 (set 0)
    if constexpr (DIRECT) {
        rows_up_to(k1);
    } else {
        load_group(std::false_type{}, std::integral_constant<int, 0>{}, 0);
    }

    uint64_t mask[RPW];
#pragma unroll
    for (int rb = 0; rb < RPW; ++rb)
        mask[rb] = p.tree_keys == 0 ? 0ull : (p.tree_mask ? p.tree_mask[(int64_t)b * p.T + node_of[rb]] : ancestor_mask(sp, node_of[rb]));

    // running reference (log2 domain, scaled), the score (not scaled) from which on it moves, and this lane's share of the sum
    // (two addends: the additions of a step do not wait for each other)
    float m2[RPW], limit[RPW], lsum[RPW], lsum2[RPW];
    const float to_score = 1.f / p.scale_log2;
    f32x16 acc[RPW][DB];
#pragma unroll
    for (int rb = 0; rb < RPW; ++rb) {
        m2[rb] = limit[rb] = -INFINITY;
        lsum[rb] = lsum2[rb] = 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[rb][db][r] = 0.f;
    }

    // per-lane LDS offsets; everything else is a compile-time immediate
    // K fragment of k-step ks: chunk 2*ks + half of row `col`
    const int k_lane[2] = {(col >> 4) * (DB * 512) + half * 128 + ((col & 15) ^ (4 * half)) * 8,
                           (col >> 4) * (DB * 512) + half * 128 + ((col & 15) ^ (8 + 4 * half)) * 8};
    const int t16 = lane & 15;
    const int v_lane = half * 128 + (t16 >> 2) * 32 + ((lane >> 4) & 1) * 16 + ((t16 >> 1) & 1) * 8 + (t16 & 1) * 4;
    uint32_t k_at[KS], v_at[DB]; // DIRECT: addresses in slot 0
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) k_at[ks] = (uint32_t)(uintptr_t)(lds_void*)&sK[0][0] + (uint32_t)(col * D + ((2 * ks + half) ^ kx(col)) * 8) * 2u;
#pragma unroll
    for (int db = 0; db < DB; ++db) {
        const int r = 4 * half + (t16 >> 2);
        v_at[db] = (uint32_t)(uintptr_t)(lds_void*)&sV[0][0] + (uint32_t)(r * D + ((4 * db + 2 * ((lane >> 4) & 1) + ((t16 >> 1) & 1)) ^ vx(r)) * 8 + (t16 & 1) * 4) * 2u;
        asm("" : "+v"(v_at[db])); // (the ring's address stays in: a read's immediate offset reaches 64 KB)
    }
    auto k_frag = [&](int slot, int ks) __attribute__((always_inline)) {
        if constexpr (DIRECT) return *(const __attribute__((address_space(3))) u32x4*)(k_at[ks] + (uint32_t)(slot * SUB * 2));
        else return *(const u32x4*)(sK[slot] + k_lane[ks & 1] + ks * 256);
    };
    auto v_frag = [&](int slot, int sl, int db) __attribute__((always_inline)) { // two transposing reads of 4 keys x 16 channels
        lds_s16x4 *lo, *hi;
        if constexpr (DIRECT) {
            lo = (lds_s16x4*)(v_at[db] + (uint32_t)(slot * SUB * 2 + sl * (16 * D * 2)));
            hi = (lds_s16x4*)(v_at[db] + (uint32_t)(slot * SUB * 2 + sl * (16 * D * 2) + 8 * D * 2));
        } else {
            const uint16_t* tV = sV[slot] + v_lane + sl * (DB * 512) + db * 512;
            lo = (lds_s16x4*)tV;
            hi = (lds_s16x4*)(tV + 256);
        }
        return __builtin_bit_cast(u32x4, __builtin_shufflevector(__builtin_amdgcn_ds_read_tr16_b64_v4i16(lo), __builtin_amdgcn_ds_read_tr16_b64_v4i16(hi), 0, 1, 2, 3, 4, 5, 6, 7));
    };

    // S^T = K . Q^T for one tile: lane (col, half) gets keys 8*(r/4) + 4*half + r%4 of row `col`
    auto qk = [&](f32x16(&s)[RPW], int kslot) __attribute__((always_inline)) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const bf16x8 a = __builtin_bit_cast(bf16x8, k_frag(kslot, ks));
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
    // O^T += V^T . P^T
    auto pv = [&](int vslot, const bf16x8(&pf)[RPW][2]) __attribute__((always_inline)) {
#pragma unroll
        for (int sl = 0; sl < 2; ++sl)
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const bf16x8 a = __builtin_bit_cast(bf16x8, v_frag(vslot, sl, db));
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
            limit[rb] = (m_new + kLazy) * to_score;
            float psum = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], p.scale_log2, -m_use)); // exp2(-inf) = 0
                psum += s[r];
            }
            lsum[rb] = lsum[rb] * alpha[rb] + psum;
            lsum2[rb] *= alpha[rb];
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
    auto scale_acc = [&](const float(&alpha)[RPW]) __attribute__((always_inline)) {
#pragma unroll
        for (int rb = 0; rb < RPW; ++rb)
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[rb][db][r] *= alpha[rb];
    };
    auto rescale = [&](const float(&alpha)[RPW]) __attribute__((always_inline)) {
        bool need = false;
#pragma unroll
        for (int rb = 0; rb < RPW; ++rb) need |= alpha[rb] != 1.f;
        if (__any(need)) scale_acc(alpha);
    };

    // One pipeline step for prefix-only tiles with every neighbour present, written slot
    // by slot so that the instruction stream alternates between the two units: slot (f, rb)
    // holds one MFMA (fragment f: the KS fragments of K for S(next), then the 2*DB
    // fragments of V^T for O += V(prev)^T . P(prev)^T), the LDS read of the fragment two
    // slots ahead, and one share of the softmax of S(cur) -> P(cur) for row block rb. The
    // softmax is cut into 16 groups per row block: 4 of running-maximum work (the last one
    // fixes the reference), 8 of two exponentials each, 4 of bf16 packing.
    // copy(0), copy(1): called in the step's second slot and in the middle, for the tile copies.
    auto fast_step = [&](auto copy, f32x16(&s_next)[RPW], int kslot, int vslot, const bf16x8(&p_prev)[RPW][2], f32x16(&s_cur)[RPW],
                         bf16x8(&p_cur)[RPW][2]) __attribute__((always_inline)) {
        constexpr int NF = KS + 2 * DB; // fragments = MFMA slots per row block
        constexpr int GPS = 16 / NF;    // softmax groups per slot
        static_assert(16 % NF == 0, "softmax groups must divide evenly over the slots");
        constexpr int PF = 2;
        u32x4 frag[PF + 1];
        // slot order: K and V^T fragments alternate, so that consecutive MFMAs never use the
        // same accumulator (a dependent MFMA issued right behind its predecessor stalls the
        // wave's whole instruction stream until the result is back)
        static_assert(KS == 2 * DB, "as many K fragments as V^T fragments");
        auto load_frag = [&](int f) __attribute__((always_inline)) {
            const int h = f >> 1;
            frag[f % (PF + 1)] = (f & 1) == 0 ? k_frag(kslot, h) : v_frag(vslot, h / DB, h % DB);
        };
        float mx[RPW], alpha[RPW];
        bool moved[RPW]; // uniform: some row's reference has moved, the accumulators are rescaled behind the step
        u32x4 pw[RPW][2];
        auto softmax_group = [&](int rb, int g) __attribute__((always_inline)) {
            f32x16& sc = s_cur[rb];
            if (g < 4) {
                mx[rb] = g == 0 ? maximum3(maximum3(sc[0], sc[1], sc[2]), sc[3], sc[3])
                                : maximum3(maximum3(mx[rb], sc[4 * g], sc[4 * g + 1]), sc[4 * g + 2], sc[4 * g + 3]);
                if (g == 3) {
                    const float top = half_maximum(mx[rb]); // finite: prefix keys are always visible
                    moved[rb] = __any(top > limit[rb]);
                    if (moved[rb]) { // rare after the first tiles, so everything that it alone needs stands here
                        const float mt = top * p.scale_log2;
                        const float m_new = (mt > m2[rb] + kLazy) ? mt : m2[rb];
                        alpha[rb] = __builtin_amdgcn_exp2f(m2[rb] - m_new);
                        m2[rb] = m_new;
                        limit[rb] = (m_new + kLazy) * to_score;
                        lsum[rb] *= alpha[rb];
                        lsum2[rb] *= alpha[rb];
                    }
                }
            } else if (g < 12) {
#pragma unroll
                for (int e = 2 * (g - 4); e < 2 * (g - 4) + 2; ++e)
                    sc[e] = __builtin_amdgcn_exp2f(fmaf(sc[e], p.scale_log2, -m2[rb]));
                // the previous group's pair joins the sum here, one group late, so that the add
                // never waits for an exponential; two running sums keep the adds independent. The
                // empty asm keeps each add in its slot (otherwise all sixteen are sunk behind the
                // step as one dependent chain, out of the MFMAs' shadow).
                if (g > 4) {
                    lsum[rb] += sc[2 * (g - 5)];
                    lsum2[rb] += sc[2 * (g - 5) + 1];
                    asm volatile("" : "+v"(lsum[rb]), "+v"(lsum2[rb]));
                }
            } else {
                const int q = g - 12, sl = q >> 1;
                if (g == 12) {
                    lsum[rb] += sc[14];
                    lsum2[rb] += sc[15];
                }
#pragma unroll
                for (int e = 2 * (q & 1); e < 2 * (q & 1) + 2; ++e) {
                    const f32x2 pr = {sc[8 * sl + 2 * e], sc[8 * sl + 2 * e + 1]};
                    pw[rb][sl][e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pr, bf16x2));
                    asm volatile("" : "+v"(pw[rb][sl][e]));
                }
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
                if (rb == 0 && f % (NF / 2) == 1) copy(f / (NF / 2));
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
        static_assert(RPW == 1, "one flag");
        if (moved[0]) scale_acc(alpha);
    };

    // Every load so far (tiles, queries, masks) has landed after this wait. Stating it here,
    // outside any branch, also keeps the compiler from re-waiting for the query registers
    // inside the loop, where such a wait would drain the tile copies in flight.
    __builtin_amdgcn_s_waitcnt(wait_vm(0));
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[0][ks] = read_q_frag<D>(sq, ks, col, half);
    if constexpr (DIRECT) {
        zero_tail(0, 0, k1);
        __syncthreads(); // every wave has its queries: their slots may be filled
        // ... with what the first iteration does not request
        if (!upper) {
            for (int t = Q_K; t <= NSLOT - 2; ++t) fetch(std::false_type{}, false, t, t);
        }
        if (!HALVES || upper) {
            for (int t = Q_V; t <= NSLOT - 4; ++t) fetch(std::false_type{}, true, t, t);
        }
    } else {
        __syncthreads(); // every wave has its queries: the rings may be filled
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
        stash_tile_live(std::false_type{}, sK[0], stage[1][0], 0);
        stash_tile_live(std::false_type{}, sK[1], stage[1][1], 1);
        stash_tile_live(std::false_type{}, sK[2], stage[1][2], 2);
        stash_tile_live(std::true_type{}, sV[0], stage[1][3], 0);
        load_group(std::false_type{}, std::integral_constant<int, 1>{}, 1);
    }
    // tiles that end at or before min(S, k1) hold prefix keys only
    const int n_plain = max(0, min(S, k1) - k0) / kTileKeys;
    const int fast_end = min(n_plain, n - 1) & ~1; // fast iterations need tiles ta + 1 (plain) and ta + 2 (present)
    // what the first fast step takes for V(-1), with probabilities of zero
    if (fast_end > (DIRECT ? 0 : 2))
        for (int i = tid * 8; i < SUB; i += NW * 64 * 8) *(u32x4*)&sV[NSLOT - 1][i] = u32x4{0u, 0u, 0u, 0u};
    if constexpr (!DIRECT) __syncthreads();

    f32x16 sa[RPW], sb[RPW];  // scores of the iteration's first / second tile
    bf16x8 pa[RPW][2], pb[RPW][2];
#pragma unroll
    for (int rb = 0; rb < RPW; ++rb)
#pragma unroll
        for (int sl = 0; sl < 2; ++sl) pb[rb][sl] = __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u});
    if (wave_active) qk(sa, 0);
    __syncthreads(); // slot 0 of the K ring is rewritten in the first iteration

    // An iteration handles tiles ta and tb = ta + 1. Fast ones have every neighbour tile present and only prefix keys; the
    // general form (two parts, the copies in between) checks and masks. slot(d): ring slot of tile ta + d.
    auto general_first = [&](int ta, auto slot) __attribute__((always_inline)) { // S(tb), O(ta - 1) | P(ta)
        float alpha[RPW];
        if (ta + 1 < n) qk(sb, slot(1));
        if (ta > 0) pv(slot(-1), pb);
        softmax(std::true_type{}, k0 + ta * kTileKeys, sa, pa, alpha);
        rescale(alpha);
    };
    auto general_second = [&](int ta, auto slot) __attribute__((always_inline)) { // S(ta + 2), O(ta) | P(tb)
        float alpha[RPW];
        if (ta + 2 < n) qk(sa, slot(2));
        pv(slot(0), pa);
        if (ta + 1 < n) {
            softmax(std::true_type{}, k0 + (ta + 1) * kTileKeys, sb, pb, alpha);
            rescale(alpha);
        }
    };
    // Through registers: iteration g = ta / 2 requests group g + 2 = tiles up to 2g + 8 and, in its middle, takes group g (requested
    // one and a half iterations ago) to LDS. The LDS writes complete under
    // the second tile's work; the barrier at the end publishes them for iteration g + 1.
    // set_tag: the register set of the copy group that this iteration stashes
    auto iteration = [&](auto active, auto cfast_tag, auto lfast_tag, auto set_tag, int ta) __attribute__((always_inline)) {
        constexpr bool FAST = decltype(cfast_tag)::value;
        const int g = ta >> 1;
        auto slot = [&](int d) __attribute__((always_inline)) { return (ta + d) & (NSLOT - 1); };
        bt_advance(2 * g + 5);
        if (active) {
            // (the very first step applies all-zero probabilities to a slot of zeros)
            if constexpr (FAST) fast_step([](int) {}, sb, slot(1), slot(-1), pb, sa, pa);
            else general_first(ta, slot);
        }
        stash_group(lfast_tag, set_tag, g);
        load_group(lfast_tag, set_tag, g + 2);
        if (active) {
            if constexpr (FAST) fast_step([](int) {}, sa, slot(2), slot(0), pa, sb, pb);
            else general_second(ta, slot);
        }
        __syncthreads();
    };
    // DIRECT, rings of N: a fast iteration requests K(ta + N - 1), K(ta + N), V(ta + N - 3), V(ta + N - 2) into the slots of tiles read in the
    // one before, whether they exist or not: so a wait for all loads but the last iterations' is one for the tiles of
    // the next, requested N / 2 - 2 iterations earlier. ph: ta % N, a constant where the loop is unrolled (the slots are then
    // part of the instructions). FULL: all tiles requested are full ones.
    auto direct_iteration = [&](auto active, auto cfast_tag, auto full_tag, auto ph, int ta) __attribute__((always_inline)) {
        constexpr bool FAST = decltype(cfast_tag)::value, FULL = decltype(full_tag)::value;
        auto slot = [&](int d) __attribute__((always_inline)) { // d: -1 .. N
            const int x = ph + d;
            return (NSLOT & (NSLOT - 1)) == 0 ? x & (NSLOT - 1) : x < 0 ? x + NSLOT : x >= NSLOT ? x - NSLOT : x;
        };
        auto request = [&](int i) __attribute__((always_inline)) { // i: 0 .. 3 (HALVES: 0 and 2)
            auto tile = [&](bool v, int j) __attribute__((always_inline)) {
                const int d = v ? NSLOT - 3 + j : NSLOT - 1 + j;
                if (FAST || ta + d < n) fetch(full_tag, v, ta + d, v ? slot(NSLOT - 3 + j) : slot(NSLOT - 1 + j));
            };
            if (!HALVES) tile(i >= 2, i & 1);
            else if (i % 2 == 0) tile(upper, i >> 1);
        };
        bt_advance(FULL ? ta + NSLOT - 3 : min(ta + NSLOT - 3, last));
        if (active) {
            // (the very first step applies all-zero probabilities to a slot of zeros)
            if constexpr (FAST) {
                fast_step([&](int i) __attribute__((always_inline)) { request(i); }, sb, slot(1), slot(-1), pb, sa, pa);
                fast_step([&](int i) __attribute__((always_inline)) { request(2 + i); }, sa, slot(2), slot(0), pa, sb, pb);
            } else {
                for (int i = 0; i < 4; ++i) request(i);
                general_first(ta, slot);
                general_second(ta, slot);
            }
        } else {
            for (int i = 0; i < 4; ++i) request(i);
        }
        if constexpr (FAST) wait_loads<(NSLOT / 2 - 2) * (HALVES ? 2 : 4)>();
        else wait_loads<0>();
        if (!FULL) {
            zero_tail(ta + 1, slot(1), k1);
            if (FAST || ta + 2 < n) zero_tail(ta + 2, slot(2), k1);
        }
        __syncthreads();
    };
    using T = std::true_type;
    using F = std::false_type;
    using S0 = std::integral_constant<int, 0>;
    using S1 = std::integral_constant<int, 1>;
    // The forms only ever get more general as ta grows (prefix tiles first, copies near the end of the range last), so three loops
    // in a row cover every case. (One loop with all forms, or one that is left in its middle, spills hundreds of registers.)
    // Through registers iterations come in pairs so that the two register sets alternate at compile time; iteration ta
    // loads group ta/2 + 2 = tiles up to ta + 8.
    auto all_tiles = [&](auto active) __attribute__((always_inline)) {
        int ta = 0;
        if constexpr (DIRECT) {
            auto turn = [&](auto full_tag) __attribute__((always_inline)) { // of the rings
                direct_iteration(active, T{}, full_tag, std::integral_constant<int, 0>{}, ta);
                direct_iteration(active, T{}, full_tag, std::integral_constant<int, 2>{}, ta + 2);
                direct_iteration(active, T{}, full_tag, std::integral_constant<int, 4>{}, ta + 4);
                if constexpr (NSLOT == 8) direct_iteration(active, T{}, full_tag, std::integral_constant<int, 6>{}, ta + 6);
            };
            for (; ta + NSLOT - 2 < fast_end && ta + 2 * NSLOT - 2 < n_full; ta += NSLOT) turn(T{});
            for (; ta + NSLOT - 2 < fast_end; ta += NSLOT) turn(F{});
            int ph = 0;
            auto next = [&]() __attribute__((always_inline)) {
                ta += 2;
                ph = ph + 2 == NSLOT ? 0 : ph + 2;
            };
            for (; ta < fast_end; next()) direct_iteration(active, T{}, F{}, ph, ta);
            for (; ta < n; next()) direct_iteration(active, F{}, F{}, ph, ta);
        } else {
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
        }
    };
    // Waves without rows only copy, in loops of their own. (Through registers all waves pass the same code: four waves of 128 channels
    // run out of registers otherwise, 32 x 60 nodes of 32 / 32 heads, 3136 keys 304 -> 377 us, and are bound by memory.)
    if constexpr (!DIRECT) all_tiles(wave_active);
    else if (wave_active) all_tiles(T{});
    else all_tiles(F{});
    if (wave_active) {
    if ((n & 1) == 0) pv((n - 1) % NSLOT, pb);

    // ---- epilogue: lane (col, half) holds, for row `col`, channels db*32 + 8*(r/4) + 4*half + r%4
    // (what depends on the lane alone is worked out again: kept over the loop it takes registers)
    int tid_end = threadIdx.x;
    asm volatile("" : "+v"(tid_end));
    const int lane = tid_end & 63, half = lane >> 5, col = lane & 31;
#pragma unroll
    for (int rb = 0; rb < RPW; ++rb) {
        const float l = half_sum(lsum[rb] + lsum2[rb]);
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
        run_piece(b, kvh, rg, split * p.keys_per_split, p.keys_per_split, split, p.num_splits == 1, 0);
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
        __shared__ int32_t s_start[NW][kBalMaxSeqs], s_len[NW][kBalMaxSeqs], s_bounds[NW][kBalMaxChunks + 1];
        s_start[wave][lane] = start;
        s_len[wave][lane] = S;
        s_bounds[wave][lane] = lane < p.bal_chunks ? bounds : total;
        if (lane == 0) s_bounds[wave][kBalMaxChunks] = total;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup"); // read by all lanes of this wave
        int p0, p1;
        const uint64_t pieces = __ballot(bal_piece(lo, hi, start, steps, p0, p1));
        const uint64_t shared = __ballot(bal_piece(lo, hi, start, steps, p0, p1) && !(p0 == 0 && p1 == steps)); // others have the rest
        if (has_rows && ((shared >> lane) & 1)) arrival_open(words + lane, seen);
        for (uint64_t left = pieces; left != 0; left &= left - 1) { // in the order of the line
            const int i = __builtin_ctzll(left);
            const int len = __builtin_amdgcn_readfirstlane(s_len[wave][i]);
            const int s0 = __builtin_amdgcn_readfirstlane(s_start[wave][i]), t = bal_steps(p, len);
            int t0, t1;
            bal_piece(lo, hi, s0, t, t0, t1);
            __syncthreads(); // the previous piece's last reads of the tile rings, the tree and the flag
            run_piece(i, kvh, rg, t0 * kIterKeys, (t1 - t0) * kIterKeys, c + i, ((shared >> i) & 1) == 0, len);
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
            const int s0 = __builtin_amdgcn_readfirstlane(s_start[wave][i]), t = bal_steps(p, __builtin_amdgcn_readfirstlane(s_len[wave][i]));
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

template <int D, int RPW, int NW, bool BAL, bool MAY>
void launch_pipe(const AttnParams& p, dim3 grid, hipStream_t s) {
    if (p.once) hipLaunchKernelGGL((attn_mfma_pipe_kernel<D, RPW, NW, false, BAL, MAY>), grid, dim3(NW * kWave), 0, s, p);
    else if (p.paged) hipLaunchKernelGGL((attn_mfma_pipe_kernel<D, RPW, NW, true, BAL, false>), grid, dim3(NW * kWave), 0, s, p);
    else hipLaunchKernelGGL((attn_mfma_pipe_kernel<D, RPW, NW, false, BAL, false>), grid, dim3(NW * kWave), 0, s, p);
}
template <int D, int RPW, int NW>
hipError_t launch_pipe(const AttnParams& p, hipStream_t s) {
    constexpr bool MAY = NW == 4; // eight waves gain 1 - 2 % from it where they are one row group, and lose 3 - 5 % where they are two
    if (p.once && (p.paged || !MAY)) return hipErrorInvalidValue;
    if (p.bal_chunks > 0) {
        const dim3 grid(((p.bal_chunks * p.Hkv + 7) / 8) * 8 * p.row_groups);
        launch_pipe<D, RPW, NW, true, MAY>(p, grid, s);
    } else {
        const dim3 grid(p.by_length ? (p.B * p.Hkv + 7) / 8 * 8 * p.row_groups : (p.total_wgs + 7) / 8 * 8);
        launch_pipe<D, RPW, NW, false, MAY>(p, grid, s);
    }
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
