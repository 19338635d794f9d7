// Tree-masked attention for fp32 storage on the fp32 matrix cores (paper Eq. 1 with a softmax scale,
// restricted to the keys a node may see: all prefix tokens + the tree slots of its ancestor-or-self
// set, Section 3.1). Products, sums and softmax are fp32 throughout.
//
// One workgroup of eight waves owns one or two sets of four query rows of one (sequence, KV head) and
// all of its keys; wave w takes the 16-key tiles w, w + 8, ... . v_mfma_f32_4x4x1_16b_f32 multiplies
// sixteen independent 4 x 4 blocks, and the blocks are laid out so that nothing moves between lanes:
//   lane = 16 * kb + 4 * cg + j       kb: four keys of the tile, cg: channels 4 cg .. 4 cg + 3 of every 16
//   scores   block (kb, cg) = keys 4 kb .. + 3 x query rows 0 .. 3 over the channels of cg; the four cg
//            blocks of a key group are added up with two row rotations (DPP)
//   output   block (kb, cg) = V's channels 16 cg + 4 i + e (register i of accumulator e) x query rows over
//            the keys of kb: the probabilities are the second operand as they stand. Every key group
//            keeps its own softmax reference, sum and accumulators; they meet at the end.
// V goes from memory straight into the operand registers (16-byte loads), K through a piece of LDS that is the
// wave's own (no barrier in the loop); the next tile's K is requested around the scores, its V after the output.
//
// Why four-row blocks: fp32 launches are small and there is no workspace, hence no key splits between
// workgroups; 16-row blocks would leave most CUs idle. With two sets a CU's matrix cores (128 instructions of
// 8 clocks per tile on four SIMDs: 256 clocks) take as long as its reads (16 KB per tile at 64 bytes per clock);
// one set per workgroup halves the matrix and vector work of a CU as long as that spreads the rows over CUs
// that would be idle otherwise (the host's choice).
// Before (one wave per row, plain fused multiply-adds): 2 x 31 nodes, 8 / 2 heads of 128 channels, 333 - 600
// keys 188 us; 8 nodes over 64 keys, 4 / 1 heads of 64 channels 19 us. Now 10.6 and 4.7 us.
#include "attn_mfma_common.h"

namespace vs {

namespace {

constexpr int kF32Waves = 8;
constexpr int kF32Tile = 16; // keys per tile
constexpr float kLazyF32 = 8.f; // log2 slack of the running softmax reference: weights stay below 2^8

// x summed over the four lanes of a 16-lane row that differ in bits 2 and 3
__device__ __forceinline__ float sum_cg(float x) {
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x124, 0xf, 0xf, false)); // row_ror:4
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x128, 0xf, 0xf, false)); // row_ror:8
    return x;
}

// x of lane J of every four
template <int J>
__device__ __forceinline__ uint32_t quad_lane(uint32_t x) { return dpp<J * 0x55>(x); }

// op over the sixteen lanes (kb, cg) that share j, in every lane
template <typename Op>
__device__ __forceinline__ float row_all(float x, Op op) {
    x = op(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x124, 0xf, 0xf, false)));
    x = op(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x128, 0xf, 0xf, false)));
    u32x2 w = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = op(__uint_as_float(w[0]), __uint_as_float(w[1]));
    w = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return op(__uint_as_float(w[0]), __uint_as_float(w[1]));
}

template <int D, int SETS, bool PAGED>
__global__ __launch_bounds__(kF32Waves * kWave, 2) void attn_f32_kernel(const AttnParams p) {
    request_args(p);
    constexpr int KJ = D / 16; // 16-byte pieces of a key row per lane
    constexpr int VM = D / 64; // ... of a value row
    constexpr int ROWS = 4 * SETS; // query rows of the workgroup
    constexpr int PITCH = D + 4; // floats per row of the exchange area (keeps its writes free of bank conflicts)
    constexpr int PARTS = kF32Waves * 4;

    __shared__ __attribute__((aligned(16))) float so[kF32Waves * ROWS * PITCH]; // the waves' results, [wave][row][channel]
    __shared__ __attribute__((aligned(16))) float sk[kF32Waves][kF32Tile * D];          // a key tile per wave
    __shared__ float sm[SETS][PARTS][4], sl[SETS][PARTS][4];             // references and sums
    __shared__ int32_t sp[VS_MAX_TREE];
    __shared__ int32_t sflag;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kb = lane >> 4, cg = (lane >> 2) & 3, j = lane & 3;

    // the row groups of a unit run on one XCD and share its L2 (one split)
    const WorkItem at = work_item(p);
    if (at.none) return;
    const int rg = at.rg, kvh = at.kvh, b = at.b;

    const int32_t S = p.prefix_len[b]; // requested first; the first tile and the queries do not wait for it
    const int64_t cache_tokens = PAGED ? (int64_t)p.max_blocks * p.block_size : p.capacity;
    const int last_slot = (int)(cache_tokens < (int64_t)p.max_prefix_len + p.tree_keys ? cache_tokens : (int64_t)p.max_prefix_len + p.tree_keys) - 1;
    const float* kbase = (const float*)p.k + (int64_t)kvh * p.stride_head + (PAGED ? 0 : (int64_t)b * p.stride_seq);
    const float* vbase = (const float*)p.v + (int64_t)kvh * p.stride_head + (PAGED ? 0 : (int64_t)b * p.stride_seq);

    f32x4 kf[KJ], vf[4][VM];
    // first slot of the tile and the largest slot that may be read, both uniform: base address and clamp
    auto tile_base = [&](int t0, int last, int64_t& base, int& lim) __attribute__((always_inline)) {
        const int t = min(t0, last & ~(kF32Tile - 1)); // a tile past the end repeats the last one (finite, unused)
        base = 0;
        int in = t;
        if (PAGED) { // blocks hold a multiple of 16 slots, so a tile lies in one
            int32_t blk = p.block_table[(int64_t)b * p.max_blocks + (t >> p.block_shift)];
            if ((uint32_t)blk >= (uint32_t)p.num_blocks) blk = 0; // reported through status
            base = (int64_t)blk * p.stride_block;
            in = t & (p.block_size - 1);
        }
        base += (int64_t)in * p.stride_tok;
        lim = last - t; // >= 0
    };
    // K: a load instruction fetches KPI whole key rows, lane q -> row q / CPR, 16-byte chunk q % CPR
    constexpr int CPR = D / 4, KPI = 64 / CPR;
    const int krow = lane / CPR, kchunk = lane % CPR;
    // this lane's key row and value row 0 of a full tile; a ragged one clamps every row
    const int64_t k_lane = (int64_t)krow * p.stride_tok + 4 * kchunk;
    const int64_t v_lane = (int64_t)(4 * kb) * p.stride_tok + 4 * (lane & 15);
    auto load_k = [&](int t0, int last) __attribute__((always_inline)) {
        int64_t base;
        int lim;
        tile_base(t0, last, base, lim);
        if (lim >= kF32Tile - 1) {
#pragma unroll
            for (int i = 0; i < KJ; ++i) kf[i] = *(const f32x4*)(kbase + (base + KPI * i * p.stride_tok) + k_lane);
        } else {
#pragma unroll
            for (int i = 0; i < KJ; ++i)
                kf[i] = *(const f32x4*)(kbase + base + (int64_t)min(KPI * i + krow, lim) * p.stride_tok + 4 * kchunk);
        }
    };
    auto load_v = [&](int t0, int last) __attribute__((always_inline)) {
        int64_t base;
        int lim;
        tile_base(t0, last, base, lim);
        if (lim >= kF32Tile - 1) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int m = 0; m < VM; ++m) vf[r][m] = *(const f32x4*)(vbase + (base + r * p.stride_tok) + v_lane + 64 * m);
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int m = 0; m < VM; ++m)
                    vf[r][m] = *(const f32x4*)(vbase + base + (int64_t)min(4 * kb + r, lim) * p.stride_tok + 64 * m + 4 * (lane & 15));
        }
    };
    load_k(kF32Tile * wave, last_slot);

    // queries: set s, row rg * 8 + 4 s + j; rows past the end repeat the last one (results discarded)
    f32x4 qf[SETS][KJ];
    int row_of[SETS], node[SETS];
#pragma unroll
    for (int s = 0; s < SETS; ++s) row_of[s] = min(rg * ROWS + 4 * s + j, p.rows - 1);
    row_nodes(p, row_of, node);
#pragma unroll
    for (int s = 0; s < SETS; ++s) {
        const float* q = (const float*)p.q + row_start<D>(p, b, kvh) + (uint64_t)row_number(row_of[s], node[s], p.row_skip) * (uint32_t)D + 4 * cg;
#pragma unroll
        for (int i = 0; i < KJ; ++i) qf[s][i] = *(const f32x4*)(q + 16 * i);
    }
    uint64_t mask[SETS];
    const bool given = p.tree_mask && p.tree_keys != 0;
#pragma unroll
    for (int s = 0; s < SETS; ++s) mask[s] = given ? p.tree_mask[(int64_t)b * p.T + node[s]] : 0ull;
    load_v(kF32Tile * wave, last_slot);

    int32_t tree_code = VS_STATUS_OK;
    if (p.tree_mask || p.tree_keys == 0) {
        if (tid == 0) sflag = 0;
        __syncthreads();
    } else {
        tree_code = load_tree(p.parent + (int64_t)b * p.T, p.T, sp, &sflag);
    }
    const bool s_ok = prefix_ok(p, S);
    if (kvh == 0 && rg == 0) report_status(p, b, tree_code, s_ok, S, &sflag);
    if (tree_code != VS_STATUS_OK || !s_ok) return;
    if (!given && p.tree_keys != 0) {
#pragma unroll
        for (int s = 0; s < SETS; ++s) mask[s] = ancestor_mask(sp, node[s]);
    }

    const int n = S + p.tree_keys;
    float m2[SETS], l[SETS]; // reference (log2 domain, scaled) and sum of this lane's key group and row
    f32x4 acc[SETS][VM][4];
#pragma unroll
    for (int s = 0; s < SETS; ++s) {
        m2[s] = -INFINITY;
        l[s] = 0.f;
#pragma unroll
        for (int m = 0; m < VM; ++m)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[s][m][e] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    for (int t0 = kF32Tile * wave; t0 < n; t0 += kF32Tile * kF32Waves) {
        f32x4 sc[SETS][2]; // two chains per set
#pragma unroll
        for (int s = 0; s < SETS; ++s)
#pragma unroll
            for (int c = 0; c < 2; ++c) sc[s][c] = f32x4{0.f, 0.f, 0.f, 0.f};
        // K through this wave's LDS area (the operand wants neighbouring lanes on different keys: read like
        // that from memory, every four lanes touch four cache lines and the address units take four times as
        // long). Chunk c of key r sits at position c ^ 4 (r % 4): writes and reads are free of bank conflicts.
#pragma unroll
        for (int i = 0; i < KJ; ++i) {
            const int r = KPI * i + krow;
            *(f32x4*)(sk[wave] + r * D + 4 * (kchunk ^ (4 * (r & 3)))) = kf[i];
        }
        if (SETS == 1 && t0 + kF32Tile * kF32Waves < n) load_k(t0 + kF32Tile * kF32Waves, n - 1);
        f32x4 ka[KJ];
#pragma unroll
        for (int i = 0; i < KJ; ++i) ka[i] = *(const f32x4*)(sk[wave] + (4 * kb + j) * D + 4 * ((4 * i + cg) ^ (4 * j)));
#pragma unroll
        for (int i = 0; i < KJ; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int s = 0; s < SETS; ++s)
                    sc[s][e & 1] = __builtin_amdgcn_mfma_f32_4x4x1f32(ka[i][e], qf[s][i][e], sc[s][e & 1], 0, 0, 0);

        // (two sets: the registers of the next tile are free only now)
        if (SETS == 2 && t0 + kF32Tile * kF32Waves < n) load_k(t0 + kF32Tile * kF32Waves, n - 1);

        float pr[SETS][4];
#pragma unroll
        for (int s = 0; s < SETS; ++s) {
            float x[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) x[r] = sum_cg(sc[s][0][r] + sc[s][1][r]) * p.scale_log2;
            if (t0 + kF32Tile > S) { // uniform: tree slots or the end of the range
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int sh = t0 + 4 * kb + r - S; // tree slot of the key (negative: prefix)
                    // (no short-circuit operators: as branches, the compiler lost one of the assignments)
                    const uint32_t bit = (uint32_t)(mask[s] >> (sh & 63)) & 1u;
                    const bool vis = (sh < 0) | ((sh < p.tree_keys) & (bit != 0));
                    x[r] = vis ? x[r] : -INFINITY;
                }
            }
            const float mx = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
            const float m_new = mx > m2[s] + kLazyF32 ? mx : m2[s]; // the reference moves in large steps only
            const float m_use = m_new == -INFINITY ? 0.f : m_new; // no visible key yet: every weight is 2^-inf = 0
            const float alpha = __builtin_amdgcn_exp2f(m2[s] - m_use);
            float sum = 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                pr[s][r] = __builtin_amdgcn_exp2f(x[r] - m_use);
                sum += pr[s][r];
            }
            l[s] = l[s] * alpha + sum;
            if (__any(m_new != m2[s])) {
#pragma unroll
                for (int m = 0; m < VM; ++m)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[s][m][e] *= alpha;
            }
            m2[s] = m_new;
        }
        if (t0 + kF32Tile > n) { // slots past the last key: whatever they hold must not meet a zero weight
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int m = 0; m < VM; ++m)
#pragma unroll
                    for (int e = 0; e < 4; ++e) vf[r][m][e] = t0 + 4 * kb + r < n ? vf[r][m][e] : 0.f;
        }
        // A value that is not finite must not meet the zero weight of a row that does not see its key. Only tree slots are hidden
        // from some rows: where one of their tiles holds such a value, the rows that see it get it here and the product a zero.
        if (t0 + kF32Tile > S) { // uniform
            f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int m = 0; m < VM; ++m)
#pragma unroll
                    for (int e = 0; e < 4; ++e) z[e] = fmaf(vf[r][m][e], 0.f, z[e]);
            const float any = (z[0] + z[1]) + (z[2] + z[3]);
            if (__builtin_expect(__any(any != any), 0)) {
                auto infinite = [](float x) { return !(fabsf(x) < INFINITY); }; // or NaN
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int sh = t0 + 4 * kb + r - S;
                    bool sees[SETS]; // this lane's row
#pragma unroll
                    for (int s = 0; s < SETS; ++s) sees[s] = (sh < 0) | ((sh < p.tree_keys) & (((uint32_t)(mask[s] >> (sh & 63)) & 1u) != 0));
#pragma unroll
                    for (int m = 0; m < VM; ++m)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const uint32_t raw = __float_as_uint(vf[r][m][e]);
                            auto channel = [&](int i, uint32_t bits) __attribute__((always_inline)) { // register i holds the channel that lane i of four fetched
                                const float x = __uint_as_float(bits);
#pragma unroll
                                for (int s = 0; s < SETS; ++s)
                                    if (infinite(x) && sees[s]) acc[s][m][e][i] = fmaf(x, pr[s][r], acc[s][m][e][i]);
                            };
                            channel(0, quad_lane<0>(raw));
                            channel(1, quad_lane<1>(raw));
                            channel(2, quad_lane<2>(raw));
                            channel(3, quad_lane<3>(raw));
                            if (infinite(vf[r][m][e])) vf[r][m][e] = 0.f;
                        }
                }
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int m = 0; m < VM; ++m)
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int s = 0; s < SETS; ++s)
                        acc[s][m][e] = __builtin_amdgcn_mfma_f32_4x4x1f32(vf[r][m][e], pr[s][r], acc[s][m][e], 0, 0, 0);
        if (t0 + kF32Tile * kF32Waves < n) load_v(t0 + kF32Tile * kF32Waves, n - 1);
    }

    // ---- merge the key groups of all waves (log-sum-exp): everybody scales by the common reference and
    // sum, the four key groups of a wave are added up in registers, the waves through LDS
    if (cg == 0) {
#pragma unroll
        for (int s = 0; s < SETS; ++s) {
            sm[s][4 * wave + kb][j] = m2[s];
            sl[s][4 * wave + kb][j] = l[s];
        }
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < SETS; ++s) {
        // two parts per lane of a row: 16 lanes (kb, cg) x 2
        const int q = 2 * (4 * kb + cg);
        const float ma = sm[s][q][j], mb = sm[s][q + 1][j];
        float M = row_all(fmaxf(ma, mb), [](float x, float y) { return fmaxf(x, y); }); // finite: a node sees itself or the prefix
        const float den = row_all(sl[s][q][j] * __builtin_amdgcn_exp2f(ma - M) + sl[s][q + 1][j] * __builtin_amdgcn_exp2f(mb - M),
                                  [](float x, float y) { return x + y; });
        const float f = __builtin_amdgcn_exp2f(m2[s] - M) / den;
        // registers in the order of their channels: 16 VM of them, halved twice
        float x[16 * VM];
#pragma unroll
        for (int m = 0; m < VM; ++m)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) x[16 * m + 4 * i + e] = acc[s][m][e][i] * f;
        // lower / upper half of the lanes keep the first / second half of the registers, then even / odd rows
#pragma unroll
        for (int i = 0; i < 8 * VM; ++i) {
            const u32x2 w = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[i]), __float_as_uint(x[i + 8 * VM]), false, false);
            x[i] = __uint_as_float(w[0]) + __uint_as_float(w[1]);
        }
#pragma unroll
        for (int i = 0; i < 4 * VM; ++i) {
            const u32x2 w = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[i]), __float_as_uint(x[i + 4 * VM]), false, false);
            x[i] = __uint_as_float(w[0]) + __uint_as_float(w[1]);
        }
        // channels (register 16 m + 4 i + e, lane): 64 m + 16 cg + 4 i + e
        const int ch = VM == 2 ? 64 * (kb >> 1) + 16 * cg + 8 * (kb & 1) : 16 * cg + 4 * kb;
#pragma unroll
        for (int i = 0; i < VM; ++i)
            *(f32x4*)(so + ((wave * SETS + s) * 4 + j) * PITCH + ch + 4 * i) = f32x4{x[4 * i], x[4 * i + 1], x[4 * i + 2], x[4 * i + 3]};
    }
    __syncthreads();
    constexpr int CPT = ROWS * D > kF32Waves * kWave ? 2 : 1; // channels per thread
    if (ROWS * D < kF32Waves * kWave && tid >= ROWS * D) return;
    const int row = tid * CPT / D, c = tid * CPT % D;
    const int r = rg * ROWS + row;
    if (r < p.rows) {
        float o[CPT];
#pragma unroll
        for (int e = 0; e < CPT; ++e) o[e] = 0.f;
#pragma unroll
        for (int w = 0; w < kF32Waves; ++w) // waves without a tile hold zeros
#pragma unroll
            for (int e = 0; e < CPT; ++e) o[e] += so[(w * ROWS + row) * PITCH + c + e];
        float* dst = (float*)p.out + row_start<D>(p, b, kvh) + (uint64_t)row_number(r, row_node(p, r), p.row_skip) * (uint32_t)D + c;
#pragma unroll
        for (int e = 0; e < CPT; ++e) dst[e] = o[e];
    }
}

template <int D, int SETS>
hipError_t launch_f32(const AttnParams& p, hipStream_t s) {
    const dim3 grid((p.total_wgs + 7) / 8 * 8), block(kF32Waves * kWave);
    if (p.paged) hipLaunchKernelGGL((attn_f32_kernel<D, SETS, true>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((attn_f32_kernel<D, SETS, false>), grid, block, 0, s, p);
    return hipGetLastError();
}

} // namespace

hipError_t launch_attention_f32(const AttnParams& p, hipStream_t s) {
    if (p.rows_per_group == 4) return p.d == 128 ? launch_f32<128, 1>(p, s) : launch_f32<64, 1>(p, s);
    return p.d == 128 ? launch_f32<128, 2>(p, s) : launch_f32<64, 2>(p, s);
}

} // namespace vs
