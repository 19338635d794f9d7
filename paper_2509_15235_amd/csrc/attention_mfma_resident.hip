// Tree-masked attention for small launches (one layer of one sequence, short sequences): the whole key range of a
// split (at most 192 keys, 256 with one or two row blocks) is resident in LDS, and the workgroup's waves share first the keys and then the channels.
//
// Math and MFMA layouts are those of attention_mfma.hip (paper Eq. 1 with a softmax scale over the prefix plus the
// ancestor-or-self tree slots, Section 3.1): S^T = K . Q^T with v_mfma_f32_32x32x16_bf16, a lane holds 16 keys of
// ONE query row, the probabilities are the B operand of O^T += V^T . P^T, V is transposed by ds_read_b64_tr_b16 on its
// way out of LDS.
//
// What bounds it: latency. Every wave runs its instructions once, one after the other, at 8 to 10 cycles each (a
// dependent vector instruction 8.5, a scalar one 8.4, an independent vector one 5.5, instructions fetched for the first
// time 2 more), so 250 of them are a microsecond; the matrix cores work for 0.3 us of ten.
// Hence: eight waves = NRB row blocks x KQ key parts. A wave scores its row block against its part of the keys and writes
// the probabilities, relative to the part's own maximum, to LDS as ready-made operands (1 KB per 16 keys, read back
// by lane); then it multiplies ALL keys with its share of the channels, part by part. Exchanging probabilities takes
// a third of the instructions of exchanging accumulators (a form that did: 0.8 us to hand them over, 1.0 to add
// them up and store). Keys are requested before the queries, values last: they arrive while the scores are
// worked out. What can be had without the sequence's length is requested before it arrives.
// (One reference for all parts would save the weights at the end, but a probability of 1 is exact in bf16, and the
// largest of every part being so is worth 2 - 4 % of the error.)
#include <type_traits>

#include "attn_mfma_common.h"

namespace vs {

namespace {

constexpr int kResWaves = 8;

template <int D, int NRB, int NT, bool PAGED>
__global__ __launch_bounds__(kResWaves * 64, 2) void attn_mfma_resident_kernel(const AttnParams p) {
    request_args(p);
    constexpr int KS = D / 16;          // k-steps of the S^T product
    constexpr int DB = D / 32;          // 32-channel blocks of the output
    constexpr int KQ = kResWaves / NRB; // key parts inside the workgroup
    constexpr int PPM = (NT + KQ - 1) / KQ; // tiles per key part: j * KQ + part
    constexpr int OWN = KQ < DB ? KQ : DB;  // waves of a row block that have channels
    constexpr int DBW = DB / OWN;           // their channel blocks each
    constexpr int SUB = kTileKeys * D;  // elements per 32-key tile of K (or V)
    constexpr int LPR = D / 8;          // lanes (16-byte chunks) per row
    constexpr int RPI = 64 / LPR;       // rows per load instruction
    constexpr int RPB = RPI * kResWaves; // rows that one load instruction of every wave fetches
    constexpr int NB = NT * kTileKeys / RPB; // such loads per tensor
    constexpr int P_ELEMS = NRB * NT * 1024;  // probabilities: [row block][tile][16-key half][64 lanes][8]
    constexpr int Q_AT = 2 * NT * SUB, Q_ELEMS = NRB * kRowBlock * D;
    constexpr bool P_OVER_K = (Q_AT + Q_ELEMS + P_ELEMS) * 2 + 8192 > kLdsBytesPerCU; // 192 keys, four row blocks of 128 channels
    constexpr int P_AT = P_OVER_K ? 0 : Q_AT + Q_ELEMS;
    constexpr int SMEM_ELEMS = Q_AT + Q_ELEMS + (P_OVER_K ? 0 : P_ELEMS);
    static_assert(NT * kTileKeys <= resident_max_keys(NRB) && NB * RPB == NT * kTileKeys, "keys of a split");
    static_assert(DB % OWN == 0 && (!P_OVER_K || P_ELEMS <= NT * SUB) && SMEM_ELEMS * 2 + 8192 <= kLdsBytesPerCU, "LDS");

    // K[t] at smem + t * SUB, V[t] at smem + (NT + t) * SUB, behind them the queries: row blocks of D-channel rows
    __shared__ __attribute__((aligned(1024))) uint16_t smem[SMEM_ELEMS];
    __shared__ float s_max[NRB][KQ][kRowBlock], s_sum[NRB][KQ][kRowBlock]; // every part's maxima and sums
    __shared__ int32_t sp[VS_MAX_TREE];
    __shared__ int32_t sflag;
    uint16_t* sK = smem;
    uint16_t* sV = smem + NT * SUB;
    uint16_t* sQ = smem + Q_AT;
    uint16_t* sP = smem + P_AT;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5;
    const int col = lane & 31;
    const int rbw = wave % NRB; // row block inside the group
    const int kq = wave / NRB;  // key part

    const WorkItem at = work_item(p);
    if (at.none) return;
    const int b = at.b, kvh = at.kvh, rg = at.rg, split = at.split;

    const int32_t S = p.prefix_len[b]; // requested first, needed last: everything below is issued before it arrives

    // ---- request the split's keys. Load u of wave w fetches rows u * RPB + w * RPI .. + RPI - 1 of the split, 1 KB of
    // consecutive memory. The loads do not wait for the prefix length: they are bounded by the longest sequence that the host
    // allows (paged: by the block table). A block-table entry outside the pool reads block 0 (reported through status).
    const uint16_t* kbase = (const uint16_t*)p.k;
    const uint16_t* vbase = (const uint16_t*)p.v;
    const int lrow = lane / LPR, lchunk = lane % LPR;
    const int k0 = split * p.keys_per_split; // the host keeps k0 below max_prefix_len + tree_keys, hence inside the cache
    const int64_t head_base = (PAGED ? 0 : (int64_t)b * p.stride_seq) + (int64_t)kvh * p.stride_head;
    const uint32_t stride = (uint32_t)p.stride_tok * 2u; // bytes; the host keeps a slice's offsets below 2^31 bytes
    u32x4 kreg[NB], vreg[NB];
    int64_t blk_base[PAGED ? NB : 1];
    uint32_t lane_off;
    if constexpr (PAGED) {
        // the RPI rows of a load lie in one cache block; past the table's last rows those are read again
        int32_t id[NB];
        int r0[NB];
        const int64_t cache_tokens = (int64_t)p.max_blocks * p.block_size, end = (int64_t)k0 + NT * kTileKeys;
        const int last = (int)(cache_tokens < end ? cache_tokens : end) - RPI;
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            r0[u] = min(k0 + u * RPB + wave * RPI, last);
            id[u] = p.block_table[(int64_t)b * p.max_blocks + (r0[u] >> p.block_shift)];
        }
        lane_off = (uint32_t)lrow * stride + lchunk * 16;
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int32_t blk = (uint32_t)id[u] < (uint32_t)p.num_blocks ? id[u] : 0;
            blk_base[u] = ((int64_t)blk * p.stride_block + head_base) * 2 + (uint32_t)(r0[u] & (p.block_size - 1)) * stride;
            kreg[u] = *(const u32x4*)((const char*)kbase + blk_base[u] + lane_off);
        }
    } else {
        lane_off = (uint32_t)(wave * RPI + lrow) * stride + lchunk * 16;
    }
    // contiguous caches: rows past the longest allowed sequence read as zeros
    const __amdgpu_buffer_rsrc_t krs = slice_of(kbase + head_base, k0, p, stride), vrs = slice_of(vbase + head_base, k0, p, stride);
    if constexpr (!PAGED) {
#pragma unroll
        for (int u = 0; u < NB; ++u)
            kreg[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(krs, lane_off + (uint32_t)(u * RPB) * stride, 0, 0));
    }
    // ---- this wave's share of its row block's queries
    const int row_base = rg * (NRB * kRowBlock) + rbw * kRowBlock;
    const bool wave_active = row_base < p.rows;
    constexpr int QPW = (KS + KQ - 1) / KQ; // pieces per wave
    u32x4 qreg[QPW];
    load_q_pieces<D>(p, b, kvh, [&](int) { return row_base; }, [&](int i) { return min(kq * QPW + i, KS - 1); }, lane, qreg);
    // the gate of the row group (thread 0 opens it below)
    uint64_t* const gate = p.gates ? p.gates + kGateWords * (int64_t)((b * p.Hkv + kvh) * p.row_groups + rg) : nullptr;
    uint64_t seen = 0;
    if (p.gates && wave == 0) seen = gate_load(gate);
    // the row's ancestor mask, when the caller supplies the masks
    const int r = min(row_base + col, p.rows - 1); // rows past the end repeat the last row (results discarded)
    const int node = row_node(p, r);
    uint64_t mask = 0;
    if (p.tree_mask && p.tree_keys != 0) mask = p.tree_mask[(int64_t)b * p.T + node];
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        if constexpr (PAGED) vreg[u] = *(const u32x4*)((const char*)vbase + blk_base[u] + lane_off);
        else vreg[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(vrs, lane_off + (uint32_t)(u * RPB) * stride, 0, 0));
    }

    const bool reports = kvh == 0 && split == 0 && rg == 0;
    int32_t tree_code = VS_STATUS_OK;
    if (!p.tree_mask && p.tree_keys != 0) {
        tree_code = load_tree(p.parent + (int64_t)b * p.T, p.T, sp, &sflag);
        if (tree_code == VS_STATUS_OK) mask = ancestor_mask(sp, node);
    } else if (reports) {
        if (tid == 0) sflag = 0;
        __syncthreads();
    }
    const bool s_ok = prefix_ok(p, S);
    if (reports) report_status(p, b, tree_code, s_ok, S, &sflag);
    if (tree_code != VS_STATUS_OK || !s_ok) return;

    const int nk = S + p.tree_keys;
    if (k0 >= nk) return;
    const bool final_rows = p.num_splits == 1 || (p.gates && nk <= p.keys_per_split); // a sequence of one split has nothing to merge
    const bool merge = p.gates && !final_rows;
    if (merge && tid == 0) merge_open(gate, seen);
    const int k1 = min(nk, k0 + p.keys_per_split);

    // ---- keys and queries into LDS. Chunk c of tile row r lands where the fragment reads expect it (same placement as
    // the streaming kernels):
    //   K: ((r/16)*DB + c/4) * 1024 + (c%4) * 256 + ((r%16) ^ 4*(c%4)) * 16
    //   V: ((r/16)*DB + c/4) * 1024 + (4*(r%16) + c%4) * 16
    const int srow = wave * RPI + lrow, rr = srow & (kTileKeys - 1); // (RPB is a multiple of a tile)
    {
        const uint32_t ko = (uint32_t)((srow / kTileKeys) * (SUB * 2) + ((rr >> 4) * DB + (lchunk >> 2)) * 1024 + (lchunk & 3) * 256 + (((rr & 15) ^ (4 * (lchunk & 3))) * 16));
#pragma unroll
        for (int u = 0; u < NB; ++u) *(u32x4*)((char*)sK + ko + u * (RPB / kTileKeys * SUB * 2)) = kreg[u];
    }
#pragma unroll
    for (int i = 0; i < QPW; ++i) store_q_piece<D>(sQ + rbw * (kRowBlock * D), qreg[i], min(kq * QPW + i, KS - 1), lane);
    __syncthreads();

    // ---- S^T = K . Q^T of this wave's key part: lane (col, half) gets keys 8*(q/4) + 4*half + q%4 of row `col`
    f32x16 s[PPM];
    {
        const int k_lane[2] = {(col >> 4) * (DB * 512) + half * 128 + ((col & 15) ^ (4 * half)) * 8,
                               (col >> 4) * (DB * 512) + half * 128 + ((col & 15) ^ (8 + 4 * half)) * 8};
        bf16x8 qf[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[ks] = read_q_frag<D>(sQ + rbw * (kRowBlock * D), ks, col, half);
#pragma unroll
        for (int j = 0; j < PPM; ++j) {
#pragma unroll
            for (int q = 0; q < 16; ++q) s[j][q] = 0.f;
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int j = 0; j < PPM; ++j) {
                const uint16_t* kt = sK + min(j * KQ + kq, NT - 1) * SUB;
                const bf16x8 a = __builtin_bit_cast(bf16x8, *(const u32x4*)(kt + k_lane[ks & 1] + ks * 256));
                s[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[ks], s[j], 0, 0, 0);
            }
    }
    // the values have arrived meanwhile; rows past the split's last key become zeros (whatever the cache holds there,
    // NaN included, must not meet a zero probability; a key of that kind only spoils its own score, which is masked)
    {
        const uint32_t vo = (uint32_t)((srow / kTileKeys) * (SUB * 2) + ((rr >> 4) * DB + (lchunk >> 2)) * 1024 + (4 * (rr & 15) + (lchunk & 3)) * 16);
        if (k0 + NT * kTileKeys > k1) { // uniform
            const u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int u = 0; u < NB; ++u) vreg[u] = k0 + u * RPB + srow < k1 ? vreg[u] : zero;
        }
#pragma unroll
        for (int u = 0; u < NB; ++u) *(u32x4*)((char*)sV + vo + u * (RPB / kTileKeys * SUB * 2)) = vreg[u];
    }
    // uniform: tree slots, the end of the range, or a last tile that this key part does not have
    if (k0 + NT * kTileKeys > min(S, k1) || (PPM - 1) * KQ + kq >= NT) {
#pragma unroll
        for (int j = 0; j < PPM; ++j) {
            const int first = k0 + (j * KQ + kq) * kTileKeys;
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
    const float m2 = half_max(mx) * p.scale_log2;    // this part's reference (log2 domain, scaled); -inf: no visible key in it
    const float m_use = m2 == -INFINITY ? 0.f : m2;
    if (P_OVER_K) __syncthreads(); // the keys have been read
    float ps0 = 0.f, ps1 = 0.f;
#pragma unroll
    for (int j = 0; j < PPM; ++j) {
#pragma unroll
        for (int q = 0; q < 16; q += 2) {
            s[j][q] = __builtin_amdgcn_exp2f(fmaf(s[j][q], p.scale_log2, -m_use)); // exp2(-inf) = 0
            s[j][q + 1] = __builtin_amdgcn_exp2f(fmaf(s[j][q + 1], p.scale_log2, -m_use));
            ps0 += s[j][q];
            ps1 += s[j][q + 1];
        }
        if (j * KQ + kq < NT) { // uniform; a part without this tile has added zeros
#pragma unroll
            for (int sl = 0; sl < 2; ++sl) {
                u32x4 w;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const f32x2 pr = {s[j][8 * sl + 2 * e], s[j][8 * sl + 2 * e + 1]};
                    w[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pr, bf16x2));
                }
                *(u32x4*)(sP + ((rbw * NT + j * KQ + kq) * 2 + sl) * 512 + lane * 8) = w;
            }
        }
    }
    const float psum = half_sum(ps0 + ps1);
    if (half == 0) {
        s_max[rbw][kq][col] = m2;
        s_sum[rbw][kq][col] = psum;
    }
    __syncthreads();

    // ---- O^T = V^T . P^T over all keys, for this wave's channel blocks; the rows leave as they are. Lane (col, half)
    // holds, for row `col`, channels db*32 + 8*(q/4) + 4*half + q%4.
    if (wave_active && kq < OWN) {
        const int t16 = lane & 15;
        const int v_lane = half * 128 + (t16 >> 2) * 32 + ((lane >> 4) & 1) * 16 + ((t16 >> 1) & 1) * 8 + (t16 & 1) * 4 + kq * (DBW * 512);
        float f[KQ], M = -INFINITY, l = 0.f; // the parts' weights, the rows' reference and sum
#pragma unroll
        for (int o = 0; o < KQ; ++o) {
            f[o] = s_max[rbw][o][col];
            M = fmaxf(M, f[o]);
        }
        const float Ms = M == -INFINITY ? 0.f : M; // no visible key in this split: every weight is 2^-inf = 0
#pragma unroll
        for (int o = 0; o < KQ; ++o) {
            f[o] = __builtin_amdgcn_exp2f(f[o] - Ms);
            l += f[o] * s_sum[rbw][o][col];
        }
        f32x16 acc[DBW], part[DBW];
#pragma unroll
        for (int o = 0; o < KQ && o < NT; ++o) {
#pragma unroll
            for (int db = 0; db < DBW; ++db)
#pragma unroll
                for (int q = 0; q < 16; ++q) part[db][q] = 0.f;
#pragma unroll
            for (int t = o; t < NT; t += KQ)
#pragma unroll
                for (int sl = 0; sl < 2; ++sl) {
                    const bf16x8 pf = __builtin_bit_cast(bf16x8, *(const u32x4*)(sP + ((rbw * NT + t) * 2 + sl) * 512 + lane * 8));
#pragma unroll
                    for (int db = 0; db < DBW; ++db) {
                        const uint16_t* vt = sV + t * SUB + sl * (DB * 512) + db * 512 + v_lane;
                        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)vt);
                        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vt + 256));
                        const bf16x8 a = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                        part[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pf, part[db], 0, 0, 0);
                    }
                }
#pragma unroll
            for (int db = 0; db < DBW; ++db)
#pragma unroll
                for (int q = 0; q < 16; ++q) acc[db][q] = o == 0 ? f[o] * part[db][q] : acc[db][q] + f[o] * part[db][q];
        }
        const float inv = l > 0.f ? 1.f / l : 0.f; // no visible key in this split (partials only): zeros, weight 0
        if (final_rows) {
            if (row_base + col < p.rows) {
                uint16_t* orow = (uint16_t*)p.out + row_offset(p, b, kvh, r, node) + kq * (DBW * 32) + 4 * half;
#pragma unroll
                for (int db = 0; db < DBW; ++db)
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4)
                        *(u32x2*)(orow + db * 32 + 8 * q4) = pack_partial(acc[db][4 * q4], acc[db][4 * q4 + 1], acc[db][4 * q4 + 2], acc[db][4 * q4 + 3], inv);
            }
        } else {
            const int64_t unit = (int64_t)b * p.Hkv + kvh;
            uint16_t* po = p.part_o + part_block<D>(p, unit, split, row_base >> 5) + piece_at(p, kq * DBW * 2);
#pragma unroll
            for (int db = 0; db < DBW; ++db) {
                if (merge) store_partial<true>(p, po, db, lane, acc[db], inv);
                else store_partial(p, po, db, lane, acc[db], inv);
            }
            if (kq == 0 && half == 0) {
                const f32x2 ml = {M, l};
                float* dst = p.part_ml + ml_block(p, unit, split, row_base >> 5) * 2;
                if (merge) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, ml), span_of(dst), col * 8, 0, kDeviceScope);
                else *(f32x2*)(dst + col * 2) = ml;
            }
        }
    }
    if (merge) {
        const int nrb = p.rows_pad / kRowBlock, rb0 = rg * NRB;
        merge_splits<D>(p, gate, b, kvh, rb0, min(rb0 + NRB, nrb), split, (nk + p.keys_per_split - 1) / p.keys_per_split, kResWaves,
                        (uint32_t*)sp);
    }
}

// NT = tiles per split (2, 4, 6 or 8 tiles of 32 keys)
template <int D, int NRB, bool PAGED>
hipError_t launch_res(const AttnParams& p, hipStream_t s) {
    const dim3 grid(((p.total_wgs + 7) / 8) * 8), block(kResWaves * kWave);
    const int nt = p.keys_per_split / kTileKeys;
    if (nt <= 2) hipLaunchKernelGGL((attn_mfma_resident_kernel<D, NRB, 2, PAGED>), grid, block, 0, s, p);
    else if (nt <= 4) hipLaunchKernelGGL((attn_mfma_resident_kernel<D, NRB, 4, PAGED>), grid, block, 0, s, p);
    else if (nt <= 6) hipLaunchKernelGGL((attn_mfma_resident_kernel<D, NRB, 6, PAGED>), grid, block, 0, s, p);
    else if constexpr (resident_max_keys(NRB) >= 8 * kTileKeys) hipLaunchKernelGGL((attn_mfma_resident_kernel<D, NRB, 8, PAGED>), grid, block, 0, s, p);
    return hipGetLastError();
}
template <int D, bool PAGED>
hipError_t launch_res_rb(const AttnParams& p, int row_blocks, hipStream_t s) {
    return row_blocks == 4 ? launch_res<D, 4, PAGED>(p, s) : row_blocks == 2 ? launch_res<D, 2, PAGED>(p, s) : launch_res<D, 1, PAGED>(p, s);
}

} // namespace

// Row blocks per workgroup: 4, 2 or 1 (the other waves split the keys).
bool attention_resident_supported(int row_blocks) { return row_blocks == 4 || row_blocks == 2 || row_blocks == 1; }

hipError_t launch_attention_mfma_resident(const AttnParams& p, int row_blocks, hipStream_t s) {
    if (!attention_resident_supported(row_blocks) || p.keys_per_split > resident_max_keys(row_blocks) || p.keys_per_split % kIterKeys) return hipErrorInvalidValue;
    if (p.d == 128) return p.paged ? launch_res_rb<128, true>(p, row_blocks, s) : launch_res_rb<128, false>(p, row_blocks, s);
    if (p.d == 64) return p.paged ? launch_res_rb<64, true>(p, row_blocks, s) : launch_res_rb<64, false>(p, row_blocks, s);
    return hipErrorInvalidValue;
}

} // namespace vs
