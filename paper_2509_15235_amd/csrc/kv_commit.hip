// Commit of the accepted path into the pre-allocated KV cache (paper Section 3.1: draft
// tokens after the first rejected one are discarded; Appendix A: the cache is allocated
// once, so keeping the accepted tokens means moving their rows inside it).
//
// Node path[k]'s row sits at logical slot S + path[k] and has to end up at slot S + k.
// One thread owns one 16-byte piece of a (layer, KV head, K-or-V) row position and moves it
// for k = 1 .. accepted_len in ascending order. Since path[k] >= k, no source is
// overwritten before it is read, whatever the other threads do: pieces never overlap
// between threads. Up to eight moves are in flight per thread (all loads, then all stores),
// which keeps the ascending order where it matters: a batch's destinations lie below the
// next batch's sources.
//
// A workgroup serves one sequence: every wave of it checks the path, the prefix length and (paged) the
// block-table entries of every slot it may touch before anything moves; a sequence that
// fails a check is reported through `status`, keeps its cache and its prefix length.
//
// Bound by latency: arguments, then path and lengths, then (paged) block ids, then rows, one trip to memory behind another.
// So a lane holds a node's path entry and a block id - no LDS, no barrier, no second look at the table for a row - and
// every trip is asked for before the last one's answer is looked at.
// us, commits in a graph, before (path and flags in LDS, loads one at a time) / so: 28 layers of 4 heads, 4 accepted 2.88 / 2.13;
// 4 sequences, 32 layers of 32 heads, up to 1 accepted 2.96 / 2.39; 6 sequences paged, up to 3 accepted 3.41 / 2.27; 13 other steps
// 0.70 - 0.98, geometric mean of all 0.77. Nothing accepted 1.7 either way: launch, arguments and lengths.
#include "vs_device.h"

namespace vs {

namespace {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
constexpr int kCommitThreads = 256;
constexpr int kCommitBatch = 8;

template <bool PAGED>
__global__ __launch_bounds__(kCommitThreads) void kv_commit_kernel(const CommitParams p) {
    request_args(p);
    const int b = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63;
    const int32_t node = p.path[(int64_t)b * p.T + min(lane, p.T - 1)];
    int32_t S = p.prefix_len[b], alen = p.accepted_len[b];
    // ---- this thread's piece: (layer, K or V, KV head, 16-byte chunk of the row). A wave's lanes past the last piece stay, since
    // path and block ids are read from lanes, whose registers nobody keeps up once they have left: they do what the last piece's lane, one of the
    // same wave, does in the same instructions. (Without their stores 1 - 6 % slower.)
    const int64_t own = (int64_t)blockIdx.x * kCommitThreads + tid, item = min(own, p.items_per_seq - 1);
    int64_t layer;
    uint32_t chunk, kvh, which;
    if (p.items_per_seq <= 0xffffffffll) { // (the 45 instructions of a division, three times, stood between the checks and the rows)
        const uint32_t pair = fast_div(fast_div((uint32_t)item, p.by_chunks, chunk), p.by_heads, kvh);
        which = pair & 1;
        layer = pair >> 1;
    } else {
        const int64_t head = item / p.chunks_per_row, pair = head / p.Hkv;
        chunk = (uint32_t)(item - head * p.chunks_per_row);
        kvh = (uint32_t)(head - pair * p.Hkv);
        which = pair & 1;
        layer = pair >> 1;
    }
    char* base = (char*)(which ? p.v : p.k) + layer * p.stride_layer_bytes + (int64_t)kvh * p.stride_head_bytes + (int64_t)chunk * 16;
    if (!PAGED) base += (int64_t)b * p.stride_seq_bytes;

    S = __builtin_amdgcn_readfirstlane(S); // the compiler does not know that the stores below change neither
    alen = __builtin_amdgcn_readfirstlane(alen);
    const int64_t have = PAGED ? (int64_t)p.max_blocks * p.block_size : p.capacity;
    const bool s_ok = S >= 0 && (int64_t)S + p.T <= have;
    const int first = S >> p.block_shift; // the blocks that the T slots touch, a lane each (blocks have 16 slots or more)
    int32_t blk = 0;
    if (PAGED && s_ok && lane <= ((S + p.T - 1) >> p.block_shift) - first) blk = p.block_table[(int64_t)b * p.max_blocks + first + lane];

    // ---- checks
    const bool alen_ok = alen >= 0 && alen < p.T;
    const int32_t before = (int32_t)dpp<0x138>((uint32_t)node); // of the lane below
    const bool node_ok = lane == 0 ? node == 0 : node > before && node < p.T;
    int32_t code = VS_STATUS_OK;
    if (!alen_ok || __any(lane <= alen && !node_ok)) code = VS_STATUS_BAD_PATH;
    else if (!s_ok) code = VS_STATUS_BAD_PREFIX;
    else if (PAGED && __any((uint32_t)blk >= (uint32_t)p.num_blocks)) code = VS_STATUS_BAD_BLOCK;
    if (blockIdx.x == 0 && tid == 0) {
        if (p.status) p.status[b] = code;
        p.new_prefix_len[b] = code == VS_STATUS_OK ? S + alen + 1 : S;
    }
    if (code != VS_STATUS_OK || own - lane >= p.items_per_seq) return; // the whole wave

    auto row = [&](int32_t tok) -> char* { // tok is the same for all lanes
        if constexpr (PAGED) {
            const int64_t in = __builtin_amdgcn_readlane(blk, (tok >> p.block_shift) - first);
            return base + (in * p.stride_block_bytes + (int64_t)(tok & (p.block_size - 1)) * p.stride_tok_bytes);
        }
        return base + (int64_t)tok * p.stride_tok_bytes;
    };
    // N moves, of which those past the path's end read its last row and write nothing: loads behind a condition wait for one another,
    // since the compiler does not know which of their registers is still on its way
    const auto move = [&](auto count, int k0) {
        constexpr int N = decltype(count)::value;
        u32x4 r[N];
#pragma unroll
        for (int u = 0; u < N; ++u) r[u] = *(const u32x4*)row(S + __builtin_amdgcn_readlane(node, min(k0 + u, alen)));
        asm volatile("" ::: "memory"); // or a load sinks to the only place that needs it, behind a condition
#pragma unroll
        for (int u = 0; u < N; ++u)
            if (k0 + u <= alen && __builtin_amdgcn_readlane(node, k0 + u) != k0 + u) *(u32x4*)row(S + k0 + u) = r[u]; // the same for all lanes
    };
    int k0 = 1;
    for (; alen - k0 >= 4; k0 += kCommitBatch) move(std::integral_constant<int, kCommitBatch>{}, k0);
    if (alen - k0 >= 2) move(std::integral_constant<int, 4>{}, k0);
    else if (alen >= k0) move(std::integral_constant<int, 2>{}, k0);
}

} // namespace

hipError_t launch_kv_commit(const CommitParams& p, hipStream_t s) {
    const dim3 grid((unsigned)((p.items_per_seq + kCommitThreads - 1) / kCommitThreads), (unsigned)p.B);
    if (p.paged) hipLaunchKernelGGL(kv_commit_kernel<true>, grid, dim3(kCommitThreads), 0, s, p);
    else hipLaunchKernelGGL(kv_commit_kernel<false>, grid, dim3(kCommitThreads), 0, s, p);
    return hipGetLastError();
}

} // namespace vs
