// What greedy and stochastic acceptance share: the scan of a logits row by workgroups of 8192 floats and the tree in
// registers. Each is two kernels, the scan and a walk of one workgroup per sequence.
// Chunks of 8192 floats on 512 threads: half as many results to merge as 4096 on 256 (16 x 60 x 152064 logits 99.1 -> 90.6 us greedy,
// 107 -> 97 stochastic; 4 x 31 x 32003 9.4 -> 8.4 and 14.3 -> 13.4). One kernel, the last workgroup of a sequence walking its
// tree, was 3 - 4 % faster still up to 256 workgroups and up to 60 % slower from 1024 on, where each lives longer than its loads
// take (pair acknowledged, counter, end): not worth a second form.
#pragma once

#include "vs_device.h"

namespace vs {

// Chunks of 4096 on 256 threads? For rows of at most one of them (half the waves), and where rows end in a short chunk (at most
// half of one), with two or eight chunks to a row, in launches of more than 1280 workgroups: with eight, ids dealt round-robin give
// all short ones to one XCD, with two the short ones are half of the launch. us, chunks of 8192 / of 4096, greedy and stochastic:
//   24 x 63 x 8960 16.3 / 13.8, 21.8 / 20.8; 30 x 60 x 12192 20.0 / 18.7, 26.8 / 26.0; 18 x 38 x 57509 30.9 / 28.7, 38.5 / 37.7
// Stochastic calls lose with the shorter ones elsewhere: 200 rows of 8292 .. 12192 0 - 6 %, three and more chunks 0 - 8 %.
inline bool scan_short_chunks(int32_t V, int64_t rows) {
    if (V <= kScanChunk / 2) return true;
    const int32_t chunks = (int32_t)(((int64_t)V + kScanChunk - 1) / kScanChunk), last = V - (chunks - 1) * kScanChunk;
    return (chunks == 2 || chunks == 8) && last <= kScanChunk / 2 && rows * chunks > 5 * kNumCUs;
}

// Workgroup id = row * chunks + chunk (the host keeps the product below 2^31); row counts over all sequences.
struct ScanItem {
    int row, chunk;
};
__device__ __forceinline__ ScanItem scan_item(FastDiv by_chunks) {
    uint32_t chunk;
    const uint32_t row = fast_div(blockIdx.x, by_chunks, chunk);
    return {(int)row, (int)chunk};
}

// A chunk of a row (THREADS: of the workgroup; a row of up to 4096 logits needs 256, and launches half as many waves): every
// thread has 16 entries and perhaps one of the up to three behind the last four.
struct ScanChunk {
    f32x4 a[kScanVec];
    float tail;
    int32_t begin, nvec, tail_at; // tail_at: >= end when this thread has none
};
template <int THREADS, int CHUNK = THREADS * kScanVec * 4>
__device__ __forceinline__ ScanChunk scan_load(const float* lg, int chunk, int V, int tid = threadIdx.x) {
    ScanChunk c;
    c.begin = chunk * CHUNK;
    const int end = V - c.begin < CHUNK ? V : c.begin + CHUNK;
    c.nvec = (end - c.begin) >> 2;
#pragma unroll
    for (int j = 0; j < kScanVec; ++j) {
        const int k = tid + j * THREADS;
        c.a[j] = k < c.nvec ? load4_stream(lg + c.begin + 4 * k) : f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    }
    c.tail_at = c.begin + 4 * c.nvec + tid;
    c.tail = c.tail_at < end ? lg[c.tail_at] : -INFINITY;
    if (c.tail_at >= end) c.tail_at = INT32_MAX;
    return c;
}

// The tree, a lane per node, in every wave that asks. Rows past the tree: parent -2.
__device__ __forceinline__ int32_t tree_lane(const int32_t* parent_row, int T) {
    const int lane = threadIdx.x & 63;
    const int32_t p = parent_row[lane < T ? lane : 0];
    return lane < T ? p : -2;
}
// parent[0] == -1, 0 <= parent[i] < i (the whole wave calls it)
__device__ __forceinline__ int32_t tree_check(int32_t parent, int T) {
    const int lane = threadIdx.x & 63;
    const bool bad_root = lane == 0 && parent != -1, bad_parent = lane > 0 && lane < T && (parent < 0 || parent >= lane);
    return __ballot(bad_root) ? VS_STATUS_BAD_ROOT : (__ballot(bad_parent) ? VS_STATUS_BAD_PARENT : VS_STATUS_OK);
}
// lane k <= alen: the ancestor of `node` at depth k (node's own depth is alen); others -1
__device__ __forceinline__ int32_t tree_path(int32_t parent, int node, int alen) {
    const int lane = threadIdx.x & 63;
    int32_t path = -1;
    for (int k = alen; k >= 0; --k) {
        if (lane == k) path = node;
        node = __builtin_amdgcn_readlane(parent, node < 0 ? 0 : node);
    }
    return path;
}

} // namespace vs
