// Index arithmetic of the kernels that can go wrong in ways no ordinary size shows: constexpr and free of HIP headers, so that
// the same definitions serve the device, the library's host code and tests that have no GPU (tests/test_index_math.py).
#pragma once

#include <stdint.h>

namespace vs {

// Bytes of one sequence's K (or V) rows of one KV head from key k0 on that a split may ask for before it knows its length: up to
// the longest sequence that the host allows (most_keys > k0), not up to the cache's capacity. The host keeps most_keys * stride
// below 2^31 bytes; the slots of a cache beyond that may lie any distance away. Rows of row_bytes, `stride` bytes apart.
constexpr uint32_t slice_bytes(int64_t most_keys, int32_t k0, int32_t keys_per_split, uint32_t stride, uint32_t row_bytes) {
    const int64_t left = most_keys - k0;
    const uint32_t rows = left < keys_per_split ? (uint32_t)left : (uint32_t)keys_per_split;
    return (rows - 1) * stride + row_bytes;
}

// End of the keys from k0 on, at most `keys` of them, that a workgroup may ask for before it knows its sequence's length.
constexpr int32_t early_end(int64_t most_keys, int32_t k0, int32_t keys) {
    const int64_t end = (int64_t)k0 + keys;
    return (int32_t)(most_keys < end ? most_keys : end);
}

// Elements from a (sequence, KV head)'s first query row to row r: a node's rows are adjacent, node_stride lies between two nodes'
// beyond that. 64 bits: 64 nodes of many rows each pass 2^32 elements.
constexpr int64_t row_elements(int32_t r, int32_t node, int64_t node_stride, int32_t d) {
    return (int64_t)((uint64_t)(uint32_t)node * (uint64_t)node_stride + (uint64_t)(uint32_t)r * (uint32_t)d);
}

} // namespace vs
