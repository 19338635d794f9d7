// Index arithmetic of the kernels that can go wrong in ways no ordinary size shows: constexpr and free of HIP headers, so that
// the same definitions serve the device, the library's host code and tests that have no GPU (tests/test_index_math.py).
#pragma once

#include <stdint.h>

namespace vs {

// Division by a number that the host knows: one multiplication and one correction instead of the 45 instructions of a
// 32-bit division (m = floor((2^32 - 1) / d): the product's upper half is the quotient or one less, for any n).
struct FastDiv {
    uint32_t d, m;
};
constexpr FastDiv fast_div_by(int32_t d) { return {(uint32_t)d, 0xffffffffu / (uint32_t)d}; }
constexpr uint32_t fast_div(uint32_t n, FastDiv by, uint32_t& rem) {
    uint32_t q = (uint32_t)(((uint64_t)n * by.m) >> 32);
    rem = n - q * by.d;
    if (rem >= by.d) {
        rem -= by.d;
        ++q;
    }
    return q;
}

// Node of query row r (r / group), inv_group = 1 / group. (r + 1/2) / group is 1 / (2 group) or more away from a whole number and the
// quotient is below 64, so up to 16384 rows a node the fp32 error, 64 * 2^-23, is too small to matter; beyond, it is off by less
// than one.
constexpr int32_t kShortGroup = 16384;
template <typename F> // (a constexpr function has to have a constant value for some arguments, a template has not)
constexpr int32_t node_of_row_short(int32_t r, F inv_group) { return (int32_t)__builtin_fmaf((float)r, inv_group, 0.5f * inv_group); }
constexpr int32_t node_of_row(int32_t r, int32_t group, float inv_group) {
    if (group <= kShortGroup) return node_of_row_short(r, inv_group);
    int32_t n = (int32_t)((float)r * inv_group);
    const int32_t rem = r - n * group;
    n += (rem >= group) - (rem < 0);
    return n;
}

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


// The same in rows, `skip` = Hq - group of them between two nodes': below T * Hq and so below 2^31. What a kernel does for several rows
// on its way to its first loads (a 64-bit product per row takes three more instructions).
constexpr uint32_t row_number(int32_t r, int32_t node, int32_t skip) { return (uint32_t)node * (uint32_t)skip + (uint32_t)r; }

// Elements from the first piece (512 elements) of a partial result to another one: those of all splits lie in between. 64 bits: a
// paged cache's table can name any number of keys, and so can the splits of 64 that a caller asks for.
constexpr int64_t piece_elements(int32_t piece, int32_t num_splits) { return (int64_t)piece * num_splits * 512; }

// Whether no two rows of `row` elements are the same memory, or parts of it, that lie at a * sa + b * sb + c * sc elements, a < na and so on:
// in the order of their strides, each index has to step over all that the ones before it reach. (Rows that interleave otherwise count as
// not apart.) In double: exact below 2^53, and no stride wraps.
constexpr bool rows_apart(int64_t row, int64_t na, int64_t sa, int64_t nb, int64_t sb, int64_t nc, int64_t sc) {
    int64_t n[3] = {na, nb, nc}, s[3] = {sa, sb, sc};
    double reach = (double)row;
    for (int i = 0; i < 3; ++i) {
        int least = i;
        for (int j = i + 1; j < 3; ++j)
            if (s[j] < s[least]) least = j;
        const int64_t count = n[least], stride = s[least];
        n[least] = n[i];
        s[least] = s[i];
        if (count <= 1) continue;
        if ((double)stride < reach) return false;
        reach += (double)stride * (double)(count - 1);
    }
    return true;
}

} // namespace vs
