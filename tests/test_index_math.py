"""The kernels' index arithmetic (csrc/index_math.h), compiled for the host and compared with whole numbers of any size."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#include "index_math.h"
using namespace vs;
extern "C" {
uint32_t t_slice_bytes(int64_t most, int32_t k0, int32_t keys, uint32_t stride, uint32_t row) { return slice_bytes(most, k0, keys, stride, row); }
void t_fast_div(const uint32_t* n, int64_t count, int32_t d, uint32_t* q, uint32_t* rem) {
    const FastDiv by = fast_div_by(d);
    for (int64_t i = 0; i < count; ++i) q[i] = fast_div(n[i], by, rem[i]);
}
void t_node_of_row(const int32_t* r, int64_t count, int32_t group, int32_t* node) {
    for (int64_t i = 0; i < count; ++i) node[i] = node_of_row(r[i], group, 1.f / (float)group);
}
int64_t t_row_elements(int32_t r, int32_t node, int64_t node_stride, int32_t d) { return row_elements(r, node, node_stride, d); }
int32_t t_early_end(int64_t most, int32_t k0, int32_t keys) { return early_end(most, k0, keys); }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    at = tmp_path_factory.mktemp("index_math")
    src, so = at / "shim.cpp", at / "shim.so"
    src.write_text(SHIM)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-fPIC", "-shared",
                           "-I" + os.path.join(ROOT, "paper_2509_15235_amd", "csrc"), str(src), "-o", str(so)])
    L = ctypes.CDLL(str(so))
    i32, u32, i64 = ctypes.c_int32, ctypes.c_uint32, ctypes.c_int64
    L.t_slice_bytes.argtypes, L.t_slice_bytes.restype = [i64, i32, i32, u32, u32], u32
    L.t_early_end.argtypes, L.t_early_end.restype = [i64, i32, i32], i32
    L.t_fast_div.argtypes = [ctypes.c_void_p, i64, i32, ctypes.c_void_p, ctypes.c_void_p]
    L.t_node_of_row.argtypes = [ctypes.c_void_p, i64, i32, ctypes.c_void_p]
    L.t_row_elements.argtypes, L.t_row_elements.restype = [i32, i32, i64, i32], i64
    return L


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("most", [1, 2, 9, 21, 31, 63, 64, 65, 128, 200, 1756, 16777215])
def test_slice_holds_every_row_that_may_live(lib, most, d):
    """A split's slice ends with its last row that a sequence can have, for every token stride that the host accepts
    (most * stride below 2^30 elements, a multiple of eight) and splits longer than the sequence."""
    top = ((1 << 30) - 1) // most // 8 * 8
    r = np.random.default_rng(most + d)
    strides = {d, top, 34087048, *(int(x) // 8 * 8 for x in r.integers(d, max(top, d + 1), size=200))}
    for stride in (s for s in strides if d <= s <= top):
        for keys in (64, 128, 192, 256):
            for k0 in {0, (most - 1) // keys * keys}:
                rows = min(most - k0, keys)
                assert lib.t_slice_bytes(most, k0, keys, 2 * stride, 2 * d) == (rows - 1) * 2 * stride + 2 * d < 1 << 31


def test_early_end(lib):
    for most, k0, keys in [(9, 0, 64), (64, 0, 64), (65, 64, 64), (1756, 1664, 128), ((1 << 31) + 62, 0, 192), ((1 << 31) + 62, (1 << 31) - 257, 192),
                           (2147483647, 2147483584, 192)]:
        assert lib.t_early_end(most, k0, keys) == min(most, k0 + keys)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("group,Hkv,T", [(1, 1, 1), (7, 4, 60), (1, 32, 64), (8, 1, 64), (16400, 1, 2), (1 << 19, 1, 64), ((1 << 19) + 3, 2, 63), (1 << 25, 1, 32)])
def test_row_elements(lib, group, Hkv, T, d):
    """Row r of a KV head, head r % group of node r / group, in a dense [T, Hkv * group, d] tensor, also past 2^32 elements."""
    for node in {0, 1, T // 2, T - 1}:
        for head in {0, group // 2, group - 1}:
            assert lib.t_row_elements(node * group + head, node, (Hkv - 1) * group * d, d) == (node * Hkv * group + head) * d


def test_division_by_multiplication(lib):
    """Quotient and remainder of 32-bit numbers by any divisor that the host passes."""
    r = np.random.default_rng(3)
    n = np.concatenate([[0, 1, 255, 256, 2 ** 31 - 1, 2 ** 31, 2 ** 32 - 1], r.integers(0, 2 ** 32, size=300)])
    q, rem = np.empty(2 * len(n), dtype=np.uint32), np.empty(2 * len(n), dtype=np.uint32)
    for d in [*range(1, 400), 2 ** 31 - 1, *(int(x) for x in r.integers(1, 2 ** 31, size=4000))]:
        m = np.concatenate([n, n // d * d]).astype(np.uint32)      # whole multiples among them
        lib.t_fast_div(m.ctypes.data, len(m), d, q.ctypes.data, rem.ctypes.data)
        assert (q == m // np.uint32(d)).all() and (rem == m % np.uint32(d)).all()


def test_node_of_row(lib):
    """The first and the last row of every node, for every group up to 16384 (the short form) and for larger ones."""
    r = np.random.default_rng(4)
    node = np.empty(128, dtype=np.int32)
    for g in [*range(1, 16386), 16400, 65537, (1 << 19) + 8, 1 << 25, *(int(x) for x in r.integers(16385, (2 ** 31 - 1) // 64, size=2000))]:
        n = np.arange(64, dtype=np.int64)
        rows = np.concatenate([n * g, n * g + g - 1]).astype(np.int32)
        lib.t_node_of_row(rows.ctypes.data, len(rows), g, node.ctypes.data)
        assert (node == np.concatenate([n, n])).all(), g
