"""The query rows' numbers that the attention kernels load and store by, run from the kernels' own header: equal to the
element offsets in 64 bits that tests/test_index_math.py checks, for every group that a call may have."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = """
#include "index_math.h"
using namespace vs;
extern "C" {
uint32_t t_row_number(int32_t r, int32_t node, int32_t skip) { return row_number(r, node, skip); }
int64_t t_row_elements(int32_t r, int32_t node, int64_t node_stride, int32_t d) { return row_elements(r, node, node_stride, d); }
int32_t t_node(int32_t r, int32_t group) { return group <= kShortGroup ? node_of_row_short(r, 1.f / (float)group) : node_of_row(r, group, 1.f / (float)group); }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    at = tmp_path_factory.mktemp("row_numbers")
    src, so = at / "shim.cpp", at / "shim.so"
    src.write_text(SHIM)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-fPIC", "-shared",
                           "-I" + os.path.join(ROOT, "paper_2509_15235_amd", "csrc"), str(src), "-o", str(so)])
    L = ctypes.CDLL(str(so))
    L.t_row_number.restype = ctypes.c_uint32
    L.t_row_elements.argtypes, L.t_row_elements.restype = [ctypes.c_int32, ctypes.c_int32, ctypes.c_int64, ctypes.c_int32], ctypes.c_int64
    return L


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("group,Hkv,T", [(1, 1, 1), (7, 4, 60), (1, 32, 64), (8, 1, 64), (16384, 3, 40), (16400, 1, 2), (1 << 19, 1, 64),
                                         ((1 << 19) + 3, 2, 31), (1 << 24, 2, 63), ((1 << 25) - 1, 1, 64)])
def test_row_numbers(lib, group, Hkv, T, d):
    skip = (Hkv - 1) * group
    r = np.random.default_rng(group + T)
    for node in {0, 1 % T, T // 2, T - 1}:
        for head in {0, group // 2, group - 1, int(r.integers(0, group))}:
            row = node * group + head
            assert lib.t_node(row, group) == node
            n = lib.t_row_number(row, node, skip)
            assert n == node * Hkv * group + head < T * Hkv * group
            assert n * d == lib.t_row_elements(row, node, skip * d, d)
