"""When K and V are loaded as data that is read once: large launches on contiguous caches in which no two rows are the same memory. Without a GPU."""
import ctypes
import itertools
import os
import subprocess

import pytest

import paper_2509_15235_amd as vs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = """
#include "index_math.h"
extern "C" int t_rows_apart(int64_t row, int64_t na, int64_t sa, int64_t nb, int64_t sb, int64_t nc, int64_t sc) {
    return vs::rows_apart(row, na, sa, nb, sb, nc, sc);
}
"""


def _once(B, T, Hq, Hkv, d, longest, **kw):
    cap = longest + T
    desc = vs.AttnDesc(B=B, T=T, Hq=Hq, Hkv=Hkv, d=d, dtype=vs.VS_BF16, softmax_scale=d ** -0.5, max_prefix_len=longest, capacity=cap,
                       stride_seq=Hkv * cap * d, stride_head=cap * d, stride_tok=d)
    for name, value in kw.items():
        setattr(desc, name, value)
    return vs.lib().vs_internal_reads_once(ctypes.byref(desc), 1)


# own tiles of one and of two row blocks, balanced shares of four waves: 79, 1049, 401 and 675 MB
LARGE = [(64, 4, 28, 4, 128, 600), (64, 4, 28, 4, 128, 8000), (8, 60, 32, 32, 128, 3000), (20, 60, 32, 32, 128, 2000)]


@pytest.mark.parametrize("c", LARGE)
def test_sequences_with_rows_of_their_own(c):
    B, T, Hq, Hkv, d, longest = c
    cap = longest + T
    assert _once(*c) == 1
    assert _once(*c, stride_seq=cap * Hkv * d, stride_tok=Hkv * d, stride_head=d) == 1  # [sequence][token][head]
    assert _once(*c, stride_seq=cap * d, stride_head=B * cap * d) == 1                  # [head][sequence][token]


@pytest.mark.parametrize("c", LARGE)
def test_shared_rows_are_left_to_the_caches(c):
    B, T, Hq, Hkv, d, longest = c
    cap = longest + T
    assert _once(*c, stride_seq=0) == 0
    assert _once(*c, stride_head=0) == 0
    assert _once(*c, stride_seq=100 * d) == 0               # windows of one line of tokens
    paged = dict(paged=1, block_size=16, max_blocks=-(-cap // 16), num_blocks=B * -(-cap // 16), stride_block=Hkv * 16 * d,
                 stride_head=16 * d, block_table=4096)
    assert _once(*c, **paged) == 0                          # the host does not know the block table


@pytest.mark.parametrize("c", [(16, 4, 28, 4, 128, 600), (64, 60, 28, 4, 128, 8000), (1, 60, 28, 4, 128, 1696), (4, 4, 28, 4, 128, 12000)])
def test_small_launches_and_shared_tiles(c):
    assert _once(*c) == 0


@pytest.fixture(scope="module")
def rows_apart(tmp_path_factory):
    at = tmp_path_factory.mktemp("rows_apart")
    (at / "shim.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-fPIC", "-shared",
                           "-I" + os.path.join(ROOT, "paper_2509_15235_amd", "csrc"), str(at / "shim.cpp"), "-o", str(at / "shim.so")])
    f = ctypes.CDLL(str(at / "shim.so")).t_rows_apart
    f.argtypes = [ctypes.c_int64] * 7
    return f


def test_rows_apart_against_all_elements(rows_apart):
    """What counts as apart is; plain layouts count; strides as large as a caller can name do not wrap."""
    row, apart = 2, 0
    for (na, nb, nc) in itertools.product([1, 2, 3], repeat=3):
        for sa, sb, sc in itertools.product([0, 1, 2, 3, 4, 6, 8, 12], repeat=3):
            if not rows_apart(row, na, sa, nb, sb, nc, sc):
                continue
            at = [a * sa + b * sb + c * sc + e for a in range(na) for b in range(nb) for c in range(nc) for e in range(row)]
            assert len(set(at)) == len(at), (na, sa, nb, sb, nc, sc)
            apart += 1
    assert apart > 1000
    for order in itertools.permutations(range(3)):  # dense, in any order
        n, s, reach = [5, 3, 4], [0, 0, 0], row
        for i in order:
            s[i] = reach
            reach *= n[i]
        assert rows_apart(row, n[0], s[0], n[1], s[1], n[2], s[2])
    big = (1 << 63) - 1
    assert rows_apart(128, 100, 128, 4, big // 2, 64, big) == 0 and rows_apart(128, 100, 128, 4, 12800, 64, big) == 1
