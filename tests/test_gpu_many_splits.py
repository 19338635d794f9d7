"""Partial results of more splits than 32-bit offsets reach: the arithmetic from the kernels' own header, and a call that has
them, over a paged cache whose table names the same few blocks again and again."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import paper_2509_15235_amd as vs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_pieces_past_32_bits(tmp_path):
    src, so = tmp_path / "shim.cpp", tmp_path / "shim.so"
    src.write_text('#include "index_math.h"\nextern "C" int64_t t_piece(int32_t piece, int32_t splits) { return vs::piece_elements(piece, splits); }\n')
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-fPIC", "-shared",
                           "-I" + os.path.join(ROOT, "paper_2509_15235_amd", "csrc"), str(src), "-o", str(so)])
    L = ctypes.CDLL(str(so))
    L.t_piece.argtypes, L.t_piece.restype = [ctypes.c_int32, ctypes.c_int32], ctypes.c_int64
    for splits in (1, 32, 299593, 699051, 2097153, 4194305, 33554431):
        for piece in range(8):
            assert L.t_piece(piece, splits) == piece * splits * 512


@pytest.mark.gpu
def test_splits_past_32_bits():
    """4.2 million splits of 64 keys. A channel's value is the same power of two in every key, which is then the result whatever
    the scores are, up to roundings: 2^-9 each for the probabilities, the partial rows and the result, and 2^22 terms of either
    sum, 2^-24 each and of either sign. A partial result that was not stored would be the NaN that the workspace is filled with,
    one in another piece's place another power of two."""
    import torch
    import gpu_util as gu
    d, T, bs, blocks, splits = 64, 3, 4096, 6, (1 << 22) + 5
    prefix = splits * 64 - T
    desc = vs.AttnDesc(B=1, T=T, Hq=1, Hkv=1, d=d, dtype=vs.VS_BF16, softmax_scale=0.125, max_prefix_len=prefix, paged=1, block_size=bs,
                       max_blocks=(prefix + T + bs - 1) // bs, num_blocks=blocks, stride_block=bs * d, stride_head=bs * d, stride_tok=d,
                       schedule=vs.VS_SCHED_RESIDENT, num_splits=10 ** 7)
    table = (torch.arange(desc.max_blocks, device="cuda", dtype=torch.int32) % blocks).contiguous()
    desc.block_table = table.data_ptr()
    rc, pl = vs.vs_attention_plan(desc)
    assert rc == 0 and pl.num_splits == splits and pl.keys_per_split == 64
    g = torch.Generator(device="cuda").manual_seed(7)
    k = torch.randn(blocks * bs * d, device="cuda", generator=g).to(torch.bfloat16)
    value = 2.0 ** (torch.arange(d, device="cuda") % 16 - 8)
    value[1::3] *= -1.0
    v = value.to(torch.bfloat16).repeat(blocks * bs).contiguous()
    q = torch.randn(T * d, device="cuda", generator=g).to(torch.bfloat16)
    out = torch.zeros(T, d, device="cuda", dtype=torch.bfloat16)
    status = torch.full((1,), -99, device="cuda", dtype=torch.int32)
    lens = torch.tensor([prefix], device="cuda", dtype=torch.int32)
    parent = torch.tensor([-1, 0, 0], device="cuda", dtype=torch.int32)
    need = vs.vs_attention_workspace_bytes(desc)
    ws = torch.full((need,), 0xff, device="cuda", dtype=torch.uint8)
    rc = vs.vs_tree_verify_attention(desc, q, k, v, lens, parent, None, out, status, ws, need, gu.stream_ptr())
    assert rc == 0, vs.vs_strerror(rc)
    torch.cuda.synchronize()
    assert status.item() == 0
    np.testing.assert_allclose(out.float().cpu().numpy(), value.cpu().numpy()[None].repeat(T, 0), rtol=3 * 2.0 ** -9 + 2 * 2.0 ** -13, atol=0)
