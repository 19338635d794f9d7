"""GPU parity on caches whose tokens are not d elements apart: token-major layouts that several sequences, heads and layers share."""
import numpy as np
import pytest
import torch

import gen
import paper_2509_15235_amd as vs

pytestmark = pytest.mark.gpu

TIGHT_LONG = (1.5e-3, 6e-3)
TIGHT_SHORT = (1.2e-2, 6e-3)


def _token_major(da, cfg, need, stride, slots):
    """Moves da's contiguous caches into one buffer of `slots` tokens, `stride` elements apart, that holds every sequence's and KV
    head's K and V side by side; NaN wherever no sequence has a key."""
    B, Hkv, d = cfg.B, cfg.Hkv, cfg.d
    assert stride >= 2 * B * Hkv * d and slots >= need
    buf = torch.full((slots * stride,), float("nan"), device="cuda", dtype=da.k.dtype)
    at = buf.as_strided((need, B, 2, Hkv, d), (stride, 2 * Hkv * d, Hkv * d, d, 1))
    for b in range(B):
        n = int(da.inp.prefix_len[b]) + cfg.T
        at[:n, b, 0] = da.k[b, :, :n].transpose(0, 1)
        at[:n, b, 1] = da.v[b, :, :n].transpose(0, 1)
    da.k, da.v = buf, buf[Hkv * d:]
    da.desc.capacity, da.desc.stride_seq, da.desc.stride_head, da.desc.stride_tok = slots, 2 * Hkv * d, d, stride


def _token_major_pool(da, cfg, gap):
    """The same for a paged cache: a block is its tokens one after the other, each with K and V of every KV head and a gap of NaN."""
    Hkv, d, bs, blocks = cfg.Hkv, cfg.d, cfg.block_size, da.desc.num_blocks
    stride = 2 * Hkv * d + gap
    buf = torch.full((blocks * bs * stride,), float("nan"), device="cuda", dtype=da.k.dtype)
    at = buf.as_strided((blocks, bs, 2, Hkv, d), (bs * stride, stride, Hkv * d, d, 1))
    at[:, :, 0] = da.k.transpose(1, 2)
    at[:, :, 1] = da.v.transpose(1, 2)
    da.k, da.v = buf, buf[Hkv * d:]
    da.desc.stride_block, da.desc.stride_head, da.desc.stride_tok = bs * stride, d, stride


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("dtype,T,Hq,Hkv,d,lens,knobs", [
    ("bf16", 3, 28, 4, 128, [170, 61, 0], {}),                     # resident: one row block,
    ("bf16", 9, 28, 4, 128, [240, 33], {}),                        # two,
    ("bf16", 60, 28, 4, 128, [700], {}),                           # four in splits
    ("bf16", 4, 28, 4, 128, [490, 300, 256], {}),                  # own tiles
    ("bf16", 8, 32, 8, 64, [450, 7], {}),
    ("bf16", 16, 28, 4, 128, [1300, 900, 640, 50], {}),            # rounds
    ("bf16", 31, 32, 8, 64, [1500, 257], {}),
    ("bf16", 60, 28, 4, 128, [1100, 900, 300, 64], {}),            # pipelined: eight waves
    ("bf16", 60, 32, 32, 128, [500], {}),                          # ... four
    ("bf16", 60, 32, 8, 64, [700, 40], {"schedule": vs.VS_SCHED_PIPELINED, "num_splits": 3}),
    ("bf16", 60, 28, 4, 128, [1100, 90, 2000], {"schedule": vs.VS_SCHED_BALANCED}),
    ("bf16", 60, 28, 4, 128, [600, 333], {"schedule": vs.VS_SCHED_LOOP}),
    ("bf16", 60, 28, 4, 128, [600, 333], {"rows_per_wave": 2, "waves_per_group": 8}),
    ("bf16", 5, 8, 2, 64, [77, 130], {"impl": vs.VS_IMPL_GENERIC}),
    ("f32", 31, 8, 2, 128, [333, 90], {}),
    ("f32", 8, 4, 1, 64, [64], {}),
])
def test_token_major(oracle_mod, dtype, T, Hq, Hkv, d, lens, knobs, paged):
    import gpu_util as gu
    B = len(lens)
    cfg = gen.Config("strided", B, Hq, Hkv, d, T, min(6, T - 1), 4, 100, 0.5, 1, dtype, prefix=None, prefix_range=(1, 2), paged=paged)
    inp = gen.attention_inputs(cfg, 950 + T + B, prefix_len=np.array(lens, dtype=np.int32))
    da = gu.DeviceAttn(inp, **knobs)
    if paged:
        _token_major_pool(da, cfg, 24)
    else:
        _token_major(da, cfg, max(lens) + T, 2 * B * Hkv * d + 24, max(lens) + T + 70)
    got = da.run()
    assert (da.status.cpu().numpy() == 0).all()
    ref = oracle_mod.tree_attention(inp, threads=8)
    for b in range(B):
        tol = (2e-5, 2e-5) if dtype == "f32" else TIGHT_LONG if lens[b] >= 256 else TIGHT_SHORT
        gu.check_close(got[b], ref[b], *tol, what=f"sequence {b} of {lens[b]}")


@pytest.mark.parametrize("T,Hq,Hkv,d,S,schedule", [
    (3, 28, 4, 128, 6, vs.VS_SCHED_AUTO),      # one row block
    (4, 28, 4, 128, 17, vs.VS_SCHED_AUTO),
    (8, 32, 8, 64, 1, vs.VS_SCHED_AUTO),
    (9, 28, 4, 128, 0, vs.VS_SCHED_AUTO),      # two
    (9, 28, 4, 128, 12, vs.VS_SCHED_AUTO),
    (16, 28, 4, 128, 5, vs.VS_SCHED_AUTO),     # four
    (16, 16, 1, 64, 5, vs.VS_SCHED_AUTO),
    (9, 28, 4, 128, 12, vs.VS_SCHED_LOOP),
    (9, 28, 4, 128, 12, vs.VS_SCHED_PIPELINED),
    (30, 32, 4, 128, 1, vs.VS_SCHED_PIPELINED),
    (9, 32, 8, 64, 7, vs.VS_SCHED_BALANCED),
])
@pytest.mark.parametrize("B", [1, 2])
def test_slots_further_apart_than_32_bits_reach(oracle_mod, B, T, Hq, Hkv, d, S, schedule):
    """Sequences of few keys in a cache of 64 slots whose last ones lie beyond 2^32 bytes: the longest allowed sequence is what offsets
    have to reach (34 087 048 elements from token to token: 63 of them are 2^32 bytes and 752)."""
    import gpu_util as gu
    stride = 34087048
    cfg = gen.Config("far", B, Hq, Hkv, d, T, min(6, T - 1), 4, 100, 0.5, 1, "bf16", prefix=None, prefix_range=(1, 2), paged=False)
    lens = np.array([S] + [max(S - 1, 0)] * (B - 1), dtype=np.int32)
    assert (S + T) * stride < 1 << 30
    inp = gen.attention_inputs(cfg, 900 + T, prefix_len=lens)
    da = gu.DeviceAttn(inp, schedule=schedule)
    _token_major(da, cfg, S + T, stride, 64)
    da.ws_bytes = vs.vs_attention_workspace_bytes(da.desc)
    da.ws = torch.randint(0, 256, (max(da.ws_bytes, 256),), device="cuda", dtype=torch.uint8)
    got = da.run()
    assert (da.status.cpu().numpy() == 0).all()
    gu.check_close(got, oracle_mod.tree_attention(inp, threads=8), *TIGHT_SHORT)
    np.testing.assert_array_equal(got, da.run())
