"""GPU parity on caches whose tokens are not d elements apart: token-major layouts that several sequences, heads and layers share."""
import numpy as np
import pytest
import torch

import gen
import paper_2509_15235_amd as vs

pytestmark = pytest.mark.gpu

TIGHT_SHORT = (1.2e-2, 6e-3)


def _token_major(da, cfg, need, stride, slots):
    """Moves da's contiguous caches into one buffer of `slots` tokens, `stride` elements apart, that holds every sequence's and KV
    head's K and V side by side; NaN wherever no sequence has a key."""
    B, Hkv, d = cfg.B, cfg.Hkv, cfg.d
    assert stride >= 2 * B * Hkv * d
    buf = torch.full((slots * stride,), float("nan"), device="cuda", dtype=torch.bfloat16)
    at = buf.as_strided((need, B, 2, Hkv, d), (stride, 2 * Hkv * d, Hkv * d, d, 1))
    for b in range(B):
        n = int(da.inp.prefix_len[b]) + cfg.T
        at[:n, b, 0] = da.k[b, :, :n].transpose(0, 1)
        at[:n, b, 1] = da.v[b, :, :n].transpose(0, 1)
    da.k, da.v = buf, buf[Hkv * d:]
    da.desc.capacity, da.desc.stride_seq, da.desc.stride_head, da.desc.stride_tok = slots, 2 * Hkv * d, d, stride


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
