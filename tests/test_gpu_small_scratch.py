"""Attention calls with less scratch than their fine cut asks for but enough for the coarser one behind it run on that; with
less still they are refused. Over the kernels that the coarser cut may belong to, for both entry points."""
import numpy as np
import pytest

import gen
import paper_2509_15235_amd as vs

pytestmark = pytest.mark.gpu


# longest prefix, bytes that the fine cut reports, least that is accepted
@pytest.mark.parametrize("B,T,Hq,Hkv,d,prefix,need,least", [
    (1, 62, 8, 1, 128, 195, 679936, 676864),      # the resident kernel's four row blocks
    (1, 56, 8, 1, 128, 1995, 2014208, 2011648),   # rounds
    (3, 64, 28, 4, 128, 259, 2860032, 2838528),   # the pipelined kernel with a combine kernel
])
def test_verification(oracle_mod, B, T, Hq, Hkv, d, prefix, need, least):
    import gpu_util as gu
    cfg = gen.Config("scratch", B, Hq, Hkv, d, T, 6, 4, 100, 0.5, 1, "bf16", prefix=None, prefix_range=(1, 2), paged=False)
    inp = gen.attention_inputs(cfg, 1300 + T, prefix_len=np.array([prefix - 70 * b for b in range(B)], dtype=np.int32))
    ref = oracle_mod.tree_attention(inp, threads=8)
    da = gu.DeviceAttn(inp)
    assert da.ws_bytes == need
    for given in (need, need - 256, least):
        da.ws_bytes = given
        da.ws.random_(0, 256)
        da.out.fill_(float("nan"))
        gu.check_close(da.run(), ref, 1.2e-2, 6e-3)
        assert (da.status.cpu().numpy() == 0).all()
    da.ws_bytes = least - 256
    with pytest.raises(AssertionError):
        da.run()


@pytest.mark.parametrize("B,T,Hq,Hkv,d,length,need,least", [
    (1, 31, 8, 1, 128, 257, 339968, 338432),
    (3, 55, 28, 4, 128, 321, 2657280, 2635776),
    (1, 56, 8, 1, 128, 1995, 3786496, 3785728),
])
def test_compression(oracle_mod, B, T, Hq, Hkv, d, length, need, least):
    import torch
    import gpu_util as gu
    inp = gen.compress_inputs(1400 + T, B, T, Hq, Hkv, d, [length - 60 * b for b in range(B)])
    ref = np.stack([oracle_mod.compress_attention_seq(inp["q"][b], inp["k"][b], inp["v"][b], int(inp["lens"][b]), inp["scale"], Hkv) for b in range(B)])
    q, k, v = (gu.dev_bf16(inp[n + "_bits"]) for n in "qkv")
    cap = inp["cap"]
    desc = vs.AttnDesc(B=B, T=T, Hq=Hq, Hkv=Hkv, d=d, dtype=vs.VS_BF16, softmax_scale=float(inp["scale"]), max_prefix_len=length, capacity=cap,
                       stride_seq=Hkv * cap * d, stride_head=cap * d, stride_tok=d)
    assert vs.vs_compress_attention_workspace_bytes(desc) == need
    ws = torch.empty(need, device="cuda", dtype=torch.uint8)
    lens = gu.dev(inp["lens"])
    for given in (need, need - 256, least, least - 256):
        ws.random_(0, 256)
        out = torch.full((B, T, Hq, d), float("nan"), device="cuda", dtype=torch.bfloat16)
        status = torch.full((B,), -99, device="cuda", dtype=torch.int32)
        rc = vs.vs_compress_attention(desc, q, k, v, lens, out, status, ws, given, gu.stream_ptr())
        assert rc == (0 if given >= least else -4)
        if rc == 0:
            torch.cuda.synchronize()
            assert (status.cpu().numpy() == 0).all()
            gu.check_close(out.float().cpu().numpy().astype(np.float64), ref, 1.2e-2, 6e-3)
