"""Launches of the pipelined kernel where shorter splits, or none, would be the faster ones: whole sequences instead of splits are taken, shorter splits
are not. Against the oracle at exactly the scratch that the plan asks for."""
import numpy as np
import pytest

import gen
import paper_2509_15235_amd as vs

pytestmark = pytest.mark.gpu


# longest prefix, splits and workgroups of the plan
@pytest.mark.parametrize("B,T,Hq,Hkv,d,longest,splits,wgs", [
    (29, 19, 8, 1, 128, 1170, 5, 145),
    (4, 37, 32, 8, 64, 801, 4, 128),
    (24, 19, 28, 4, 128, 366, 1, 96),
    (13, 50, 28, 4, 128, 516, 1, 104),    # two row groups
    (6, 35, 8, 2, 128, 1567, 7, 84),
])
def test_against_the_oracle(oracle_mod, B, T, Hq, Hkv, d, longest, splits, wgs):
    import gpu_util as gu
    cfg = gen.Config("short_splits", B, Hq, Hkv, d, T, 6, 4, 100, 0.5, 1, "bf16", prefix=None, prefix_range=(1, 2), paged=False)
    lens = np.array([longest] + [(longest * 7 * b) // 31 % min(longest, 640) for b in range(1, B)], dtype=np.int32)
    inp = gen.attention_inputs(cfg, 2700 + T, prefix_len=lens)
    ref = oracle_mod.tree_attention(inp, threads=8)
    da = gu.DeviceAttn(inp)
    pl = da.plan()
    assert (pl.schedule, pl.num_splits, pl.workgroups) == (vs.VS_SCHED_PIPELINED, splits, wgs)
    assert (da.ws_bytes > 0) == (splits > 1)
    if splits > 1:
        da.ws.random_(0, 256)
    da.out.fill_(float("nan"))
    gu.check_close(da.run(), ref, 1.2e-2, 6e-3)
    assert (da.status.cpu().numpy() == 0).all()
