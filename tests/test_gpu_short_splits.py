"""Launches whose splits the planner makes shorter, fewer or the pipelined kernel's own where coarser ones would do: at the scratch
that the plan asks for, and at what the coarser plan behind it needs, which is accepted too."""
import numpy as np
import pytest

import gen
import paper_2509_15235_amd as vs

pytestmark = pytest.mark.gpu


# longest prefix, schedule, splits and workgroups of the plan, bytes that the coarser plan needs
@pytest.mark.parametrize("B,T,Hq,Hkv,d,longest,schedule,splits,wgs,coarser", [
    (29, 19, 8, 1, 128, 1170, vs.VS_SCHED_PIPELINED, 7, 203, 6124800),     # five
    (4, 37, 32, 8, 64, 801, vs.VS_SCHED_PIPELINED, 7, 224, 2785280),       # four
    (24, 19, 28, 4, 128, 366, vs.VS_SCHED_PIPELINED, 1, 96, 8110080),      # two
    (6, 35, 8, 2, 128, 1567, vs.VS_SCHED_RESIDENT, 7, 252, 3551232),       # seven of the pipelined kernel
])
def test_against_the_oracle(oracle_mod, B, T, Hq, Hkv, d, longest, schedule, splits, wgs, coarser):
    import gpu_util as gu
    cfg = gen.Config("short_splits", B, Hq, Hkv, d, T, 6, 4, 100, 0.5, 1, "bf16", prefix=None, prefix_range=(1, 2), paged=False)
    lens = np.array([longest] + [(longest * 7 * b) // 31 % min(longest, 640) for b in range(1, B)], dtype=np.int32)
    inp = gen.attention_inputs(cfg, 2700 + T, prefix_len=lens)
    ref = oracle_mod.tree_attention(inp, threads=8)
    da = gu.DeviceAttn(inp)
    pl = da.plan()
    assert (pl.schedule, pl.num_splits, pl.workgroups) == (schedule, splits, wgs)
    for given in {da.ws_bytes, min(da.ws_bytes, coarser)}:
        da.ws_bytes = given
        if given:
            da.ws.random_(0, 256)
        da.out.fill_(float("nan"))
        gu.check_close(da.run(), ref, 1.2e-2, 6e-3)
        assert (da.status.cpu().numpy() == 0).all()
