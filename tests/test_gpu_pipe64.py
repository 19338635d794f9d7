"""GPU parity of the pipelined attention kernel with eight waves and 64 channels (half of its waves copy keys, the other
half values): lengths around tiles, iterations and the loop's forms, waves without rows, both cache layouts, whole
sequences, splits and balanced shares."""
import numpy as np
import pytest

import gen
import paper_2509_15235_amd as vs

pytestmark = pytest.mark.gpu

TIGHT_LONG = (1.5e-3, 6e-3)
TIGHT_SHORT = (1.2e-2, 6e-3)
LENS = [1, 31, 64, 96, 127, 160, 256, 289, 352, 415, 640, 1000, 1313, 2048]


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("T,Hq,Hkv", [(40, 12, 3), (64, 4, 1), (33, 8, 2)])   # five, eight and five of eight waves with rows
@pytest.mark.parametrize("kw", [dict(schedule=vs.VS_SCHED_PIPELINED, num_splits=1), dict(schedule=vs.VS_SCHED_PIPELINED, num_splits=3),
                                dict(schedule=vs.VS_SCHED_BALANCED, num_splits=9)])
def test_eight_waves_of_64_channels(oracle_mod, paged, T, Hq, Hkv, kw):
    import gpu_util as gu
    cfg = gen.Config("pipe64", len(LENS), Hq, Hkv, 64, T, 6, 4, 100, 0.5, 1, "bf16", prefix=None, prefix_range=(1, 2), paged=paged)
    inp = gen.attention_inputs(cfg, 660 + T, prefix_len=np.array(LENS, dtype=np.int32))
    da = gu.DeviceAttn(inp, waves_per_group=8, **kw)
    da.ws.random_(0, 256)
    if not paged:
        for b, n in enumerate(LENS):                              # nothing behind a sequence's last key counts
            da.k[b, :, n + T:] = float("nan")
            da.v[b, :, n + T:] = float("nan")
    got = da.run()
    assert (da.status.cpu().numpy() == 0).all()
    ref = oracle_mod.tree_attention(inp, threads=8)
    for b, n in enumerate(LENS):
        gu.check_close(got[b], ref[b], *(TIGHT_LONG if n >= 256 else TIGHT_SHORT), what=f"sequence {b} of {n}")
    np.testing.assert_array_equal(got, da.run())
