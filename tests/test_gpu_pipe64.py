"""GPU parity of the pipelined attention kernel with 64 channels: eight waves (half of them copy keys, the other half
values) at lengths around tiles, iterations and the loop's forms, with waves without rows, as whole sequences, splits
and balanced shares; four waves where three workgroups share a CU. Both cache layouts."""
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


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("B,T,hi", [(33, 43, 1000), (48, 64, 400)])              # 528 and 768 workgroups: the ends of the range
def test_three_workgroups_per_cu(oracle_mod, paged, B, T, hi):
    import gpu_util as gu
    lens = np.random.default_rng(B).integers(1, hi, size=B).astype(np.int32)
    lens[:8] = [1, 31, 32, 63, 96, 129, 255, hi]
    cfg = gen.Config("pipe64", B, 16, 16, 64, T, 6, 4, 100, 0.5, 1, "bf16", prefix=None, prefix_range=(1, 2), paged=paged)
    inp = gen.attention_inputs(cfg, 670 + T, prefix_len=lens)
    da = gu.DeviceAttn(inp)
    pl = da.plan()
    assert pl.schedule == vs.VS_SCHED_PIPELINED and pl.waves_per_group == 4 and 512 < pl.workgroups <= 768 and pl.num_splits == 1
    got = da.run()
    assert (da.status.cpu().numpy() == 0).all()
    seqs = list(range(10)) + [B // 2, B - 1]
    ref = oracle_mod.tree_attention(inp, threads=8, seqs=seqs)
    for b in seqs:
        gu.check_close(got[b], ref[b], *(TIGHT_LONG if lens[b] >= 256 else TIGHT_SHORT), what=f"sequence {b} of {lens[b]}")
    assert np.isfinite(got).all()
    np.testing.assert_array_equal(got, da.run())
