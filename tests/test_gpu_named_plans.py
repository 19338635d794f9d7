"""A reported LDS-resident plan that is asked for by name - its schedule alone, with its number of splits, with its waves and row
blocks as well - is the plan that was reported, and gives its results bit for bit."""
import numpy as np
import pytest

import gen
import paper_2509_15235_amd as vs

HEADS = [(28, 4, 128), (32, 32, 128), (8, 2, 128), (8, 1, 128), (40, 8, 128), (32, 8, 64), (16, 16, 64), (28, 4, 64)]


def _names(pl):
    return [dict(schedule=pl.schedule), dict(schedule=pl.schedule, num_splits=pl.num_splits),
            dict(schedule=pl.schedule, num_splits=pl.num_splits, rows_per_wave=pl.rows_per_wave, waves_per_group=pl.waves_per_group)]


def _plan(desc):
    rc, pl = vs.vs_attention_plan(desc)
    assert rc == 0
    return pl, [getattr(pl, f) for f, _ in pl._fields_] + [vs.vs_attention_workspace_bytes(desc)]


def test_reported_plans():
    r = np.random.default_rng(5)
    seen = 0
    for _ in range(6000):
        Hq, Hkv, d = HEADS[r.integers(len(HEADS))]
        B, T, keys = int(2 ** r.uniform(0, 6)), int(r.integers(1, 65)), int(2 ** r.uniform(3, 12))
        sizes = dict(B=B, T=T, Hq=Hq, Hkv=Hkv, d=d, dtype=vs.VS_BF16, softmax_scale=0.1, max_prefix_len=keys, capacity=keys + T,
                     stride_seq=Hkv * (keys + T) * d, stride_head=(keys + T) * d, stride_tok=d)
        pl, all_of_it = _plan(vs.AttnDesc(**sizes))
        if pl.schedule != vs.VS_SCHED_RESIDENT:
            continue
        seen += 1
        for kw in _names(pl):
            assert _plan(vs.AttnDesc(**sizes, **kw))[1] == all_of_it, (sizes, kw)
        for n in {1, 2, pl.num_splits + 1, 10 ** 6} - {pl.num_splits}:  # any other number: splits of 192 keys at most
            assert _plan(vs.AttnDesc(**sizes, schedule=pl.schedule, num_splits=n))[0].keys_per_split <= 192
    assert seen > 1000


@pytest.mark.gpu
@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("B,T,Hq,Hkv,d,keys", [(4, 60, 28, 4, 128, 128), (4, 39, 28, 4, 128, 601), (8, 47, 40, 8, 128, 369), (4, 14, 32, 8, 64, 190)])
def test_results(oracle_mod, B, T, Hq, Hkv, d, keys, paged):
    import gpu_util as gu
    cfg = gen.Config("named", B, Hq, Hkv, d, T, min(6, T - 1), 4, 100, 0.5, 1, "bf16", prefix=None, prefix_range=(1, 2), paged=paged)
    inp = gen.attention_inputs(cfg, 1200 + T, prefix_len=np.array([keys - T - 9 * b for b in range(B)], dtype=np.int32))
    da = gu.DeviceAttn(inp)
    pl = da.plan()
    assert pl.schedule == vs.VS_SCHED_RESIDENT
    want = da.run()
    ref = oracle_mod.tree_attention(inp, threads=8)
    gu.check_close(want, ref, 1.2e-2, 6e-3)
    for kw in _names(pl):
        np.testing.assert_array_equal(want, gu.DeviceAttn(inp, **kw).run())
