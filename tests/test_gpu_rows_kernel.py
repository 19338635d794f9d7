"""GPU parity of the attention kernel whose waves have key tiles of their own (the planner's choice for one row block
and, where splits are long or there is one short one, two of 128 channels): lengths around tiles, rounds and splits,
fewer keys than waves, block-table windows, cached garbage behind the last key, more sequences than run at once."""
import numpy as np
import pytest

import gen
import paper_2509_15235_amd as vs

pytestmark = pytest.mark.gpu

TIGHT_LONG = (1.5e-3, 6e-3)
TIGHT_SHORT = (1.2e-2, 6e-3)


@pytest.mark.parametrize("B,T,Hq,Hkv,d,paged,lens", [
    (3, 4, 28, 4, 128, True, [1, 31, 300]),                       # waves without a tile, tiles without a prefix key
    (4, 1, 8, 8, 128, False, [0, 32, 255, 256]),
    (5, 32, 4, 4, 128, True, [224, 225, 480, 481, 512]),          # 32 rows; ends around rounds of eight tiles
    (6, 20, 16, 16, 64, False, [100, 1, 513, 767, 768, 1100]),
    (1, 3, 8, 1, 128, True, [40001]),                             # more splits than one, table windows of 32 tiles
    (1, 3, 8, 1, 64, True, [33000]),
    (2, 7, 8, 2, 128, False, [3000, 90]),                         # a sequence of one live split
    (20, 2, 16, 16, 128, True, [37 * i + 1 for i in range(20)]),  # four waves, in order
    (20, 2, 16, 16, 64, False, [61 * i + 5 for i in range(20)]),  # four waves, longest first
    (3, 9, 28, 4, 128, True, [190, 3, 255]),                      # two row blocks, one split
    (16, 60, 8, 8, 128, False, [2500 - 97 * i for i in range(16)]),  # two row blocks, splits of more than 1024 keys
])
def test_rows(oracle_mod, B, T, Hq, Hkv, d, paged, lens):
    import gpu_util as gu
    cfg = gen.Config("rows", B, Hq, Hkv, d, T, min(6, T - 1) if T > 1 else 1, 4, 100, 0.5, 1, "bf16", prefix=None, prefix_range=(1, 2), paged=paged)
    inp = gen.attention_inputs(cfg, 700 + T, prefix_len=np.array(lens, dtype=np.int32))
    da = gu.DeviceAttn(inp)
    pl = da.plan()
    assert pl.schedule == vs.VS_SCHED_LOOP and pl.row_groups == 1 and pl.waves_per_group == (4 if B * Hkv > 256 else 8)
    da.ws.random_(0, 256)
    if not paged:
        for b in range(B):                                        # nothing behind a sequence's last key counts
            da.k[b, :, lens[b] + T:] = float("nan")
            da.v[b, :, lens[b] + T:] = float("nan")
    got = da.run()
    assert (da.status.cpu().numpy() == 0).all()
    ref = oracle_mod.tree_attention(inp, threads=8)
    for b in range(B):
        gu.check_close(got[b], ref[b], *(TIGHT_LONG if lens[b] >= 256 else TIGHT_SHORT), what=f"sequence {b} of {lens[b]}")
    for _ in range(3):
        np.testing.assert_array_equal(got, da.run())
