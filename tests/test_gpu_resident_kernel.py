"""GPU parity of the attention kernel that keeps a split's keys in LDS: one, two and four row blocks, one to eight tiles of
32 keys, ends around tiles, cached garbage behind the last key, splits of 64, 128 and 192 keys."""
import numpy as np
import pytest

import gen
import paper_2509_15235_amd as vs

TIGHT_LONG = (1.5e-3, 6e-3)
TIGHT_SHORT = (1.2e-2, 6e-3)


@pytest.mark.gpu
@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("B,T,Hq,Hkv,d,lens,splits", [
    (5, 3, 28, 4, 128, [61, 1, 29, 30, 0], 1),                    # one row block: a single tile of 64 keys,
    (6, 3, 8, 1, 128, [125, 62, 93, 0, 124, 31], 1),              # two,
    (6, 4, 32, 8, 64, [188, 187, 124, 1, 63, 64], 1),             # three
    (7, 9, 28, 4, 128, [247, 246, 215, 216, 183, 1, 0], 1),       # two row blocks: one split of up to 256 keys
    (4, 9, 28, 4, 128, [55, 54, 23, 0], 1),
    (5, 50, 8, 8, 128, [14, 13, 1, 0, 5], 1),
    (2, 3, 28, 4, 128, [700, 61], 11),                            # splits of 64 keys
    (3, 2, 8, 1, 64, [1022, 959, 3], 16),
    (4, 3, 28, 4, 128, [1200, 1100, 127, 128], 10),               # of 128
    (1, 6, 8, 2, 128, [3900], 31),                                # ... more than sixteen of them
    (16, 3, 28, 4, 128, [597 - 31 * i for i in range(16)], 4),    # of 192
    (3, 16, 28, 4, 128, [1900, 1800, 191], 15),                   # four row blocks, of 128 and, with one more workgroup to a row
    (4, 14, 28, 4, 128, [2300, 192, 193, 1000], 13),              # group, of 192
    (2, 50, 8, 8, 128, [2046, 64], 11),                           # two row blocks, of 192
])
def test_resident(oracle_mod, B, T, Hq, Hkv, d, lens, splits, paged):
    import gpu_util as gu
    cfg = gen.Config("resident", B, Hq, Hkv, d, T, min(6, T - 1) if T > 1 else 1, 4, 100, 0.5, 1, "bf16", prefix=None, prefix_range=(1, 2), paged=paged)
    inp = gen.attention_inputs(cfg, 600 + T, prefix_len=np.array(lens, dtype=np.int32))
    da = gu.DeviceAttn(inp)
    pl = da.plan()
    assert pl.num_splits == splits and pl.waves_per_group == 8 and pl.keys_per_split <= 256
    if splits > 1:
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


@pytest.mark.gpu
def test_many_rows_to_a_node(oracle_mod):
    """More rows to a node than the short form of the row arithmetic covers."""
    import gpu_util as gu
    cfg = gen.Config("wide", 1, 16400, 1, 64, 2, 1, 4, 100, 0.5, 1, "bf16", prefix=None, prefix_range=(1, 2), paged=False)
    inp = gen.attention_inputs(cfg, 650, prefix_len=np.array([70], dtype=np.int32))
    got = gu.DeviceAttn(inp).run()
    gu.check_close(got, oracle_mod.tree_attention(inp, threads=8), *TIGHT_SHORT)
