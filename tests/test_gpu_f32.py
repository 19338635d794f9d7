"""GPU parity of the fp32 attention kernel: lengths around its 16-key tiles and one round of eight waves (128
keys), row counts around its eight-row workgroups, both cache layouts, both head sizes."""
import numpy as np
import pytest

import gen

pytestmark = pytest.mark.gpu

TIGHT_F32 = (2e-5, 2e-5)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("T,Hq,Hkv,lens,paged,masks", [
    (1, 1, 1, [0], False, False),                         # one key, one row
    (8, 4, 1, [7, 8, 9], False, True),                    # n = 15, 16, 17
    (3, 6, 2, [109, 125, 126, 141], True, False),         # one tile per wave, one more
    (9, 7, 7, [255, 256, 257, 0], False, False),          # rows 8 + 1
    (64, 2, 1, [1, 400, 64], True, True),
    (31, 8, 2, [600, 333], False, True),
])
def test_tile_edges(oracle_mod, d, T, Hq, Hkv, lens, paged, masks):
    import gpu_util as gu
    cfg = gen.Config("f32", len(lens), Hq, Hkv, d, T, min(6, T - 1), 4, 100, 0.5, 1, "f32", prefix=None, prefix_range=(1, 2),
                     paged=paged)
    inp = gen.attention_inputs(cfg, 800 + T, prefix_len=np.array(lens, dtype=np.int32))
    mask = gu.run_mask(inp.parent)[3] if masks else None
    da = gu.DeviceAttn(inp)
    got = da.run(tree_mask=mask)
    assert (da.status.cpu().numpy() == 0).all()
    gu.check_close(got, oracle_mod.tree_attention(inp, threads=8), *TIGHT_F32, what=f"d {d} T {T}")
    np.testing.assert_array_equal(got, da.run(tree_mask=mask))


def test_bad_inputs_are_reported_and_isolated(oracle_mod):
    import gpu_util as gu
    cfg = gen.Config("f32", 3, 4, 2, 64, 12, 5, 4, 100, 0.5, 1, "f32", prefix=None, prefix_range=(1, 2), paged=True)
    inp = gen.attention_inputs(cfg, 811, prefix_len=np.array([50, 90, 70], dtype=np.int32))
    da = gu.DeviceAttn(inp)
    da.prefix[0] = 91                                     # beyond the host bound
    da.table[1, 2] = inp.n_blocks + 7
    got = da.run()
    assert list(da.status.cpu().numpy()) == [3, 4, 0]
    gu.check_close(got[2], oracle_mod.tree_attention(inp, threads=4)[2], *TIGHT_F32, what="the good sequence")
