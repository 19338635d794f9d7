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


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,Hq,Hkv,paged", [(1, 4, 1, False), (6, 32, 8, True)])   # four rows per workgroup, eight
@pytest.mark.parametrize("S", [300, 6, 0])                                        # the tree in two tiles, from a tile's middle on
def test_non_finite_values_stay_with_the_rows_that_see_them(oracle_mod, d, B, Hq, Hkv, paged, S):
    """K and V rows of tree slots with Inf and NaN: a node that does not see such a slot is as if it held zeros."""
    import gpu_util as gu
    T = 24
    cfg = gen.Config("f32", B, Hq, Hkv, d, T, 5, 3, 100, 0.5, 1, "f32", prefix=None, prefix_range=(1, 2), paged=paged)
    inp = gen.attention_inputs(cfg, 812, prefix_len=np.full(B, S, dtype=np.int32))
    _, mask, _ = oracle_mod.tree_mask(inp.parent[0])
    slots = [T - 2, T - 9]
    hides = [i for i in range(T) if not any(int(mask[i]) >> x & 1 for x in slots)]
    sees = [i for i in range(T) if i not in hides]
    assert hides and sees
    for x, k, v in zip(slots, (1.0, np.nan), (np.inf, -np.inf)):
        at = (0, slice(None), S + x) if not paged else (inp.block_table[0, (S + x) // cfg.block_size], slice(None), (S + x) % cfg.block_size)
        inp.k_cache[at] *= np.float32(k)
        inp.v_cache[at + (7,)] = v
        inp.v_cache[at + (d - 1,)] = np.nan
    ref = oracle_mod.tree_attention(inp, threads=8)
    got = gu.DeviceAttn(inp).run()
    gu.check_close(got[0, hides], ref[0, hides], *TIGHT_F32, what="rows that do not see the slots")
    assert np.isnan(got[0, sees][..., d - 1]).all() and not np.isfinite(got[0, sees][..., 7]).any()
    only = [i for i in sees if not int(mask[i]) >> slots[1] & 1]                   # an ordinary key with an infinite value
    other = [c for c in range(d) if c not in (7, d - 1)]
    gu.check_close(got[0, only][..., other], ref[0, only][..., other], *TIGHT_F32, what="their other channels")
    assert (got[0, only][..., 7] == np.inf).all()
    if B > 1:
        gu.check_close(got[1:], ref[1:], *TIGHT_F32, what="the other sequences")
