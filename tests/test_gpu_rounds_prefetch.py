"""GPU parity of the kernel that runs a split in rounds of 128 keys with two rounds on their way: one to many rounds, ends around
a round, whatever the cache holds behind the last key (NaN), block tables longer than a window, blocks of 16 and 64 tokens."""
import numpy as np
import pytest

import gen
import paper_2509_15235_amd as vs

pytestmark = pytest.mark.gpu

TIGHT_LONG = (1.5e-3, 6e-3)
TIGHT_SHORT = (1.2e-2, 6e-3)


def _run(oracle_mod, B, T, Hq, Hkv, d, paged, lens, seed, block_size=16):
    import gpu_util as gu
    cfg = gen.Config("rounds", B, Hq, Hkv, d, T, min(6, T - 1), 4, 100, 0.5, 1, "bf16", prefix=None, prefix_range=(1, 2), paged=paged)
    if paged:
        cfg.block_size = block_size
    inp = gen.attention_inputs(cfg, seed, prefix_len=np.array(lens, dtype=np.int32))
    da = gu.DeviceAttn(inp)
    pl = da.plan()
    assert pl.schedule == vs.VS_SCHED_LOOP and pl.keys_per_split > 192
    da.ws.random_(0, 256)
    if not paged:
        for b in range(B):                                         # nothing behind a sequence's last key counts
            da.k[b, :, lens[b] + T:] = float("nan")
            da.v[b, :, lens[b] + T:] = float("nan")
    got = da.run()
    assert (da.status.cpu().numpy() == 0).all()
    ref = oracle_mod.tree_attention(inp, threads=8)
    for b in range(B):
        gu.check_close(got[b], ref[b], *(TIGHT_LONG if lens[b] >= 256 else TIGHT_SHORT), what=f"sequence {b} of {lens[b]}")
    for _ in range(3):
        np.testing.assert_array_equal(got, da.run())


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("Hq,Hkv,d,T", [(16, 4, 128, 32), (32, 8, 64, 30), (16, 16, 64, 50), (8, 8, 128, 40)])
def test_ends(oracle_mod, Hq, Hkv, d, T, paged):
    """Last rounds of every kind: full, one key, one tile and a key, none behind a full one."""
    lens = [640 - T + k for k in (0, 1, 127, 128, 129)] + [5, 256 - T, 257 - T, 33, 600, 470, 384 - T, 385 - T, 128 - T, 129 - T, 639 - T]
    lens += [1100 - T] * (1 if Hq != 16 else 0)
    _run(oracle_mod, len(lens), T, Hq, Hkv, d, paged, lens, 410 + T)


@pytest.mark.parametrize("B,T,Hq,Hkv,d,lens,block_size", [
    (16, 16, 28, 4, 128, [5000 - 311 * i for i in range(16)], 16),  # splits of more than a window of 64 blocks
    (16, 31, 32, 8, 64, [4700 - 290 * i for i in range(16)], 64),
    (2, 60, 28, 4, 128, [1696, 1500], 64),
])
def test_tables(oracle_mod, B, T, Hq, Hkv, d, lens, block_size):
    _run(oracle_mod, B, T, Hq, Hkv, d, True, lens, 430 + T, block_size)
