"""GPU parity of the balanced schedule's merge (the wave that comes last to a row block's pieces): one to many pieces per
sequence, more shares than steps, sequences without a usable length in between, arrival words that hold anything at
first, and one workspace used by calls of different shapes in turn."""
import numpy as np
import pytest

import gen
import paper_2509_15235_amd as vs

pytestmark = pytest.mark.gpu

TIGHT_SHORT = (1.2e-2, 6e-3)


def _inputs(B, T, Hq, Hkv, d, paged, lens, seed):
    cfg = gen.Config("balanced", B, Hq, Hkv, d, T, min(6, T - 1) if T > 1 else 1, 4, 100, 0.5, 1, "bf16", prefix=None, prefix_range=(1, 2),
                     paged=paged)
    return gen.attention_inputs(cfg, seed, prefix_len=np.array(lens, dtype=np.int32))


@pytest.mark.parametrize("B,T,Hq,Hkv,d,paged,lens,shares,waves", [
    (1, 60, 28, 4, 128, True, [4000], 64, 8),                     # one sequence of 64 pieces
    (2, 13, 8, 2, 128, False, [3000, 40], 7, 4),                  # more than three pieces; a ragged last row block
    (2, 9, 8, 1, 64, True, [500, 1500], 4, 8),                    # two and three pieces, three row blocks of 64 channels
    (3, 40, 28, 4, 128, False, [100, 130, 64], 64, 4),            # more shares than steps, three row groups
    (64, 3, 4, 4, 128, True, [37 * i % 900 + 1 for i in range(64)], 64, 4),  # a word for every lane
    (33, 20, 16, 16, 64, False, [61 * i % 700 + 1 for i in range(33)], 11, 4),
    (6, 60, 8, 8, 128, False, [900, 1, 900, 2000, 0, 333], 12, 8),  # a multiple of the sequences: both cuts are priced
])
def test_merge(oracle_mod, B, T, Hq, Hkv, d, paged, lens, shares, waves):
    import gpu_util as gu
    inp = _inputs(B, T, Hq, Hkv, d, paged, lens, 600 + T)
    da = gu.DeviceAttn(inp, schedule=vs.VS_SCHED_BALANCED, num_splits=shares, waves_per_group=waves)
    da.ws.random_(0, 256)
    got = da.run()
    assert (da.status.cpu().numpy() == 0).all()
    gu.check_close(got, oracle_mod.tree_attention(inp, threads=8), *TIGHT_SHORT, what="balanced")
    for _ in range(3):                                             # whoever comes last, the pieces are summed in one order
        np.testing.assert_array_equal(got, da.run())


def test_one_workspace_for_different_shapes(oracle_mod):
    """The arrival words of one call lie among the partial results of another; a bad length and a bad tree in one round."""
    import torch
    import gpu_util as gu
    runs = []
    for k, (B, T, Hq, Hkv, d, lens, shares) in enumerate([(3, 60, 28, 4, 128, [1500, 700, 64], 9), (2, 31, 8, 8, 64, [900, 1111], 5),
                                                          (4, 24, 8, 2, 128, [400, 50, 1111, 800], 16)]):
        inp = _inputs(B, T, Hq, Hkv, d, k == 2, lens, 650 + k)
        runs.append((gu.DeviceAttn(inp, schedule=vs.VS_SCHED_BALANCED, num_splits=shares), oracle_mod.tree_attention(inp, threads=8)))
    ws = torch.zeros(max(da.ws_bytes for da, _ in runs), device="cuda", dtype=torch.uint8)
    for rep in range(4):
        for da, ref in runs:
            da.ws = ws
            if rep == 2:
                good = da.prefix.clone(), da.parent.clone()
                da.prefix[0] = -5
                da.parent[-1, 0] = 3
            got = da.run()
            if rep == 2:
                st = da.status.cpu().numpy()
                assert st[0] == 3 and st[-1] == 1
                da.prefix.copy_(good[0])
                da.parent.copy_(good[1])
            else:
                gu.check_close(got, ref, *TIGHT_SHORT, what=f"pass {rep}")
