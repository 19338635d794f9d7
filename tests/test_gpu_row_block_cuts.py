"""Cuts of short calls into few row blocks per workgroup of the LDS-resident kernel, or of the one whose waves have tiles of their
own: every number of row blocks with every number of tiles, one split or several merged by their workgroups, row blocks and keys that end inside the last one, on a workspace
of garbage and on one without room for the gates of the finer cut."""
import numpy as np
import pytest

import gen
import paper_2509_15235_amd as vs

TIGHT_LONG = (1.5e-3, 6e-3)
TIGHT_SHORT = (1.2e-2, 6e-3)

CUTS = [  # B, T, Hq, Hkv, d, keys, (row groups, keys per split, splits)
    (1, 5, 28, 4, 128, 60, (2, 64, 1)),         # one row block, one split: a tile,
    (4, 60, 28, 4, 128, 128, (14, 128, 1)),     # two,
    (3, 37, 32, 8, 64, 129, (5, 192, 1)),       # three,
    (1, 60, 32, 32, 128, 255, (2, 256, 1)),     # four
    (16, 28, 8, 2, 128, 250, (4, 256, 1)),
    (26, 37, 8, 1, 128, 39, (5, 64, 1)),        # two row blocks, one split: a tile,
    (17, 61, 8, 1, 128, 72, (8, 128, 1)),       # two,
    (8, 43, 28, 4, 128, 129, (5, 192, 1)),      # three, four
    (16, 31, 32, 8, 64, 256, (2, 256, 1)),
    (1, 25, 28, 4, 128, 350, (6, 64, 6)),       # one row block, splits of a tile,
    (2, 20, 28, 4, 128, 700, (5, 128, 6)),      # two,
    (1, 28, 8, 2, 128, 2133, (4, 128, 17)),
    (4, 44, 8, 2, 128, 711, (6, 192, 4)),       # three,
    (1, 32, 28, 4, 64, 2195, (7, 256, 9)),      # four
    (1, 60, 28, 4, 128, 460, (7, 64, 8)),       # two row blocks, splits of a tile,
    (8, 29, 8, 2, 128, 439, (2, 64, 7)),
    (2, 30, 28, 4, 128, 1000, (4, 128, 8)),     # two,
    (4, 45, 40, 8, 128, 309, (4, 192, 2)),      # three, in place of the pipelined kernel,
    (4, 39, 28, 4, 128, 601, (5, 256, 3)),      # four
    (8, 47, 40, 8, 128, 369, (2, 192, 2)),      # four row blocks in place of the pipelined kernel;
    (10, 60, 28, 4, 64, 64, (4, 64, 1)),        # one split: a tile,
    (34, 61, 8, 1, 128, 65, (4, 128, 1)),       # two,
    (34, 62, 8, 1, 128, 134, (4, 192, 1)),      # three;
    (11, 63, 8, 1, 128, 279, (4, 64, 5)),       # splits of a tile,
    (11, 61, 8, 1, 128, 323, (4, 128, 3)),      # two,
    (2, 60, 8, 1, 128, 2068, (4, 128, 17)),     # ... more than sixteen of them
    (16, 9, 28, 4, 128, 257, (2, 320, 1)),      # one row block, tiles of the wave's own
    (4, 40, 32, 32, 128, 320, (2, 320, 1)),
]


def _desc(B, T, Hq, Hkv, d, keys):
    cap = keys + 16
    return vs.AttnDesc(B=B, T=T, Hq=Hq, Hkv=Hkv, d=d, dtype=vs.VS_BF16, softmax_scale=0.1, max_prefix_len=keys - T, capacity=cap,
                       stride_seq=Hkv * cap * d, stride_head=cap * d, stride_tok=d)


def test_the_cuts():
    for *shape, cut in CUTS:
        desc = _desc(*shape)
        rc, pl = vs.vs_attention_plan(desc)
        assert rc == 0 and (pl.row_groups, pl.keys_per_split, pl.num_splits) == cut, (shape, pl.row_groups, pl.keys_per_split, pl.num_splits)
        assert pl.workgroups == shape[0] * shape[3] * cut[0] * cut[2] <= 256
        B, T, Hq, Hkv, d, _ = shape
        rows = -(-T * Hq // Hkv // 32) * 32
        assert vs.vs_attention_workspace_bytes(desc) == (B * Hkv * (cut[2] * rows * (2 * d + 8) + cut[0] * 256) if cut[2] > 1 else 0)


@pytest.mark.gpu
@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("B,T,Hq,Hkv,d,keys,cut", CUTS)
def test_results(oracle_mod, B, T, Hq, Hkv, d, keys, cut, paged):
    import gpu_util as gu
    lens = np.array([max(0, keys - T - 65 * b) for b in range(B)], dtype=np.int32)
    cfg = gen.Config("cuts", B, Hq, Hkv, d, T, min(6, T - 1), 4, 100, 0.5, 1, "bf16", prefix=None, prefix_range=(1, 2), paged=paged)
    inp = gen.attention_inputs(cfg, 1100 + T, prefix_len=lens)
    da = gu.DeviceAttn(inp)
    assert (da.plan().row_groups, da.plan().keys_per_split, da.plan().num_splits) == cut
    if not paged:
        for b in range(B):                                        # nothing behind a sequence's last key counts
            da.k[b, :, lens[b] + T:] = float("nan")
            da.v[b, :, lens[b] + T:] = float("nan")
    ref = oracle_mod.tree_attention(inp, threads=8)

    def check():
        da.ws.random_(0, 256)
        got = da.run()
        assert (da.status.cpu().numpy() == 0).all()
        for b in range(B):
            gu.check_close(got[b], ref[b], *(TIGHT_LONG if lens[b] >= 256 else TIGHT_SHORT), what=f"sequence {b} of {lens[b]}")
        np.testing.assert_array_equal(got, da.run())
    check()
    gates = B * Hkv * 256 * cut[0]
    if cut[2] > 1 and cut[:2] == (5, 256):                        # the cut that it replaced: no gates, as many splits
        da.ws_bytes -= gates
        check()
        da.ws_bytes -= 256
        with pytest.raises(AssertionError):
            da.run()
