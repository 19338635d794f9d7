"""GPU parity of the attention kernel that runs a split in rounds of 128 keys (the planner's choice for few units
or few row blocks): lengths around rounds and splits, one to several row groups, block-table windows, and the
merge of the splits by their own workgroups on a workspace full of garbage."""
import numpy as np
import pytest

import gen
import paper_2509_15235_amd as vs

pytestmark = pytest.mark.gpu

TIGHT_LONG = (1.5e-3, 6e-3)
TIGHT_SHORT = (1.2e-2, 6e-3)


@pytest.mark.parametrize("B,T,Hq,Hkv,d,paged,lens", [
    (2, 60, 28, 4, 128, False, [1696, 1500]),                    # four row groups, two rounds per split
    (2, 60, 28, 4, 128, True, [1600, 1]),                        # most splits without a key
    (4, 33, 12, 4, 64, False, [1100, 127, 128, 129]),             # four row blocks, 64 channels
    (4, 16, 28, 4, 128, True, [1296, 1000, 3, 511]),
    (2, 50, 8, 8, 128, False, [2000, 1234]),                     # two row blocks
    (3, 33, 6, 6, 64, True, [900, 77, 640]),
    (1, 9, 8, 1, 128, True, [40001]),                            # splits beyond a block-table window
    (1, 9, 8, 1, 64, True, [33000]),
    (1, 64, 9, 1, 128, False, [5000]),                           # five row groups
    (16, 20, 16, 4, 128, False, [37 * i + 1 for i in range(16)]),  # one split per unit or a few, ends everywhere
    (3, 60, 28, 4, 128, False, [196, 133, 0]),                   # one split of two rounds, four row groups
    (8, 31, 32, 8, 64, True, [225, 162, 163, 96, 97, 98, 1, 33]),  # ... four row blocks of 64 channels, ends around a round
])
def test_rounds(oracle_mod, B, T, Hq, Hkv, d, paged, lens):
    import gpu_util as gu
    cfg = gen.Config("rounds", B, Hq, Hkv, d, T, min(6, T - 1), 4, 100, 0.5, 1, "bf16", prefix=None, prefix_range=(1, 2),
                     paged=paged)
    inp = gen.attention_inputs(cfg, 900 + T, prefix_len=np.array(lens, dtype=np.int32))
    da = gu.DeviceAttn(inp)
    assert da.plan().schedule == vs.VS_SCHED_LOOP and da.plan().waves_per_group == 8
    da.ws.random_(0, 256)                                        # the merge's words start as anything
    got = da.run()
    assert (da.status.cpu().numpy() == 0).all()
    ref = oracle_mod.tree_attention(inp, threads=8)
    for b in range(B):
        gu.check_close(got[b], ref[b], *(TIGHT_LONG if lens[b] >= 256 else TIGHT_SHORT), what=f"sequence {b} of {lens[b]}")
    for _ in range(3):
        np.testing.assert_array_equal(got, da.run())


@pytest.mark.parametrize("B,T,Hq,Hkv,d,paged,lens", [
    (12, 62, 28, 4, 128, False, [76, 1, 130, 40, 64, 100, 2, 99, 63, 65, 128, 127]),  # one split, many units
    (4, 14, 28, 4, 128, True, [120, 0, 178, 33]),
    (8, 10, 32, 8, 64, False, [120, 1, 60, 182, 64, 65, 100, 3]),                      # two row blocks
    (1, 60, 28, 4, 128, True, [400]),                                                  # splits of 64 keys
    (2, 9, 28, 4, 128, False, [1400, 70]),
    (1, 19, 8, 1, 64, True, [2029]),                                                   # 32 of them
])
def test_short_sequences(oracle_mod, B, T, Hq, Hkv, d, paged, lens):
    """The resident kernel with one split, or splits of 64 keys."""
    import gpu_util as gu
    cfg = gen.Config("short", B, Hq, Hkv, d, T, min(6, T - 1), 4, 100, 0.5, 1, "bf16", prefix=None, prefix_range=(1, 2), paged=paged)
    inp = gen.attention_inputs(cfg, 800 + T, prefix_len=np.array(lens, dtype=np.int32))
    da = gu.DeviceAttn(inp)
    pl = da.plan()
    tiles = (max(lens) + T + 63) // 64
    assert pl.schedule == vs.VS_SCHED_RESIDENT and pl.num_splits == (1 if tiles <= 3 else tiles)
    da.ws.random_(0, 256)
    got = da.run()
    assert (da.status.cpu().numpy() == 0).all()
    ref = oracle_mod.tree_attention(inp, threads=8)
    for b in range(B):
        gu.check_close(got[b], ref[b], *(TIGHT_LONG if lens[b] >= 256 else TIGHT_SHORT), what=f"sequence {b} of {lens[b]}")
    for _ in range(3):
        np.testing.assert_array_equal(got, da.run())


def test_merge_words_between_calls(oracle_mod):
    """Calls of different shapes and lengths in turn on one workspace (the words of one lie in the partial results
    of the other), sequences with a bad length or tree among them, then the good ones again."""
    import torch
    import gpu_util as gu
    runs = []
    for k, (B, T, Hq, Hkv, lens) in enumerate([(2, 60, 28, 4, [1696, 900]), (1, 60, 28, 4, [1696]), (3, 24, 8, 2, [400, 50, 1111])]):
        cfg = gen.Config("mix", B, Hq, Hkv, 128, T, 5, 4, 100, 0.5, 1, "bf16", prefix=None, prefix_range=(1, 2), paged=False)
        inp = gen.attention_inputs(cfg, 950 + k, prefix_len=np.array(lens, dtype=np.int32))
        runs.append((gu.DeviceAttn(inp), oracle_mod.tree_attention(inp, threads=8)))
    ws = torch.zeros(max(da.ws_bytes for da, _ in runs), device="cuda", dtype=torch.uint8)
    good = None
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
                assert (st[0] == 3 or len(st) == 1) and st[-1] in (1, 3)
                da.prefix.copy_(good[0])
                da.parent.copy_(good[1])
            else:
                for b in range(len(ref)):
                    gu.check_close(got[b], ref[b], *TIGHT_SHORT, what=f"pass {rep} sequence {b}")


def _hand_over(da, gates, want):
    """Four calls in which nobody waits, equal to `want`, with shares handed over; and one as usual."""
    import torch
    words = da.ws[da.ws_bytes - gates * 256:da.ws_bytes].view(torch.int64).view(gates, 32)   # behind the partial results, 256 bytes each
    handed = []
    try:
        vs.lib().vs_internal_set_merge_wait(0)
        for _ in range(4):
            words.zero_()
            np.testing.assert_array_equal(da.run(), want)
            handed.append(int(words[:, 24].sum()))   # every gate's count of shares handed over
            at_rest = words[:, 0] == (0xffc3a9 << 40) - (1 << 64)
            assert (at_rest | (words[:, 0] == 0)).all() and at_rest.any()   # (sequences of one split leave theirs alone)
    finally:
        vs.lib().vs_internal_set_merge_wait(2000)
    assert sum(handed) > 0, handed   # (in every call but where all splits arrive within a trip to memory)
    np.testing.assert_array_equal(da.run(), want)


@pytest.mark.parametrize("kw", [{}, dict(schedule=vs.VS_SCHED_RESIDENT), dict(schedule=vs.VS_SCHED_PIPELINED, waves_per_group=8, num_splits=10),
                                dict(schedule=vs.VS_SCHED_PIPELINED, waves_per_group=4, num_splits=7)])
def test_shares_handed_over(oracle_mod, kw):
    """Nobody waits at the gate: every workgroup but a row group's last one leaves its share of the merge to it."""
    import gpu_util as gu
    cfg = gen.Config("handover", 2, 28, 4, 128, 60, 6, 4, 100, 0.5, 1, "bf16", prefix=None, prefix_range=(1, 2), paged=False)
    inp = gen.attention_inputs(cfg, 970, prefix_len=np.array([1100, 421], dtype=np.int32))
    da = gu.DeviceAttn(inp, **kw)
    pl = da.plan()
    assert pl.num_splits > 1 and pl.combine == 1
    assert da.ws_bytes == 2 * 4 * pl.num_splits * 448 * (128 * 2 + 8) + 2 * 4 * pl.row_groups * 256   # partial results and gates
    want = da.run()
    _hand_over(da, 2 * 4 * pl.row_groups, want)


@pytest.mark.parametrize("Hq,Hkv,T,lens,wgs", [(28, 4, 60, [1100, 421, 2000], 216),      # eight waves, nine splits, two row groups
                                               (28, 4, 60, [3000, 421, 64, 1100, 2900, 2100, 3136, 1], 256),  # four splits
                                               (32, 32, 60, [2900], 256)])                # four waves
def test_shares_of_the_pipelined_kernel_handed_over(oracle_mod, Hq, Hkv, T, lens, wgs):
    """The same where the planner lets the pipelined kernel merge its own splits."""
    import gpu_util as gu
    cfg = gen.Config("handover", len(lens), Hq, Hkv, 128, T, 6, 4, 100, 0.5, 1, "bf16", prefix=None, prefix_range=(1, 2), paged=False)
    inp = gen.attention_inputs(cfg, 971, prefix_len=np.array(lens, dtype=np.int32))
    da = gu.DeviceAttn(inp)
    pl = da.plan()
    assert pl.schedule == vs.VS_SCHED_PIPELINED and pl.workgroups == wgs and pl.combine == 1
    partials = len(lens) * Hkv * pl.num_splits * (-(-T * Hq // Hkv // 32) * 32) * (128 * 2 + 8)
    assert da.ws_bytes == partials + len(lens) * Hkv * pl.row_groups * 256   # the gates
    da.ws.random_(0, 256)
    want = da.run()
    ref = oracle_mod.tree_attention(inp, threads=8)
    for b in range(len(lens)):
        gu.check_close(want[b], ref[b], *(TIGHT_LONG if lens[b] >= 256 else TIGHT_SHORT), what=f"sequence {b} of {lens[b]}")
    _hand_over(da, len(lens) * Hkv * pl.row_groups, want)


@pytest.mark.parametrize("T,Hq,Hkv,d,paged,lens", [(62, 16, 1, 128, True, [7875]), (58, 8, 1, 64, False, [7879, 1001]),        # four row blocks,
                                                   (19, 28, 4, 128, True, [7662]),                                             # a last split of one key
                                                   (8, 8, 1, 128, False, [11897, 3, 640, 11513, 1000, 7850, 2, 5000]),         # two
                                                   (3, 28, 4, 128, True, [15870, 1200]), (4, 8, 1, 64, False, [15869] * 3 + [900, 1, 15357, 15356, 3000])])  # own tiles
def test_crowds_at_a_gate(oracle_mod, T, Hq, Hkv, d, paged, lens):
    """28 splits and more on nearly all CUs, whose workgroups look at a second word."""
    import torch
    import gpu_util as gu
    cfg = gen.Config("crowd", len(lens), Hq, Hkv, d, T, min(6, T - 1), 4, 100, 0.5, 1, "bf16", prefix=None, prefix_range=(1, 2), paged=paged)
    inp = gen.attention_inputs(cfg, 980, prefix_len=np.array(lens, dtype=np.int32))
    da = gu.DeviceAttn(inp)
    pl = da.plan()
    assert pl.schedule == vs.VS_SCHED_LOOP and pl.waves_per_group == 8 and pl.num_splits >= 28 and pl.workgroups >= 224
    assert pl.keys_per_split >= (320 if T == 8 else 256)   # fewer keys are the resident kernel's
    da.ws.random_(0, 256)
    want = da.run()
    ref = oracle_mod.tree_attention(inp, threads=8)
    for b in range(len(lens)):
        gu.check_close(want[b], ref[b], *(TIGHT_LONG if lens[b] >= 256 else TIGHT_SHORT), what=f"sequence {b} of {lens[b]}")
    for _ in range(3):
        np.testing.assert_array_equal(want, da.run())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        for _ in range(2):                           # the second one finds the words as the first one left them
            assert vs.vs_tree_verify_attention(da.desc, da.q, da.k, da.v, da.prefix, da.parent, None, da.out, da.status, da.ws, da.ws_bytes,
                                               torch.cuda.current_stream().cuda_stream) == 0
    for rep in range(4):
        da.out.fill_(float("nan"))
        if rep % 2:
            da.ws.random_(0, 256)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(want, da.out.float().cpu().numpy().astype(np.float64), err_msg=f"replay {rep}")
        np.testing.assert_array_equal(want, da.run())
    _hand_over(da, len(lens) * Hkv * pl.row_groups, want)
