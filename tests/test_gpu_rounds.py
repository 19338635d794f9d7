"""GPU parity of launches with more whole sequences than run at once: the workgroups take the sequences
longest first."""
import numpy as np
import pytest

import gen
import paper_2509_15235_amd as vs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,Hq,Hkv,d,paged,lens", [
    (40, 60, 28, 4, 128, True, "ragged"),    # eight-wave workgroups, 320 of them
    (64, 40, 28, 4, 64, False, "ragged"),    # a full wave of sequences
    (43, 9, 13, 13, 128, False, "ties"),     # four-wave workgroups, a unit count off the eight XCDs
    (64, 33, 9, 9, 128, True, "one bad"),
])
def test_longest_first(oracle_mod, B, T, Hq, Hkv, d, paged, lens):
    import gpu_util as gu
    r = np.random.default_rng(B + T)
    S = r.integers(1, 400, size=B).astype(np.int32) if lens != "ties" else r.choice([7, 130, 131], size=B).astype(np.int32)
    S[B // 3] = 800                                    # shorter ones are taken in order
    cfg = gen.Config("rounds", B, Hq, Hkv, d, T, min(6, T - 1), 4, 100, 0.5, 1, "bf16", prefix=None, prefix_range=(1, 400),
                     paged=paged)
    inp = gen.attention_inputs(cfg, 700 + B, prefix_len=S)
    da = gu.DeviceAttn(inp, schedule=vs.VS_SCHED_PIPELINED, num_splits=1)
    pl = da.plan()
    assert pl.num_splits == 1 and pl.workgroups > (256 if pl.waves_per_group == 8 else 512)
    bad = None
    if lens == "one bad":
        bad = 11
        da.prefix[bad] = 10 ** 6
    got = da.run()
    st = da.status.cpu().numpy()
    assert [int(x) for x in st] == [3 if b == bad else 0 for b in range(B)]
    seqs = [b for b in sorted({0, 1, B // 2, B - 1, int(S.argmax()), int(S.argmin())}) if b != bad]
    ref = oracle_mod.tree_attention(inp, threads=8, seqs=seqs)
    for b in seqs:
        gu.check_close(got[b], ref[b], 1.2e-2, 6e-3, what=f"sequence {b} of length {S[b]}")
    rest = np.array([b for b in range(B) if b != bad])
    assert np.isfinite(got[rest]).all()
