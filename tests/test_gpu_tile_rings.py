"""GPU parity of the pipelined kernel's tile rings: every length of the loop's forms (turns of the rings, what is left of one, the
general iterations), block tables longer than a window of 64 tiles, references that move in the middle of the loop, and
shares that end in a sequence whose tree is malformed while its tiles are on their way."""
import numpy as np
import pytest

import gen
import paper_2509_15235_amd as vs

pytestmark = pytest.mark.gpu

TIGHT_LONG = (1.5e-3, 6e-3)
TIGHT_SHORT = (1.2e-2, 6e-3)
# 28 / 4-like heads in eight waves, four waves of 64 channels (rings of six tiles), four of 128 (through registers)
SHAPES = [(128, 16, 2, 33, 8), (64, 16, 2, 33, 8), (64, 4, 2, 40, 4), (128, 4, 2, 40, 4)]


def _inputs(lens, d, Hq, Hkv, T, paged, seed, block_size=16):
    cfg = gen.Config("rings", len(lens), Hq, Hkv, d, T, 6, 4, 100, 0.5, 1, "bf16", prefix=None, prefix_range=(1, 2), paged=paged)
    if paged:
        cfg.block_size = block_size
    return gen.attention_inputs(cfg, seed, prefix_len=np.array(lens, dtype=np.int32))


def _check(oracle_mod, inp, skip=(), tol=None, **kw):
    import gpu_util as gu
    da = gu.DeviceAttn(inp, **kw)
    da.ws.random_(0, 256)
    got = da.run()
    status = da.status.cpu().numpy()
    ref = oracle_mod.tree_attention(inp, threads=8, seqs=[b for b in range(len(inp.prefix_len)) if b not in skip])
    for b, n in enumerate(inp.prefix_len):
        if b in skip:
            assert status[b] != 0
            continue
        assert status[b] == 0
        gu.check_close(got[b], ref[b], *(tol or (TIGHT_LONG if n >= 256 else TIGHT_SHORT)), what=f"sequence {b} of {n}")
    keep = [b for b in range(len(inp.prefix_len)) if b not in skip]
    np.testing.assert_array_equal(got[keep], da.run()[keep])


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("d,Hq,Hkv,T,waves", SHAPES)
def test_every_number_of_tiles(oracle_mod, d, Hq, Hkv, T, waves, paged):
    """0 .. 26 tiles of prefix, whole and with a key less or more: one to three turns of either ring and all that can be left."""
    lens = [max(0, 32 * i + (i % 3) - 1) for i in range(27)] + [32 * i for i in (7, 8, 9, 15, 16, 17, 22, 23, 24)]
    inp = _inputs(lens, d, Hq, Hkv, T, paged, 900 + d + T)
    _check(oracle_mod, inp, schedule=vs.VS_SCHED_PIPELINED, waves_per_group=waves, num_splits=1)


@pytest.mark.parametrize("block_size", [16, 128, 4096])
@pytest.mark.parametrize("d,Hq,Hkv,T,waves", SHAPES)
def test_windows_of_the_block_table(oracle_mod, d, Hq, Hkv, T, waves, block_size):
    """Windows of 64 tiles move on every 32: 1024, 2048 and 3072 keys lie around where they do, in blocks smaller and larger."""
    lens = [1000, 1024, 1183, 2015, 2048, 2207, 3300]
    inp = _inputs(lens, d, Hq, Hkv, T, True, 920 + d + T, block_size)
    _check(oracle_mod, inp, schedule=vs.VS_SCHED_PIPELINED, waves_per_group=waves, num_splits=1)
    _check(oracle_mod, inp, schedule=vs.VS_SCHED_BALANCED, waves_per_group=waves, num_splits=9)


@pytest.mark.parametrize("d,Hq,Hkv,T,waves", SHAPES)
def test_references_that_move(oracle_mod, d, Hq, Hkv, T, waves):
    """Keys that grow along the sequence: the largest score passes the reference by 2^8 over and over."""
    inp = _inputs([900, 700], d, Hq, Hkv, T, False, 940 + d + T)
    k = inp.k_cache * (1.0 + np.arange(inp.k_cache.shape[2], dtype=np.float32)[:, None] / 40.0)
    inp.k_cache, inp.k_bits = gen._store(k, "bf16")
    # a few keys carry all of the weight, so their probabilities' rounding does not average out: half a unit of bf16's last
    # place each, 2^-9, of weights that add up to one, next to the output's own
    tol = (2.0 ** -9 * float(np.nanmax(np.abs(inp.v_cache))) + 1.5e-3, 6e-3)
    _check(oracle_mod, inp, tol=tol, schedule=vs.VS_SCHED_PIPELINED, waves_per_group=waves, num_splits=1)


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("d,Hq,Hkv,T,waves", SHAPES)
def test_shares_with_a_malformed_tree(oracle_mod, d, Hq, Hkv, T, waves, paged):
    lens = [700, 300, 1500, 90, 1100]
    inp = _inputs(lens, d, Hq, Hkv, T, paged, 960 + d + T)
    inp.parent = inp.parent.copy()
    for b in (1, 4):
        inp.parent[b, 5] = 9
    _check(oracle_mod, inp, skip=(1, 4), schedule=vs.VS_SCHED_BALANCED, waves_per_group=waves, num_splits=7)


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("d,Hq,Hkv,T,waves", [(128, 4, 2, 64, 4), (64, 4, 2, 64, 4), (128, 8, 2, 64, 8)])
def test_merges_behind_a_malformed_tree(oracle_mod, d, Hq, Hkv, T, waves, paged):
    """Shares that begin in a sequence which they share and end in a malformed one: all waves have rows, and merge them in LDS
    where the last piece's queries and tiles were on their way to when its tree turned out to be malformed."""
    lens = [n for i in range(8) for n in (700 + 64 * i, 130 + i)]
    inp = _inputs(lens, d, Hq, Hkv, T, paged, 980 + d + waves)
    inp.parent = inp.parent.copy()
    bad = tuple(range(1, 16, 2))
    for b in bad:
        inp.parent[b, 5] = 9
    for shares in (16, 23, 41):
        _check(oracle_mod, inp, skip=bad, schedule=vs.VS_SCHED_BALANCED, waves_per_group=waves, num_splits=shares)
