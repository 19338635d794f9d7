"""GPU parity of both acceptance calls at the ends of their chunks of 8192 logits (and of the 4096 that 256 threads scan), and of the
stochastic walk over wide trees: many siblings, repeated and impossible tokens, a rejected token that holds nearly all the mass."""
import numpy as np
import pytest

import test_gpu_accept_sample as base

pytestmark = pytest.mark.gpu
gu = base.gu

EDGES = [1, 2, 3, 4, 5, 15, 17, 4093, 4095, 4096, 4097, 8189, 8191, 8192, 8193, 8195, 16383, 16386, 24577]


@pytest.mark.parametrize("V", EDGES)
def test_greedy_at_chunk_ends(gu, oracle_mod, V):
    r = np.random.default_rng(V)
    B, T = 3, 5
    parent = np.tile(np.array([-1, 0, 0, 1, 1], dtype=np.int32), (B, 1))
    logits = r.standard_normal((B, T, V)).astype(np.float32)
    at = [i for i in (0, 1, 4095, 4096, 8191, 8192, 16383, 16384, V - 2, V - 1) if 0 <= i < V]
    for b in range(B):
        for t in range(T):                                        # equal maxima around the ends: the first counts
            logits[b, t, r.choice(at, size=min(2, len(at)), replace=False)] = 9.0
    logits[0, 4, :] = -np.inf                                     # nothing above -inf: index 0
    logits[1, 2, 0] = np.nan                                      # a NaN in column 0 is never displaced
    tokens = np.zeros((B, T), dtype=np.int32)
    tokens[:, 1] = logits[:, 0].argmax(-1)
    tokens[:, 3] = logits[:, 1].argmax(-1)
    for ld, off in ((V, 0), (V + 3, 1)):
        got = gu.run_accept(logits, tokens, parent, ld=ld, offset_elems=off)
        want = oracle_mod.tree_accept(logits, tokens, parent)
        for g, w in zip(got, want):
            np.testing.assert_array_equal(g, w)


@pytest.mark.parametrize("T,V", [(16, 1024), (16, 1023), (17, 1024), (16, 1025), (5, 3072), (5, 3073), (1, 16384), (1, 16385), (8, 2047), (3, 4099)])
def test_greedy_of_few_logits(gu, oracle_mod, T, V):
    """One kernel up to sixteen pieces of 1024 logits, and just beyond: chains and wide trees, maxima at the pieces' ends."""
    r = np.random.default_rng(T * V)
    B = 5
    parent = np.stack([np.array([-1] + [int(r.integers(max(0, i - 1 - b), i)) for i in range(1, T)], dtype=np.int32) for b in range(B)])
    logits = r.standard_normal((B, T, V)).astype(np.float32)
    at = [i for k in range(0, V + 1024, 1024) for i in (k - 1, k, k + 1) if 0 <= i < V] + [V - 1]
    for b in range(B):
        for t in range(T):
            logits[b, t, r.choice(at, size=min(2, len(at)), replace=False)] = 9.0
    logits[0, T - 1, :] = -np.inf
    logits[1, T // 2, 0] = np.nan
    tokens = np.zeros((B, T), dtype=np.int32)
    tokens[:, 1:] = np.take_along_axis(logits.argmax(-1), np.maximum(parent[:, 1:], 0), axis=1)
    tokens[2, T // 2] += 1
    for ld, off in ((V, 0), (V + 3, 1)):
        got = gu.run_accept(logits, tokens, parent, ld=ld, offset_elems=off)
        want = oracle_mod.tree_accept(logits, tokens, parent)
        for g, w in zip(got, want):
            np.testing.assert_array_equal(g, w)


@pytest.mark.parametrize("V", EDGES)
def test_sampling_at_chunk_ends(gu, oracle_mod, V):
    B, T = 6, 5 if V >= 5 else 1
    if T > 1:
        parent, tokens, logits, ua, ub = base._case(500 + V, B, T, V, max_depth=2, max_children=2)
    else:
        r = np.random.default_rng(V)
        parent, tokens = np.full((B, 1), -1, dtype=np.int32), np.zeros((B, 1), dtype=np.int32)
        logits, ua, ub = r.standard_normal((B, 1, V)).astype(np.float32), r.random((B, 1)), r.random(B)
    ua, ub = np.asarray(ua, dtype=np.float32), np.asarray(ub, dtype=np.float32)
    ub[0], ub[1] = 0.0, np.float32(1.0 - 2.0 ** -24)               # the first and the last token with weight
    for ld, off in ((V, 0), (V + 3, 1)):
        base._check(gu, oracle_mod, logits, tokens, parent, 0.9, ua, ub, min_exact_frac=0.6, ld=ld, offset_elems=off)


@pytest.mark.parametrize("V,heavy", [(700, False), (700, True), (20000, False), (20000, True)])
def test_wide_trees(gu, oracle_mod, V, heavy):
    """A root with 40 children and one of them with 20 more; tokens repeat and some are no tokens at all. heavy: a child that holds
    99 % of the root's mass is rejected, so that the masses behind it come from the chunks."""
    r = np.random.default_rng(V + heavy)
    B, T = 12, 61
    parent = np.array([[-1] + [0] * 40 + [7] * 20] * B, dtype=np.int32)
    tokens = r.integers(0, V, size=(B, T)).astype(np.int32)
    tokens[:, 12], tokens[:, 30], tokens[:, 55] = tokens[:, 5], tokens[:, 5], tokens[:, 50]
    tokens[:, 20], tokens[:, 45] = -1, V
    logits = (2 * r.standard_normal((B, T, V))).astype(np.float32)
    for b in range(B):
        logits[b, 0, tokens[b, 7]] = np.log(V) + 2.0 + b % 3
        if heavy:
            logits[b, 0, tokens[b, 3]] = np.log(V) + 9.0
    ua, ub = r.random((B, T)).astype(np.float32), r.random(B).astype(np.float32)
    ua[:, 3] = 0.9999
    ua[: B // 2, 1:41] = np.maximum(ua[: B // 2, 1:41], np.float32(0.98))  # most are rejected
    base._check(gu, oracle_mod, logits, tokens, parent, 1.0, ua, ub, min_exact_frac=0.6)


@pytest.mark.parametrize("T,V", [(64, 262144), (16, 130 * 8192), (16, 130 * 8192 + 1)])
def test_sampling_at_the_end_of_the_walks_own_memory(gu, oracle_mod, T, V):
    """The walk keeps 2080 chunk results of a sequence in LDS and reads more than that from memory: 2048, 2080 and 2096 of them."""
    parent, tokens, logits, ua, ub = base._case(700 + T, 1, T, V)
    base._check(gu, oracle_mod, logits, tokens, parent, 1.0, ua, ub, min_exact_frac=0.0)


@pytest.mark.parametrize("B,T,V", [(11, 60, 8193), (10, 64, 8193), (11, 60, 12288), (11, 60, 12289), (11, 59, 8995), (3, 54, 57345), (3, 53, 57345),
                                   (3, 54, 61440), (3, 54, 61441)])
def test_large_launches_of_rows_that_end_in_a_short_chunk(gu, oracle_mod, B, T, V):
    """Two or eight chunks of 8192 a row, the last at most half full, and more than 1280 of them in all: chunks of 4096 instead."""
    parent, tokens, logits, ua, ub = base._case(800 + T, B, T, V)
    r = np.random.default_rng(V)
    ub[0], ub[1] = 0.0, np.float32(1.0 - 2.0 ** -24)
    base._check(gu, oracle_mod, logits, tokens, parent, 1.0, ua, ub, min_exact_frac=0.6, ld=V + 3, offset_elems=1)
    at = [i for k in range(0, V + 4096, 4096) for i in (k - 1, k, k + 1) if 0 <= i < V] + [V - 1]
    for b in range(B):
        for t in range(T):                                        # equal maxima around the ends: the first counts
            logits[b, t, r.choice(at, size=2, replace=False)] = 19.0
    tokens[:, 1:] = np.take_along_axis(logits.argmax(-1), np.maximum(parent[:, 1:], 0), axis=1)
    got = gu.run_accept(logits, tokens, parent, ld=V + 3, offset_elems=1)
    for g, w in zip(got, oracle_mod.tree_accept(logits, tokens, parent)):
        np.testing.assert_array_equal(g, w)
