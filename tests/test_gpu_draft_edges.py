"""GPU parity of the draft expansion around the edges of its 8192-float chunks, at the largest frontiers, with
signed zeros and banned tokens, and of the final selection where few or very many candidates reach its bound."""
import numpy as np
import pytest

import gen
from test_gpu_draft_tree import _check_build, _grow_both

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gu():
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("V,K,D,N,ld,offset", [
    (8192, 3, 2, 9, 8192, 0), (8193, 16, 3, 63, 8193, 3), (8189, 8, 2, 20, 8191, 1), (16387, 13, 2, 40, 16388, 2),
    (300001, 16, 2, 63, 300001, 1),                          # merged lists of more than 256 entries
])
def test_chunk_edges(gu, oracle_mod, V, K, D, N, ld, offset):
    dd = _grow_both(gu, oracle_mod, 900 + K, 2, V, K, D, ld=ld, offset_elems=offset)
    _check_build(gu, oracle_mod, dd, N)


def test_largest_frontier(gu, oracle_mod):
    """64 rows of 16 children: 1024 candidates in one step, on a workspace full of garbage."""
    F, K, V = 64, 16, 700
    dd = gu.DeviceDraft(2, K, F * K)
    logits = np.stack([gen.draft_logits(31, b, 1, F, V) for b in range(2)])
    cum = -np.arange(F, dtype=np.float32)[None].repeat(2, 0) * 0.01
    nf, nc = dd.expand(logits, gu.dev(cum), gu.dev(np.arange(2 * F, dtype=np.int32).reshape(2, F)), garbage=True)
    for b in range(2):
        rc, tok, sc, fr, gap = oracle_mod.draft_expand_seq(logits[b], cum[b], K)
        assert rc == 0
        np.testing.assert_array_equal(dd.tok.cpu().numpy()[b], tok)
        np.testing.assert_allclose(dd.score.cpu().numpy()[b], sc, rtol=0, atol=3e-5)
        if gap > 6e-5:
            np.testing.assert_array_equal(nf.cpu().numpy()[b], fr)


def test_zeros_and_banned_tokens(gu, oracle_mod):
    """Signed zeros are ties (lower token first); rows with hardly a finite entry."""
    def mutate(level, logits):
        logits[:, :, :] = -np.inf
        logits[:, :, 5000:5006] = [-0.0, 0.0, -0.0, 1.0, 0.0, -2.0]
        logits[:, 0, 17] = 3.0
    dd = _grow_both(gu, oracle_mod, 41, 2, 9000, 5, 2, mutate=mutate)
    _check_build(gu, oracle_mod, dd, 12)


@pytest.mark.parametrize("M,N,kind", [(2048, 63, "plateau"), (700, 63, "plateau"), (2048, 1, "distinct"), (64, 63, "distinct"), (63, 63, "distinct")])
def test_selection_bounds(gu, oracle_mod, M, N, kind):
    r = np.random.default_rng(M + N)
    dd = gu.DeviceDraft(1, 4, M)
    dd.M = M
    sc = np.full((1, M), -1.5, np.float32) if kind == "plateau" else -np.abs(r.standard_normal((1, M))).astype(np.float32)
    dd.tok.copy_(gu.dev(r.integers(0, 999, (1, M)).astype(np.int32)))
    dd.score.copy_(gu.dev(sc))
    dd.par.copy_(gu.dev(np.full((1, M), -1, np.int32)))
    _check_build(gu, oracle_mod, dd, N)


@pytest.mark.parametrize("scores,N", [
    ([-0.0, 0.0, 0.0, -1.0], 2),                                 # the first two of three equal scores
    ([-0.0] * 70 + [0.0] * 70, 63),
    ([0.0, -0.0] * 1024, 63),                                    # a plateau of more entries than are ranked as a list
    ([-1.0] * 300 + [0.0, -0.0, -0.0, 0.0, -0.0] * 9, 40),
])
def test_signed_zero_scores(gu, oracle_mod, scores, N):
    """Scores -0 and +0 are equal: the earlier candidate comes first whichever sign it has, also as the
    parent of a later one."""
    M = len(scores)
    dd = gu.DeviceDraft(1, 4, M)
    dd.M = M
    par = np.full((1, M), -1, np.int32)
    par[0, M // 2:] = np.arange(M - M // 2) // 2 if M <= 4 else -1
    dd.tok.copy_(gu.dev(np.arange(M, dtype=np.int32)[None]))
    dd.score.copy_(gu.dev(np.array([scores], np.float32)))
    dd.par.copy_(gu.dev(par))
    _check_build(gu, oracle_mod, dd, N)
