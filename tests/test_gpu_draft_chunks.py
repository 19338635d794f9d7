"""GPU parity of the draft expansion where a chunk of logits takes another way to its first K entries: short last chunks
(one wave), plateaus of more entries than the candidate list holds, rows with fewer finite entries than K, NaN."""
import numpy as np
import pytest

from test_gpu_draft_tree import _check_build, _grow_both

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gu():
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("K", [1, 8, 16])
@pytest.mark.parametrize("V", [16, 1023, 1027, 1028, 8192 + 3, 8192 + 1027, 8192 + 1030, 2 * 8192 - 1])
def test_last_chunk(gu, oracle_mod, V, K):
    dd = _grow_both(gu, oracle_mod, 300 + K, 2, V, K, 2)
    _check_build(gu, oracle_mod, dd, 20)


@pytest.mark.parametrize("B,K,V", [
    (3, 16, 4 * 10240 + 1283), (3, 16, 4 * 10240 + 1284), (3, 16, 5 * 10240),     # the second level's 48 rows: chunks of 10240 logits
    (5, 8, 5 * 12288 + 1539), (5, 8, 5 * 12288 + 1540), (5, 8, 5 * 12288 + 1),    # ... 40 rows: chunks of 12288
    (1, 7, 33 * 8192 - 5), (1, 9, 17 * 8192 + 2), (2, 1, 30000),                  # more lists than are on their way at once; lists of one
])
def test_long_chunks(gu, oracle_mod, B, K, V):
    dd = _grow_both(gu, oracle_mod, 330 + K, B, V, K, 2)
    _check_build(gu, oracle_mod, dd, min(40, K + K * K))


@pytest.mark.parametrize("V,count", [(8192, 127), (8192, 128), (8192, 129), (1000, 129), (9000, 8192)])
def test_plateaus(gu, oracle_mod, V, count):
    """`count` equal maxima in the first chunk: around the list's 128 entries."""
    def mutate(level, logits):
        logits[:, :, :min(count, V)] = np.float32(30.0)
        logits[:, 1:, 5] = np.float32(31.0)
    dd = _grow_both(gu, oracle_mod, 310, 2, V, 12, 2, mutate=mutate)
    _check_build(gu, oracle_mod, dd, 30)


@pytest.mark.parametrize("V,finite", [(9000, 16), (9000, 17), (8192, 40), (700, 16)])
def test_few_finite(gu, oracle_mod, V, finite):
    def mutate(level, logits):
        keep = logits[:, :, 3:3 + finite].copy()
        logits[:] = -np.inf
        # far below 0, but not so far that the log-sum-exp, a float near the entries, is rounded by what a score may differ
        # by: at most 2^-18 = 4e-6 below 128 (3e-5 at 1000)
        logits[:, :, 3:3 + finite] = -90.0 + keep
    dd = _grow_both(gu, oracle_mod, 320, 2, V, 16, 2, mutate=mutate)
    _check_build(gu, oracle_mod, dd, 30)


def test_nan_is_never_taken(gu, oracle_mod):
    """A row with a NaN has NaN scores (as in the sum of exp), its tokens are those of the other entries, and the next
    frontier is what the other rows give."""
    import gen
    F, K, V = 4, 4, 9000
    dd = gu.DeviceDraft(1, K, F * K)
    logits = gen.draft_logits(33, 0, 1, F, V)[None].copy()
    clean = logits.copy()
    logits[0, 2, 4321] = np.nan
    clean[0, 2, 4321] = -np.inf
    cum = np.zeros((1, F), np.float32)
    nf, nc = dd.expand(logits, gu.dev(cum), gu.dev(np.arange(F, dtype=np.int32)[None]), garbage=True)
    rc, tok, sc, fr, gap = oracle_mod.draft_expand_seq(clean[0], cum[0], K)
    np.testing.assert_array_equal(dd.tok.cpu().numpy()[0], tok)
    got = dd.score.cpu().numpy()[0].reshape(F, K)
    assert np.isnan(got[2]).all() and np.isfinite(got[[0, 1, 3]]).all()
    others = [c for c in range(F * K) if c // K != 2]
    best = sorted(sorted(others, key=lambda c: (-got.reshape(-1)[c], c))[:K])
    np.testing.assert_array_equal(nf.cpu().numpy()[0], best)
