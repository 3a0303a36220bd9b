"""The encoder where its pieces meet: chunks so crowded that their codes do not fit their words, unary
runs over many words, words that several chunks share, streams of one word, and calls around the numbers
of chunks at which the scan over them changes its form.  Every round against the oracle, bit for bit."""
import numpy as np
import pytest

from parity_util import DeviceRun, check_round

pytestmark = pytest.mark.gpu

CHUNK = 8192


def _planted(n, at, seed):
    """Small values everywhere, the entries `at` far larger (positive side)."""
    g = np.random.default_rng(seed)
    x = (g.standard_normal(n) * 1e-3).astype(np.float32)
    x[at] = (1.0 + g.random(len(at))).astype(np.float32)
    return x


def _spread(n, k, seed):
    return np.sort(np.random.default_rng(seed).choice(n, k, replace=False))


def _at(kind, n, k):
    if kind == "first_chunk":                             # all kept entries in one chunk: far more bits than it has words
        return np.arange(k)
    if kind == "last_entries":                            # a unary run over the whole tensor, then no gaps
        return np.arange(n - k, n)
    if kind == "middle_chunk":
        return CHUNK * 17 + 100 + np.arange(k)
    if kind == "crowded_and_sparse":                      # crowded chunks next to ones with an entry or none
        a = np.concatenate([np.arange(CHUNK * 3, CHUNK * 3 + k // 2), np.arange(CHUNK * 5 + 1, CHUNK * 5 + 1 + k // 2 - 2),
                            [CHUNK * 4 + 8191, CHUNK * 30]])
        return np.concatenate([a, CHUNK * 20 + np.arange(k - len(a))])
    return np.minimum(np.arange(k) * (n // k) + np.random.default_rng(k).integers(0, n // k, k), n - 1)     # one every n / k entries


@pytest.mark.parametrize("p,chunks", [(0.02, 40), (0.1, 33), (0.45, 5), (1.2e-4, 200), (3e-5, 400), (1e-3, 300)])
@pytest.mark.parametrize("kind", ["first_chunk", "last_entries", "middle_chunk", "crowded_and_sparse", "even"])
def test_chunks_crowded_and_empty(p, chunks, kind):
    n = CHUNK * chunks - 13
    k = max(1, int(np.floor(p * n)))
    if kind in ("middle_chunk", "crowded_and_sparse") and (k > CHUNK - 200 or k < 8 or chunks < 33):
        pytest.skip("does not fit the pattern")
    sizes = [n, 700, 1]
    with DeviceRun(sizes) as run:
        R = [np.zeros(s, np.float32) for s in sizes]
        for r in range(2):
            dWs = [_planted(n, _at(kind, n, k), r), _planted(700, _spread(700, 3, r), r), np.ones(1, np.float32)]
            R = [x.R_new for x in check_round(run, dWs, R, p, check_decode=(r == 0))]


@pytest.mark.parametrize("chunks", [2, 255, 257, 1024, 1025, 4095, 4096, 4097])
def test_calls_of_many_small_tensors(chunks):
    g = np.random.default_rng(chunks)
    sizes = [int(s) for s in g.integers(1, 60, chunks)]
    if chunks > 100:                                      # a few longer ones in between, the number of chunks kept
        for i, extra in ((7, 2), (50, 5)):
            sizes[i] = CHUNK * extra + 11
            del sizes[60:60 + extra]
    assert sum((s + CHUNK - 1) // CHUNK for s in sizes) == chunks
    with DeviceRun(sizes) as run:
        R = [np.zeros(s, np.float32) for s in sizes]
        for r in range(2):
            dWs = [(g.standard_normal(s) * 1e-3).astype(np.float32) for s in sizes]
            R = [x.R_new for x in check_round(run, dWs, R, 0.03, check_decode=(chunks < 1000))]
