"""The encoder where its pieces meet: chunks so crowded that their codes do not fit their words, unary
runs over many words, words that several chunks share, streams of one word, and calls around the numbers
of chunks at which the scan over them changes its form.  Every round against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

from paper_1805_08768_amd import binding as sbc
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


@pytest.mark.parametrize("p,chunks", [(1e-3, 1100), (2e-4, 4099)])
@pytest.mark.parametrize("pattern", ["full", "ends", "two_thirds"])
def test_full_chunks_in_calls_of_many_chunks(p, chunks, pattern):
    """Chunks that are kept whole, at the chunk's ends or with gaps: their codes take several stretches of what a
    wavefront puts together at a time, in the one launch for 1100 chunks and behind the scan for 4099."""
    n = CHUNK * chunks - 77
    k = max(1, int(np.floor(p * n)))
    at = torch.arange(CHUNK * 5, CHUNK * 6)
    if pattern == "ends":
        at = torch.cat([at[:3000], at[-(k - 3000):]]) if k < CHUNK else at
    elif pattern == "two_thirds":
        at = at[at % 3 != 1]
    rest = k - len(at)
    assert rest >= 0 or k < CHUNK
    at = at[:k] if rest < 0 else torch.cat([at, CHUNK * 6 + 40 + torch.arange(rest) * 5])      # the rest just behind it
    assert len(at) == k
    g = torch.Generator("cuda:0").manual_seed(chunks)
    x = torch.randn(n, device="cuda:0", generator=g) * 1e-3
    x[at.cuda()] = 1.0 + torch.rand(k, device="cuda:0", generator=g)
    ctx = sbc.sbc_create(0, n, 1)
    try:
        R = torch.zeros_like(x)
        msg = torch.zeros(sbc.sbc_msg_bound([n], p), dtype=torch.uint8, device="cuda:0")
        nbytes = sbc.sbc_compress(ctx, [x], [R], p, msg)
        out = torch.zeros_like(x)
        sbc.sbc_decompress_accumulate(ctx, msg, nbytes, p, 1.0, [out])
        assert torch.equal(torch.nonzero(out).flatten().cpu(), at)
        assert torch.equal(R, x - out)
        bits = np.unpackbits(sbc.sbc_last_mask(ctx, 0, n).numpy().view(np.uint8), bitorder="little")[:n]
        assert np.array_equal(np.flatnonzero(bits), at.numpy())
    finally:
        sbc.sbc_destroy(ctx)
