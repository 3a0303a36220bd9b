"""Candidate lists and the selection from them at the places where they change their form: lists in one
piece and in segments, lists that stay in registers and longer ones, bins of the k-th entry from one entry
to more than are ranked one against the others, lists long enough for sweeps, and a compact context whose
segment overflows while the list as a whole would not.  Against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

from paper_1805_08768_amd import binding as sbc, synth
from parity_util import DeviceRun, check_round

pytestmark = pytest.mark.gpu

CHUNK = 8192


@pytest.mark.parametrize("chunks,short", [(63, 5), (64, 0), (64, 8191), (65, 1), (71, 17), (72, 0), (80, 4000)])
def test_lists_in_segments(chunks, short):
    sizes = [CHUNK * chunks - short, 3000]
    with DeviceRun(sizes) as run:
        R = [np.zeros(n, np.float32) for n in sizes]
        for r in range(3):
            dWs = [synth.gaussian_update(n, round_=r, tensor=i) for i, n in enumerate(sizes)]
            if r == 2:                                    # everything interesting in one segment's chunks
                x = dWs[0].reshape(-1)
                x[CHUNK * 11:CHUNK * 12] *= 6.0
                x[CHUNK * 19:CHUNK * 20] *= 6.0
            res = check_round(run, dWs, R, 0.004, check_decode=(r == 0))
            R = [x.R_new for x in res]


@pytest.mark.parametrize("p", [0.1, 0.13, 0.3])
def test_list_lengths_around_what_registers_hold(p):
    """Lists of a single piece: all of them longer than the 16384 keys held, one just below, one beyond."""
    sizes = [120001, 131072, 200003, 16384, 16400]
    with DeviceRun(sizes) as run:
        R = [np.zeros(n, np.float32) for n in sizes]
        for r in range(2):
            dWs = [synth.gaussian_update(n, round_=r, tensor=i) for i, n in enumerate(sizes)]
            R = [x.R_new for x in check_round(run, dWs, R, p, check_decode=False)]


@pytest.mark.parametrize("m", [1, 2, 16, 17, 63, 64, 65, 128, 129, 255, 256, 257, 300, 1500])
@pytest.mark.parametrize("ties", [False, True])
def test_entries_in_the_bin_of_the_kth(m, ties):
    """m entries of each side share the leading 20 key bits with the k-th, which is the middle one of them."""
    n, p = 60000, 0.03
    k = int(np.floor(p * n))
    g = np.random.default_rng(m)
    x = (g.standard_normal(n) * 1e-3).astype(np.float32)
    at = g.permutation(n)
    base = np.float32(1.5).view(np.uint32)
    low = g.integers(0, 4096, m) if not ties else g.integers(0, 3, m)
    bin_ = (np.uint32(base) + low.astype(np.uint32)).view(np.float32)
    beyond = max(0, k - (m + 1) // 2)
    if m > 2 * k:
        pytest.skip("more entries than fit")
    for side, sign in ((0, 1.0), (1, -1.0)):
        a = at[side * 2 * n // 5: side * 2 * n // 5 + beyond + m]
        x[a[:beyond]] = sign * (2.0 + g.random(beyond)).astype(np.float32) * (1.0 if side == 0 else 0.9)
        x[a[beyond:]] = sign * bin_
    sizes = [n, 500]
    with DeviceRun(sizes) as run:
        R = [np.zeros(s, np.float32) for s in sizes]
        for r in range(2):
            small = (g.standard_normal(500) * 1e-3).astype(np.float32)
            R = [y.R_new for y in check_round(run, [x, small], R, p, check_decode=False)]


@pytest.mark.parametrize("k", [8191, 8192, 32767, 32768])
def test_kept_entries_around_the_limits_of_long_lists(k):
    p = 0.02
    n = next(n for n in range(int(k / p) - 2, int(k / p) + 60) if int(np.floor(p * n)) == k)
    with DeviceRun([n]) as run:
        R = [np.zeros(n, np.float32)]
        for r in range(2):
            res = check_round(run, [synth.gaussian_update(n, round_=r)], R, p, check_decode=(r == 0))
            assert res[0].k == k
            assert bool(sbc.sbc_last_route(run.ctx) & sbc.SBC_ROUTE_WIDE) == (k >= 32768)
            R = [x.R_new for x in res]


def test_compact_context_whose_segment_overflows():
    """4100 chunks; 1.2e6 equal entries, all in chunks of one segment, which holds 1.05e6: the histogram route
    takes the list in one piece, and the first k of them are kept."""
    n, p = CHUNK * 4100, 0.001
    k = int(np.floor(p * n))
    ctx = sbc.sbc_create_compact(0, n, 1)
    try:
        x = torch.randn(n, dtype=torch.float32, device="cuda:0", generator=torch.Generator("cuda:0").manual_seed(1)) * 1e-3
        x.view(-1, CHUNK)[3::8, :2400] = 1.0
        planted = torch.nonzero(x == 1.0).flatten()
        assert 1_050_000 < len(planted) < n // 4
        want = planted[:k]
        R = torch.zeros_like(x)
        msg = torch.zeros(sbc.sbc_msg_bound([n], p), dtype=torch.uint8, device="cuda:0")
        nbytes = sbc.sbc_compress(ctx, [x], [R], p, msg)
        assert sbc.sbc_last_route(ctx) & sbc.SBC_ROUTE_HISTOGRAM
        out = torch.zeros_like(x)
        sbc.sbc_decompress_accumulate(ctx, msg, nbytes, p, 1.0, [out])
        assert torch.equal(torch.nonzero(out).flatten(), want)
        assert torch.equal(R, x - out)
    finally:
        sbc.sbc_destroy(ctx)


def test_keys_left_by_a_sampled_call_on_data_of_two_scales():
    """Three chunks of 256 hold entries fifty times as large as all others, fewer than are kept: a sampled
    call's list ends near the k-th entry, far below the first of the large ones, and says nothing about what
    follows it.  The key it leaves for the next call must not let half the tensor pass."""
    n, p = CHUNK * 256, 0.01
    with DeviceRun([n]) as run:
        R = [np.zeros(n, np.float32)]
        for r in range(8):
            x = synth.gaussian_update(n, round_=r).reshape(-1, CHUNK)
            x[40:43] *= 50.0
            res = check_round(run, [x.reshape(-1)], R, p, check_decode=False)
            assert max(sbc.sbc_last_candidates(run.ctx, 0)) < n // 8, (r, sbc.sbc_last_route(run.ctx))
            R = [v.R_new for v in res]


@pytest.mark.parametrize("sweeps", [False, True])
@pytest.mark.parametrize("segments,ties", [((3,), False), ((3,), True), ((0, 7), False), ((0, 7), True)])
def test_lists_crowded_into_few_segments(sweeps, segments, ties):
    """All candidates of a list but a few in one or two of its eight segments: shares are cut from the list as
    a whole, across the segments' borders."""
    n, p = CHUNK * 91 - 77, 0.03
    with DeviceRun([n, 700]) as run:
        sbc.sbc_set_option(run.ctx, sbc.SBC_OPT_WIDE_MIN_KEPT, 9000 if sweeps else 1 << 30)
        R = [np.zeros(n, np.float32), np.zeros(700, np.float32)]
        for r in range(3):
            x = synth.gaussian_update(CHUNK * 91, round_=r).reshape(-1, CHUNK)
            for g in segments:
                x[g::8] *= 40.0
                if ties:                                  # a few values, most of them at the threshold
                    x[g::8] = np.sign(x[g::8]) * np.float32(0.04) * np.float32(1 + r) * (1 + (np.abs(x[g::8]) > 0.09))
            x[44, ::1000] = 3.0                           # (a segment with a few entries of its own)
            dWs = [np.ascontiguousarray(x.reshape(-1)[:n]), synth.gaussian_update(700, round_=r, tensor=1)]
            res = check_round(run, dWs, R, p, check_decode=False)
            R = [v.R_new for v in res]


@pytest.mark.parametrize("carry", [0, 1])
def test_lists_left_by_the_streaming_kernel(carry):
    """With the fused step: tensors whose long lists are full of equal values are left to the kernels behind it,
    which read their lists in pairs, at odd list capacities, beside tensors that it finishes and one that keeps
    too many entries for it (its lists in two arrays)."""
    sizes = [200001, 60007, 700001, 9001, 130000]
    p, taken_over = 0.012, 0
    with DeviceRun(sizes) as run:
        sbc.sbc_set_option(run.ctx, sbc.SBC_OPT_FUSED_STEP, 1)
        sbc.sbc_set_option(run.ctx, sbc.SBC_OPT_CARRY_FILTER_KEYS, carry)
        R = [np.zeros(n, np.float32) for n in sizes]
        for r in range(3):
            dWs = [synth.gaussian_update(n, round_=r, tensor=i) if i in (2, 3) else synth.palette_update(n, round_=r, tensor=i)
                   for i, n in enumerate(sizes)]
            res = check_round(run, dWs, R, p, check_decode=(r == 0))
            taken_over += bool(sbc.sbc_last_route(run.ctx) & sbc.SBC_ROUTE_TAKEN_OVER)
            R = [x.R_new for x in res]
    assert taken_over
