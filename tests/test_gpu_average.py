"""The server step for all messages at once against one message after another (which the oracle's
decoder checks elsewhere) and against the oracle itself: every width of the state functions and a
remainder width beyond them, blocks of 2048 and chunks of 8192 entries on both sides of their edges,
streams for a wavefront, for a workgroup and for neither, more messages than a pass takes, blocks of
more entries than lanes, messages of more positions than there is room for, and corrupt ones."""
import numpy as np
import pytest
import torch

from oracle import sbc_oracle as o
from paper_1805_08768_amd import binding as sbc, synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _messages(sizes, p, count, seed):
    ctx = sbc.sbc_create(0, sum(sizes), len(sizes))
    try:
        out = []
        for m in range(count):
            g = np.random.default_rng(seed + m)
            dW = [torch.from_numpy((g.standard_normal(n) * 2.0 ** (m % 5)).astype(np.float32)).to(DEV) for n in sizes]
            R = [torch.zeros(n, dtype=torch.float32, device=DEV) for n in sizes]
            msg = torch.zeros(sbc.sbc_msg_bound(sizes, p), dtype=torch.uint8, device=DEV)
            out.append((msg, sbc.sbc_compress(ctx, dW, R, p, msg)))
        return out
    finally:
        sbc.sbc_destroy(ctx)


def _outputs(sizes, offset=0):
    flat = torch.full((sum(sizes) + 8,), float("nan"), dtype=torch.float32, device=DEV)
    views, at = [], offset
    for n in sizes:
        views.append(flat[at:at + n])
        at += n
    return flat, views


def _in_turn(ctx, messages, p, scale, sizes):
    out = [torch.zeros(n, dtype=torch.float32, device=DEV) for n in sizes]
    for msg, nbytes in messages:
        sbc.sbc_decompress_accumulate(ctx, msg, nbytes, p, scale, out)
    return out


def _same(got, want):
    return all(torch.equal(a.view(torch.int32), b.view(torch.int32)) for a, b in zip(got, want))


EDGES = [1, 2, 63, 2047, 2048, 2049, 6143, 8191, 8192, 8193, 40961]


@pytest.mark.parametrize("p, sizes, counts", [
    (0.45, EDGES, (1, 2, 7, 8, 9)),
    (0.2, EDGES + [300_007], (1, 5)),
    (0.12, EDGES + [170_003], (1, 3, 66)),
    (0.02, EDGES + [300_007, 1_200_001], (1, 63, 64, 65, 130)),
    (0.03, EDGES + [90_001], (47, 48, 49)),           # half a block at a time, and whole ones
    (0.004, EDGES + [1_200_001], (3,)),
    (2e-4, EDGES + [2_500_003], (1, 9)),
    (1.2e-5, EDGES + [2_500_003], (9,)),
    (1e-6, EDGES + [2_500_003], (9,)),                # remainders wider than the packed decoder's
    (0.02, [7_000_001, 2049], (2,)),                  # a stream of more tiles than one workgroup takes
])
def test_same_bits_as_one_after_another(p, sizes, counts):
    ctx = sbc.sbc_create(0, sum(sizes), len(sizes))
    try:
        messages = _messages(sizes, p, max(counts), 100)
        for count in counts:
            for offset, scale in ((0, 1.0 / count), (3, 1e-39)):
                want = _in_turn(ctx, messages[:count], p, scale, sizes)
                flat, out = _outputs(sizes, offset)
                sbc.sbc_decompress_average(ctx, messages[:count], p, scale, out)
                assert _same(out, want), (p, count, offset)
                assert torch.isnan(flat[:offset]).all() and torch.isnan(flat[offset + sum(sizes):]).all()
    finally:
        sbc.sbc_destroy(ctx)


def test_against_the_oracle_and_other_calls_between():
    sizes, p = [2049, 8192, 50_000], 0.01
    messages = _messages(sizes, p, 3, 7)
    want = [np.zeros(n, np.float32) for n in sizes]
    for msg, nbytes in messages:
        o.decode_accumulate(bytes(msg[:nbytes].cpu().numpy().tobytes()), sizes, np.float32(1.0 / 3.0), want)
    ctx = sbc.sbc_create(0, sum(sizes), len(sizes))
    try:
        dW = [torch.from_numpy(x).to(DEV) for x in synth.small_model_update(sizes)]
        R = [torch.zeros(n, dtype=torch.float32, device=DEV) for n in sizes]
        own = torch.zeros(sbc.sbc_msg_bound(sizes, p), dtype=torch.uint8, device=DEV)
        side = torch.cuda.Stream()
        for _ in range(3):                            # client steps on another stream share the scratch memory
            side.wait_stream(torch.cuda.current_stream())
            sbc.sbc_compress(ctx, dW, R, p, own, side)
            _, out = _outputs(sizes)
            sbc.sbc_decompress_average(ctx, messages, p, 1.0 / 3.0, out)
            assert all(np.array_equal(x.cpu().numpy().view(np.uint32), w.view(np.uint32)) for x, w in zip(out, want))
        # with a client step pending the messages are taken in turn
        sbc.sbc_compress_begin(ctx, dW, R, p, own)
        _, out = _outputs(sizes)
        sbc.sbc_decompress_average(ctx, messages, p, 1.0 / 3.0, out)
        sbc.sbc_compress_end(ctx)
        assert all(np.array_equal(x.cpu().numpy().view(np.uint32), w.view(np.uint32)) for x, w in zip(out, want))
    finally:
        sbc.sbc_destroy(ctx)


def test_more_positions_than_room_and_corrupt_messages():
    sizes = [40_000, 500]
    ctx = sbc.sbc_create(0, sum(sizes), len(sizes))
    try:
        # 5 % of the entries in a message with the remainder width of p = 0.04
        wide_p, p = 0.05, 0.04
        assert sbc.sbc_golomb_bstar(wide_p) == sbc.sbc_golomb_bstar(p)
        messages = _messages(sizes, wide_p, 3, 50)
        want = _in_turn(ctx, messages, p, 0.5, sizes)
        _, out = _outputs(sizes)
        sbc.sbc_decompress_average(ctx, messages, p, 0.5, out)
        assert _same(out, want)
        for at in (0, 36, 40, 32 + 24 * 2 + 5):       # magic, count, bit length, payload
            broken = [(m.clone(), nb) for m, nb in messages]
            broken[1][0][at] ^= 0x41
            status = []
            for call in (lambda: _in_turn(ctx, broken, p, 0.5, sizes),
                         lambda: sbc.sbc_decompress_average(ctx, broken, p, 0.5, out)):
                try:
                    call()
                    status.append(0)
                except sbc.SbcError as e:
                    status.append(e.code)
            assert status[0] == status[1], at
            if at < 40:
                assert status[1] == sbc.SBC_ECORRUPT
            sbc.sbc_decompress_average(ctx, messages, p, 0.5, out)      # the context is none the worse
            assert _same(out, want)
    finally:
        sbc.sbc_destroy(ctx)
