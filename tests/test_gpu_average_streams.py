"""The server average returns when its status is known, before its last kernel has ended: what follows at once, on the same
stream or another, with the same context, must not meet it half way."""
import numpy as np
import pytest
import torch

from paper_1805_08768_amd import binding as sbc, synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _messages(sizes, p, count, seed):
    ctx = sbc.sbc_create(0, sum(sizes), len(sizes))
    try:
        out = []
        for c in range(count):
            dW = [torch.from_numpy(synth.gaussian_update(n, client=c, round_=seed, tensor=t)).to(DEV) for t, n in enumerate(sizes)]
            msg = torch.zeros(sbc.sbc_msg_bound(sizes, p), dtype=torch.uint8, device=DEV)
            n = sbc.sbc_compress(ctx, dW, [torch.zeros_like(x) for x in dW], p, msg)
            torch.cuda.synchronize()
            out.append((msg, n))
        return out
    finally:
        sbc.sbc_destroy(ctx)


def _reference(messages, sizes, p):
    """One message after another, waited for."""
    ctx = sbc.sbc_create(0, sum(sizes), len(sizes))
    try:
        out = [torch.zeros(n, device=DEV) for n in sizes]
        for m, n in messages:
            sbc.sbc_decompress_accumulate(ctx, m, n, p, 1.0 / len(messages), out)
            torch.cuda.synchronize()
        return out
    finally:
        sbc.sbc_destroy(ctx)


@pytest.mark.parametrize("then", ["average", "compress", "corrupt", "decode"])
@pytest.mark.parametrize("same_stream", [True, False])
@pytest.mark.parametrize("p", [0.002, 0.004])
def test_what_follows_an_average(then, same_stream, p):
    # (at 0.002 an average whose last kernel stores 36 MB; at 0.004 the longest stream has more tiles than the averaging
    # kernels take, and the messages are decoded in turn)
    sizes = [9000000, 300, 70001]
    small = [400000, 5]
    a, b = _messages(sizes, p, 3, 1), _messages(small, p, 2, 2)
    want_a, want_b = _reference(a, sizes, p), _reference(b, small, p)
    dW = [torch.from_numpy(synth.gaussian_update(n, round_=7, tensor=t)).to(DEV) for t, n in enumerate(sizes)]
    ctx = sbc.sbc_create(0, sum(sizes), len(sizes))
    other = sbc.sbc_create(0, sum(sizes), len(sizes))
    try:
        msg2 = torch.zeros(sbc.sbc_msg_bound(sizes, p), dtype=torch.uint8, device=DEV)
        n2 = sbc.sbc_compress(other, dW, [torch.zeros_like(x) for x in dW], p, msg2)
        first = torch.cuda.Stream()
        second = first if same_stream else torch.cuda.Stream()
        bad = b[0][0].clone()
        bad[32 + 24 * len(small):] = 255
        torch.cuda.synchronize()
        for _ in range(4):
            out_a, out_b = [torch.full((n,), 7.0, device=DEV) for n in sizes], [torch.full((n,), 7.0, device=DEV) for n in small]
            R = [torch.zeros_like(x) for x in dW]
            msg = torch.zeros_like(msg2)
            torch.cuda.synchronize()
            with torch.cuda.stream(first):
                sbc.sbc_decompress_average(ctx, a, p, 1.0 / len(a), out_a)
            with torch.cuda.stream(second):
                if then == "average":
                    sbc.sbc_decompress_average(ctx, b, p, 1.0 / len(b), out_b)
                elif then == "corrupt":
                    with pytest.raises(sbc.SbcError):
                        sbc.sbc_decompress_average(ctx, [(bad, b[0][1]), b[1]], p, 0.5, out_b)
                    sbc.sbc_decompress_average(ctx, b, p, 1.0 / len(b), out_b)
                elif then == "compress":
                    n = sbc.sbc_compress(ctx, dW, R, p, msg)
                else:
                    out_b = [torch.zeros(n, device=DEV) for n in small]
                    for m, nb in b:
                        sbc.sbc_decompress_accumulate(ctx, m, nb, p, 1.0 / len(b), out_b)
            torch.cuda.synchronize()
            assert all(torch.equal(x, y) for x, y in zip(out_a, want_a))
            if then == "compress":
                assert n == n2 and torch.equal(msg[:n], msg2[:n])
            else:
                assert all(torch.equal(x, y) for x, y in zip(out_b, want_b))
    finally:
        sbc.sbc_destroy(ctx)
        sbc.sbc_destroy(other)


def test_stream_of_an_average_that_is_destroyed():
    """A context whose last average ran on a stream that its caller has destroyed goes on working on others."""
    import ctypes
    with open("/proc/self/maps") as f:
        hip = ctypes.CDLL([line.split()[-1] for line in f if "libamdhip64" in line][0])
    sizes, p = [3000000, 70001], 0.004
    a = _messages(sizes, p, 3, 1)
    want = _reference(a, sizes, p)
    dW = [torch.from_numpy(synth.gaussian_update(n, round_=7, tensor=t)).to(DEV) for t, n in enumerate(sizes)]
    ctx = sbc.sbc_create(0, sum(sizes), len(sizes))
    try:
        msg = torch.zeros(sbc.sbc_msg_bound(sizes, p), dtype=torch.uint8, device=DEV)
        for synchronized in (True, False):
            out, again = [[torch.full((n,), 7.0, device=DEV) for n in sizes] for _ in range(2)]
            torch.cuda.synchronize()
            handle = ctypes.c_void_p()
            assert hip.hipStreamCreateWithFlags(ctypes.byref(handle), 1) == 0          # (non-blocking)
            with torch.cuda.stream(torch.cuda.ExternalStream(handle.value)):
                sbc.sbc_decompress_average(ctx, a, p, 1.0 / len(a), out)
            if synchronized:
                assert hip.hipStreamSynchronize(handle) == 0
            assert hip.hipStreamDestroy(handle) == 0
            with torch.cuda.stream(torch.cuda.Stream()):
                sbc.sbc_decompress_average(ctx, a, p, 1.0 / len(a), again)
                n = sbc.sbc_compress(ctx, dW, [torch.zeros_like(x) for x in dW], p, msg)
                torch.cuda.current_stream().synchronize()
                one = [torch.zeros(n, device=DEV) for n in sizes]
                sbc.sbc_decompress_accumulate(ctx, msg, n, p, 1.0, one)
            torch.cuda.synchronize()
            assert all(torch.equal(x, y) for x, y in zip(out, want)) and all(torch.equal(x, y) for x, y in zip(again, want))
            assert all(int((x != 0).sum()) == max(1, int(p * n)) for x, n in zip(one, sizes))
    finally:
        sbc.sbc_destroy(ctx)


def test_decode_recorded_while_an_average_runs():
    """A deferred decode in a graph whose recording begins before the average's last kernel on another stream has ended."""
    sizes, p = [9000000, 70001], 0.002
    a = _messages(sizes, p, 3, 1)
    want = _reference(a, sizes, p)
    ctx = sbc.sbc_create(0, sum(sizes), len(sizes))
    try:
        sbc.sbc_set_option(ctx, sbc.SBC_OPT_DEFER_DECODE_STATUS, 1)
        out, one = [[torch.zeros(n, device=DEV) for n in sizes] for _ in range(2)]
        first, second = torch.cuda.Stream(), torch.cuda.Stream()
        torch.cuda.synchronize()
        with torch.cuda.stream(second):
            sbc.sbc_decompress_accumulate(ctx, a[0][0], a[0][1], p, 0.5, one)           # (the tables are there)
        sbc.sbc_decode_status(ctx, second)
        with torch.cuda.stream(second):
            sbc.sbc_decompress_accumulate(ctx, a[0][0], a[0][1], p, 0.5, one)           # (and the status word is clean)
        torch.cuda.synchronize()
        want_one = [x * 0.5 for x in one]
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.stream(first):
            sbc.sbc_decompress_average(ctx, a, p, 1.0 / len(a), out)
        with torch.cuda.stream(second):
            graph.capture_begin()
            try:
                sbc.sbc_decompress_accumulate(ctx, a[0][0], a[0][1], p, 0.5, one)
            finally:
                graph.capture_end()
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(out, want))
        for _ in range(3):
            with torch.cuda.stream(second):
                for x in one:
                    x.zero_()
                graph.replay()
            torch.cuda.synchronize()
            assert all(torch.equal(x, y) for x, y in zip(one, want_one))
        sbc.sbc_decode_status(ctx, second)
    finally:
        sbc.sbc_destroy(ctx)


def test_what_an_average_has_stored_is_there_for_the_host_and_other_streams():
    """Right after the stream has been waited for: in pinned host memory, in a copy to the host, and for another stream behind an
    event of the caller's.  Averages of different messages in turn, so that whatever is missing shows as the one before's."""
    sizes, p = [9000000, 300, 70001], 0.002               # (36 MB: more than the caches closest to the compute units hold)
    rounds = [_messages(sizes, p, 3, r) for r in range(2)]
    want = [[x.cpu() for x in _reference(m, sizes, p)] for m in rounds]
    want_dev = [[x.to(DEV) for x in w] for w in want]
    ctx = sbc.sbc_create(0, sum(sizes), len(sizes))
    try:
        stream, other = torch.cuda.Stream(), torch.cuda.Stream()
        flat = torch.zeros(sum(sizes) + 64, pin_memory=True)
        out = [torch.zeros(n, device=DEV) for n in sizes]
        host = [torch.zeros(n, pin_memory=True) for n in sizes]
        class Pinned:                                     # (the binding takes device tensors; the library any device-visible memory)
            ptrs = (sbc.ctypes.c_void_p * len(sizes))()
            numel_arr = (sbc.ctypes.c_int64 * len(sizes))(*sizes)
            tensors = sizes
        at = 0
        for t, n in enumerate(sizes):
            Pinned.ptrs[t] = flat.data_ptr() + 4 * at
            at += (n + 15) // 16 * 16
        torch.cuda.synchronize()
        for r in range(24):
            messages, w, w_dev = rounds[r % 2], want[r % 2], want_dev[r % 2]
            with torch.cuda.stream(stream):
                arr = (sbc.ctypes.c_void_p * len(messages))(*[m.data_ptr() for m, _ in messages])
                lens = (sbc.ctypes.c_size_t * len(messages))(*[n for _, n in messages])
                rc = sbc.load().sbc_decompress_average(ctx, stream.cuda_stream, arr, lens, len(messages), Pinned.numel_arr, len(sizes), p,
                                                       1.0 / len(messages), Pinned.ptrs)
                assert rc == sbc.SBC_OK
            stream.synchronize()
            at = 0
            for n, x in zip(sizes, w):
                assert torch.equal(flat[at:at + n], x), "pinned, round %d" % r
                at += (n + 15) // 16 * 16
            with torch.cuda.stream(stream):
                sbc.sbc_decompress_average(ctx, messages, p, 1.0 / len(messages), out)
            stream.synchronize()
            for h, x in zip(host, out):
                h.copy_(x, non_blocking=True)
            torch.cuda.current_stream().synchronize()
            assert all(torch.equal(h, x) for h, x in zip(host, w)), "copied, round %d" % r
            messages, w, w_dev = rounds[(r + 1) % 2], want[(r + 1) % 2], want_dev[(r + 1) % 2]
            with torch.cuda.stream(stream):
                sbc.sbc_decompress_average(ctx, messages, p, 1.0 / len(messages), out)
                behind = torch.cuda.Event()
                behind.record(stream)
            with torch.cuda.stream(other):
                other.wait_event(behind)
                same = torch.stack([(x == y).all() for x, y in zip(out, w_dev)])
                for h, x in zip(host, out):
                    h.copy_(x, non_blocking=True)
            other.synchronize()
            assert bool(same.all()) and all(torch.equal(h, x) for h, x in zip(host, w)), "other stream, round %d" % r
    finally:
        sbc.sbc_destroy(ctx)
