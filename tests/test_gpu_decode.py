"""The server step against the oracle's bit-serial decoder at every width of the state functions
(b from 0 to 19), with streams just below, at and above whole tiles of 512 segments, one workgroup
and the tile kernels, and with sub-normal accumulators and addends (the update is an fp32 addition
that rounds once and flushes nothing)."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import sbc_oracle as o
from paper_1805_08768_amd import binding as sbc, synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
TILE_BITS = 64 * 512


def _sizes(p):
    """Tensor sizes whose streams are about 1 and 2 tiles long, on both sides of the boundary, as far
    as that stays below four million entries; and small ones."""
    b = sbc.sbc_golomb_bstar(p)
    out = [1, 70, 8192]
    for bits in (TILE_BITS - 40, TILE_BITS + 40, 2 * TILE_BITS + 700):
        n = int(bits / (p * (b + 1.6)))
        if n <= 4_000_000:
            out.append(n)
    return out if len(out) > 3 else out + [3_000_001]


@pytest.mark.parametrize("p", [0.45, 0.2, 0.05, 0.02, 0.01, 0.004, 0.001, 2e-4, 6e-5, 1.2e-5, 1e-6])
def test_every_state_function_width_at_tile_edges(p):
    sizes = _sizes(p)
    ctx = sbc.sbc_create(0, sum(sizes), len(sizes))
    try:
        dW = [torch.from_numpy(x).to(DEV) for x in synth.small_model_update(sizes)]
        R = [torch.zeros(n, dtype=torch.float32, device=DEV) for n in sizes]
        msg = torch.zeros(sbc.sbc_msg_bound(sizes, p), dtype=torch.uint8, device=DEV)
        nbytes = sbc.sbc_compress(ctx, dW, R, p, msg)
        data = bytes(msg[:nbytes].cpu().numpy().tobytes())
        g = np.random.default_rng(int(1e7 * p))
        for scale, unit in ((1.0, 1.0), (1e-37, 1e-39)):
            base = [(g.standard_normal(n) * unit).astype(np.float32) for n in sizes]
            want = [x.copy() for x in base]
            o.decode_accumulate(data, sizes, scale, want)
            for wide_min in (0, 20):                     # one workgroup a stream / long ones tile by tile
                sbc.sbc_set_option(ctx, sbc.SBC_OPT_WIDE_MIN_KEPT, wide_min)
                out = [torch.from_numpy(x).to(DEV) for x in base]
                sbc.sbc_decompress_accumulate(ctx, msg, nbytes, p, scale, out)
                for t, (x, w) in enumerate(zip(out, want)):
                    assert np.array_equal(x.cpu().numpy().view(np.uint32), w.view(np.uint32)), (p, t, scale, wide_min)
    finally:
        sbc.sbc_destroy(ctx)


def test_into_pinned_host_memory():
    """The accumulator may be any memory the device can read and write."""
    sizes, p = [20000, 64, 8193, 300000], 0.01
    ctx = sbc.sbc_create(0, sum(sizes), len(sizes))
    try:
        dW = [torch.from_numpy(x).to(DEV) for x in synth.small_model_update(sizes)]
        R = [torch.zeros(n, dtype=torch.float32, device=DEV) for n in sizes]
        msg = torch.zeros(sbc.sbc_msg_bound(sizes, p), dtype=torch.uint8, device=DEV)
        nbytes = sbc.sbc_compress(ctx, dW, R, p, msg)
        want = [torch.full((n,), 0.5, dtype=torch.float32, device=DEV) for n in sizes]
        sbc.sbc_decompress_accumulate(ctx, msg, nbytes, p, 0.25, want)
        status = torch.full((1,), -9, dtype=torch.int32, device=DEV)
        lib, vp = sbc.load(), ctypes.c_void_p
        for call in ("context", "no allocation"):
            host = [torch.full((n,), 0.5, dtype=torch.float32, pin_memory=True) for n in sizes]
            numel = (ctypes.c_int64 * len(sizes))(*sizes)
            out = (vp * len(sizes))(*[h.data_ptr() for h in host])
            if call == "context":
                rc = lib.sbc_decompress_accumulate(ctx, None, vp(msg.data_ptr()), nbytes, numel, len(sizes), p, 0.25, out)
            else:
                rc = lib.sbc_decompress_accumulate_noalloc(0, None, vp(msg.data_ptr()), nbytes, numel, len(sizes), p, 0.25,
                                                           out, vp(status.data_ptr()))
            torch.cuda.synchronize()
            assert rc == sbc.SBC_OK and all(torch.equal(h, w.cpu()) for h, w in zip(host, want)), call
        assert int(status[0]) == sbc.SBC_OK
    finally:
        sbc.sbc_destroy(ctx)


@pytest.mark.parametrize("at", [0, 17, 34])
def test_more_long_streams_than_the_tile_kernels_take(at):
    """34 streams of two or three tiles and one several times as long anywhere in the list: the same bits as
    from the context-free call, which gives every stream one workgroup."""
    sizes, p = [70_001] * 20 + [110_003] * 14, 0.2
    sizes.insert(at, 640_001)
    ctx = sbc.sbc_create(0, sum(sizes), len(sizes))
    try:
        dW = [torch.from_numpy(x).to(DEV) for x in synth.small_model_update(sizes)]
        R = [torch.zeros(n, dtype=torch.float32, device=DEV) for n in sizes]
        msg = torch.zeros(sbc.sbc_msg_bound(sizes, p), dtype=torch.uint8, device=DEV)
        nbytes = sbc.sbc_compress(ctx, dW, R, p, msg)
        want = [torch.full((n,), 0.5, dtype=torch.float32, device=DEV) for n in sizes]
        out = [x.clone() for x in want]
        status = torch.full((1,), -9, dtype=torch.int32, device=DEV)
        sbc.sbc_decompress_accumulate_noalloc(msg, nbytes, p, 0.25, want, status)
        sbc.sbc_decompress_accumulate(ctx, msg, nbytes, p, 0.25, out)
        assert int(status[0]) == sbc.SBC_OK
        assert all(torch.equal(x, w) for x, w in zip(out, want))
    finally:
        sbc.sbc_destroy(ctx)
