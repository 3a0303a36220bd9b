"""The streaming pass around the sizes at which it changes its way through the caches and how many of its workgroups share a
compute unit, and around whole runs of chunks, at aligned and odd offsets, in steps that follow at once and that do not:
every entry's sum and every kept entry against torch on the device."""
import time

import pytest
import torch

from paper_1805_08768_amd import binding as sbc

pytestmark = pytest.mark.gpu

CHUNK = 8192
PAST = 160 * (1 << 20) // 12             # the most entries of a step that stays in the cache


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("n", [31 * CHUNK, 32 * CHUNK, 32 * CHUNK + 1, 63 * CHUNK + 5, 65 * CHUNK, PAST, PAST + 1, 23999999, 24000000,
                               (1 << 28) // 12 + 1])
def test_sums_and_kept_entries(n, offset):
    p = 0.001
    k = max(1, int(p * n))
    g = torch.Generator("cuda:0").manual_seed(n + offset)
    dW = [torch.randn(n + 1, device="cuda:0", generator=g)[offset:offset + n] for _ in range(2)]
    R = (torch.randn(n + 1, device="cuda:0", generator=g) * 0.5)[offset:offset + n]
    out = torch.zeros(n, device="cuda:0")
    msg = torch.zeros(sbc.sbc_msg_bound([n], p), dtype=torch.uint8, device="cuda:0")
    ctx = sbc.sbc_create(0, n, 1)
    try:
        for step in range(4):
            A = R + dW[step % 2]
            torch.cuda.synchronize()
            if step % 2:
                time.sleep(0.002)                         # (else the step follows the one before at once)
            nbytes = sbc.sbc_compress(ctx, [dW[step % 2]], [R], p, msg)
            out.zero_()
            sbc.sbc_decompress_accumulate(ctx, msg, nbytes, p, 1.0, [out])
            kept = torch.nonzero(out).flatten()
            assert kept.numel() == k
            side = 1.0 if float(out[kept[0]]) > 0 else -1.0
            want = torch.topk(A * side, k).indices.sort().values
            assert torch.equal(kept, want)
            assert torch.equal(R, A - out)
            mean = float(A[kept].double().mean())
            assert abs(float(out[kept[0]]) - mean) <= 1e-6 * abs(mean)       # (fp32 of a sum in fp64)
    finally:
        sbc.sbc_destroy(ctx)
