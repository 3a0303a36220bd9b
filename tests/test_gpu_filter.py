"""The streaming pass at the places where its vector loads, masks and float comparisons could go
wrong: operands at every 4-byte offset (each its own), sizes around whole chunks and vectors, and
data whose filter keys fall on zero, on sub-normal values and on both sides of it, with the filter
keys carried over several rounds.  Every round against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import sbc_oracle as o
from paper_1805_08768_amd import binding as sbc, synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SIZES = [1, 2, 3, 4, 5, 8191, 8192, 8193, 8194, 16383, 16387, 24575, 40001]


def _placed(n, offset):
    """A tensor of n entries that starts `offset` entries after a 16-byte boundary."""
    return torch.zeros(n + offset + 4, dtype=torch.float32, device=DEV)[offset:offset + n]


def _rounds(updates, sizes, p, off_dw, off_r, sampled=False):
    dW = [_placed(n, off_dw) for n in sizes]
    R = [_placed(n, off_r) for n in sizes]
    assert all((x.data_ptr() >> 2) & 3 == off_dw & 3 for x in dW)
    ctx = sbc.sbc_create(0, sum(sizes), len(sizes))
    try:
        msg = torch.zeros(sbc.sbc_msg_bound(sizes, p), dtype=torch.uint8, device=DEV)
        R_host = [np.zeros(n, np.float32) for n in sizes]
        for r, ups in enumerate(updates):
            for d, u in zip(dW, ups):
                d.copy_(torch.from_numpy(u))
            want = o.compress_model(ups, R_host, p)
            nbytes = sbc.sbc_compress(ctx, dW, R, p, msg)
            assert bytes(msg[:nbytes].cpu().numpy().tobytes()) == o.build_message(want), "round %d" % r
            for t, (x, w) in enumerate(zip(R, want)):
                assert np.array_equal(x.cpu().numpy(), w.R_new.astype(np.float32)), (r, t)
            R_host = [w.R_new for w in want]
    finally:
        sbc.sbc_destroy(ctx)


@pytest.mark.parametrize("off_dw,off_r", [(0, 0), (1, 1), (0, 2), (3, 1)])
def test_offsets_and_ragged_sizes(off_dw, off_r):
    ups = [synth.small_model_update(SIZES, round_=r) for r in range(2)]
    _rounds(ups, SIZES, 0.02, off_dw, off_r)


@pytest.mark.parametrize("case", ["few_nonzero", "subnormal", "one_sign", "zeros"])
def test_filter_keys_at_zero_and_among_subnormals(case):
    sizes = [30000, 9000, 500]
    g = np.random.default_rng(5)
    ups = []
    for r in range(4):
        ups.append([])
        for n in sizes:
            x = np.zeros(n, np.float32)
            if case == "few_nonzero":                    # fewer non-zero entries per side than are kept (k = n / 50)
                at = g.choice(n, n // 60, replace=False)
                x[at] = g.standard_normal(len(at)).astype(np.float32)
            elif case == "subnormal":                    # the k-th entry is sub-normal, and there are zeros
                x = (g.standard_normal(n) * 1e-41).astype(np.float32)
                x[g.random(n) < 0.3] = 0.0
                x[:3] = [1.0, -2.0, 3.0]
            elif case == "one_sign":                     # nothing on the other side but zeros and -0.0
                x = np.abs(g.standard_normal(n)).astype(np.float32) * np.float32(-1.0 if r % 2 else 1.0)
                x[g.random(n) < 0.9] = -0.0
            ups[-1].append(x)
    _rounds(ups, sizes, 0.02, 0, 0)
