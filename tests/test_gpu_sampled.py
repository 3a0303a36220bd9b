"""Parity of the subsampled variant ("Sparse Binarization": threshold from a random subsample,
noisy amount of sparsity; SBC_OPT_SAMPLED_THRESHOLD) with the oracle's sparse_binary_compress_sampled
on the same seeded inputs, to the same bar as the exact mode: mask, counts, bitstream, message
bytes, side and decoded update bit exact; mu+, mu- and the residual within 1e-5 relative."""
import numpy as np
import pytest
import torch

from oracle import sbc_oracle as o
from paper_1805_08768_amd import binding as sbc, synth
from parity_util import DeviceRun, check_round

pytestmark = pytest.mark.gpu


def run_rounds(sizes, gen, p, rounds=1, wide_min_kept=None):
    with DeviceRun(sizes, sampled=True) as run:
        if wide_min_kept is not None:
            sbc.sbc_set_option(run.ctx, sbc.SBC_OPT_WIDE_MIN_KEPT, wide_min_kept)
        R = [np.zeros(n, np.float32) for n in sizes]
        routes = []
        for r in range(rounds):
            print("sampled round", r, "sizes", sizes[:4], "p", p, flush=True)
            res = check_round(run, gen(r), R, p)
            R = [x.R_new for x in res]
            routes.append(sbc.sbc_last_route(run.ctx))
        return res, routes


@pytest.mark.parametrize("p", [0.1, 0.01, 0.001])
def test_sampled_small_ragged_model(p):
    sizes = [64, 1000, 8192, 8193, 20000, 5, 1, 16384, 16385, 40001, 300000]
    res, _ = run_rounds(sizes, lambda r: synth.small_model_update(sizes, round_=r), p, rounds=2)
    if p == 0.01:       # the count is the sample's, not k, once the tensor is larger than the sample
        assert any(len(x.kept) != x.k for x in res if x.n > o.SAMPLE_MAX)
        assert all(len(x.kept) == x.k for x in res if x.n <= o.SAMPLE_MAX)


def test_sampled_ties_hit_the_cap():
    sizes = [300000, 777, 50000]
    res, _ = run_rounds(sizes, lambda r: [synth.palette_update(n, round_=r, tensor=i) for i, n in enumerate(sizes)],
                        0.01, rounds=2)
    assert any(len(x.kept) == o.sampled_cap(x.n, x.k) for x in res)
    zeros = [np.zeros(5000, np.float32), np.zeros(64, np.float32), np.zeros(40000, np.float32)]
    res, _ = run_rounds([5000, 64, 40000], lambda r: zeros, 0.01)
    assert [len(x.kept) for x in res] == [164, 64, 864]


def test_sampled_degenerate_tensors():
    onehot = np.zeros(100000, np.float32); onehot[99999] = -2.0
    cases = [
        ("constant", [np.full(90000, -0.25, np.float32)], 0.05),
        ("all negative", [-np.abs(synth.gaussian_update(90000))], 0.01),
        ("one hot at the end", [onehot], 0.001),
        ("single element", [np.array([-3.5], np.float32)], 0.5),
        ("keep almost everything", [synth.gaussian_update(50000)], 0.9),
        ("denormals", [(synth.gaussian_update(40000) * 1e-36).astype(np.float32)], 0.01),
    ]
    for name, dWs, p in cases:
        print("case", name, flush=True)
        run_rounds([len(d) for d in dWs], lambda r: dWs, p, rounds=2)


def test_sampled_resnet50_shaped_round():
    """The benchmark's workload: bitstream and message against the oracle for the whole model."""
    shapes = synth.resnet50_shapes()
    sizes = synth.numels(shapes)
    res, _ = run_rounds(sizes, lambda r: synth.resnet50_update(round_=r), 1e-3, rounds=1)
    ratio = sum(len(x.kept) for x in res) / sum(x.k for x in res)
    assert 0.8 < ratio < 1.25


def test_sampled_bitmap_and_grid_wide_routes():
    sizes = [1000000, 300, 65536]
    gen = lambda r: [synth.gaussian_update(n, round_=r, tensor=i) for i, n in enumerate(sizes)]
    _, routes = run_rounds(sizes, gen, 0.1, rounds=2, wide_min_kept=1 << 30)     # one workgroup per tensor
    assert not any(rt & sbc.SBC_ROUTE_WIDE for rt in routes)
    _, routes = run_rounds(sizes, gen, 0.1, rounds=2, wide_min_kept=6500)        # sweeps first
    assert all(rt & sbc.SBC_ROUTE_WIDE for rt in routes)
    # ties beyond the cap on a tensor with sweeps
    sizes = [200000, 70000]
    dWs = [synth.palette_update(200000), synth.palette_update(70000, tensor=1)]
    run_rounds(sizes, lambda r: dWs, 0.1, rounds=2, wide_min_kept=6500)


def test_sampled_option_switches_back_and_message_capacity():
    sizes = [100000, 5000]
    p = 0.01
    with DeviceRun(sizes, sampled=True) as run:
        dWs = synth.small_model_update(sizes, round_=1)
        R0 = [np.zeros(n, np.float32) for n in sizes]
        check_round(run, dWs, R0, p)
        # a buffer of the exact mode's bound is refused: the sampled variant may send more
        small = torch.zeros(sbc.sbc_msg_bound(sizes, p), dtype=torch.uint8, device="cuda:0")
        d_dW = [torch.from_numpy(x).to("cuda:0") for x in dWs]
        with pytest.raises(sbc.SbcError) as e:
            sbc.sbc_compress(run.ctx, d_dW, run.R, p, small)
        assert e.value.code == sbc.SBC_ECAPACITY
        # back to the exact mode on the same context
        sbc.sbc_set_option(run.ctx, sbc.SBC_OPT_SAMPLED_THRESHOLD, 0)
        run.sampled = False
        for r in run.R:
            r.zero_()
        res = check_round(run, dWs, R0, p)
        assert all(len(x.kept) == x.k for x in res)
