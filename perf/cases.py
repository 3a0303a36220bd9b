"""What a user of this library has it do, as cases that can be timed and compared: client steps
(sbc_compress with the residual carried from round to round), server steps
(sbc_decompress_accumulate, Server.average) and a whole round of several clients, from one small
model to a flat update of 1.5e9 entries.

Results are exact by specification (mask and bit stream from integer comparisons, sums of the kept
values as exact integers rounded once), so every case is compared bit for bit.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_1805_08768_amd import binding as sbc
from paper_1805_08768_amd import rounds, synth

DEV = "cuda:0"


# ------------------------------------------------------------------- cases ----

def listed():
    return [
        # The smallest calls: a model of four small tensors (a one-chunk one, a 64-entry one, a ragged
        # one), client step and context-free server step in turn.  Launches and host time decide.
        dict(name="step_small_model", op="step", model="small", data="laplace", p=0.01),
        # One tensor of 2^20 Gaussian entries at the paper's p = 1 %: 10,485 kept entries per side.
        dict(name="compress_gauss_2p20", op="compress", model="flat", entries=1 << 20, data="gauss", p=0.01),
        # One tensor of 4 Mi heavy-tailed entries with exact duplicates (ties), p = 0.1 %.
        dict(name="compress_student_4m", op="compress", model="flat", entries=4194304, data="student", p=0.001),
        # A framework that hands over one packed gradient buffer: 24 tensors of odd sizes, each at
        # whatever 4-byte offset it falls on.
        dict(name="compress_ragged_packed", op="compress", model="ragged", entries=12000000, tensors=24,
             shape_seed=5, data="laplace", p=0.01, packed=True),
        # The ResNet-50-shaped model at the paper's two sparsities: the ordinary client step.
        dict(name="compress_resnet50_p001", op="compress", model="resnet50", data="laplace", p=0.001),
        dict(name="compress_resnet50_p01", op="compress", model="resnet50", data="laplace", p=0.01),
        # The LSTM language model (embedding rows mostly zero) at p = 0.01 %.
        dict(name="compress_lstm_p0001", op="compress", model="lstm", vocab=10000, hidden=1500, data="gauss", p=0.0001),
        # The subsampled variant (thresholds from a random subsample, noisy count) on the same model.
        dict(name="compress_lstm_sampled", op="compress", model="lstm", vocab=10000, hidden=1500, data="gauss",
             p=0.001, sampled=True),
        # The largest: one flat update of 1.5e9 entries on a context with short candidate lists.
        dict(name="compress_flat_1p5e9", op="compress", model="flat", entries=1500000000, data="gauss", p=0.001,
             compact=True),
        # Server: one message with long streams (up to 150,000 codes each), waited for.
        dict(name="decode_lstm_p01", op="decode", model="lstm", vocab=10000, hidden=1500, data="gauss", p=0.01),
        # Server: the average over 32 clients' messages of the ResNet-50-shaped model.
        dict(name="average_resnet50_32", op="average", model="resnet50", data="laplace", p=0.001, clients=32),
        # A whole round of Alg. 1, everything in device memory: four clients in parallel, the server's
        # average, the weight update.
        dict(name="round_resnet50_4", op="round", model="resnet50", data="laplace", p=0.01, clients=4),
    ]


def draw(rng):
    def log_uniform(lo, hi):
        return math.exp(rng.uniform(math.log(lo), math.log(hi)))

    case = {"p": float("%.3g" % log_uniform(1e-4, 0.05))}
    op = case["op"] = rng.choices(["compress", "step", "decode", "average", "round"], [10, 3, 3, 2, 2])[0]
    one = op in ("compress", "step", "decode")
    model = case["model"] = rng.choices(["flat", "ragged", "resnet50", "lstm"], [5, 6, 2, 2] if one else [1, 5, 1, 2])[0]
    if model == "flat":
        case["entries"] = int(log_uniform(3e4, 4e8 if op == "compress" else 1e8 if one else 1e7)) | rng.randrange(2)
    elif model == "ragged":
        case["entries"] = int(log_uniform(1e5, 6e7 if one else 1e7))
        case["tensors"] = rng.randrange(3, 80)
        case["shape_seed"] = rng.randrange(1000)
        case["packed"] = rng.random() < 0.4
    elif model == "lstm":
        case["vocab"], case["hidden"] = int(log_uniform(1000, 20000)), int(log_uniform(100, 1500 if one else 600))
    case["data"] = rng.choice(["laplace", "gauss", "student"])
    if op in ("average", "round"):
        case["clients"] = rng.randrange(2, 17 if op == "average" else 7)
    if op == "compress":
        case["sampled"] = rng.random() < 0.15
        case["compact"] = rng.random() < 0.2
    return case


def _sizes(case):
    model = case["model"]
    if model == "flat":
        return [int(case["entries"])]
    if model == "small":
        return [20000, 64, 8193, 300000]
    if model == "resnet50":
        return synth.numels(synth.resnet50_shapes())
    if model == "lstm":
        return synth.numels(synth.lstm_lm_shapes(case["vocab"], case["hidden"]))
    # ragged: sizes spread over three orders of magnitude, mostly odd, scaled to the total
    r = random.Random(int(case["shape_seed"]))
    raw = [math.exp(r.uniform(0.0, math.log(1000.0))) for _ in range(int(case["tensors"]))]
    scale = case["entries"] / sum(raw)
    return [max(1, int(x * scale)) | 1 for x in raw]


def _offsets(case, sizes):
    """Where each tensor starts in its flat buffer: at multiples of 64 entries, or packed."""
    offs, total = [], 0
    for n in sizes:
        offs.append(total)
        total += n if case.get("packed") else (n + 63) // 64 * 64
    return offs, total


def _views(flat, offs, sizes):
    return [flat[o:o + n] for o, n in zip(offs, sizes)]


# ------------------------------------------------------------------ inputs ----

def _generator(seed, what):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + int(what)) & ((1 << 62) - 1))
    return g


def _draw_into(x, data, g):
    """Unit-scale values of one family, in place."""
    if data == "laplace":
        x.exponential_(1.0, generator=g)
        x.mul_(torch.randint(0, 2, x.shape, generator=g, device=DEV, dtype=torch.int8).mul_(2).sub_(1))
    elif data == "student":                       # Student-t(3)
        chi2 = torch.zeros_like(x)
        for _ in range(3):
            x.normal_(generator=g)
            chi2.addcmul_(x, x)
        x.normal_(generator=g)
        x.div_(chi2.div_(3.0).sqrt_().clamp_(min=1e-6))
        m = x.numel() // 100                      # exact duplicates of values elsewhere in the tensor
        dst = torch.randint(0, x.numel(), (m,), generator=g, device=DEV)
        src = torch.randint(0, x.numel(), (m,), generator=g, device=DEV)
        x[torch.unique(dst)] = x[src[:torch.unique(dst).numel()]]
    else:
        x.normal_(generator=g)
    return x


def _layers(case, seed, sizes):
    """Per-tensor scale 10^U(-4,-2), the same in every round and client; 1e-3 for the Gaussian models."""
    r = np.random.RandomState(int(seed) % (1 << 31))
    s = 10.0 ** r.uniform(-4.0, -2.0, len(sizes))
    return [1e-3] * len(sizes) if case["data"] == "gauss" else [float(v) for v in s]


def _update(case, seed, what, sizes, offs, total, scales):
    """One client's update of one round as a flat buffer (padding zero)."""
    g = _generator(seed, what)
    flat = torch.zeros(total, dtype=torch.float32, device=DEV)
    if len(sizes) == 1:
        _draw_into(flat[:sizes[0]], case["data"], g).mul_(scales[0])
        return flat
    whole = _draw_into(torch.empty(total, dtype=torch.float32, device=DEV), case["data"], g)
    for t, (o, n) in enumerate(zip(offs, sizes)):
        torch.mul(whole[o:o + n], scales[t], out=flat[o:o + n])
    if case["model"] == "lstm":                   # 5 % of the embedding's rows were seen in this round
        v, h = case["vocab"], case["hidden"]
        idle = torch.rand(v, generator=g, device=DEV) >= 0.05
        flat[offs[0]:offs[0] + v * h].view(v, h)[idle] = 0.0
    return flat


def _residual(case, seed, what, sizes, offs, total, scales):
    """A residual in mid-training: what several rounds left behind, its tails already sent."""
    flat = _update(dict(case, model="flat" if len(sizes) == 1 else "ragged"), seed, what, sizes, offs, total, scales)
    for t, x in enumerate(_views(flat, offs, sizes)):
        x.mul_(2.0).clamp_(-3.0 * scales[t], 3.0 * scales[t])
    return flat


ROUNDS = 3       # updates a client goes through in turn (two for the flat ones beyond 1e8 entries)


def _updates_of(case):
    return 2 if case["model"] == "flat" and case["entries"] > 100000000 else ROUNDS


class _Context:
    """A context of the library, destroyed with the object."""

    def __init__(self, sizes, sampled=False, compact=False):
        self.handle = None
        self.handle = (sbc.sbc_create_compact if compact else sbc.sbc_create)(0, sum(sizes), len(sizes))
        if sampled:
            sbc.sbc_set_option(self.handle, sbc.SBC_OPT_SAMPLED_THRESHOLD, 1)

    def __del__(self):
        if self.handle is not None:
            sbc.sbc_destroy(self.handle)
            self.handle = None


class _State:
    pass


def _client(case, seed, client, sizes, offs, total, scales, n_updates, zero_residual):
    """Flat updates and the residual of one client."""
    ups = [_update(case, seed, 100 * client + r + 1, sizes, offs, total, scales) for r in range(n_updates)]
    res = (torch.zeros(total, dtype=torch.float32, device=DEV) if zero_residual
           else _residual(case, seed, 100 * client + 99, sizes, offs, total, scales))
    return ups, res


def _messages(case, seed, count, sizes, offs, total, scales):
    """First-round messages of `count` clients: (message tensor, size) pairs."""
    ctx = _Context(sizes)
    out = []
    for c in range(count):
        (up,), res = _client(case, seed, c, sizes, offs, total, scales, 1, True)
        msg = torch.zeros(sbc.sbc_msg_bound(sizes, case["p"]), dtype=torch.uint8, device=DEV)
        n = sbc.sbc_compress(ctx.handle, _views(up, offs, sizes), _views(res, offs, sizes), case["p"], msg)
        torch.cuda.synchronize()
        out.append((msg[:(n + 7) // 8 * 8].clone(), n))
    return out


def prepare(case, seed):
    s = _State()
    s.case, s.p, s.turn = case, float(case["p"]), 0
    op = case["op"]
    sizes = _sizes(case)
    offs, total = _offsets(case, sizes)
    scales = _layers(case, seed, sizes)
    if op in ("compress", "step"):
        ups, s.residual = _client(case, seed, 0, sizes, offs, total, scales, _updates_of(case), False)
        s.updates = [sbc.TensorList(_views(u, offs, sizes)) for u in ups]
        s.residual_list = sbc.TensorList(_views(s.residual, offs, sizes))
        sampled = bool(case.get("sampled"))
        bound = (sbc.sbc_msg_bound_sampled if sampled else sbc.sbc_msg_bound)(sizes, s.p)
        s.msg = sbc.MessageBuffer(torch.zeros(bound, dtype=torch.uint8, device=DEV))
        s.ctx = _Context(sizes, sampled, bool(case.get("compact")))
        if op == "step":
            s.out = torch.zeros(total, dtype=torch.float32, device=DEV)
            s.out_list = sbc.TensorList(_views(s.out, offs, sizes))
            s.status = torch.zeros(1, dtype=torch.int32, device=DEV)
    elif op == "decode":
        (msg, s.nbytes), = _messages(case, seed, 1, sizes, offs, total, scales)
        s.msg = sbc.MessageBuffer(msg)
        s.out = torch.zeros(total, dtype=torch.float32, device=DEV)
        s.out_list = sbc.TensorList(_views(s.out, offs, sizes))
        s.ctx = _Context(sizes)
    elif op == "average":
        s.server = _Closing(rounds.Server(sizes, s.p, DEV))
        s.messages = [(sbc.MessageBuffer(m), n) for m, n in _messages(case, seed, case["clients"], sizes, offs, total, scales)]
    else:
        s.server = _Closing(rounds.Server(sizes, s.p, DEV))
        s.clients = []
        for c in range(case["clients"]):
            (up,), res = _client(case, seed, c, sizes, offs, total, scales, 1, False)
            cl = _Closing(rounds.Client(sizes, s.p, DEV))
            for dst, src in zip(cl.it.dW, _views(up, offs, sizes)):
                dst.copy_(src)
            for dst, src in zip(cl.it.R, _views(res, offs, sizes)):
                dst.copy_(src)
            s.clients.append(cl)
        s.weights = torch.zeros_like(s.server.it.acc_flat)
    torch.cuda.synchronize()
    return s


class _Closing:
    """A client or server of the round loop, closed with this object."""

    def __init__(self, it):
        self.it = it

    def __del__(self):
        self.it.close()


# ---------------------------------------------------------------- one pass ----

def run(s):
    op = s.case["op"]
    if op in ("compress", "step"):
        dW = s.updates[s.turn]
        s.turn = (s.turn + 1) % len(s.updates)
        n = sbc.sbc_compress(s.ctx.handle, dW, s.residual_list, s.p, s.msg)
        if op == "compress":
            return {"bytes": n, "message": s.msg.tensor, "residual": s.residual}
        sbc.sbc_decompress_accumulate_noalloc(s.msg, n, s.p, 1.0, s.out_list, s.status)
        return {"bytes": n, "message": s.msg.tensor, "residual": s.residual, "out": s.out, "status": s.status}
    if op == "decode":
        sbc.sbc_decompress_accumulate(s.ctx.handle, s.msg, s.nbytes, s.p, 1.0, s.out_list)
        return {"out": s.out}
    server = s.server.it
    if op == "average":
        server.average(s.messages)
        return {"out": server.acc_flat}
    clients = [c.it for c in s.clients]
    now = torch.cuda.current_stream()
    for c in clients:
        c.stream.wait_stream(now)                 # this round's weights
        c.begin_upload()
    messages = [c.end_upload() for c in clients]
    server.average(messages)
    s.weights.add_(server.acc_flat)
    return {"bytes": [n for _, n in messages], "messages": [m for m, _ in messages],
            "residuals": [c.R_flat for c in clients], "average": server.acc_flat, "weights": s.weights}


# ------------------------------------------------------------- what it takes ----

def work(case):
    """Bytes: update and residual read, residual written; messages; dense outputs of the server."""
    sizes = _sizes(case)
    n, p = sum(sizes), case["p"]
    kept = sum(sbc.sbc_num_kept(x, p) for x in sizes)
    message = 32 + 24 * len(sizes) + kept * (sbc.sbc_golomb_bstar(p) + 1.6) / 8.0
    client, server = 12.0 * n + message, message + 8.0 * kept     # (a decoded entry is read and written)
    op, c = case["op"], case.get("clients", 1)
    if op == "compress":
        return {"bytes": client, "flops": float(n)}
    if op == "step":
        return {"bytes": client + server, "flops": float(n + kept)}
    if op == "decode":
        return {"bytes": server, "flops": float(kept)}
    if op == "average":
        return {"bytes": c * message + 4.0 * n, "flops": float(c * kept)}
    return {"bytes": c * (client + message) + 12.0 * n, "flops": float(c * (n + kept) + n)}


def tolerance(case):
    return "exact"


# --------------------------------------------------- the same in 64 bits ----

def _kept(n, p):
    return min(n, max(1, int(math.floor(p * float(n)))))


def _mix32(x):
    m = 0xFFFFFFFF
    x = x ^ (x >> 16)
    x = (x * 0x7FEB352D) & m
    x = x ^ (x >> 15)
    x = (x * 0x846CA68B) & m
    return x ^ (x >> 16)


def _sample(n, t):
    """Positions of the stratified sample of the subsampled variant."""
    if n <= 16384:
        return np.arange(n)
    slots, out = n // 64, []
    for r in range(256):
        lo, hi = r * slots // 256, (r + 1) * slots // 256
        h = _mix32((r * 0x9E3779B9 + t * 0x85EBCA6B + 1) & 0xFFFFFFFF)
        out.append((lo + ((h * (hi - lo)) >> 32)) * 64 + np.arange(64))
    return np.concatenate(out)


def _side(x, count, floor_value):
    """Mask of the `count` largest entries of x (equal values to the lowest index), and their mean;
    with a threshold, of every entry at or beyond it, at most `count` of them."""
    if floor_value is not None:
        mask = x >= floor_value
        if int(mask.sum()) <= count:
            return mask, float(x[mask].double().mean())
    tau = torch.topk(x, count).values[-1]
    mask = x > tau
    ties = torch.nonzero(x == tau).flatten()
    mask[ties[:count - int(mask.sum())]] = True
    return mask, float(x[mask].double().mean())


def _step64(case, dW, R, t):
    """Alg. 2 and the residual line on one tensor: (dense binarized update, new residual), fp64."""
    A = R + dW                                    # fp32, one rounding, by definition
    n, p = A.numel(), case["p"]
    k = _kept(n, p)
    floors = (None, None)
    if case.get("sampled"):
        smp = torch.sort(A[torch.from_numpy(_sample(n, t)).to(DEV)], descending=True).values
        m = smp.numel()
        r = max(1, int(math.floor(p * float(m))))
        floors = (smp[r - 1], -smp[m - r])
        k = min(n, 2 * k + 64)
    mp, up = _side(A, k, floors[0])
    mn, un = _side(-A, k, floors[1])
    mask, mu = (mp, up) if up >= un else (mn, -un)
    sent = mask.double() * mu
    return sent, A.double() - sent


def exact(case, seed):
    sizes = _sizes(case)
    c = case.get("clients", 1)
    if c * sum(sizes) > 900000000 or c * len(sizes) > 8000:
        return None
    offs, total = _offsets(case, sizes)
    scales = _layers(case, seed, sizes)
    op = case["op"]
    zero = op in ("decode", "average")

    def padded(parts, o, n):
        flat = torch.zeros(n, dtype=torch.float64, device=DEV)
        for x, at in zip(parts, o):
            flat[at:at + x.numel()] = x
        return flat

    sent, left = [], []
    for i in range(c):
        ups, res = _client(case, seed, i, sizes, offs, total, scales, 1, zero)
        got = [_step64(case, dw, r, t) for t, (dw, r) in enumerate(zip(_views(ups[0], offs, sizes), _views(res, offs, sizes)))]
        sent.append([a for a, _ in got])
        left.append([b for _, b in got])
    if op == "compress":
        return {"bytes": None, "message": None, "residual": padded(left[0], offs, total)}
    if op == "step":
        return {"bytes": None, "message": None, "residual": padded(left[0], offs, total),
                "out": padded(sent[0], offs, total), "status": None}
    if op == "decode":
        return {"out": padded(sent[0], offs, total)}
    # (the round loop's own buffers start every tensor at a multiple of 64 entries)
    offs64, total64 = _offsets({}, sizes)
    avg = padded([sum(x) / c for x in zip(*sent)], offs64, total64)
    if op == "average":
        return {"out": avg}
    return {"bytes": [None] * c, "messages": [None] * c, "residuals": [padded(x, offs64, total64) for x in left],
            "average": avg, "weights": avg}
