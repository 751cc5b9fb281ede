"""What a user of the library has it do, as cases that can be timed: forward passes of the model families over the sizes
they come in, and one iteration of the mask update between them.

listed() names the cases, draw() gives more of the same ranges, prepare() builds what a user's program holds before the
call (weights set, device buffers, workspace), run() is one pass through the public entry points on the caller's stream.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1901_10997_amd import binding as B

# Model widths of the latency profile, speech- and language-model batches, utterance lengths (10 ms frames) and word
# sequences: the ranges draw() covers.
WIDTHS = (64, 2048)
INPUTS = (32, 2048)
STEPS = (8, 300)
MAX_BATCH = {"f32": 64, "bf16": 256}
KEPT = (0.05, 0.40)        # fraction of the weights that grow-and-prune masks leave
PRUNED_ROWS = (256, 6000)  # of a gate matrix, and its columns
PRUNED_COLS = (200, 3000)
MAX_PRUNED = 9_000_000
MAX_FLOPS = 3.0e11         # a drawn forward (dense count); below the listed speech and throughput models
MAX_PARAMS = 30_000_000    # ... and its weights, so that a model is packed quickly


def _forward(name, cell, layers, bidir, D, H, T, batch, dtype="f32", keep=None, state=False):
    c = dict(kind="forward", cell=cell, layers=layers, bidir=bidir, D=D, H=H, T=T, B=batch, dtype=dtype, keep=keep,
             state=state)
    return dict(c, name=name) if name else c


def listed():
    return [
        # smallest model of the configurations, one sequence: the latency of a single dense layer
        _forward("lstm_1x200_dense_b1", "lstm", 1, False, 200, 200, 35, 1),
        # a wide layer of the latency-versus-width profile (off the 32-grid)
        _forward("lstm_1x1900_dense_b1", "lstm", 1, False, 1900, 1900, 35, 1),
        # the pruned language model answering one user: states carried from call to call
        _forward("lm_2x1500_masked_b1", "lstm", 2, False, 1500, 1500, 35, 1, keep=0.10, state=True),
        # the same model scoring a batch of sequences
        _forward("lm_2x1500_masked_b20", "lstm", 2, False, 1500, 1500, 35, 20, keep=0.10, state=True),
        # the pruned speech model over a batch of utterances
        _forward("speech_5x800_masked_b16", "lstm", 5, True, 640, 800, 300, 16, keep=0.15),
        # the same model before pruning (and what row/column pruning plus compaction leaves: dense, smaller)
        _forward("speech_5x800_dense_b16", "lstm", 5, True, 640, 800, 300, 16),
        # offline throughput in bf16
        _forward("lstm_2x1024_bf16_b256", "lstm", 2, False, 1024, 1024, 128, 256, dtype="bf16"),
        # the row/column-compacted language model (1500/400 -> 1197/317) in bf16 at a serving batch
        _forward("lm_2x1197_bf16_b20", "lstm", 2, False, 317, 1197, 70, 20, dtype="bf16", state=True),
        # H-LSTM language model, one user
        _forward("hlstm_lm_1x1500_masked_b1", "hlstm", 1, False, 400, 1500, 35, 1, keep=0.10, state=True),
        # H-LSTM speech model, pruned
        _forward("hlstm_3x800_masked_b16", "hlstm", 3, True, 640, 800, 300, 16, keep=0.20),
        # H-LSTM speech model grown to a hardware-favoured width, dense
        _forward("hlstm_3x640_dense_b16", "hlstm", 3, True, 640, 640, 300, 16),
        # one pruning iteration on a gate matrix: connections, then rows and columns, then the smaller matrix
        dict(name="prune_6000x1500", kind="prune", M=6000, N=1500, keep=0.8, p_w=0.35, p_r=0.05, p_c=0.05),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    family = rng.choice(["lstm_dense", "lstm_masked", "lstm_masked", "lstm_bf16", "lstm_bf16", "hlstm_masked",
                         "hlstm_dense", "prune"])
    if family == "prune":
        N = _log_int(rng, *PRUNED_COLS)
        return dict(kind="prune", M=min(_log_int(rng, *PRUNED_ROWS), MAX_PRUNED // N), N=N, keep=round(rng.uniform(0.2, 1.0), 3),
                    p_w=round(rng.uniform(0.05, 0.7), 3), p_r=round(rng.uniform(0.01, 0.2), 3),
                    p_c=round(rng.uniform(0.01, 0.2), 3))
    dtype = "bf16" if family == "lstm_bf16" else "f32"
    cell = "hlstm" if family.startswith("hlstm") else "lstm"
    keep = round(rng.uniform(*KEPT), 3) if family.endswith("masked") else None
    batch = 1 if rng.random() < 0.3 else _log_int(rng, 2, MAX_BATCH[dtype])
    bidir = rng.random() < 0.4
    c = _forward(None, cell, rng.randint(1, 5), bidir, _log_int(rng, *INPUTS), _log_int(rng, *WIDTHS),
                 _log_int(rng, *STEPS), batch, dtype, keep, state=rng.random() < 0.5)
    while _params(c) > MAX_PARAMS and c["layers"] > 1:
        c["layers"] -= 1
    while _params(c) > MAX_PARAMS:
        c["H"] = c["H"] * 7 // 8
    c["T"] = max(1, min(c["T"], int(MAX_FLOPS / (2.0 * c["B"] * _params(c)))))
    return c


def _matrices(c):
    """(name, rows, columns) of every weight matrix of every (layer, direction)."""
    H, ndir = c["H"], 2 if c["bidir"] else 1
    for l in range(c["layers"]):
        D = c["D"] if l == 0 else ndir * H
        for d in range(ndir):
            if c["cell"] == "hlstm":    # gate hidden layers as wide as the hidden state
                yield (l, d), (("W1x", 4 * H, D), ("W1h", 4 * H, H), ("W2", 4 * H, H))
            else:
                yield (l, d), (("Wx", 4 * H, D), ("Wh", 4 * H, H))


def _params(c):
    return sum(r * k for _, mats in _matrices(c) for _, r, k in mats)


def prepare(case, seed):
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)

    def uniform(shape, a):
        return (torch.rand(shape, generator=gen, device=dev) * 2 - 1) * a

    if case["kind"] == "prune":
        M, N = case["M"], case["N"]
        # rows and columns of different importance, as training leaves them
        W = torch.randn((M, N), generator=gen, device=dev)
        W *= torch.exp(0.5 * torch.randn((M, 1), generator=gen, device=dev))
        W *= torch.exp(0.5 * torch.randn((1, N), generator=gen, device=dev))
        mask = (torch.rand((M, N), generator=gen, device=dev) < case["keep"]).to(torch.uint8)
        return dict(case=case, W0=W, mask0=mask, W=torch.empty_like(W), mask=torch.empty_like(mask), Wc=torch.empty_like(W),
                    mask_c=torch.empty_like(mask), rows=torch.empty(M, dtype=torch.int32, device=dev),
                    cols=torch.empty(N, dtype=torch.int32, device=dev))

    H, T, Bn, keep = case["H"], case["T"], case["B"], case["keep"]
    ndir = 2 if case["bidir"] else 1
    bf16 = case["dtype"] == "bf16"
    weights = {}
    for key, mats in _matrices(case):
        p = {}
        fan_in = sum(k for n, _, k in mats if n != "W2") * (keep or 1.0)
        a = min(0.4, 1.0 / math.sqrt(fan_in))
        for name, rows, cols in mats:
            W = uniform((rows, cols), a)
            p[name] = (W.bfloat16().float() if bf16 else W).cpu().numpy()
            p["M" + name[1:]] = (None if keep is None else
                                 (torch.rand((rows, cols), generator=gen, device=dev) < keep).to(torch.uint8).cpu().numpy())
        for name in (("b1", "b2") if case["cell"] == "hlstm" else ("b",)):
            p[name] = uniform(4 * H, a).cpu().numpy()
        weights[key] = p
    model = B.Lstm(case["layers"], case["D"], H, case["bidir"], B.LSTM_BF16 if bf16 else B.LSTM_F32,
                   gate_hidden=H if case["cell"] == "hlstm" else 0)
    model.set_weights_from(weights)
    x = torch.randn((T, Bn, case["D"]), generator=gen, device=dev)
    if bf16:
        x = x.to(torch.bfloat16)
    n = case["layers"] * ndir
    h0 = uniform((n, Bn, H), 0.5) if case["state"] else None
    c0 = uniform((n, Bn, H), 0.5) if case["state"] else None
    ws_bytes = B.lstm_workspace_bytes(model.handle, T, Bn)
    return dict(case=case, model=model, x=x, h0=h0, c0=c0, y=torch.empty((T, Bn, ndir * H), device=dev),
                hT=torch.empty((n, Bn, H), device=dev), cT=torch.empty((n, Bn, H), device=dev),
                ws=torch.empty(ws_bytes, dtype=torch.uint8, device=dev))


def run(s):
    c = s["case"]
    stream = torch.cuda.current_stream().cuda_stream
    if c["kind"] == "prune":
        M, N = c["M"], c["N"]
        W, mask = s["W"], s["mask"]
        W.copy_(s["W0"])            # the unpruned matrix is kept for the roll-back
        mask.copy_(s["mask0"])
        before, after = B.lstm_prune_weights(W.data_ptr(), mask.data_ptr(), M * N, c["p_w"], stream)
        rows, _ = B.lstm_prune_rows_cols(W.data_ptr(), mask.data_ptr(), M, N, c["p_r"], 0.0, stream)
        _, cols = B.lstm_prune_rows_cols(W.data_ptr(), mask.data_ptr(), M, N, 0.0, c["p_c"], stream)
        Rc, Nc = B.lstm_compact_rows_cols(W.data_ptr(), mask.data_ptr(), 1, M, N, s["rows"].data_ptr(), s["cols"].data_ptr(),
                                          s["Wc"].data_ptr(), s["mask_c"].data_ptr(), stream)
        return dict(before=before, after=after, rows=rows, cols=cols, Rc=Rc, Nc=Nc, W=W, mask=mask, row_index=s["rows"],
                    col_index=s["cols"], Wc=s["Wc"].view(-1)[:Rc * Nc], mask_c=s["mask_c"].view(-1)[:Rc * Nc])
    B.lstm_forward(s["model"].handle, c["T"], c["B"], s["x"].data_ptr(),
                   None if s["h0"] is None else s["h0"].data_ptr(), None if s["c0"] is None else s["c0"].data_ptr(),
                   s["y"].data_ptr(), s["hT"].data_ptr(), s["cT"].data_ptr(), s["ws"].data_ptr(), s["ws"].numel(), stream)
    return s["y"], s["hT"], s["cT"]


def work(case):
    if case["kind"] == "prune":
        n = case["M"] * case["N"]
        # weights and mask read, both written back, the compacted matrix and its mask written; one addition per sum
        return {"bytes": 15.0 * n, "flops": 2.0 * n}
    keep = case["keep"] or 1.0
    size = 2 if case["dtype"] == "bf16" else 4
    ndir = 2 if case["bidir"] else 1
    kept = _params(case) * keep
    TB, H, n = case["T"] * case["B"], case["H"], case["layers"] * ndir
    states = (2 if case["state"] else 0) + 2
    # a kept weight of a masked matrix carries its 16-bit column
    return {"bytes": kept * (size + (0 if case["keep"] is None else 2)) + TB * case["D"] * size + TB * ndir * H * 4
            + states * n * case["B"] * H * 4, "flops": 2.0 * TB * kept}


def tolerance(case):
    if case["kind"] == "prune":
        return "exact"
    # fp32 sums of at most a few thousand terms through contracting gates; bf16 rounds the recurrent operand every step
    return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 1e-5}
