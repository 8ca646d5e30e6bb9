"""The work a user of this library has it do, as measurable cases through the public entry points.

A case is a pruned recurrent layer (cell, hidden units, samples advanced together, timesteps, density of the recurrent
matrix, how nonzeros are spread over its rows) and one of four kinds of call:

  forward   the recurrence over b' that is already there (forward / forward_lstm / forward_gru)
  layer     a whole layer from raw inputs: the dense input projection, then the recurrence
  backward  gradients of a vanilla layer whose forward outputs are kept: backward pass and recurrent weight gradient
  train     a whole training step: forward pass that keeps what the backward pass needs, backward pass, weight gradient

``weights`` says how a training user gets the weight gradient: "fused" asks the backward call for it,
"separate" calls weight_gradient on the forward handle.  ``activations`` is the library's option of that name.
Patterns are uniform random (the unstructured pruning the library is built for), weights N(0, 1/nonzeros of the row)
times a gain below one, b' and inputs N(0, 1).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1804_10223_amd import binding

GATES = {"lstm": 4, "gru": 3}
VANILLA = ("relu", "tanh", "identity")


def _case(name, kind, cell, hidden, batch, steps, density, rows="fixed", inputs=0, weights="", activations="binary32", h0=False):
    return {"name": name, "kind": kind, "cell": cell, "hidden": hidden, "batch": batch, "steps": steps, "density": density,
            "rows": rows, "inputs": inputs, "weights": weights, "activations": activations, "h0": h0}


def listed():
    return [
        # one short request on a small layer: launch and latency
        _case("rnn_256_b1_t16", "forward", "relu", 256, 1, 16, 0.10),
        # the shape of the paper's ablation table: an ordinary layer that fits a few compute units
        _case("rnn_1152_b4", "forward", "relu", 1152, 4, 256, 0.10, h0=True),
        # the headline layer
        _case("rnn_2304_b4", "forward", "relu", 2304, 4, 256, 0.30),
        # the largest layer, with rows of unequal length
        _case("rnn_5760_b2", "forward", "relu", 5760, 2, 128, 0.10, rows="poisson"),
        # a gated layer at the largest batch
        _case("lstm_1024_b8", "forward", "lstm", 1024, 8, 128, 0.20),
        # a translation layer over one sentence, from its inputs: small product, small recurrence
        _case("lstm_layer_512_b1_t50", "layer", "lstm", 512, 1, 50, 0.0625, inputs=512),
        # a speech layer over a long utterance, from its inputs, with binary16 activations
        _case("speech_layer_2560_b8_half", "layer", "relu", 2560, 8, 512, 0.12, inputs=2560, activations="binary16"),
        # sizes that divide nothing, inputs that no wide load can take
        _case("gru_layer_771_b4_t100", "layer", "gru", 771, 4, 100, 0.15, rows="poisson", inputs=333, h0=True),
        # gradients of the headline layer, weight gradient asked of the backward call
        _case("backward_2304_b4", "backward", "relu", 2304, 4, 256, 0.30, weights="fused"),
        # a training step of the gated layer, weight gradient on the forward handle
        _case("train_lstm_1024_b8", "train", "lstm", 1024, 8, 128, 0.20, weights="separate"),
        # a training step of a GRU layer from its inputs, weight gradient asked of the backward call
        _case("train_gru_1024_b4", "train", "gru", 1024, 4, 128, 0.20, inputs=1024, weights="fused"),
        # a training step of odd sizes
        _case("train_tanh_701_b2_t77", "train", "tanh", 701, 2, 77, 0.15, rows="poisson", weights="separate", h0=True),
    ]


def _log_uniform(rng, low, high):
    return math.exp(rng.uniform(math.log(low), math.log(high)))


def draw(rng):
    """One more case: cell, kind, sizes and density spread over the ranges of the listed ones."""
    while True:
        kind = rng.choice(["forward", "forward", "layer", "layer", "backward", "train", "train"])
        cell = rng.choice({"backward": ["relu", "tanh"], "train": ["tanh", "lstm", "gru"]}.get(kind, ["relu", "relu", "tanh", "lstm", "gru"]))
        gates = GATES.get(cell, 1)
        batch = rng.choice([1, 2, 4, 8])
        hidden = int(round(_log_uniform(rng, 160, 5760 if gates == 1 else 2048)))
        if rng.random() < 0.5:
            hidden = max(160, hidden // 64 * 64)
        steps = int(round(_log_uniform(rng, 16, 256)))
        density = round(_log_uniform(rng, 0.04, 0.30), 4)
        inputs = int(round(_log_uniform(rng, 80, 2560))) if kind == "layer" or (kind == "train" and rng.random() < 0.5) else 0
        if inputs and rng.random() < 0.6:
            inputs = max(80, inputs // 8 * 8)
        half = kind in ("forward", "layer") and cell in VANILLA and batch >= 4 and rng.random() < 0.3
        gradients = kind in ("backward", "train")
        # what fits on the chip with room to spare, and no more work than the largest listed case
        if gates * hidden * hidden * density > (1.6e6 if gradients else 3.4e6):
            continue
        if hidden * batch > (8192 if gates > 1 else 20480) or (gradients and hidden * batch * gates > 32768):
            continue
        if 2.0 * inputs * gates * hidden * steps * batch > 3e10:
            continue
        # (asking the backward call for the weight gradient is not offered for every mapping: drawn where it always is)
        fused = gradients and gates > 1 and hidden * batch * gates <= 8192 and rng.random() < 0.6
        return _case("", kind, cell, hidden, batch, steps, density, rows=rng.choice(["fixed", "poisson"]), inputs=inputs,
                     weights=("fused" if fused else "separate") if gradients else "",
                     activations="binary16" if half else "binary32", h0=rng.random() < 0.5)


def _pruned(gen, rows, cols, density, spread, gain):
    """CSR arrays of a rows x cols matrix with a uniform random pattern, drawn on the GPU."""
    mean = int(round(density * cols))
    if spread == "poisson":   # rows of Poisson length, given their total (which fixes the shape of the weight gradient)
        picks = torch.randint(rows, (rows * mean,), device="cuda", generator=gen)
        counts = torch.bincount(picks, minlength=rows).clamp_(max=cols)
    else:
        counts = torch.full((rows,), mean, device="cuda", dtype=torch.long)
    row_ptr = torch.zeros(rows + 1, dtype=torch.long, device="cuda")
    torch.cumsum(counts, 0, out=row_ptr[1:])
    most = int(counts.max())
    col_parts = []
    for first in range(0, rows, 2048):
        last = min(rows, first + 2048)
        order = torch.rand((last - first, cols), device="cuda", generator=gen).argsort(dim=1, stable=True)[:, :most]
        keep = torch.arange(most, device="cuda")[None, :] < counts[first:last, None]
        order = order.masked_fill(~keep, cols).sort(dim=1).values
        col_parts.append(order[order < cols])
    per_row = torch.repeat_interleave(counts, counts).float()
    val = torch.randn(int(row_ptr[-1]), device="cuda", generator=gen) / per_row.sqrt() * gain
    return (row_ptr.int().cpu().numpy(), torch.cat(col_parts).int().cpu().numpy(),
            val.half().cpu().numpy().view(np.uint16))


def prepare(case, seed):
    """Handles made once per model, and the device tensors a user's program holds before the call."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    cell, hidden, batch, steps, kind = case["cell"], case["hidden"], case["batch"], case["steps"], case["kind"]
    rows = hidden * GATES.get(cell, 1)

    def normal(*shape):
        return torch.randn(shape, device="cuda", generator=gen)

    csr = _pruned(gen, rows, hidden, case["density"], case["rows"], 0.9 if cell in VANILLA else 1.0)
    state = {"case": case}
    if kind != "backward" or case["weights"] == "separate":
        options = {"activations": case["activations"]} if case["activations"] != "binary32" else {}
        state["rnn"] = binding.SparseRNN(hidden, batch, cell, *csr, **options)
    if kind in ("backward", "train"):
        state["bwd"] = binding.SparseRNN(hidden, batch, cell if cell in VANILLA else cell + "_backward",
                                         *binding.transpose_csr(rows, hidden, *csr))
        state["dh"] = normal(steps, batch, hidden)
    if kind == "backward":
        kept = normal(steps, batch, hidden)
        state["h"] = kept.clamp_(min=0.0) if cell == "relu" else kept.tanh_()
    elif case["inputs"]:
        state["x_in"] = normal(steps, batch, case["inputs"])
        state["w_in"] = (normal(rows, case["inputs"]) / math.sqrt(case["inputs"])).half()
        state["bias"] = normal(rows) * 0.1
    else:
        state["x"] = normal(steps, batch, rows)
    state["h0"] = normal(batch, hidden) * 0.1 if case["h0"] else None
    state["c0"] = normal(batch, hidden) * 0.1 if case["h0"] and cell == "lstm" else None
    state["b_hn"] = normal(hidden) * 0.5 if cell == "gru" else None
    return state


def run(state):
    case, h0 = state["case"], state["h0"]
    cell, kind = case["cell"], case["kind"]
    rnn, bwd = state.get("rnn"), state.get("bwd")
    fused = case["weights"] == "fused"
    if kind == "backward":
        if fused:
            return bwd.backward_with_weights(state["dh"], state["h"], h0)
        delta, dh0 = bwd.backward(state["dh"], state["h"])
        return delta, dh0, rnn.weight_gradient(delta, state["h"], h0)
    x = rnn.project(state["x_in"], state["w_in"], state["bias"]) if case["inputs"] else state["x"]
    if kind != "train":
        if cell == "lstm":
            return rnn.forward_lstm(x, h0, state["c0"])
        if cell == "gru":
            return rnn.forward_gru(x, state["b_hn"], h0)
        return rnn.forward(x, h0)
    if cell == "lstm":
        c0 = state["c0"]
        h, c, gates = rnn.forward_lstm_train(x, h0, c0)
        if fused:
            return (h, c) + tuple(bwd.backward_lstm_with_weights(state["dh"], gates, c, h, c0, h0))
        d, dh0, dc0 = bwd.backward_lstm(state["dh"], gates, c, c0)
        return h, c, d, dh0, dc0, rnn.weight_gradient(d, h, h0)
    if cell == "gru":
        h, gates = rnn.forward_gru_train(x, state["b_hn"], h0)
        if fused:
            return (h,) + tuple(bwd.backward_gru_with_weights(state["dh"], gates, h, h0))
        d, d_rec, dh0 = bwd.backward_gru(state["dh"], gates, h, h0)
        return h, d, d_rec, dh0, rnn.weight_gradient(d_rec, h, h0)
    h = rnn.forward(x, h0)
    if fused:
        return (h,) + tuple(bwd.backward_with_weights(state["dh"], h, h0))
    delta, dh0 = bwd.backward(state["dh"], h)
    return h, delta, dh0, rnn.weight_gradient(delta, h, h0)


def work(case):
    """Least bytes (inputs read once, outputs written once; a nonzero is a binary16 value and a 16-bit index) and operations."""
    gates = GATES.get(case["cell"], 1)
    hidden, steps, batch, kind = case["hidden"], case["steps"], case["batch"], case["kind"]
    rows, vectors = gates * hidden, steps * batch
    nnz = rows * int(round(case["density"] * hidden))
    size = flops = 0
    if case["inputs"]:
        size += 4 * vectors * case["inputs"] + 2 * rows * case["inputs"]
        flops += 2 * vectors * rows * case["inputs"]
    if kind != "backward":
        size += 4 * nnz + (0 if case["inputs"] else 4 * vectors * rows)            # weights, b'
        size += 4 * vectors * hidden * (2 if case["cell"] == "lstm" else 1)        # h (and c)
        flops += 2 * vectors * nnz
    if kind in ("backward", "train"):
        size += 4 * nnz + 4 * vectors * hidden + 4 * vectors * rows                # weights, incoming and outgoing gradients
        size += 4 * vectors * hidden if kind == "backward" else 0                  # forward outputs
        size += 4 * vectors * rows if case["cell"] == "gru" else 0                 # gradient of the recurrent sums
        size += 4 * nnz                                                            # weight gradient
        flops += 4 * vectors * nnz
    return {"bytes": size, "flops": flops}


def tolerance(case):
    """About four times what the same passes show when the products of a row are added in another order (twice or half the
    lanes per row): at most 3.6e-7 and 5.8e-6 over the listed and forty drawn cases.  binary16 activations round every h
    once, and a sum that falls on the other side of a rounding boundary moves it by one unit of binary16: 1.9e-4, 1.8e-3."""
    if case["activations"] == "binary16":
        return {"rel": 8e-4, "max": 8e-3}
    return {"rel": 2e-6, "max": 3e-5}
