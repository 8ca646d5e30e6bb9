"""Handles with nothing fixed about the mapping, which sprnn_create chooses by measuring: what may not depend on its choice.

Shapes that are divided into parts by themselves on an otherwise idle device (the tests hold whatever is chosen)."""
import numpy as np
import pytest
import torch

from paper_1804_10223_amd import binding, workloads as wl

pytestmark = pytest.mark.gpu
GATES = {"lstm": 4, "gru": 3}


def _dev(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _normal(rng, *shape):
    return _dev(rng.standard_normal(shape).astype(np.float32))


def _offered(handle, cell):
    """Which calls a handle offers: asked without a place for the result, so that what is offered is refused as INVALID (or, with
    no steps, done) before anything is launched, and the rest as UNSUPPORTED."""
    lib, h, none = binding.load_library(), handle._h, [None]
    codes = {"weight_gradient": lib.sprnn_weight_gradient(h, 0, *none * 5)}
    if cell == "lstm_backward":
        codes["with_weights"] = lib.sprnn_backward_lstm_with_weights(h, 0, *none * 11)
    elif cell == "gru_backward":
        codes["with_weights"] = lib.sprnn_backward_gru_with_weights(h, 0, *none * 9)
    elif cell not in GATES:
        codes["with_weights"] = lib.sprnn_backward_with_weights(h, 0, *none * 7)
        codes["backward"] = lib.sprnn_backward(h, 0, *none * 5)
        codes["noalloc"] = lib.sprnn_forward_noalloc(h, 0, *none * 4)
    return {k for k, code in codes.items() if code in (binding.SPRNN_OK, binding.SPRNN_ERR_INVALID)}


@pytest.mark.parametrize("cell,H,B,dens", [("relu", 1152, 4, 0.1), ("relu", 4096, 4, 0.01), ("tanh", 2000, 8, 0.03), ("lstm", 1024, 8, 0.05),
                                           ("lstm_backward", 1024, 8, 0.2), ("lstm_backward", 1024, 4, 0.05), ("gru_backward", 1500, 4, 0.1)])
def test_no_call_is_lost_to_a_faster_mapping(cell, H, B, dens):
    w = wl.make_workload("offer", cell.replace("_backward", ""), H, B, 1, dens, seed=H + B)
    csr = (w.row_ptr, w.col_idx, w.val_bits)
    if cell.endswith("_backward"):
        csr = binding.transpose_csr(w.rows, H, *csr)[:3]
    with binding.SparseRNN(H, B, cell, *csr, xcd="spread") as own, binding.SparseRNN(H, B, cell, *csr) as chosen:
        print("case", cell, H, B, "lanes", own.info()["lanes_per_row"], chosen.info()["lanes_per_row"], "parts", chosen.info()["parts"], flush=True)
        assert _offered(own, cell) <= _offered(chosen, cell)


LONG = 160


@pytest.mark.parametrize("cell,H,B,dens,rows,options", [
    ("relu", 1152, 4, 0.1, "fixed", {}),
    ("tanh", 701, 2, 0.15, "poisson", {}),
    ("relu", 2304, 4, 0.3, "fixed", {}),
    ("relu", 2560, 8, 0.12, "fixed", {"activations": "binary16"}),
    ("lstm", 837, 2, 0.1, "poisson", {}),
    ("lstm", 1024, 8, 0.2, "fixed", {}),
    ("gru", 771, 4, 0.15, "poisson", {}),
])
def test_calls_of_every_length_have_the_bits_of_any_handle_with_these_lanes(cell, H, B, dens, rows, options):
    """A divided handle runs short calls undivided (from which length on, creation measures): calls on both sides of that, in
    turn, against one long call, and that against a handle with these lanes that is not divided."""
    w = wl.make_workload("length", cell, H, B, LONG, dens, seed=H, row_nnz=rows, h0_std=0.5)
    csr = (w.row_ptr, w.col_idx, w.val_bits)
    rng = np.random.Generator(np.random.PCG64(2))
    x, h0, b_hn = _dev(w.x), _dev(w.h0), _dev(getattr(w, "b_hn", None))
    c0, e = _normal(rng, B, H), _normal(rng, LONG, B, H)
    gated, half = cell in GATES, bool(options)

    def forward(rnn, steps):
        xs = x[:steps].contiguous()
        if cell == "lstm":
            return rnn.forward_lstm_train(xs, h0, c0)
        return rnn.forward_gru_train(xs, b_hn, h0) if cell == "gru" else (rnn.forward(xs, h0),)

    def backward(bwd, kept, steps):   # of the last `steps` of the long call: nothing flows in from beyond its end
        tail = lambda a: a[LONG - steps:].contiguous()
        before = lambda a, first: first if steps == LONG else a[LONG - steps - 1].contiguous()
        if cell == "lstm":
            h, c, gates = kept
            return bwd.backward_lstm(tail(e), tail(gates), tail(c), before(c, c0))[:1]
        if cell == "gru":
            h, gates = kept
            return bwd.backward_gru(tail(e), tail(gates), tail(h), before(h, h0))[:2]
        return bwd.backward(tail(e), tail(kept[0]))[:1]

    name = cell + "_backward" if gated else cell
    t_csr = None if half else binding.transpose_csr(w.rows, H, *csr)[:3]
    with binding.SparseRNN(H, B, cell, *csr, **options) as rnn:
        info = rnn.info()
        print("case", cell, H, B, {k: info[k] for k in ("parts", "one_xcd", "lanes_per_row", "grid", "block")}, flush=True)
        want = forward(rnn, LONG)
        for steps in (1, 90, 2, 3, 60, 5, 8, 40, 13, 22, 30, LONG):
            for k, (a, b) in enumerate(zip(forward(rnn, steps), want)):
                assert torch.equal(a, b[:steps]), (steps, k)
        assert rnn.check() == binding.SPRNN_OK
    with binding.SparseRNN(H, B, cell, *csr, lanes_per_row=info["lanes_per_row"], jitter=3, **options) as fixed:
        assert fixed.info()["parts"] == 1
        for a, b in zip(forward(fixed, LONG), want):
            assert torch.equal(a, b)
        assert fixed.check() == binding.SPRNN_OK
    if half:
        return
    with binding.SparseRNN(H, B, name, *t_csr) as bwd:
        info = bwd.info()
        print("   backward", {k: info[k] for k in ("parts", "one_xcd", "lanes_per_row", "grid", "block")}, flush=True)
        grads = backward(bwd, want, LONG)
        for steps in (1, 90, 2, 60, 5, 40, 13, 22, 30, LONG):
            for k, (a, b) in enumerate(zip(backward(bwd, want, steps), grads)):
                assert torch.equal(a, b[LONG - steps:]), (steps, k)
        assert bwd.check() == binding.SPRNN_OK
    with binding.SparseRNN(H, B, name, *t_csr, lanes_per_row=info["lanes_per_row"], jitter=3) as fixed:
        for a, b in zip(backward(fixed, want, LONG), grads):
            assert torch.equal(a, b)
        assert fixed.check() == binding.SPRNN_OK


@pytest.mark.parametrize("cell,H,B,dens,lengths", [
    # lengths on both sides of where the product behind the recurrence takes over from the sums inside it, and between that and
    # where it would if the time that a division saves were counted
    ("tanh", 1152, 4, 0.1, (3, 12, 40)),
    ("relu", 701, 2, 0.15, (5, 20, 80)),
    ("lstm", 1024, 8, 0.2, (2, 3, 12)),
    ("gru", 1024, 4, 0.2, (4, 12, 40)),
])
def test_the_weight_gradient_of_a_backward_call_has_the_bits_of_any_handle_with_these_lanes(cell, H, B, dens, lengths):
    w = wl.make_workload("default", cell, H, B, 1, dens, seed=H)
    t_csr = binding.transpose_csr(w.rows, H, w.row_ptr, w.col_idx, w.val_bits)
    name = cell + "_backward" if cell in GATES else cell
    rng = np.random.Generator(np.random.PCG64(11))
    T = max(lengths)
    e, h, h0 = _normal(rng, T, B, H), _normal(rng, T, B, H).tanh_(), _normal(rng, B, H)
    gates, c, c0 = _normal(rng, T, B, 4 * H).sigmoid_(), _normal(rng, T, B, H), _normal(rng, B, H)

    def passes(bwd, steps):
        head = lambda a: a[:steps].contiguous()
        if cell == "lstm":
            return bwd.backward_lstm_with_weights(head(e), head(gates), head(c), head(h), c0, h0)
        if cell == "gru":
            return bwd.backward_gru_with_weights(head(e), head(gates), head(h), h0)
        return bwd.backward_with_weights(head(e), head(h), h0)

    with binding.SparseRNN(H, B, name, *t_csr) as chosen:
        info = chosen.info()
        print("case", cell, H, B, "parts", info["parts"], "lanes", info["lanes_per_row"], flush=True)
        with binding.SparseRNN(H, B, name, *t_csr, lanes_per_row=info["lanes_per_row"]) as fixed:
            for steps in lengths:
                for k, (a, b) in enumerate(zip(passes(chosen, steps), passes(fixed, steps))):
                    assert torch.equal(a, b), (steps, k, (a - b).abs().max().item())
            assert chosen.check() == binding.SPRNN_OK and fixed.check() == binding.SPRNN_OK
