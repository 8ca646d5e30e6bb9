"""The persistent kernel's forms without run-time options give, bit for bit, what its general form gives.

A handle with pauses (options.jitter) runs the general form, one without the form for its number of copy rounds; with the same
lanes per row both add a row's products in the same order.  Shapes: each number of rounds (one piece of 16 bytes per lane and
round), two groups of eight, one workgroup; word counts at both ends of the instantiations and in wavefronts of unequal
length; sequences of every length modulo the unrolled loops.  The pauses are the general form's; the forms without options are
made to wait, or not to, by their back-off.
"""
import numpy as np
import pytest
import torch

from paper_1804_10223_amd import binding, workloads as wl

pytestmark = pytest.mark.gpu
GATES = {"lstm": 4, "gru": 3}


def _dev(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()


CASES = [
    # cell, hidden, batch, density, rows, options (with them: pieces of 16 bytes / lanes = copy rounds)
    ("relu", 96, 1, 0.3, "poisson", {"lanes_per_row": 2}),                               # one workgroup
    ("tanh", 190, 2, 0.06, "fixed", {"lanes_per_row": 2}),
    ("identity", 100, 4, 0.3, "poisson", {"lanes_per_row": 4, "grid": 1}),
    ("relu", 60, 8, 0.5, "fixed", {"lanes_per_row": 8}),
    ("lstm", 40, 1, 0.4, "poisson", {"lanes_per_row": 1}),
    ("lstm", 30, 8, 0.4, "fixed", {"lanes_per_row": 8}),
    ("gru", 48, 4, 0.3, "poisson", {"lanes_per_row": 4}),
    ("relu", 512, 4, 0.1, "poisson", {"lanes_per_row": 16, "waves": 8}),                  # one round; 2 to 5 words
    ("tanh", 333, 1, 0.35, "poisson", {"lanes_per_row": 8, "waves": 4}),                  # one; 10 to 20 words
    ("relu", 801, 4, 0.14, "fixed", {"lanes_per_row": 8, "waves": 8}),                    # two; 14 words
    ("identity", 1500, 2, 0.05, "poisson", {"lanes_per_row": 4, "waves": 8, "balance": 2}),   # two; words of very unequal rows
    ("relu", 1400, 4, 0.02, "fixed", {"lanes_per_row": 4, "waves": 8}),                   # three; 7 words
    ("relu", 2000, 4, 0.2, "fixed", {"lanes_per_row": 16, "waves": 8}),                   # four; 25 words
    ("tanh", 1900, 4, 0.3, "fixed", {"lanes_per_row": 16, "waves": 4}),                   # eight; 36 words
    ("relu", 3000, 8, 0.01, "poisson", {"lanes_per_row": 8, "waves": 8, "compact": 2}),    # twelve: two groups
    ("relu", 700, 8, 0.1, "fixed", {"lanes_per_row": 8, "waves": 8}),
    ("lstm", 300, 4, 0.2, "poisson", {"lanes_per_row": 8, "waves": 6}),
    ("lstm", 512, 8, 0.1, "fixed", {"lanes_per_row": 8, "waves": 4}),
    ("gru", 420, 2, 0.25, "poisson", {"lanes_per_row": 8, "waves": 7}),
    ("gru", 1000, 8, 0.1, "fixed", {"lanes_per_row": 8, "waves": 8}),
    ("relu", 1000, 4, 0.1, "poisson", {"lanes_per_row": 16, "waves": 8, "activations": "binary16"}),
    ("tanh", 2560, 8, 0.05, "fixed", {"lanes_per_row": 16, "waves": 8, "activations": "binary16"}),
]


@pytest.mark.parametrize("cell,H,B,dens,rows,opts", CASES)
def test_forms_without_options_have_the_bits_of_the_general_form(cell, H, B, dens, rows, opts):
    T = 9
    w = wl.make_workload("forms", cell, H, B, T, dens, seed=H, row_nnz=rows, h0_std=0.5)
    rng = np.random.Generator(np.random.PCG64(3))
    x, h0, e = _dev(w.x), _dev(w.h0), _dev(rng.standard_normal((T, B, H)).astype(np.float32))
    c0, b_hn = _dev(rng.standard_normal((B, H)).astype(np.float32)), _dev(getattr(w, "b_hn", None))
    half = opts.get("activations") == "binary16"
    t_csr = binding.transpose_csr(w.rows, H, w.row_ptr, w.col_idx, w.val_bits)
    bopts = {k: v for k, v in opts.items() if cell not in GATES or k == "compact"}
    if cell in GATES:
        bopts.update(lanes_per_row=16, waves=8)
    print("case", cell, H, B, opts, flush=True)
    results = []
    for jitter in (0, 5):
        out = []
        with binding.SparseRNN(H, B, cell, w.row_ptr, w.col_idx, w.val_bits, jitter=jitter, **opts) as rnn:
            for steps in (1, 2, 3, 4, 5, 6, 7, 8, T):
                if cell == "lstm":
                    out += list(rnn.forward_lstm(x[:steps].contiguous(), h0, c0))
                elif cell == "gru":
                    out.append(rnn.forward_gru(x[:steps].contiguous(), b_hn, h0))
                else:
                    out.append(rnn.forward(x[:steps].contiguous(), h0))
            if cell == "lstm":
                h, c, gates = rnn.forward_lstm_train(x, h0, c0)
                out += [h, c, gates]
            elif cell == "gru":
                h, gates = rnn.forward_gru_train(x, b_hn, h0)
                out += [h, gates]
            else:
                h = out[-1]
            assert rnn.check() == binding.SPRNN_OK
        if not half:
            with binding.SparseRNN(H, B, cell + "_backward" if cell in GATES else cell, *t_csr, jitter=jitter, **bopts) as bwd:
                for steps in (1, 2, 4, T):
                    head = lambda a: a[:steps].contiguous()
                    for want_dh0 in (True, False):
                        if cell == "lstm":
                            got = bwd.backward_lstm(head(e), head(gates), head(c), c0, want_dh0=want_dh0)
                        elif cell == "gru":
                            got = bwd.backward_gru(head(e), head(gates), head(h), h0, want_dh0=want_dh0)
                        else:
                            got = bwd.backward(head(e), head(h), want_dh0=want_dh0)
                        out += [g for g in got if g is not None]
                assert bwd.check() == binding.SPRNN_OK
        results.append(out)
    assert len(results[0]) == len(results[1])
    for k, (a, b) in enumerate(zip(*results)):
        assert torch.equal(a, b), (k, (a - b).abs().max().item())


@pytest.mark.parametrize("cell,H,B,dens,rows,opts", [c for c in CASES if c[1] > 200])
def test_forms_without_options_that_poll_at_once_or_late(cell, H, B, dens, rows, opts):
    """No back-off: the first polls of a step come before the data, every wavefront loads again and again.  A back-off of several
    steps' time: the data is there at the first poll."""
    T = 40
    w = wl.make_workload("polls", cell, H, B, T, dens, seed=H, row_nnz=rows, h0_std=0.5)
    rng = np.random.Generator(np.random.PCG64(3))
    x, h0, e = _dev(w.x), _dev(w.h0), _dev(rng.standard_normal((T, B, H)).astype(np.float32))
    c0, b_hn = _dev(rng.standard_normal((B, H)).astype(np.float32)), _dev(getattr(w, "b_hn", None))
    half, gated = opts.get("activations") == "binary16", cell in GATES
    t_csr = None if half else binding.transpose_csr(w.rows, H, w.row_ptr, w.col_idx, w.val_bits)
    bopts = dict(lanes_per_row=16, waves=8) if gated else opts
    print("case", cell, H, B, opts, flush=True)
    results = []
    for kw in ({"poll_delay": -1}, {"poll_delay": 100}, {"jitter": 2}):
        with binding.SparseRNN(H, B, cell, w.row_ptr, w.col_idx, w.val_bits, **opts, **kw) as rnn:
            if cell == "lstm":
                out = list(rnn.forward_lstm_train(x, h0, c0))
            elif cell == "gru":
                out = list(rnn.forward_gru_train(x, b_hn, h0))
            else:
                out = [rnn.forward(x, h0)]
            assert rnn.check() == binding.SPRNN_OK
        if not half:
            with binding.SparseRNN(H, B, cell + "_backward" if gated else cell, *t_csr, **bopts, **kw) as bwd:
                if cell == "lstm":
                    out += bwd.backward_lstm(e, out[2], out[1], c0)
                elif cell == "gru":
                    out += bwd.backward_gru(e, out[1], out[0], h0)
                else:
                    out += bwd.backward(e, out[0])
                assert bwd.check() == binding.SPRNN_OK
        results.append(out)
    for other in results[1:]:
        for k, (a, b) in enumerate(zip(results[0], other)):
            assert torch.equal(a, b), (k, (a - b).abs().max().item())


def test_weights_beyond_a_wavefronts_own_do_not_read_h():
    """A row's sum sees no element of h that the row does not name: infinities elsewhere stay elsewhere, whatever the words per
    lane are rounded up to.  (One nonzero per row and lane: nothing is padded but what the kernel itself adds.)"""
    H = 256
    row_ptr = np.arange(H + 1, dtype=np.int32)
    col = np.arange(H, dtype=np.int32)
    one = np.full(H, 0x3C00, np.uint16)
    h0 = torch.ones((1, H), device="cuda")
    h0[0, :2] = float("inf")
    x = torch.zeros((3, 1, H), device="cuda")
    for opts in ({}, {"waves": 1}):                    # one workgroup; four
        with binding.SparseRNN(H, 1, "identity", row_ptr, col, one, lanes_per_row=1, **opts) as rnn:
            h = rnn.forward(x, h0)
            assert rnn.check() == binding.SPRNN_OK
        assert torch.isinf(h[:, 0, :2]).all() and (h[:, 0, 2:] == 1).all(), opts
