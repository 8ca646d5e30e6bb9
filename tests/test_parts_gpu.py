"""Samples shared out to several groups of workgroups (SPRNN_XCD_PARTS): the results must be, bit for bit, those of a handle
with the same lanes per row and all samples in one group, whatever the pass, the placement and the pauses.  (Handles of the
latter kind are compared with the CPU oracle by the other test files.)

Shapes: one workgroup per part, rows and chunks that divide nothing, one XCD per part, parts that fill the chip, a batch
whose whole and shared layouts differ in the width of a gather, binary16.
"""
import numpy as np
import pytest
import torch

from paper_1804_10223_amd import binding, workloads as wl

pytestmark = pytest.mark.gpu
GATES = {"lstm": 4, "gru": 3}


def _dev(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _passes(rnn, bwd, cell, s):
    """Every pass of the layer on the samples in `s`; a dict of [T][B].. or [B].. tensors, the samples of [B].. on axis 0."""
    out = {}
    if cell == "lstm":
        out["h"], out["c"] = rnn.forward_lstm(s["x"], s["h0"], s["c0"])
        out["ht"], out["ct"], out["gates"] = rnn.forward_lstm_train(s["x"], s["h0"], s["c0"])
        out["d"], out["dh0"], out["dc0"] = bwd.backward_lstm(s["e"], out["gates"], out["ct"], s["c0"])
    elif cell == "gru":
        out["h"] = rnn.forward_gru(s["x"], s["b_hn"], s["h0"])
        out["ht"], out["gates"] = rnn.forward_gru_train(s["x"], s["b_hn"], s["h0"])
        out["d"], out["v"], out["dh0"] = bwd.backward_gru(s["e"], out["gates"], out["ht"], s["h0"])
    else:
        out["h"] = rnn.forward(s["x"], s["h0"])
        if bwd is not None:
            out["noalloc"] = torch.empty_like(out["h"])
            rnn.forward_noalloc(s["x"], s["h0"], out["noalloc"])
            out["d"], out["dh0"] = bwd.backward(s["e"], out["h"])
    out["again"] = out["h"].clone() if "ht" not in out else out["ht"]
    return out


CASES = [
    # cell, hidden, batch, parts, steps, density, rows, options of both handles
    ("relu", 96, 4, 4, 9, 0.3, "fixed", {"lanes_per_row": 8}),                                                   # one workgroup a part: nothing is exchanged
    ("tanh", 333, 4, 2, 8, 0.2, "poisson", {"lanes_per_row": 8, "waves": 3}),
    ("identity", 701, 2, 2, 7, 0.15, "poisson", {"lanes_per_row": 16, "waves": 6, "xcd": "one"}),
    ("relu", 1152, 4, 4, 30, 0.1, "fixed", {"lanes_per_row": 16, "waves": 9, "xcd": "one"}),    # four XCDs, one part each
    ("relu", 1001, 8, 8, 12, 0.1, "poisson", {"lanes_per_row": 16, "waves": 8, "xcd": "one", "jitter": 5}),
    ("relu", 2304, 4, 2, 20, 0.3, "fixed", {"lanes_per_row": 32, "waves": 9}),                 # both halves of the chip
    ("tanh", 1000, 8, 2, 12, 0.1, "poisson", {"lanes_per_row": 16, "jitter": 3}),
    ("tanh", 2000, 8, 4, 6, 0.02, "fixed", {"lanes_per_row": 8, "waves": 8, "compact": 2}),
    ("lstm", 150, 8, 8, 9, 0.2, "poisson", {"lanes_per_row": 8, "waves": 5}),
    ("lstm", 1024, 8, 2, 10, 0.2, "fixed", {"lanes_per_row": 16, "waves": 8}),
    ("lstm", 1024, 8, 4, 10, 0.2, "fixed", {"lanes_per_row": 8, "waves": 8, "jitter": 7}),
    ("gru", 771, 4, 2, 11, 0.15, "poisson", {"lanes_per_row": 16, "waves": 7}),
    ("gru", 200, 2, 2, 9, 0.2, "fixed", {"lanes_per_row": 16, "waves": 8, "xcd": "one"}),
    ("relu", 2560, 8, 2, 10, 0.12, "fixed", {"lanes_per_row": 32, "waves": 10, "activations": "binary16"}),
]


@pytest.mark.parametrize("cell,H,B,P,T,dens,rows,opts", CASES)
def test_the_results_do_not_depend_on_how_the_samples_are_shared_out(cell, H, B, P, T, dens, rows, opts):
    w = wl.make_workload("parts", cell, H, B, T, dens, seed=H + B, row_nnz=rows, h0_std=0.5)
    R = w.rows
    rng = np.random.Generator(np.random.PCG64(7))
    s = {"x": _dev(w.x), "h0": _dev(w.h0), "e": _dev(rng.standard_normal((T, B, H)).astype(np.float32)),
         "c0": _dev(rng.standard_normal((B, H)).astype(np.float32)), "b_hn": _dev(getattr(w, "b_hn", None))}
    half = opts.get("activations") == "binary16"
    with_backward = not half
    t_csr = binding.transpose_csr(R, H, w.row_ptr, w.col_idx, w.val_bits)
    # (the transposed matrix of a gated cell has one row group per unit, and its passes are not confined to one XCD)
    bopts = opts if cell not in GATES else {k: v for k, v in opts.items() if k not in ("xcd", "lanes_per_row", "waves")}
    if cell in GATES:
        bopts = dict(bopts, lanes_per_row=32, waves=8)

    def handles(batch, extra):
        rnn = binding.SparseRNN(H, batch, cell, w.row_ptr, w.col_idx, w.val_bits, **dict(opts, **extra))
        bwd = binding.SparseRNN(H, batch, cell + "_backward" if cell in GATES else cell, *t_csr, **dict(bopts, **extra)) if with_backward else None
        return rnn, bwd

    print("case", cell, H, B, P, T, opts, flush=True)
    rnn, bwd = handles(B, {"parts": P})
    assert rnn.info()["parts"] == P and rnn.info()["batch"] == B
    got = _passes(rnn, bwd, cell, s)
    twice = _passes(rnn, bwd, cell, s)                                   # the ring goes on where the first calls left it
    assert rnn.check() == binding.SPRNN_OK and (bwd is None or bwd.check() == binding.SPRNN_OK)
    for k in got:
        assert torch.equal(got[k], twice[k]), k
    assert torch.equal(got["again"], got["h"])                           # the pass that keeps gate values: the same h
    if "noalloc" in got:
        assert torch.equal(got["noalloc"], got["h"])
    whole, whole_bwd = handles(B, {"grid": 0, "waves": 0, "xcd": 0})
    assert whole.info()["parts"] == 1
    want = _passes(whole, whole_bwd, cell, s)
    for k in want:
        assert torch.equal(got[k], want[k]), (k, (got[k] - want[k]).abs().max().item())
    if with_backward:
        # weight gradient, asked of either handle: the sum over the samples of all parts.  A chain of T B terms in any order,
        # factors split into parts that keep 24 bits: within (T B + 16) 2^-24 of the sum of magnitudes.
        factor = got["v"] if cell == "gru" else got["d"]
        before = torch.cat([s["h0"][None], got["h"][:-1]])
        r = torch.from_numpy(np.repeat(np.arange(R), np.diff(w.row_ptr))).cuda()
        c = torch.from_numpy(np.asarray(w.col_idx, dtype=np.int64)).cuda()
        dense = factor.double().reshape(T * B, R).T @ before.double().reshape(T * B, H)
        bound = factor.double().abs().reshape(T * B, R).T @ before.double().abs().reshape(T * B, H)
        allowed = (T * B + 16) * 2.0 ** -24 * bound[r, c] + 1e-30
        assert ((rnn.weight_gradient(factor, got["h"], s["h0"]).double() - dense[r, c]).abs() <= allowed).all()
        source = torch.from_numpy(binding.transpose_csr(R, H, w.row_ptr, w.col_idx, w.val_bits, with_source=True)[3].astype(np.int64)).cuda()
        if cell == "lstm":
            sums = bwd.backward_lstm_with_weights(s["e"], got["gates"], got["ct"], got["h"], s["c0"], s["h0"])
        elif cell == "gru":
            sums = bwd.backward_gru_with_weights(s["e"], got["gates"], got["h"], s["h0"])
        else:
            sums = bwd.backward_with_weights(s["e"], got["h"], s["h0"])
        assert torch.equal(sums[0], got["d"])
        assert ((sums[-1].double() - dense[r, c][source]).abs() <= allowed[source]).all()
        assert bwd.check() == binding.SPRNN_OK
    for hnd in (rnn, bwd, whole, whole_bwd):
        if hnd is not None:
            hnd.close()


NO_PLACEMENT = 1 << 30   # options.jitter: as if the dispatcher had put too few workgroups on every XCD


@pytest.mark.parametrize("cell,H,B,P,dens,opts", [
    ("relu", 1152, 4, 1, 0.1, {"lanes_per_row": 16, "waves": 9}),
    ("tanh", 1152, 4, 2, 0.1, {"lanes_per_row": 16, "waves": 9}),
    ("relu", 1152, 4, 4, 0.1, {"lanes_per_row": 16, "waves": 9}),
    ("relu", 1001, 8, 8, 0.1, {"lanes_per_row": 16, "waves": 8}),
    ("lstm", 256, 4, 4, 0.1, {"lanes_per_row": 8, "waves": 8}),
    ("gru", 200, 2, 2, 0.2, {"lanes_per_row": 16, "waves": 8}),
    ("relu", 1000, 8, 2, 0.1, {"lanes_per_row": 16, "waves": 8, "activations": "binary16"}),
])
def test_one_xcd_launches_with_too_few_workgroups_on_every_xcd(cell, H, B, P, dens, opts):
    """The workgroups then take their places by index and the exchange leaves the XCDs: the same results, with and without
    pauses (the general form and the one without options), also right behind a launch on one XCD with the same ring."""
    T = 12
    w = wl.make_workload("places", cell, H, B, T, dens, seed=H, h0_std=0.5)
    rng = np.random.Generator(np.random.PCG64(9))
    s = {"x": _dev(w.x), "h0": _dev(w.h0), "e": _dev(rng.standard_normal((T, B, H)).astype(np.float32)),
         "c0": _dev(rng.standard_normal((B, H)).astype(np.float32)), "b_hn": _dev(getattr(w, "b_hn", None))}
    csr = (w.row_ptr, w.col_idx, w.val_bits)
    vanilla = cell not in GATES and "activations" not in opts
    t_csr = binding.transpose_csr(H, H, *csr)[:3] if vanilla else None
    print("case", cell, H, B, P, opts, flush=True)

    def passes(jitter):
        extra = dict(opts, xcd="one", jitter=jitter, **({"parts": P} if P > 1 else {}))
        out = {}
        with binding.SparseRNN(H, B, cell, *csr, **extra) as rnn:
            info = rnn.info()
            assert info["one_xcd"] == 1 and info["parts"] == P and 2 <= info["grid"] <= 32
            bwd = binding.SparseRNN(H, B, cell, *t_csr, **extra) if vanilla else None
            for again in range(3):
                if cell == "lstm":
                    out["h", again], out["c", again] = rnn.forward_lstm(s["x"], s["h0"], s["c0"])
                elif cell == "gru":
                    out["h", again] = rnn.forward_gru(s["x"], s["b_hn"], s["h0"])
                else:
                    out["h", again] = rnn.forward(s["x"], s["h0"])
                if bwd:
                    out["d", again], out["dh0", again] = bwd.backward(s["e"], out["h", again])
                    out["noalloc", again] = torch.empty_like(out["h", again])
                    rnn.forward_noalloc(s["x"], s["h0"], out["noalloc", again])
            assert rnn.check() == binding.SPRNN_OK and (bwd is None or bwd.check() == binding.SPRNN_OK)
            if bwd:
                bwd.close()
        return out

    want = passes(0)
    for jitter in (NO_PLACEMENT, NO_PLACEMENT + 5):
        got = passes(jitter)
        for k in want:
            assert torch.equal(got[k], want[k]), (jitter, k)


SHORT_UNDIVIDED = 1 << 29   # options.jitter: calls of fewer than 20 steps run on the handle with all samples


@pytest.mark.parametrize("cell,H,B,P,dens,opts", [
    ("relu", 1152, 4, 4, 0.1, {"lanes_per_row": 16, "waves": 9, "xcd": "one"}),
    ("tanh", 1000, 8, 2, 0.1, {"lanes_per_row": 16}),
    ("lstm", 512, 8, 4, 0.2, {"lanes_per_row": 8, "waves": 8}),
    ("gru", 771, 4, 2, 0.15, {"lanes_per_row": 16, "waves": 7}),
    ("relu", 1000, 8, 2, 0.1, {"lanes_per_row": 16, "waves": 8, "activations": "binary16"}),
])
@pytest.mark.parametrize("pauses", [0, 5])
def test_calls_that_change_between_the_parts_and_the_undivided_handle(cell, H, B, P, dens, opts, pauses):
    """Calls on both sides of the change, in turn, every one on from where its own ring was left: the same bits."""
    T = 48
    w = wl.make_workload("turns", cell, H, B, T, dens, seed=H, h0_std=0.5)
    rng = np.random.Generator(np.random.PCG64(4))
    x, h0, e = _dev(w.x), _dev(w.h0), _dev(rng.standard_normal((T, B, H)).astype(np.float32))
    c0, b_hn = _dev(rng.standard_normal((B, H)).astype(np.float32)), _dev(getattr(w, "b_hn", None))
    csr = (w.row_ptr, w.col_idx, w.val_bits)
    vanilla = cell not in GATES and "activations" not in opts
    extra = dict(opts, parts=P, jitter=SHORT_UNDIVIDED + pauses)
    print("case", cell, H, B, P, opts, pauses, flush=True)

    def forward(rnn, steps):
        xs = x[:steps].contiguous()
        if cell == "lstm":
            return rnn.forward_lstm_train(xs, h0, c0)
        return rnn.forward_gru_train(xs, b_hn, h0) if cell == "gru" else (rnn.forward(xs, h0),)

    with binding.SparseRNN(H, B, cell, *csr, **extra) as rnn:
        want = forward(rnn, T)
        for steps in (1, 19, 20, 2, 21, 5, 40, 18, 3, T):
            for k, (a, b) in enumerate(zip(forward(rnn, steps), want)):
                assert torch.equal(a, b[:steps]), (steps, k)
            if vanilla:
                out = torch.empty_like(want[0][:steps])
                rnn.forward_noalloc(x[:steps].contiguous(), h0, out)
                assert torch.equal(out, want[0][:steps]), steps
        assert rnn.check() == binding.SPRNN_OK
    if vanilla:
        with binding.SparseRNN(H, B, cell, *binding.transpose_csr(H, H, *csr)[:3], **extra) as bwd:
            grads = bwd.backward(e, want[0])[0]
            for steps in (1, 19, 20, 2, 40, 18, T):   # the last steps of the long call: nothing flows in from beyond its end
                tail = lambda a: a[T - steps:].contiguous()
                assert torch.equal(bwd.backward(tail(e), tail(want[0]))[0], grads[T - steps:]), steps
            assert bwd.check() == binding.SPRNN_OK


@pytest.mark.parametrize("H,B,P,lanes,dens", [(2000, 8, 4, 8, 0.005), (4096, 4, 2, 8, 0.01)])
def test_sparse_parts_copy_h_whole_unless_told_otherwise(H, B, P, lanes, dens):
    """Layers whose workgroups would copy only some columns if all samples were in one part: with parts they copy h whole, so that
    the weight gradients are offered and the bits are those of a handle with these lanes that copies h whole."""
    T = 5
    w = wl.make_workload("sparse", "tanh", H, B, T, dens, seed=H, h0_std=0.5)
    rng = np.random.Generator(np.random.PCG64(5))
    x, h0, e = _dev(w.x), _dev(w.h0), _dev(rng.standard_normal((T, B, H)).astype(np.float32))
    csr = (w.row_ptr, w.col_idx, w.val_bits)
    t_csr = binding.transpose_csr(H, H, *csr)
    with binding.SparseRNN(H, B, "tanh", *csr, lanes_per_row=lanes) as auto:
        assert auto.info()["compact"] == 1
    results = []
    for extra in ({"parts": P}, {"compact": 2}):
        with binding.SparseRNN(H, B, "tanh", *csr, lanes_per_row=lanes, **extra) as rnn, \
             binding.SparseRNN(H, B, "tanh", *t_csr, lanes_per_row=lanes, **extra) as bwd:
            assert rnn.info()["compact"] == bwd.info()["compact"] == 0
            h = rnn.forward(x, h0)
            delta, dh0 = bwd.backward(e, h)
            results.append([h, delta, dh0, rnn.weight_gradient(delta, h, h0)] + list(bwd.backward_with_weights(e, h, h0)))
            assert rnn.check() == bwd.check() == binding.SPRNN_OK
    for k, (a, b) in enumerate(zip(*results)):
        assert torch.equal(a, b), (k, (a - b).abs().max().item())


def test_refusals():
    w = wl.make_workload("refuse", "relu", 64, 2, 1, 0.2, seed=1)
    for kw, code in (({"parts": 4}, binding.SPRNN_ERR_UNSUPPORTED), ({"parts": 2, "layout": 2}, binding.SPRNN_ERR_UNSUPPORTED),
                     ({"parts": 2, "sync": "barrier"}, binding.SPRNN_ERR_UNSUPPORTED), ({"parts": 2, "timeline": 1}, binding.SPRNN_ERR_UNSUPPORTED),
                     ({"parts": 3}, binding.SPRNN_ERR_INVALID), ({"xcd": 3}, binding.SPRNN_ERR_INVALID)):
        with pytest.raises(binding.SprnnError) as e:
            binding.SparseRNN(64, 2, "relu", w.row_ptr, w.col_idx, w.val_bits, **kw)
        assert e.value.code == code, kw
