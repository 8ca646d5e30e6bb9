"""The weight gradient at the edges of its tiles (64 or 128 rows and columns, slabs of 32 vectors), against a binary64
product sampled at the nonzeros.

Bound per entry: the kernel's products are exact to 2^-26 of |a b| and its sums binary32, so with n = T * B terms
    |got - want| <= (n + 8) 2^-24 sum_m |a[m][row] b[m][col]|.
"""
import ctypes

import numpy as np
import pytest
import torch

from paper_1804_10223_amd import binding, workloads as wl

pytestmark = pytest.mark.gpu


def _dev(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("cell,H,B,T,dens,rownnz,with_h0", [
    ("identity", 1, 1, 1, 1.0, "fixed", True),            # one row, one column, one vector
    ("relu", 63, 1, 31, 0.3, "poisson", True),            # just short of a tile and of a slab
    ("relu", 64, 4, 8, 0.3, "fixed", True),               # exactly one tile, exactly one slab
    ("tanh", 65, 1, 33, 0.3, "poisson", False),           # one beyond both
    ("relu", 129, 8, 13, 1.0, "fixed", True),             # dense, three tiles of 64 with one row left
    ("tanh", 700, 2, 49, 0.05, "poisson", True),          # no multiple of anything, three slabs and two vectors
    ("lstm", 200, 8, 9, 0.2, "fixed", True),              # more rows than columns
    ("gru", 171, 2, 17, 0.15, "poisson", False),
    ("relu", 2304, 4, 9, 0.3, "fixed", True),             # tiles of 128 x 192
    ("relu", 1800, 1, 70, 0.02, "poisson", True),         # tiles of 128 x 128 with empty rows in them
])
def test_weight_gradient_at_tile_edges(cell, H, B, T, dens, rownnz, with_h0):
    w = wl.make_workload("wg-edge", cell, H, B, T, dens, seed=H + T, row_nnz=rownnz)
    rng = np.random.default_rng(H * 31 + T)
    R = w.rows
    delta = (rng.standard_normal((T, B, R)) * 10.0 ** rng.uniform(-6, 2, size=(1, 1, R))).astype(np.float32)   # rows of very different size
    h = rng.standard_normal((T, B, H)).astype(np.float32)
    h0 = rng.standard_normal((B, H)).astype(np.float32) if with_h0 else None
    print("case", cell, H, "B", B, "T", T, dens, flush=True)
    with binding.SparseRNN(H, B, cell, w.row_ptr, w.col_idx, w.val_bits, poll_delay=-1) as rnn:
        dU = torch.full((w.nnz + 3,), 77.0, device="cuda")
        got = rnn.weight_gradient(_dev(delta), _dev(h), _dev(h0), dU).cpu().numpy()
        assert rnn.check() == binding.SPRNN_OK
        assert (dU[w.nnz:] == 77.0).all()                 # nothing beyond the last nonzero is written
    before = np.concatenate([np.zeros((1, B, H), np.float32) if h0 is None else h0[None], h[:-1]]).reshape(T * B, H).astype(np.float64)
    d64 = delta.reshape(T * B, R).astype(np.float64)
    rows = np.repeat(np.arange(R), np.diff(w.row_ptr))
    want = (d64.T @ before)[rows, w.col_idx]
    size = (np.abs(d64).T @ np.abs(before))[rows, w.col_idx]
    assert np.all(np.abs(got - want) <= (T * B + 8) * 2.0 ** -24 * size)


def _chain(delta, before, rows, cols, order):
    """The sums as one binary32 multiply-add per vector gives them, vectors in `order`.  (Rounded through binary64: an entry in
    some 2^29 differs from a true multiply-add.)"""
    out = np.zeros(len(rows), np.float32)
    for m in order:
        out = (out + delta[m][rows].astype(np.float64) * before[m][cols]).astype(np.float32)
    return out


def _wide_csr(rows, cols, per_row, rng):
    """A pattern for wide matrices, drawn without looking at every element: at most one nonzero in each of `per_row` equal parts
    of a row, a quarter of them left out."""
    col = np.arange(per_row) * (cols // per_row) + rng.integers(0, cols // per_row, (rows, per_row))
    keep = rng.random((rows, per_row)) < 0.75
    row_ptr = np.concatenate([[0], np.cumsum(keep.sum(axis=1))]).astype(np.int32)
    return row_ptr, col[keep].astype(np.int32), np.full(row_ptr[-1], 0x2C00, np.uint16)


@pytest.mark.parametrize("cell,H,B,T,per_row,with_h0,lanes", [
    ("relu", 11520, 1, 21, 24, True, True),                # wide and sparse: one accumulator per lane and nonzero
    ("tanh", 8190, 4, 5, 8, False, True),                  # ... four batches of copy rounds, a column a piece
    ("relu", 20001, 2, 5, 12, True, True),                 # ... an odd size: the last piece of h is ragged
    ("lstm", 4095, 1, 9, 8, True, True),                   # ... ragged, four rows a unit
    ("gru", 4096, 2, 7, 8, False, True),
    ("relu", 4096, 8, 2, 16, True, True),                  # ... both planes of batch 8
    ("identity", 40000, 1, 9, 8, True, True),              # ... about the widest layer whose h the LDS holds
    ("relu", 1152, 4, 1, 115, True, True),                 # one step: too little for the product's tiles
    ("relu", 1152, 4, 16, 115, True, False),
    ("lstm", 1024, 8, 6, 50, True, False),
])
def test_weight_gradient_takes_the_way_the_shape_asks_for(cell, H, B, T, per_row, with_h0, lanes):
    """Right either way; and which way it took shows in the bits: the lanes add one vector after the other."""
    rng = np.random.default_rng(H + B)
    R = H * binding.GATES.get(cell, 1)
    row_ptr, col, val = _wide_csr(R, H, per_row, rng)
    nnz = len(col)
    delta, h = rng.standard_normal((T, B, R)).astype(np.float32), rng.standard_normal((T, B, H)).astype(np.float32)
    h0 = rng.standard_normal((B, H)).astype(np.float32) if with_h0 else None
    print("case", cell, H, "B", B, "T", T, per_row, flush=True)
    with binding.SparseRNN(H, B, cell, row_ptr, col, val, poll_delay=-1, compact=2) as rnn:
        dU = torch.full((nnz + 3,), 77.0, device="cuda")
        got = rnn.weight_gradient(_dev(delta), _dev(h), _dev(h0), dU).cpu().numpy()
        assert rnn.check() == binding.SPRNN_OK
        assert (dU[nnz:] == 77.0).all()
    before = np.concatenate([np.zeros((1, B, H), np.float32) if h0 is None else h0[None], h[:-1]]).reshape(T * B, H)
    delta = delta.reshape(T * B, R)
    rows = np.repeat(np.arange(R), np.diff(row_ptr))
    terms = delta[:, rows].astype(np.float64) * before[:, col]
    assert np.all(np.abs(got - terms.sum(axis=0)) <= (T * B + 8) * 2.0 ** -24 * np.abs(terms).sum(axis=0))
    same = np.mean(got == _chain(delta, before, rows, col, range(T * B)))
    assert same > 0.999 if lanes else same < 0.9


@pytest.mark.parametrize("cell,H,B,T,dens,with_h0", [
    # long enough for the product behind the recurrence to be the chosen way ...
    ("relu", 130, 8, 80, 0.3, True), ("tanh", 65, 4, 150, 0.5, False), ("lstm", 100, 8, 70, 0.3, True),
    ("lstm", 257, 2, 90, 0.2, False), ("gru", 129, 4, 90, 0.25, True),
    # ... and too short for it: summed inside the recurrence
    ("relu", 130, 8, 3, 0.3, True), ("lstm", 100, 8, 2, 0.3, True), ("gru", 129, 4, 2, 0.25, False),
])
def test_weight_gradient_asked_of_the_backward_call(cell, H, B, T, dens, with_h0):
    """dL/dU of the call's own delta, within the bound above; the product leaves the plain backward call's outputs as they are."""
    w = wl.make_workload("wg-asked", cell, H, B, T, dens, seed=H + T, row_nnz="poisson")
    rng = np.random.default_rng(H + B)
    normal = lambda *shape: _dev(rng.standard_normal(shape).astype(np.float32))
    h0 = normal(B, H) if with_h0 else None
    t_row_ptr, t_col, t_val, source = binding.transpose_csr(w.rows, H, w.row_ptr, w.col_idx, w.val_bits, with_source=True)
    gated = cell in ("lstm", "gru")
    dh, h = normal(T, B, H), normal(T, B, H).tanh_()
    print("case", cell, H, "B", B, "T", T, dens, flush=True)
    with binding.SparseRNN(H, B, cell + "_backward" if gated else cell, t_row_ptr, t_col, t_val) as bwd:
        if gated:
            saved = normal(T, B, 4 * H).sigmoid_()
            c = normal(T, B, H)
        if cell == "lstm":
            plain = bwd.backward_lstm(dh, saved, c)
            asked = bwd.backward_lstm_with_weights(dh, saved, c, h, None, h0)
        elif cell == "gru":
            plain = bwd.backward_gru(dh, saved, h, h0)
            asked = bwd.backward_gru_with_weights(dh, saved, h, h0)
        else:
            plain = bwd.backward(dh, h)
            asked = bwd.backward_with_weights(dh, h, h0)
        torch.cuda.synchronize()
        assert bwd.check() == binding.SPRNN_OK
    if T >= 70:
        for a, b in zip(plain, asked):
            assert torch.equal(a, b)
    delta = asked[1 if cell == "gru" else 0].reshape(T * B, w.rows).double().cpu().numpy()
    before = torch.cat([torch.zeros(1, B, H) if h0 is None else h0[None].cpu(), h[:-1].cpu()]).reshape(T * B, H).double().numpy()
    rows, cols = np.repeat(np.arange(w.rows), np.diff(w.row_ptr)), w.col_idx
    want, size = (delta.T @ before)[rows, cols], (np.abs(delta).T @ np.abs(before))[rows, cols]
    got = asked[-1].cpu().numpy()
    assert np.all(np.abs(got - want[source]) <= (T * B + 8) * 2.0 ** -24 * size[source])
    back = [t * B + b for t in range(T - 1, -1, -1) for b in range(B)]
    inside = np.mean(got == _chain(delta.astype(np.float32), before.astype(np.float32), rows, cols, back)[source])
    assert inside < 0.9 if T >= 70 else inside > 0.999


@pytest.mark.parametrize("H,B,T", [(70, 4, 9), (300, 8, 12), (1152, 1, 40), (1800, 2, 17), (2304, 4, 9)])   # each shape of tile
def test_weight_gradient_over_the_whole_range_of_binary32(H, B, T):
    """Rows and columns of every size binary32 has, and some with an infinity, a NaN or a number next to the largest.

    Bound per finite entry: the one above, and what numbers below the normal range lose, 2^-149 a term.  Entries whose terms
    hold an infinity or a NaN are what binary64 makes of them.  Left out: entries whose finite terms leave binary32's range."""
    w = wl.make_workload("wg-range", "relu", H, B, T, 0.1, seed=H, row_nnz="poisson")
    rng = np.random.default_rng(H)
    delta, h = rng.standard_normal((T, B, H)).astype(np.float32), rng.standard_normal((T, B, H)).astype(np.float32)
    size = np.zeros(H)
    size[1::3] = rng.uniform(-45, -28, size=size[1::3].shape)        # down to the smallest number there is
    size[2::3] = rng.uniform(0, 30, size=size[2::3].shape)
    delta *= np.float64(10.0) ** size
    h[:, :, 5::7] *= np.float32(1e-36)
    h[:, :, 6::7] *= np.float32(1e5)
    h[h < -1.0] = 0.0                                                # exact zeros, as after a ReLU
    top = np.finfo(np.float32).max
    delta[2, 0, 4::50], delta[3, 0, 10::50], delta[4, 0, 16::50], delta[5, 0, 22::50] = np.inf, -np.inf, top, np.nan
    h[1, 0, 3::60], h[6, 0, 9::60] = np.inf, -top                    # (delta_t pairs with h_{t-1}: the first meets delta[2])
    print("case", H, B, T, flush=True)
    with binding.SparseRNN(H, B, "relu", w.row_ptr, w.col_idx, w.val_bits, poll_delay=-1) as rnn:
        got = rnn.weight_gradient(_dev(delta), _dev(h)).cpu().numpy().astype(np.float64)
    before = np.concatenate([np.zeros((1, B, H), np.float32), h[:-1]]).reshape(T * B, H)
    rows = np.repeat(np.arange(H), np.diff(w.row_ptr))
    with np.errstate(invalid="ignore"):
        terms = delta.reshape(T * B, H)[:, rows].astype(np.float64) * before[:, w.col_idx].astype(np.float64)
        want = terms.sum(axis=0)
    magnitude = np.abs(np.where(np.isfinite(terms), terms, 0.0)).sum(axis=0)
    in_range = magnitude < top / 2                                    # (beyond that binary32 sums may overflow)
    special, fine = in_range & ~np.isfinite(want), in_range & np.isfinite(want)
    assert np.isnan(want[special]).any() and np.isinf(want[special]).any() and fine.sum() > len(rows) // 2
    np.testing.assert_array_equal(got[special], want[special])
    assert np.all(np.abs(got[fine] - want[fine]) <= (T * B + 8) * (2.0 ** -24 * magnitude[fine] + 2.0 ** -149))


def test_an_error_the_caller_left_behind_is_not_taken_for_the_librarys():
    H, B, T = 300, 4, 40
    w = wl.make_workload("wg-error", "relu", H, B, T, 0.2, seed=2)
    hip = ctypes.CDLL(sorted(binding.hip_runtimes_mapped())[0])
    t_csr = binding.transpose_csr(H, H, w.row_ptr, w.col_idx, w.val_bits)
    x, out = torch.randn((T, B, H), device="cuda"), torch.empty((T, B, H), device="cuda")
    w_in, dU, dh0 = torch.randn((H, H), device="cuda").half(), torch.empty(w.nnz, device="cuda"), torch.empty((B, H), device="cuda")
    long_x, long_out = torch.randn((700, B, H), device="cuda"), torch.empty((700, B, H), device="cuda")
    torch.cuda.synchronize()

    def leave_one():
        assert hip.hipSetDevice(9999) != 0

    try:
        leave_one()
        with binding.SparseRNN(H, B, "relu", *t_csr) as rnn:
            for call in (lambda: rnn.weight_gradient(x, x, None, dU), lambda: rnn.backward_with_weights(x, x, None, out, dh0=dh0, dU=dU),
                         lambda: rnn.project(x, w_in, None, out), lambda: rnn.project(long_x, w_in, None, long_out)):
                leave_one()
                call()
    finally:
        hip.hipGetLastError()


def test_a_layer_whose_calls_never_take_the_product_keeps_no_table_for_it():
    H = 40000                                  # the table would be 34 MB, the packed weights 1.3
    row_ptr, col, val = _wide_csr(H, H, 8, np.random.default_rng(1))
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    with binding.SparseRNN(H, 1, "relu", row_ptr, col, val, poll_delay=-1, compact=2) as rnn:
        used = free - torch.cuda.mem_get_info()[0]
        assert rnn.check() == binding.SPRNN_OK
    print("bytes of the handle", used, flush=True)
    assert used < 24 << 20


# Calls short or wide enough for the weight gradient to be summed inside the backward recurrence (the others of this file and of
# the backward tests that are longer take the product): every kernel of that kind, with pauses in the hand-off.
@pytest.mark.parametrize("cell,H,B,T,dens,opts", [
    ("relu", 96, 4, 6, 0.3, {}),
    ("tanh", 257, 1, 7, 0.2, {}),
    ("identity", 130, 8, 5, 0.1, {}),
    ("tanh", 64, 4, 4, 0.4, {"grid": 1}),
    ("relu", 640, 1, 12, 0.5, {"lanes_per_row": 16, "jitter": 5}),        # 24 slots per lane in 512 threads
    ("relu", 640, 4, 3, 0.5, {"lanes_per_row": 8, "jitter": 5}),          # 48 slots per lane in 256 threads
    ("tanh", 2048, 4, 40, 0.02, {"lanes_per_row": 16, "jitter": 5}),      # wide and sparse: inside at any length
    ("tanh", 2048, 4, 40, 0.02, {"lanes_per_row": 16, "jitter": 11, "sync": "barrier"}),
    ("relu", 4096, 4, 24, 0.08, {}),
    ("relu", 2304, 4, 8, 0.3, {"jitter": 5}),
    ("relu", 1500, 8, 8, 0.05, {"lanes_per_row": 16, "jitter": 11}),
    ("tanh", 1152, 4, 8, 0.1, {"layout": "lane_pool", "jitter": 5}),
    ("relu", 333, 2, 6, 0.15, {"layout": "lane_pool"}),
    ("lstm", 1024, 4, 20, 0.05, {"lanes_per_row": 32, "jitter": 5}),
    ("lstm", 1024, 8, 4, 0.2, {"jitter": 11}),
    ("lstm", 2000, 1, 24, 0.05, {}),
    ("lstm", 300, 2, 6, 0.5, {"lanes_per_row": 16, "jitter": 5}),         # 32 slots
    ("gru", 1200, 2, 30, 0.1, {"lanes_per_row": 32, "jitter": 11}),
    ("gru", 1024, 8, 4, 0.2, {"jitter": 5}),
])
def test_weight_gradient_summed_inside_the_recurrence(cell, H, B, T, dens, opts):
    """dL/dU bit for bit as multiply-adds from the last timestep to the first give it from the call's own delta, and delta bit
    for bit that of the plain call without pauses."""
    rng = np.random.default_rng(H + T)
    R = H * binding.GATES.get(cell, 1)
    per_row = int(round(dens * H))
    row_ptr, col, val = _wide_csr(R, H, per_row, rng)
    row_ptr_t, col_t, val_t, source = binding.transpose_csr(R, H, row_ptr, col, val, with_source=True)
    normal = lambda *shape: _dev(rng.standard_normal(shape).astype(np.float32))
    dh, h, h0 = normal(T, B, H), normal(T, B, H).tanh_(), normal(B, H)
    gates, c, c0 = (normal(T, B, 4 * H).sigmoid_(), normal(T, B, H), normal(B, H)) if cell in binding.GATES else (None, None, None)
    outs = {}
    for name, options in (("plain", {k: v for k, v in opts.items() if k != "jitter"}), ("asked", opts)):
        print("case", cell, H, "B", B, "T", T, dens, name, options, flush=True)
        with binding.SparseRNN(H, B, cell + "_backward" if cell in binding.GATES else cell, row_ptr_t, col_t, val_t, poll_delay=6, compact=2, **options) as bwd:
            if name == "plain":
                out = (bwd.backward_lstm(dh, gates, c, c0) if cell == "lstm" else
                       bwd.backward_gru(dh, gates, h, h0) if cell == "gru" else bwd.backward(dh, h))
            else:
                out = (bwd.backward_lstm_with_weights(dh, gates, c, h, c0, h0) if cell == "lstm" else
                       bwd.backward_gru_with_weights(dh, gates, h, h0) if cell == "gru" else bwd.backward_with_weights(dh, h, h0))
            assert bwd.check() == binding.SPRNN_OK
            outs[name] = [o.cpu().numpy() for o in out]
    for a, b in zip(outs["plain"], outs["asked"]):
        assert np.array_equal(a, b)
    delta = outs["asked"][1 if cell == "gru" else 0].reshape(T * B, R)
    before = np.concatenate([h0[None].cpu(), h[:-1].cpu()]).reshape(T * B, H)
    rows = np.repeat(np.arange(R), np.diff(row_ptr))
    back = [t * B + b for t in range(T - 1, -1, -1) for b in range(B)]
    same = outs["asked"][-1] == _chain(delta, before, rows, col, back)[source]
    assert same.mean() > 0.999, same.mean()


@pytest.mark.parametrize("cell,what", [("tanh", "delta over h"), ("tanh", "dh0 over h0"), ("lstm", "dh0 over h0"), ("gru", "dh0 over h0"),
                                       ("gru", "dh0 over a gate")])
def test_backward_with_weights_where_an_output_takes_the_place_of_a_state(cell, what):
    """The sums read h and h_0 before the recurrence writes there, also in calls long enough for the product behind it."""
    H, B, T = 257, 4, 90
    rng = np.random.default_rng(5)
    R = H * binding.GATES.get(cell, 1)
    row_ptr, col, val = _wide_csr(R, H, 60, rng)
    csr_t = binding.transpose_csr(R, H, row_ptr, col, val)
    normal = lambda *shape: _dev(rng.standard_normal(shape).astype(np.float32))
    dh, h, h0 = normal(T, B, H), normal(T, B, H).tanh_(), normal(B, H)
    gates, c, c0 = (normal(T, B, 4 * H).sigmoid_(), normal(T, B, H), normal(B, H)) if cell in binding.GATES else (None, None, None)
    print("case", cell, what, flush=True)
    with binding.SparseRNN(H, B, cell + "_backward" if cell in binding.GATES else cell, *csr_t) as bwd:
        def call(h, h0, **outputs):
            if cell == "lstm":
                return bwd.backward_lstm_with_weights(dh, gates, c, h, c0, h0, **outputs)
            if cell == "gru":
                return bwd.backward_gru_with_weights(dh, gates, h, h0, **outputs)
            return bwd.backward_with_weights(dh, h, h0, **outputs)
        apart = call(h, h0)
        in_h, in_h0 = h.clone(), h0.clone()
        if what == "dh0 over a gate":           # (gates of the first timestep, read when dh0 is not yet written)
            d, v, dh0, dU = call(h, h0, dh0=gates[0, :1].view(4, H)[:B], want_recurrent=False)
            placed = d, apart[1], dh0.clone(), dU
        else:
            placed = call(in_h, in_h0, **({"d_bprime": in_h} if what == "delta over h" else {"dh0": in_h0}))
        assert bwd.check() == binding.SPRNN_OK
    for a, b in zip(apart[:-1], placed[:-1]):
        assert torch.equal(a, b)
    factor = apart[1 if cell == "gru" else 0].reshape(T * B, R).double().abs()
    before = torch.cat([h0[None], h[:-1]]).reshape(T * B, H).double().abs()
    rows = np.repeat(np.arange(R), np.diff(row_ptr))
    bound = 2 * (T * B + 8) * 2.0 ** -24 * (factor.T @ before).cpu().numpy()[rows, col]   # each of the two within half of it
    source = binding.transpose_csr(R, H, row_ptr, col, val, with_source=True)[3]
    assert np.all(np.abs((apart[-1] - placed[-1]).cpu().numpy()) <= bound[source])


def test_weight_gradient_has_the_same_bits_on_handles_of_different_mapping():
    H, B, T = 8192, 4, 110                     # where both ways take about the same time
    row_ptr, col, val = _wide_csr(H, H, 8, np.random.default_rng(3))
    delta, h = torch.randn((T, B, H), device="cuda"), torch.randn((T, B, H), device="cuda")
    outs = []
    for waves in (8, 12):
        with binding.SparseRNN(H, B, "relu", row_ptr, col, val, poll_delay=-1, compact=2, waves=waves, lanes_per_row=4) as rnn:
            print("case", waves, rnn.info()["block"], flush=True)
            outs.append(rnn.weight_gradient(delta, h))
            assert rnn.check() == binding.SPRNN_OK
    assert torch.equal(*outs)


@pytest.mark.parametrize("H,B,T,per_row", [(300, 4, 40, 60), (8192, 1, 12, 16)])   # the product, the sums of the lanes
def test_weight_gradient_captured_in_a_graph(H, B, T, per_row):
    row_ptr, col, val = _wide_csr(H, H, per_row, np.random.default_rng(4))
    delta, h, dU = torch.randn((T, B, H), device="cuda"), torch.randn((T, B, H), device="cuda"), torch.empty(len(col), device="cuda")
    with binding.SparseRNN(H, B, "relu", row_ptr, col, val, poll_delay=-1, compact=2) as rnn:
        rnn.weight_gradient(delta, h, None, dU)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            rnn.weight_gradient(delta, h, None, dU)
        for i in range(4):
            delta.normal_(), h.normal_(), dU.fill_(float(i))
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(dU, rnn.weight_gradient(delta, h))
