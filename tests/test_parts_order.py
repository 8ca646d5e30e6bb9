"""The order of a row's nonzeros is one for every way of sharing out the samples (CPU): which lane of the row holds which
nonzero in which slot may depend on the lanes per row only, because that is the order in which the products are added."""
import zlib

import numpy as np
import pytest

from paper_1804_10223_amd import binding, workloads as wl


def _slots(w, batch, **options):
    """{(row, lane of the row, slot): (column, value bits)} of the packed image, padding left out."""
    words, lane_row, lane_words, info = binding.pack_host(w.hidden, batch, w.cell, w.row_ptr, w.col_idx, w.val_bits, **options)
    share = batch // info["parts"] // (2 if info["activations"] == 2 else 1)
    stride = 4 * min(share, 4)
    plane = w.hidden * stride
    shift = 0 if plane <= 65536 else int(np.log2(stride))
    L, held = info["lanes_per_row"], {}
    for wg in range(words.shape[0]):
        for k in range(words.shape[1]):
            for tid in np.nonzero(words[wg, k] & 0x7FFF)[0]:
                word = int(words[wg, k, tid])
                held[int(lane_row[wg, tid]), int(tid) % L, k] = (((word >> 16) << shift) // stride, word & 0xFFFF)
    return held, info


@pytest.mark.parametrize("cell,H,batch,parts,L,dens,rows,opts", [
    ("relu", 300, 2, 2, 16, 0.2, "fixed", {}),
    ("tanh", 333, 4, 4, 64, 0.3, "poisson", {}),
    ("relu", 257, 8, 8, 8, 0.1, "poisson", {}),
    ("lstm", 130, 8, 4, 8, 0.2, "fixed", {}),
    ("gru", 97, 4, 2, 16, 0.3, "poisson", {}),
    ("relu", 5000, 4, 2, 8, 0.002, "fixed", {"compact": 2}),      # packed indices count columns in one geometry, bytes in the other
    ("relu", 320, 8, 2, 32, 0.2, "fixed", {"activations": "binary16"}),
])
def test_every_share_of_the_batch_has_the_order_of_the_whole(cell, H, batch, parts, L, dens, rows, opts):
    w = wl.make_workload("order", cell, H, batch, 1, dens, seed=H, row_nnz=rows)
    whole, info = _slots(w, batch, lanes_per_row=L, **opts)
    shared, shared_info = _slots(w, batch, lanes_per_row=L, parts=parts, **opts)
    assert info["parts"] == 1 and shared_info["parts"] == parts and info["batch"] == shared_info["batch"] == batch
    assert len(whole) == np.count_nonzero(w.val_bits & 0x7FFF) and whole == shared


@pytest.mark.parametrize("H,batch,parts,L,dens", [(4096, 4, 2, 8, 0.01), (6000, 8, 2, 8, 0.004), (2000, 8, 4, 8, 0.005)])
def test_parts_copy_h_whole_where_it_fits(H, batch, parts, L, dens):
    """Column compaction (here the choice for all samples in one part) orders a row's nonzeros by their columns' places in LDS."""
    w = wl.make_workload("sparse", "relu", H, batch, 1, dens, seed=H)
    options = dict(lanes_per_row=L)
    assert binding.pack_host(H, batch, "relu", w.row_ptr, w.col_idx, w.val_bits, **options)[3]["compact"] == 1
    assert binding.pack_host(H, batch, "relu", w.row_ptr, w.col_idx, w.val_bits, parts=parts, **options)[3]["compact"] == 0
    assert binding.pack_host(H, batch, "relu", w.row_ptr, w.col_idx, w.val_bits, parts=parts, compact=1, **options)[3]["compact"] == 1


def test_binary16_activations_keep_their_order():
    """A result with binary16 activations moves by 2^-11 of h where a sum taken in another order falls on the other side of a
    rounding boundary, so the order is fixed: which slot of which lane holds which nonzero is pinned here, for both batch sizes."""
    H = 320
    per_row = np.array([24 + (5 * r) % 17 for r in range(H)])
    row_ptr = np.concatenate([[0], np.cumsum(per_row)]).astype(np.int32)
    col = np.concatenate([np.sort((np.arange(n) * 53 + 7 * r) % H) for r, n in enumerate(per_row)]).astype(np.int32)
    val = (0x3000 + np.arange(col.size) % 0x0800).astype(np.uint16)
    w = wl.Workload("pinned", "relu", H, 8, 1, row_ptr, col, val, None, None)
    for batch, parts, want in ((8, 1, 2550844915), (4, 1, 3065920774), (8, 2, 2550844915)):
        held, info = _slots(w, batch, lanes_per_row=16, activations="binary16", compact=2, **({"parts": parts} if parts > 1 else {}))
        assert info["parts"] == parts and info["activations"] == 2 and len(held) == col.size
        order = np.array([key + value for key, value in sorted(held.items())], dtype=np.int64)
        assert zlib.crc32(order.tobytes()) == want, (batch, parts)
