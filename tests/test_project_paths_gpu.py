"""The input projection's kernels and tile widths at the edges of each, at input sizes that no 16-byte row holds and from
addresses that are aligned to one element only, against a binary64 product.

Bound per output (products exact, binary32 sums, x split into two binary16 halves exact to 2^-21, K = input size):
    |got - want| <= (K + 8) 2^-24 (sum_k |W[r][k] x[k]| + |bias[r]|) + 2^-26 sum_k |W[r][k]|.
"""
import numpy as np
import pytest
import torch

from paper_1804_10223_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,batch,T,K,offset", [
    # K shared out inside a workgroup (at most 256 tiles of 32 x 32)
    (1, 1, 1, 1, 0), (33, 1, 33, 15, 1), (32, 4, 8, 16, 0), (65, 1, 31, 17, 1), (200, 2, 50, 129, 0),
    (90, 1, 3, 1037, 1), (40, 8, 9, 96, 0), (2000, 1, 50, 200, 0),
    # tiles of 64 x 64 (too many of the above, about one per CU)
    (1111, 4, 100, 333, 0), (2304, 1, 400, 64, 1), (60, 8, 900, 70, 0), (1024, 1, 1024, 897, 0), (1024, 8, 136, 896, 0),
    # 64 x 128 and 64 x 192
    (1024, 8, 136, 897, 0), (1100, 1, 1100, 77, 1), (1100, 4, 275, 128, 0), (1100, 4, 525, 70, 0), (1100, 1, 2100, 193, 1),
])
def test_projection_paths(rows, batch, T, K, offset):
    print("case", rows, batch, T, K, offset, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rows + K)
    M = T * batch
    x = torch.randn(M * K + offset, device="cuda", generator=gen)[offset:].reshape(T, batch, K)
    w = torch.randn(rows * K + offset, device="cuda", generator=gen).half()[offset:].reshape(rows, K)
    bias = torch.randn(rows, device="cuda", generator=gen)
    row_ptr, col_idx = np.arange(rows + 1, dtype=np.int32), np.arange(rows, dtype=np.int32)
    out = torch.full((M * rows + 5,), 77.0, device="cuda")
    with binding.SparseRNN(rows, batch, "relu", row_ptr, col_idx, np.full(rows, 0x3800, np.uint16), poll_delay=-1) as rnn:
        rnn.project(x, w, bias, out[:M * rows].reshape(T, batch, rows))
        torch.cuda.synchronize()
    got = out.cpu().numpy().astype(np.float64)
    assert (got[M * rows:] == 77.0).all()
    x64, w64, b64 = x.reshape(M, K).double().cpu().numpy(), w.double().cpu().numpy(), bias.double().cpu().numpy()
    bound = (K + 8) * 2.0 ** -24 * (np.abs(x64) @ np.abs(w64).T + np.abs(b64)) + 2.0 ** -26 * np.abs(w64).sum(axis=1)
    assert np.all(np.abs(got[:M * rows].reshape(M, rows) - (x64 @ w64.T + b64)) <= bound)
