"""The order in which an aggregation adds a row, bit for bit: eight chains (sixteen in passes of at most
64 bytes) by the position of the entry in the matrix, combined in a tree, and the pieces of a row that
crosses a span of entries added in order.  Its rounding error is about that of an eighth of the row
added one by one.  With the weights of the sum aggregator (all 1) every step is one fp32 addition, which
numpy rounds the same way."""
import numpy as np
import pytest
import torch

import graphgen as gg

pytestmark = pytest.mark.gpu


def span_entries(chains, entries, n_slices):
    batches = 256
    while batches * chains > 256 and -(-entries // (batches * chains)) * n_slices < 8192:
        batches //= 2
    return batches * chains


def row_sums(rowptr, col, h, chains, span):
    out = np.zeros((len(rowptr) - 1, h.shape[1]), np.float32)
    for r in range(len(out)):
        e, end = int(rowptr[r]), int(rowptr[r + 1])
        total = None
        while e < end:
            stop = min(end, (e // span + 1) * span)
            acc = np.zeros((chains, h.shape[1]), np.float32)
            for k in range(e, stop):
                acc[k % chains] += h[col[k]]
            while len(acc) > 1:
                acc = acc[0::2] + acc[1::2]
            total = acc[0] if total is None else total + acc[0]
            e = stop
        if total is not None:
            out[r] = total
    return out


@pytest.mark.parametrize("f,bf,chains,slices", [(16, False, 16, 1), (40, False, 8, 2), (24, True, 16, 1),
                                                (136, True, 8, 3)])
def test_whole_matrix_calls_add_rows_in_eight_chains_and_a_tree(f, bf, chains, slices):
    import paper_2501_01951_amd as mg

    mg.load_library()
    n = 2500
    lens = np.random.default_rng(f).choice([0, 1, 3, 8, 17, 32, 33, 64, 70], n)
    lens[7], lens[1200] = 2000, 300
    src = np.repeat(np.arange(n), lens)
    dst = (src * 7 + np.arange(len(src)) - np.repeat(np.cumsum(lens) - lens, lens)) % n
    g = mg.build_csr(torch.from_numpy(src.astype(np.int32)).cuda(), torch.from_numpy(dst.astype(np.int32)).cuda(),
                     n, 0)
    mg.normalize(g, mg.NORM_SUM)
    a = g.arrays()
    rowptr, col = a["rowptr"].cpu().numpy(), a["col"].cpu().numpy()
    dt = torch.bfloat16 if bf else torch.float32
    h = torch.from_numpy(gg.normal(3, f, n, f)).cuda().to(dt)
    z = torch.full((n, f), 7.0, device="cuda", dtype=dt)
    mg.aggregate(g, h, z)
    want = row_sums(rowptr, col, h.float().cpu().numpy(), chains, span_entries(chains, g.nnz, slices))
    assert torch.equal(z.cpu(), torch.from_numpy(want).to(dt))
    g.free()
