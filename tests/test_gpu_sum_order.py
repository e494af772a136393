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


@pytest.mark.parametrize("ends", [1, 7, 8, 9, 16, 17, 255, 256])
@pytest.mark.parametrize("bf", [False, True])
def test_rows_that_wait_to_be_written(ends, bf):
    """Finished rows wait until every sub-group has one: spans in which just less, just as many and just more
    rows end than fill that place (and some of them by a row that began in the span before), ranges of rows
    and columns, every epilogue; what lies outside a range keeps its bits."""
    import paper_2501_01951_amd as mg

    mg.load_library()
    lens = []
    for span in range(6):  # `ends` rows per 256 entries, the last one reaching into the next span
        over = 3 if lens and ends < 255 else 0
        lens += [1] * (ends - 1) + [256 - over - (ends - 1) + (3 if ends < 255 else 0)]
    lens = np.array(lens + [0, 2, 0, 0, 5])
    n, f = len(lens) + 40, 44
    src = np.repeat(np.arange(len(lens)), lens)
    start = np.repeat(np.cumsum(lens) - lens, lens)
    dst = (src * 7 + np.arange(len(src)) - start) % n
    keep = np.unique(src * n + dst)  # long rows of small graphs repeat columns
    src, dst = keep // n, keep % n
    g = mg.build_csr(torch.from_numpy(src.astype(np.int32)).cuda(), torch.from_numpy(dst.astype(np.int32)).cuda(),
                     n, 0)
    mg.normalize(g, mg.NORM_SUM)
    a = g.arrays()
    rowptr, col = a["rowptr"].cpu().numpy(), a["col"].cpu().numpy()
    dt = torch.bfloat16 if bf else torch.float32
    ld = 48
    h = torch.zeros(n, ld, device="cuda", dtype=dt)
    h[:, :f] = torch.from_numpy(gg.normal(5, f, n, f)).cuda().to(dt)
    old = torch.from_numpy(gg.normal(6, f, n, ld)).cuda().to(dt)
    slices = 1 if bf else 2
    sums = torch.from_numpy(row_sums(rowptr, col, h[:, :f].float().cpu().numpy(), 8, span_entries(8, g.nnz, slices)))
    for relu, acc in ((False, False), (True, False), (False, True), (True, True)):
        z = old.clone()
        mg.aggregate(g, h[:, :f], z[:, :f], relu=relu, accumulate=acc)
        want = sums + old[:, :f].float().cpu() if acc else sums.clone()
        want = want.clamp(min=0) if relu else want
        empty = torch.from_numpy(rowptr[1:n + 1] == rowptr[:n])
        if acc and not relu:
            want[empty] = old[:, :f].float().cpu()[empty]
        assert torch.equal(z[:, :f].cpu(), want.to(dt)), (relu, acc)
        assert torch.equal(z[:, f:], old[:, f:])
    mask = mg.dropout_bitmap(9, n, f, 0.5)
    z = old.clone()
    mg.aggregate_masked(g, h[:, :f], z[:, :f], mask)
    bits = torch.from_numpy(np.unpackbits(mask.cpu().numpy().view(np.uint8), bitorder="little").reshape(n, -1)[:, :f])
    assert torch.equal(z[:, :f].cpu(), (sums * bits).to(dt))
    z = old.clone()
    mg.aggregate(g, h[:, :f], z[:, :f], 3, 41, 2, len(lens) - 2)
    got, was = z.cpu(), old.cpu()
    assert torch.equal(got[:2], was[:2]) and torch.equal(got[len(lens) - 2:], was[len(lens) - 2:])
    assert torch.equal(got[:, :3], was[:, :3]) and torch.equal(got[:, 41:], was[:, 41:])
    inner = slice(2, len(lens) - 2)
    tol = 1e-2 if bf else 1e-5  # a range may cut other pieces: only the order of the sums differs
    assert torch.allclose(got[inner, 3:41].float(), sums[inner, 3:41], rtol=tol, atol=tol * 16)
    g.free()
