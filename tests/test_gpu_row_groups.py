"""Aggregation over whole matrices against the oracle: row lengths around the limits of the row groups
that the bands of dense graphs use (32, 64, 256, 1024 entries, windows of 4096 rows) in matrices without
bands, both gather widths, and dense graphs on both sides of the rule for bands, the kernel that takes a
call asserted."""
import numpy as np
import pytest
import torch

import graphgen as gg
import oracle
from parity import RTOL_BF16, RTOL_F32, assert_close, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mg():
    import paper_2501_01951_amd as m

    assert torch.cuda.is_available()
    m.load_library()
    return m


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def check(mg, g, og, f, bf, tr, desc):
    """Plain, accumulating, clamped and masked calls against the oracle."""
    rtol, dt = (RTOL_BF16, torch.bfloat16) if bf else (RTOL_F32, torch.float32)
    ld = (f + 7) // 8 * 8
    h, z0 = (dev(gg.normal(7, s, og.n, ld)).to(dt) for s in (1, 2))
    agg = oracle.spmm(og, h[:, :f].float().cpu().numpy().astype(np.float64), transposed=tr)
    old = z0[:, :f].float().cpu().numpy().astype(np.float64)
    for relu, acc in ((False, False), (True, False), (False, True), (True, True)):
        say(f"{desc} f={f} bf16={bf} transpose={tr} relu={relu} accumulate={acc}")
        z = z0.clone()
        mg.aggregate(g, h[:, :f], z[:, :f], transpose=tr, relu=relu, accumulate=acc)
        want = agg + old if acc else agg
        assert_close(z[:, :f].float().cpu().numpy(), np.maximum(want, 0) if relu else want, rtol, desc)
        assert torch.equal(z[:, f:], z0[:, f:])
    bits = oracle.dropout_bitmap(3, og.n, f, 0.5)
    keep = ((bits[:, np.arange(f) // 32] >> (np.arange(f) % 32).astype(np.uint32)) & 1).astype(bool)
    z = z0.clone()
    mg.aggregate_masked(g, h[:, :f], z[:, :f], dev(bits.view(np.int32)), transpose=tr)
    assert_close(z[:, :f].float().cpu().numpy(), np.where(keep, agg, 0.0), rtol, desc + " masked")


@pytest.mark.parametrize("n,repeat", [(257, 1), (4095, 1), (4097, 3), (9000, 8)])
def test_row_lengths_around_groups_pieces_and_windows(mg, n, repeat):
    some = [0, 1, 2, 7, 8, 9, 31, 32, 33, 63, 64, 65, 127, 255, 256, 257]
    some += [v for v in (511, 513, 1023, 1024, 1025, 2049, 4000) if v <= n]
    lens = np.ones(n, dtype=np.int64)
    lens[np.random.default_rng(n).permutation(n)[:len(some) * repeat]] = some * repeat
    if n == 9000:
        lens[4090:4900] = 5000  # more than 4 M entries: the limits of large matrices
    src = np.repeat(np.arange(n), lens)
    dst = (src * 7 + np.arange(len(src)) - np.repeat(np.cumsum(lens) - lens, lens)) % n
    src, dst = src.astype(np.uint32), dst.astype(np.uint32)
    g = mg.build_csr(dev(src.view(np.int32)), dev(dst.view(np.int32)), n, mg.BUILD_TRANSPOSE)
    mg.normalize(g, mg.NORM_MEAN)
    og = oracle.transpose(oracle.normalize_mean(oracle.build_csr(src, dst, n, False, False)))
    for f, bf in ((5, False), (16, False), (33, False), (24, True), (100, True)):
        check(mg, g, og, f, bf, False, f"n={n} nnz={og.nnz}")
    check(mg, g, og, 48, False, True, f"n={n} nnz={og.nnz}")
    g.free()


@pytest.mark.parametrize("mean", [False, True])
def test_dense_graph_whose_columns_form_bands(mg, mean):
    n, degree = 60_000, 60
    rng = np.random.default_rng(5)
    src, dst = (rng.integers(0, n, n * degree // 2).astype(np.uint32) for _ in range(2))
    dst[:n // 2] = rng.integers(0, 40, n // 2)  # a few rows long enough to be cut
    g = mg.build_csr(dev(src.view(np.int32)), dev(dst.view(np.int32)), n,
                     mg.SYMMETRIZE | (0 if mean else mg.ADD_SELF_LOOPS))
    mg.normalize(g, mg.NORM_MEAN if mean else mg.NORM_SYM)
    og = oracle.build_csr(src, dst, n, True, not mean)
    og = oracle.transpose((oracle.normalize_mean if mean else oracle.normalize)(og))
    for f, bf in ((16, False), (40, False), (72, True)):
        in_bands = mg.load_library().mixgcn_aggregate_bands(g._h, int(mean), mg.BF16 if bf else mg.F32, f) > 1
        assert in_bands == (f == 40)
        check(mg, g, og, f, bf, mean, f"bands n={n} nnz={og.nnz}")
    g.free()


@pytest.mark.parametrize("mean_len", [85, 105, 160, 200])
def test_both_sides_of_the_dispatch(mg, mean_len):
    """A directed graph of 28 k columns, which never has bands: short rows and rows of 5000 entries, which
    cross many spans."""
    n = 28_000
    lens = np.full(n, 3, dtype=np.int64)
    long_rows = np.random.default_rng(mean_len).permutation(n)[:n * (mean_len - 3) // 5000]
    lens[long_rows] = 5000
    src = np.repeat(np.arange(n), lens)
    dst = (src * 7 + np.arange(len(src)) - np.repeat(np.cumsum(lens) - lens, lens)) % n
    src, dst = src.astype(np.uint32), dst.astype(np.uint32)
    g = mg.build_csr(dev(src.view(np.int32)), dev(dst.view(np.int32)), n, 0)
    mg.normalize(g, mg.NORM_MEAN)
    og = oracle.normalize_mean(oracle.build_csr(src, dst, n, False, False))
    for f, bf in ((16, False), (33, False), (40, True)):
        check(mg, g, og, f, bf, False, f"mean length {mean_len} nnz={og.nnz}")
    g.free()


def test_bands_of_narrow_and_bf16_passes(mg):
    """A graph with bands whose narrow and bf16 passes do not take them."""
    n, degree = 80_000, 300
    rng = np.random.default_rng(6)
    src, dst = (rng.integers(0, n, n * degree // 2).astype(np.uint32) for _ in range(2))
    g = mg.build_csr(dev(src.view(np.int32)), dev(dst.view(np.int32)), n)
    mg.normalize(g)
    og = oracle.normalize(oracle.build_csr(src, dst, n, True, True))
    for f, bf in ((16, False), (72, True)):
        assert mg.load_library().mixgcn_aggregate_bands(g._h, 0, mg.BF16 if bf else mg.F32, f) == 0
        check(mg, g, og, f, bf, False, f"bands n={n} nnz={og.nnz}")
    g.free()
