"""Aggregations of dense graphs whose columns are dealt to bands: which calls take them, and what holds
for their results."""
import numpy as np
import pytest

import oracle
from parity import RTOL_F32, assert_close, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def mg():
    import paper_2501_01951_amd as m

    assert torch.cuda.is_available()
    m.load_library()
    return m


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def bands(mg, g, f, dtype=None, transpose=0):
    return mg.load_library().mixgcn_aggregate_bands(g._h, transpose, mg.F32 if dtype is None else dtype, f)


def edges(n, degree, seed, hubs=0):
    """Uniform columns; hubs > 0: a part of the edges ends in that many nodes."""
    rng = np.random.default_rng(seed)
    src, dst = (rng.integers(0, n, n * degree // 2).astype(np.uint32) for _ in range(2))
    if hubs:
        dst[:n // 2] = rng.integers(0, hubs, n // 2)
    return src, dst


def graph(mg, src, dst, n, mean=False):
    g = mg.build_csr(dev(src.view(np.int32)), dev(dst.view(np.int32)), n,
                     mg.SYMMETRIZE | (0 if mean else mg.ADD_SELF_LOOPS))
    mg.normalize(g, mg.NORM_MEAN if mean else mg.NORM_SYM)
    return g


@pytest.mark.parametrize("n,degree,f,bf", [(60_000, 61, 72, True), (80_000, 300, 256, True),
                                           (80_000, 300, 256, False), (80_000, 300, 300, False)])
def test_fixed_scratch_gives_the_same_bits(mg, n, degree, f, bf):
    """mixgcn_aggregate_static takes the same kernel whatever scratch the graph's own slots have."""
    g = graph(mg, *edges(n, degree, 5, 40), n)
    say(f"static and own scratch n={n} nnz={g.nnz} f={f} bf16={bf}")
    assert (bands(mg, g, f, mg.BF16 if bf else mg.F32) > 1) == (not bf)
    h = torch.randn(n, (f + 7) // 8 * 8, device="cuda").to(torch.bfloat16 if bf else torch.float32)
    z, z_static = torch.zeros_like(h), torch.zeros_like(h)
    mg.aggregate(g, h, z, col_end=f)
    mg.aggregate_static(g, h, z_static, col_end=f)
    assert torch.equal(z, z_static)
    g.free()


@pytest.mark.parametrize("n,degree", [(60_000, 61), (100_000, 100), (180_000, 100)])
def test_rounding_error_is_that_of_the_row_ranges(mg, n, degree):
    """Against 64 bits, a call in bands is no further off than one that takes the entry-balanced kernel
    (row ranges do).  The ratio of the two rms errors over n * 64 sums varies by less than 0.2 %."""
    f = 64
    g = graph(mg, *edges(n, degree, 8), n)
    say(f"rounding error n={n} nnz={g.nnz}")
    assert bands(mg, g, f) > 1
    h = torch.randn(n, f, device="cuda", generator=torch.Generator("cuda").manual_seed(n))
    z, z_ranges = torch.empty_like(h), torch.empty_like(h)
    mg.aggregate(g, h, z)
    for r in (0, n // 2):
        mg.aggregate(g, h, z_ranges, row_begin=r, row_end=r + n // 2)
    a = g.arrays()
    rows = torch.repeat_interleave(torch.arange(n, device="cuda"), a["rowptr"].diff())
    exact = torch.zeros(n, f, dtype=torch.float64, device="cuda")
    for e in range(0, g.nnz, 1 << 21):
        part = slice(e, e + (1 << 21))
        exact.index_add_(0, rows[part], h[a["col"][part].long()].double() * a["val"][part, None].double())
    ratio = (z.double() - exact).norm() / (z_ranges.double() - exact).norm()
    assert ratio < 1.002, float(ratio)
    g.free()


@pytest.mark.parametrize("degree,hubs", [(120, 0), (100, 40)])
def test_launches_with_eight_gathers_in_flight(mg, degree, hubs):
    """256 columns make launches large enough for eight gathers in flight per wavefront, 64 do not (2.4 M batches of
    eight entries and 32 columns lie between them).  Element by element against 64 bits: a row of d entries is at most
    d / 4 multiply-adds to a chain, and a few more additions that join chains, sub-groups, pieces and bands."""
    n, f = 60_000, 256
    g = graph(mg, *edges(n, degree, 21, hubs), n)
    # of uniform columns a band of 26 k has 26 / 60 of the entries; 8 slices of 32 columns, and 2
    assert bands(mg, g, f) == bands(mg, g, 64) > 1 and g.nnz * 26 / 60 > 2.4e6 > g.nnz / 8 * 2
    h = torch.randn(n, f, device="cuda", generator=torch.Generator("cuda").manual_seed(n))
    arr = g.arrays()
    a = torch.sparse_csr_tensor(arr["rowptr"], arr["col"].long(), arr["val"].double(), (n, n))
    d = (arr["rowptr"][1:] - arr["rowptr"][:-1])[:, None].double()
    ref, bound = a @ h.double(), (a @ h.abs().double()) * (d / 4 + 24) * 2.0 ** -24  # (the values are positive)
    z, masked, parts = torch.empty_like(h), torch.empty_like(h), torch.empty_like(h)
    mg.aggregate(g, h, z)
    assert ((z.double() - ref).abs() <= bound).all()
    m = mg.dropout_bitmap(7, n, f, 0.5)
    keep = ((m[:, torch.arange(f, device="cuda") // 32] >> (torch.arange(f, device="cuda") % 32)) & 1).bool()
    mg.aggregate_masked(g, h, masked, m)
    assert torch.equal(masked, torch.where(keep, z, torch.zeros_like(z)))
    for c in range(0, f, 64):
        mg.aggregate(g, h, parts, col_begin=c, col_end=c + 64)
    assert ((parts.double() - ref).abs() <= bound).all()
    g.free()


def test_which_passes_take_the_bands(mg):
    """Wide fp32 passes of dense symmetrised graphs; not rows of 64 bytes or less, which the bands slow
    down, and not bf16."""
    g = graph(mg, *edges(80_000, 300, 9), 80_000)
    for f in (1, 8, 16, 19):
        assert bands(mg, g, f) == 0
    for f in (20, 128, 600):
        assert bands(mg, g, f) > 1 and bands(mg, g, f, mg.BF16) == 0
    sparse = graph(mg, *edges(80_000, 20, 9), 80_000)
    assert bands(mg, sparse, 128) == 0
    src, dst = edges(80_000, 150, 9)
    directed = mg.build_csr(dev(src.view(np.int32)), dev(dst.view(np.int32)), 80_000, mg.BUILD_TRANSPOSE)
    mg.normalize(directed)
    assert bands(mg, directed, 128) == 0 and bands(mg, directed, 128, transpose=1) == 0
    for x in (g, sparse, directed):
        x.free()


@pytest.mark.parametrize("n,degree,mean", [(4096, 10, False), (80_000, 300, False), (80_000, 300, True)])
def test_first_normalisation_does_not_wait_for_its_stream(mg, n, degree, mean):
    src, dst = edges(n, degree, 10)
    g = mg.build_csr(dev(src.view(np.int32)), dev(dst.view(np.int32)), n,
                     mg.SYMMETRIZE | (0 if mean else mg.ADD_SELF_LOOPS))
    stream, done = torch.cuda.Stream(), torch.cuda.Event()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        torch.cuda._sleep(1_000_000_000)  # half a second or more of the stream's time
        mg.normalize(g, mg.NORM_MEAN if mean else mg.NORM_SYM, stream=stream)
        done.record()
    assert not done.query()
    done.synchronize()
    want = oracle.build_csr(src, dst, n, True, not mean)
    want = (oracle.normalize_mean if mean else oracle.normalize)(want)
    # three fp32 roundings at most
    np.testing.assert_allclose(g.arrays()["val"].cpu().numpy(), want.val, rtol=2e-7, atol=0)
    g.free()


def test_no_second_layout_where_it_cannot_be_used(mg):
    """Row pointers apart, a graph without bands takes 16 bytes per entry: columns, values, and both
    together.  Blocks are at most an eighth larger than what is in them."""
    n, degree = 300_000, 100
    src, dst = (dev(e.view(np.int32)) for e in edges(n, degree, 11))
    mg.release_memory()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    g = mg.build_csr(src, dst, n)
    mg.normalize(g)
    torch.cuda.synchronize()
    mg.release_memory()
    taken = before - torch.cuda.mem_get_info()[0]
    assert bands(mg, g, 256) == 0
    scratch = mg.load_library().mixgcn_aggregate_scratch_bytes(g.nnz)
    assert taken < 1.125 * (16 * g.nnz + scratch) + 64 * n, (taken, g.nnz, scratch)
    g.free()


@pytest.mark.parametrize("mean", [False, True])
def test_bands_against_the_oracle(mg, mean):
    """Rows cut into pieces in several bands; column ranges that start and end inside a 16-byte group, with
    ReLU, accumulating and masked; feature rows so far apart that offsets need 64 bits."""
    n, f = 80_000, 48
    src, dst = edges(n, 150, 12, hubs=30)
    g = graph(mg, src, dst, n, mean)
    tr = int(mean)
    assert bands(mg, g, f, transpose=tr) > 1
    og = oracle.build_csr(src, dst, n, True, not mean)
    og = oracle.transpose((oracle.normalize_mean if mean else oracle.normalize)(og))
    gen = torch.Generator("cuda").manual_seed(12)
    wide = torch.empty(n, 13440, device="cuda")  # 4.3 GB
    wide[:, :f] = torch.randn(n, f, device="cuda", generator=gen)
    z0 = torch.randn(n, f, device="cuda", generator=gen)
    agg = oracle.spmm(og, wide[:, :f].cpu().numpy().astype(np.float64), transposed=bool(tr))
    old = z0.cpu().numpy().astype(np.float64)
    near = wide[:, :f].contiguous()
    for h in (near, wide):
        for c0, c1 in ((0, f), (3, 45)):
            for relu, acc in ((False, False), (True, False), (True, True)):
                say(f"bands mean={mean} pitch={h.stride(0)} columns [{c0},{c1}) relu={relu} accumulate={acc}")
                z = z0.clone()
                mg.aggregate(g, h, z, c0, c1, transpose=tr, relu=relu, accumulate=acc)
                want = agg + old if acc else agg
                want = np.maximum(want, 0) if relu else want
                assert_close(z[:, c0:c1].cpu().numpy(), want[:, c0:c1], RTOL_F32, "bands")
                assert torch.equal(z[:, :c0], z0[:, :c0]) and torch.equal(z[:, c1:], z0[:, c1:])
    bits = oracle.dropout_bitmap(3, n, f, 0.5)
    keep = ((bits[:, np.arange(f) // 32] >> (np.arange(f) % 32).astype(np.uint32)) & 1).astype(bool)
    z = z0.clone()
    mg.aggregate_masked(g, near, z, dev(bits.view(np.int32)), transpose=tr)
    assert_close(z.cpu().numpy(), np.where(keep, agg, 0.0), RTOL_F32, "masked")
    g.free()


def test_bands_on_several_streams(mg):
    """Column slices of one graph on four streams at once give the bits of the same calls in a row."""
    n, f = 80_000, 128
    g = graph(mg, *edges(n, 150, 13, hubs=30), n)
    assert bands(mg, g, f) > 1
    h = torch.randn(n, 4 * f, device="cuda")
    want, z = torch.zeros_like(h), torch.zeros_like(h)
    for i in range(4):
        mg.aggregate(g, h, want, i * f, (i + 1) * f)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(4)]
    for _ in range(3):
        for i, s in enumerate(streams):
            mg.aggregate(g, h, z, i * f, (i + 1) * f, stream=s)
        torch.cuda.synchronize()
        assert torch.equal(z, want)
        z.zero_()
        torch.cuda.synchronize()
    g.free()


def test_transpose_without_memory_for_its_bands(mg):
    """Room for the mean weights of the transpose (16 bytes per entry in all) but not for their streams
    (8 more): its aggregations take the entry-balanced kernel, those of the matrix the bands."""
    n, f = 80_000, 40
    src, dst = edges(n, 300, 14)
    g = mg.build_csr(dev(src.view(np.int32)), dev(dst.view(np.int32)), n, mg.SYMMETRIZE)
    mg.release_memory()
    torch.cuda.empty_cache()
    torch.cuda.synchronize()
    # blocks are at most a sixteenth larger than what is in them
    need = int(17 * g.nnz) + 2 * mg.load_library().mixgcn_aggregate_scratch_bytes(g.nnz) + (32 << 20)
    hog = []
    while torch.cuda.mem_get_info()[0] > need + (64 << 20):
        hog.append(torch.empty(min(32 << 30, torch.cuda.mem_get_info()[0] - need), dtype=torch.uint8, device="cuda"))
    assert need - (8 << 20) <= torch.cuda.mem_get_info()[0] < need + (64 << 20)
    mg.normalize(g, mg.NORM_MEAN)
    torch.cuda.synchronize()
    del hog
    torch.cuda.empty_cache()
    assert bands(mg, g, f) > 1 and bands(mg, g, f, transpose=1) == 0
    og = oracle.transpose(oracle.normalize_mean(oracle.build_csr(src, dst, n, True, False)))
    h = torch.randn(n, f, device="cuda")
    for tr in (0, 1):
        z = torch.empty_like(h)
        mg.aggregate(g, h, z, transpose=tr)
        assert_close(z.cpu().numpy(), oracle.spmm(og, h.cpu().numpy().astype(np.float64), transposed=bool(tr)),
                     RTOL_F32, f"transpose={tr}")
    g.free()
