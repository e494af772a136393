"""Reuse of the memory of freed graphs and finished builds: blocks pass between sizes, streams and
threads, and the results are those of first builds."""
import ctypes
import threading

import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _check(mg, case, stream):
    src, dst, n, want = case
    with torch.cuda.stream(stream):
        g = mg.build_csr(src, dst, n, stream=stream)
        mg.normalize(g, stream=stream)
        h = torch.ones(n, 40, device="cuda")
        z = torch.empty_like(h)
        mg.aggregate(g, h, z, stream=stream)
        stream.synchronize()
        a = g.arrays()
    assert np.array_equal(a["rowptr"].cpu().numpy(), want.rowptr)
    assert np.array_equal(a["col"].cpu().numpy().view(np.uint32), want.col)
    assert np.array_equal(a["deg"].cpu().numpy().view(np.uint32), np.diff(want.rowptr))
    np.testing.assert_allclose(a["val"].cpu().numpy(), want.val, rtol=2e-7)  # three fp32 roundings
    # positive sums of fewer than 2^12 values, in eight chains
    sums = np.add.reduceat(want.val, want.rowptr[:-1])
    np.testing.assert_allclose(z[:, 0].cpu().numpy(), sums, rtol=512 * 6e-8)
    assert torch.equal(z, z[:, :1].expand_as(z))
    g.free()


@pytest.mark.parametrize("n_threads", [1, 4])
def test_builds_in_reused_memory(n_threads):
    """Each thread builds and frees graphs of different sizes on a stream of its own; the cache is
    given back in the middle."""
    import paper_2501_01951_amd as mg

    mg.load_library()
    graphs = [gg.config_graph("c2", scale_override=scale) for scale in (6, 9, 12, 13)]
    rng = np.random.default_rng(4)  # and one whose columns form bands
    graphs.append((*(rng.integers(0, 60_000, 1_830_000).astype(np.uint32) for _ in range(2)), 60_000))
    cases = []
    for src, dst, n in graphs:
        cases.append((torch.from_numpy(src.view(np.int32)).cuda(), torch.from_numpy(dst.view(np.int32)).cuda(),
                      n, oracle.normalize(oracle.build_csr(src, dst, n))))
    torch.cuda.synchronize()
    errors = []

    def work(t):
        try:
            stream = torch.cuda.Stream()
            for k in range(12):
                _check(mg, cases[(t + k) % len(cases)], stream)
                if k == 6 and t == 0:
                    mg.release_memory()
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    threads = [threading.Thread(target=work, args=(t,)) for t in range(n_threads)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors


def _small_graph(mg, seed):
    src, dst = (np.random.default_rng(seed + i).integers(0, 5000, 40_000).astype(np.uint32) for i in (0, 1))
    return torch.from_numpy(src.view(np.int32)).cuda(), torch.from_numpy(dst.view(np.int32)).cuda()


@pytest.mark.parametrize("capturing", [False, True])
def test_arrays_of_a_freed_graph_wait_for_work_on_any_stream(capturing):
    """A graph is dropped with aggregations of it queued on a stream, and another one is built on a
    second stream at once: it must not get the arrays of the first before they are read.  While a
    stream is being captured the device cannot be waited for."""
    import paper_2501_01951_amd as mg

    n = 5000
    ends, other = _small_graph(mg, 1), _small_graph(mg, 3)
    h, z = torch.randn(n, 64, device="cuda"), torch.zeros(n, 64, device="cuda")
    x = torch.zeros(8, device="cuda")
    reader, builder, captured = (torch.cuda.Stream() for _ in range(3))
    g = mg.build_csr(*ends, n)
    mg.normalize(g)
    want = torch.zeros_like(z)
    mg.aggregate(g, h, want)
    torch.cuda.synchronize()

    def drop_and_build(g):
        with torch.cuda.stream(reader):
            torch.cuda._sleep(200_000_000)
            mg.aggregate(g, h, z, stream=reader)
        g.free()
        with torch.cuda.stream(builder):
            second = mg.build_csr(*other, n, stream=builder)
            mg.normalize(second, stream=builder)
        return second

    if capturing:
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=captured, capture_error_mode="relaxed"):
            x.add_(1)
            second = drop_and_build(g)
        graph.replay()
    else:
        second = drop_and_build(g)
    torch.cuda.synchronize()
    assert torch.equal(z, want)
    fresh = mg.build_csr(*other, n)
    mg.normalize(fresh)
    a, b = second.arrays(), fresh.arrays()
    for name in ("rowptr", "col", "val", "deg", "dinv"):
        assert torch.equal(a[name], b[name]), name
    mg.aggregate(second, h, z)
    mg.aggregate(fresh, h, want)
    assert torch.equal(z, want)
    second.free()
    fresh.free()


def test_cached_memory_makes_room_for_other_allocations_of_the_library():
    """With the device nearly full, a call that allocates past the cache (8 GiB for the peaks) gets what
    the cache holds."""
    import paper_2501_01951_amd as mg

    n = 300_000
    gen = torch.Generator("cuda").manual_seed(1)
    src, dst = (torch.randint(0, n, (45_000_000,), device="cuda", dtype=torch.int32, generator=gen) for _ in range(2))
    mg.release_memory()
    mg.measure_peaks()  # what the runtime itself needs for its kernels is there
    g = mg.build_csr(src, dst, n)
    g.free()
    torch.cuda.empty_cache()
    torch.cuda.synchronize()
    gib = 1 << 30
    hog = []
    while torch.cuda.mem_get_info()[0] > 8 * gib - (gib >> 1):
        hog.append(torch.empty(min(32 * gib, torch.cuda.mem_get_info()[0] - 7 * gib), dtype=torch.uint8, device="cuda"))
    free = torch.cuda.mem_get_info()[0]
    assert 6 * gib < free < 8 * gib
    assert mg.measure_peaks()
    assert torch.cuda.mem_get_info()[0] > free + gib
    del hog
    torch.cuda.empty_cache()


@pytest.mark.parametrize("n,degree,mean", [(5000, 16, False), (60_000, 61, True)])
def test_first_normalisation_can_be_captured(n, degree, mean):
    """Its arrays come from the driver or from blocks without pending work: a stream being captured
    cannot wait for events of others.  Replays give the values of an eager call."""
    import paper_2501_01951_amd as mg

    rng = np.random.default_rng(5)
    src, dst = (torch.from_numpy(rng.integers(0, n, n * degree // 2).astype(np.int32)).cuda() for _ in range(2))
    flags = mg.SYMMETRIZE | (0 if mean else mg.ADD_SELF_LOOPS)
    kind = mg.NORM_MEAN if mean else mg.NORM_SYM
    g, want = (mg.build_csr(src, dst, n, flags) for _ in range(2))
    mg.build_csr(src, dst, n, flags).free()  # blocks of its work arrays wait in the cache
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side, capture_error_mode="relaxed"):
        mg.normalize(g, kind, stream=side)
    mg.normalize(want, kind)
    h = torch.randn(n, 40, device="cuda")
    z, z_want = torch.empty_like(h), torch.empty_like(h)
    mg.aggregate(want, h, z_want, transpose=mean)
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(g.arrays()["val"], want.arrays()["val"])
        mg.aggregate(g, h, z, transpose=mean)
        assert torch.equal(z, z_want)
        z.zero_()
    g.free()
    want.free()


@pytest.mark.parametrize("n,degree", [(1000, 3), (30_000, 30), (200_000, 8)])
def test_row_pointers_on_the_host_belong_to_their_graph(n, degree):
    """The pinned host copies of row pointers go from one graph to the next: calls over row ranges, which take their
    first and last entries from them, while graphs of the same size come and go (and after the cache has been emptied)."""
    import paper_2501_01951_amd as mg

    gen = torch.Generator(device="cuda").manual_seed(n)
    held = []
    for i in range(4):
        src, dst = (torch.randint(0, n, (n * degree // 2,), device="cuda", dtype=torch.int32, generator=gen)
                    for _ in range(2))
        g = mg.build_csr(src, dst, n)
        mg.normalize(g)
        held.append(g)
        if i == 1:
            held.pop(0).free()
        if i == 2:
            mg.release_memory()
        for k in held:
            h = torch.randn(n, 8, device="cuda", generator=gen)
            z, parts = torch.empty_like(h), torch.empty_like(h)
            mg.aggregate(k, h, z)
            for r0, r1 in ((0, 1), (1, n // 3), (n // 3, n)):
                mg.aggregate(k, h, parts, row_begin=r0, row_end=r1)
            assert torch.allclose(z, parts, rtol=1e-5, atol=1e-6)  # (spans of another length: sums in another order)
    for k in held:
        k.free()


@pytest.mark.parametrize("mode", ["sym", "mean", "sum"])
@pytest.mark.parametrize("first,last,n", [(0, 300, 301), (100_000, 100_257, 400_000), (399_000, 400_000, 400_000)])
def test_values_of_rows_between_empty_ones(mode, first, last, n):
    """Groups of 256 entries that cover one row, many rows, and long runs of empty rows; a last group that is not full."""
    import paper_2501_01951_amd as mg

    gen = torch.Generator(device="cuda").manual_seed(last)
    src = torch.randint(first, last, (3001,), device="cuda", dtype=torch.int32, generator=gen)
    dst = torch.cat([src.new_full((700,), last - 1),
                     torch.randint(first, last, (2301,), device="cuda", dtype=torch.int32, generator=gen)])
    g = mg.build_csr(src, dst, n, mg.SYMMETRIZE)
    mg.normalize(g, {"sym": mg.NORM_SYM, "mean": mg.NORM_MEAN, "sum": mg.NORM_SUM}[mode], eps=0.25)
    for transpose in (False, True):
        a = g.arrays(transpose)
        deg = a["rowptr"][1:] - a["rowptr"][:-1]
        row = torch.repeat_interleave(torch.arange(n, device="cuda"), deg)
        col = a["col"].long()
        root = (1 / deg.double().sqrt()).float()
        want = {"sym": root[row] * root[col], "sum": torch.ones_like(a["val"]),
                "mean": (1 / deg.double()).float()[col if transpose else row]}[mode]
        assert torch.equal(a["val"], want)
    g.free()


@pytest.fixture
def host_memory():
    """mixgcn::host_alloc and host_free, and whether an address is pinned host memory."""
    import paper_2501_01951_amd as mg

    lib = mg.load_library()
    alloc, free = lib._ZN6mixgcn10host_allocEPPvm, lib._ZN6mixgcn9host_freeEPv
    alloc.argtypes, free.argtypes, free.restype = [ctypes.c_void_p, ctypes.c_size_t], [ctypes.c_void_p], None
    with open("/proc/self/maps") as maps:
        runtime = ctypes.CDLL(next(line.split()[-1] for line in maps if "libamdhip64" in line))

    def take(size):
        p = ctypes.c_void_p()
        assert alloc(ctypes.byref(p), size) == 0
        return p

    def pinned(p):
        attr = (ctypes.c_int * 64)()  # the memory type comes first; 1 is host memory
        ok = runtime.hipPointerGetAttributes(attr, p) == 0 and attr[0] == 1
        runtime.hipGetLastError()
        return ok

    mg.release_memory()
    yield take, free, pinned
    mg.release_memory()


def test_pinned_memory_that_is_too_large_to_keep(host_memory):
    """A block above the bound of 512 MB goes back alone; others leave when they are together more, the oldest first."""
    take, free, pinned = host_memory
    blocks = [take(size << 20) for size in (8, 300, 9, 600, 300)]
    assert all(pinned(p) for p in blocks)
    for p in blocks[:4]:
        free(p)
    assert [pinned(p) for p in blocks[:4]] == [True, True, True, False]
    free(blocks[4])
    assert [pinned(p) for p in blocks] == [False, False, True, False, True]
    assert take(9 << 20).value == blocks[2].value
    free(blocks[2])


@pytest.mark.parametrize("thread", [False, True])
def test_pinned_memory_goes_back_while_a_stream_is_captured(host_memory, thread):
    """Freeing a graph is allowed then in every mode of capture: a release that the runtime refuses would end it."""
    take, free, pinned = host_memory
    large, x = take(600 << 20), torch.zeros(8, device="cuda")
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, capture_error_mode="global"):
        x.add_(1)
        if thread:
            t = threading.Thread(target=free, args=(large,))
            t.start()
            t.join()
        else:
            free(large)
    for _ in range(3):
        graph.replay()
    assert (x == 3).all() and not pinned(large)
