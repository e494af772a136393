"""The update products (forward, data gradient, fp32 weight gradient) at the edges of their kernels: 32-row tiles, reduction steps
of 128 bytes of a row, weights that stay in LDS and weights that stream through it, output tiles of 16, 32,
64 and 128 columns; what rows hold past their columns, infinities and NaN."""
import ctypes

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mg():
    import paper_2501_01951_amd as m

    m.load_library()
    return m


def padded(n, cols, dtype, gen):
    """n x cols on a pitch of its own, NaN past the columns."""
    per = 16 // torch.empty(0, dtype=dtype).element_size()
    t = torch.full((n, (cols + per - 1) // per * per + per), float("nan"), device="cuda", dtype=dtype)
    t[:, :cols] = torch.randn(n, cols, device="cuda", generator=gen)
    return t


def check(got, a, w, dtype, steps, what):
    """Element by element.  A term's dropped partial products are below 2^-23 (fp32) or the weights' third
    term below 2^-16 (bf16) of |a| |w|; a step adds its products with a few fp32 roundings of sums no larger
    than its sum of |a| |w| (a 2^-24 each, 12 MFMAs of two), then rounds the running sum once; a bf16 result
    is rounded to 8 bits."""
    ref = a.double() @ w.double()
    mag = a.double().abs() @ w.double().abs()
    bound = mag * ((26 + steps) * 2.0 ** -24)
    if dtype == torch.bfloat16:
        bound = bound + mag * 2.0 ** -16 + ref.abs() * 2.0 ** -8
    bad = (got.double() - ref).abs() > bound + 1e-30
    assert not bad.any(), (what, int(bad.sum()))


def chain(a, w):
    """Multiply-adds of fp32 in the order of the reduction index.  A product of two floats is exact in 64 bits; the sum is
    rounded to odd there (what it loses, exactly, says which way), so that rounding it once more is rounding it once."""
    s = torch.zeros(a.shape[0], w.shape[1], device="cuda")
    for k in range(a.shape[1]):
        p, q = a[:, k:k + 1].double() * w[k:k + 1].double(), s.double()
        t = p + q
        lost = (p - (t - (t - p))) + (q - (t - p))
        bits = t.view(torch.int64)
        even = (bits & 1 == 0) & ((lost > 0) | (lost < 0))  # (not a NaN)
        s = torch.where(even, bits + torch.where((lost > 0) == (t > 0), 1, -1), bits).view(torch.float64).float()
    return s


# The general kernel: tiles of 128 rows, 32 and 128 columns and steps of 16, inside the matrices and at their edges; every
# tile inside (its fast path) alone, and beside others of the last rows.
GENERAL = [(1, 1, 1), (128, 16, 32), (129, 15, 33), (300, 100, 64), (70, 1281, 31), (20003, 37, 250), (4096, 64, 32),
           (33000, 64, 64), (16512, 64, 256), (33000, 128, 256), (262150, 200, 47), (16397, 160, 4001)]
# The weights in LDS.  Column tiles of 32: below, at and past a tile of 32 rows and a step of 32 indices, the deepest,
# several column tiles, the last one whole or not, two rounds of workgroups, two tiles to a wavefront; of 64, whole and
# not, rows left over; of 128, 32 of them, rows and columns left over
IN_LDS = [(1, 64, 1), (256, 64, 128), (255, 128, 65), (384, 256, 256), (260, 602, 129), (70, 1280, 31), (4000, 96, 40),
          (12000, 70, 120), (300, 64, 1500), (262144, 64, 31), (262144, 192, 64), (300010, 200, 47), (17900, 160, 4001),
          (131072, 128, 512)]


@pytest.mark.parametrize("n,k,m,in_lds", [(*c, False) for c in GENERAL] + [(*c, True) for c in IN_LDS])
def test_fp32_forward_sums_are_the_fp32_chain(mg, n, k, m, in_lds):
    """Bit for bit: the sums of a forward product decide the sign of an activation, so they keep their
    rounding from release to release."""
    applies = mg.load_library()._ZN6mixgcn20forward_rows_appliesElii
    applies.argtypes, applies.restype = [ctypes.c_int64, ctypes.c_int, ctypes.c_int], ctypes.c_bool
    assert applies(n, k, m) == in_lds
    gen = torch.Generator(device="cuda").manual_seed(n + k)
    z = padded(n, k, torch.float32, gen)
    w = torch.randn(k, (m + 3) // 4 * 4 + 4, device="cuda", generator=gen)[:, :m]
    want = chain(z[:, :k], w)
    for op, ref in ((mg.OP_FWD, want), (mg.OP_FWD_RELU, want.clamp(min=0))):
        out = padded(n, m, torch.float32, gen)
        mg.update(op, z[:, :k], w, out[:, :m], n, k, m)
        assert torch.equal(out[:, :m], ref) and out[:, m:].isnan().all()


# rows: one, around a tile and a workgroup's rows; depths: below, at and past a step; columns: around every tile width
SHAPES = [(1, 1, 1), (31, 3, 16), (32, 32, 17), (33, 31, 33), (255, 33, 64), (257, 64, 65), (64, 160, 128),
          (100, 161, 129), (300, 256, 127), (290, 257, 100), (520, 320, 47), (45, 602, 41), (8200, 16, 96),
          (129, 1027, 130)]
# the deepest products whose weights stay in LDS and the next deeper ones, for every tile width: fp32 192, 416, 832 and
# 1696 indices of 128, 64, 32 and 16 columns (data gradient), bf16 320, 640, 1280 and 2560 (both)
SHAPES += [(150, k, m + d) for k, m in ((128, 192), (50, 416), (20, 832), (9, 1696), (100, 320), (60, 640), (20, 1280),
                                        (10, 2560)) for d in (0, 1)]
SHAPES += [(150, k + d, m) for k, m in ((320, 100), (640, 60), (1280, 20), (2560, 10)) for d in (0, 1)]
# more column tiles than compute units of an XCD: several rounds of workgroups
SHAPES += [(20000, 32, 4130), (20000, 4130, 32)]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n,k,m", SHAPES)
def test_row_products_element_by_element(mg, dtype, n, k, m):
    gen = torch.Generator(device="cuda").manual_seed(n + k + m)
    z, g, h = padded(n, k, dtype, gen), padded(n, m, dtype, gen), padded(n, m, dtype, gen)
    w = torch.randn(k, (m + 3) // 4 * 4 + 4, device="cuda", generator=gen)[:, :m]
    step = 32 if dtype == torch.float32 else 64
    out = torch.full_like(g, 7.0)
    mg.update(mg.OP_FWD, z[:, :k], w, out[:, :m], n, k, m)
    check(out[:, :m], z[:, :k], w, dtype, -(-k // step), "forward")
    plain = out.clone()
    mg.update(mg.OP_FWD_RELU, z[:, :k], w, out[:, :m], n, k, m)
    assert torch.equal(out[:, :m], plain[:, :m].clamp(min=0)) and (out[:, m:] == 7.0).all()
    for ref in (None, h[:, :m]):
        dz = torch.full_like(z, 7.0)
        mg.update(mg.OP_DGRAD, g[:, :m], w, dz[:, :k], n, k, m, relu_ref=ref)
        dp = g[:, :m] if ref is None else torch.where(ref > 0, g[:, :m], torch.zeros_like(g[:, :m]))
        check(dz[:, :k], dp, w.t(), dtype, -(-m // step), "data gradient")
        assert (dz[:, k:] == 7.0).all()


@pytest.mark.parametrize("k,m", [(64, 128), (300, 40)])
def test_fp32_values_that_are_not_finite(mg, k, m):
    """An infinity, NaN and a value whose first term rounds to infinity reach the same outputs as in a
    product of plain floats, and the finite rows around them keep their accuracy."""
    n = 200
    gen = torch.Generator(device="cuda").manual_seed(k)
    z = torch.randn(n, k, device="cuda", generator=gen)
    w = torch.randn(k, m, device="cuda", generator=gen)
    w[1] = 0.5
    z[3, 5], z[40, 2], z[70, 1], z[71, 1] = float("inf"), float("nan"), 3.4e38, -3.4e38
    out = torch.empty(n, m, device="cuda")
    mg.update(mg.OP_FWD, z, w, out, n, k, m)
    ref = (z.double() @ w.double()).float()
    assert torch.equal(out.isnan(), ref.isnan()) and torch.equal(out.isposinf(), ref.isposinf())
    assert torch.equal(out.isneginf(), ref.isneginf())
    rest = torch.ones(n, dtype=torch.bool, device="cuda")
    rest[[3, 40, 70, 71]] = False
    check(out[rest], z[rest], w, torch.float32, k, "finite rows")
    assert (out[70] - ref[70]).abs().max() <= 1e-6 * ref[70].abs().max()
    w[2, 0] = float("inf")
    z = torch.rand(n, k, device="cuda", generator=gen) + 0.5
    mg.update(mg.OP_FWD, z, w, out, n, k, m)
    assert out[:, 0].isposinf().all() and not out[:, 1:].isinf().any() and not out.isnan().any()


@pytest.mark.parametrize("product", ["forward of three terms", "data gradient"])
@pytest.mark.parametrize("k,m", [(64, 128), (304, 72)])
def test_fp32_values_that_are_not_finite_in_three_terms(mg, k, m, product):
    """As above in the products that split their operands, and the activation of what is not finite."""
    n = 200
    gen = torch.Generator(device="cuda").manual_seed(k)
    z = torch.randn(n, k, device="cuda", generator=gen)
    w = torch.randn(k, m, device="cuda", generator=gen)

    def run(op):
        out = torch.empty(n, m, device="cuda")
        if product == "data gradient":
            mg.update(mg.OP_DGRAD, z, w.t().contiguous(), out, n, m, k)
            return out
        mg.set_update_arith(mg.ARITH_BF16X3)
        try:
            mg.update(op, z, w, out, n, k, m)
        finally:
            mg.set_update_arith(mg.ARITH_FP32)
        return out

    w[1] = 0.5
    z[3, 5], z[40, 2], z[70, 1], z[71, 1] = float("inf"), float("nan"), 3.4e38, -3.4e38
    out = run(mg.OP_FWD)
    ref = (z.double() @ w.double()).float()
    assert torch.equal(out.isnan(), ref.isnan()) and torch.equal(out.isposinf(), ref.isposinf())
    assert torch.equal(out.isneginf(), ref.isneginf())
    rest = torch.ones(n, dtype=torch.bool, device="cuda")
    rest[[3, 40, 70, 71]] = False
    check(out[rest], z[rest], w, torch.float32, k, "finite rows")
    assert (out[70] - ref[70]).abs().max() <= 1e-6 * ref[70].abs().max()
    if product != "data gradient":  # the activation of NaN is 0
        active = run(mg.OP_FWD_RELU)
        assert torch.equal(active, torch.where(out > 0, out, torch.zeros_like(out)))
    w[2, 0] = float("inf")
    z = torch.rand(n, k, device="cuda", generator=gen) + 0.5
    out = run(mg.OP_FWD)
    assert out[:, 0].isposinf().all() and not out[:, 1:].isinf().any() and not out.isnan().any()


@pytest.mark.parametrize("values", ["normal", "half zero", "positive"])
@pytest.mark.parametrize("depth", [1, 2, 3, 4, 8, 16, 32, 128, 1024])
def test_fp32_gradients_are_no_further_from_64_bits_than_the_chain(mg, depth, values):
    """2-norm over 4096 x 100 results of the data gradient and 100 x 100 of the weight gradient; the two errors
    are the same number of roundings at depth 4 with half of the values zero (5 % for the sample)."""
    gen = torch.Generator(device="cuda").manual_seed(depth)
    rows, cols = 4096, 100
    g = torch.randn(rows, depth, device="cuda", generator=gen)
    w = torch.randn(depth, cols, device="cuda", generator=gen) * 0.1
    if values == "half zero":
        g.clamp_(min=0)
    elif values == "positive":
        g.abs_(), w.abs_()

    def aligned(t):
        out = torch.zeros(t.shape[0], (t.shape[1] + 3) // 4 * 4, device="cuda")
        out[:, :t.shape[1]] = t
        return out[:, :t.shape[1]]

    def error(x, a, b):
        ref = a.double() @ b.double()
        return ((x.double() - ref).norm() / ref.norm()).item()

    dz = torch.empty(rows, cols, device="cuda")
    mg.update(mg.OP_DGRAD, aligned(g), aligned(w.t()), dz, rows, cols, depth)
    assert error(dz, g, w) <= 1.05 * error(chain(g, w), g, w)
    a = g[:cols].contiguous()  # as [cols x depth]: features of `depth` nodes, transposed
    dw = torch.empty(cols, cols, device="cuda")
    mg.update(mg.OP_WGRAD, aligned(a.t()), aligned(w), dw, depth, cols, cols)
    assert error(dw, a, w) <= 1.05 * error(chain(a, w), a, w)


@pytest.mark.parametrize("size", [1e-33, 1e-35, 1e-37, 1e-39, 1e20, 1e30, 1e35])
@pytest.mark.parametrize("depth", [4, 33, 200])
def test_fp32_gradients_keep_their_accuracy_at_every_magnitude(mg, depth, size):
    """The smallest bf16 is 2^-133: terms of a float below 1e-33 end above its last bits, unless it is scaled.
    Subnormal operands and results, a small operand next to a large one, and sums that a scaling carries past
    the largest float; error as above."""
    gen = torch.Generator(device="cuda").manual_seed(depth)
    rows, cols = 1000, 100
    g = torch.randn(rows, depth, device="cuda", generator=gen) * size
    w = torch.randn(depth, (cols + 3) // 4 * 4, device="cuda", generator=gen) * 0.1

    def aligned(t):
        out = torch.zeros(t.shape[0], (t.shape[1] + 3) // 4 * 4, device="cuda")
        out[:, :t.shape[1]] = t
        return out[:, :t.shape[1]]

    def error(x, a, b):
        ref = a.double() @ b.double()
        return ((x.double() - ref).norm() / ref.norm()).item()

    for a, b in ((g, w), (g * 1e10, w * 1e-10) if size < 1 else (g * 1e-10, w * 1e10)):
        dz = torch.empty(rows, cols, device="cuda")
        mg.update(mg.OP_DGRAD, aligned(a), aligned(b.t()), dz, rows, cols, depth)
        assert error(dz, a, b) <= 1.05 * error(chain(a, b), a, b)
        z = a[:cols].contiguous()
        dw = torch.empty(cols, cols, device="cuda")
        mg.update(mg.OP_WGRAD, aligned(z.t()), aligned(b), dw, depth, cols, cols)
        assert error(dw, z, b) <= 1.05 * error(chain(z, b), z, b)


@pytest.mark.parametrize("n,k,m", [(1, 1, 1), (1000, 3, 2), (777, 64, 3), (333, 129, 1), (2048, 256, 2), (50, 602, 3),
                                   (40, 1100, 2), (2200003, 1, 3)])
def test_fp32_data_gradient_of_few_columns_is_the_fp32_chain(mg, n, k, m):
    gen = torch.Generator(device="cuda").manual_seed(n + k)
    g, h = (padded(n, m, torch.float32, gen) for _ in range(2))
    w = padded(k, m, torch.float32, gen)[:, :m]
    g[n // 2, 0], h[n // 3, 0] = float("inf"), float("nan")
    for ref in (None, h[:, :m]):
        dz = padded(n, k, torch.float32, gen)
        mg.update(mg.OP_DGRAD, g[:, :m], w, dz[:, :k], n, k, m, relu_ref=ref)
        dp = g[:, :m] if ref is None else torch.where(ref > 0, g[:, :m], torch.zeros_like(g[:, :m]))
        want = chain(dp, w.t())
        assert torch.equal(dz[:, :k].nan_to_num(7.0), want.nan_to_num(7.0)) and dz[:, k:].isnan().all()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("k,m", [(64, 128), (128, 40), (256, 128), (330, 130)])
def test_values_that_are_not_finite_stay_in_their_rows(mg, dtype, k, m):
    """With more rows than the chip walks at a time: what is not finite in a few of the first rows must not
    change a bit of any other row, of the same tile or of the next one of the same wavefront."""
    n, bad = 200000, [0, 5, 37, 70]
    gen = torch.Generator(device="cuda").manual_seed(k + m)
    z, g = (padded(n, c, dtype, gen) for c in (k, m))
    w = torch.randn(k, (m + 3) // 4 * 4, device="cuda", generator=gen)[:, :m]
    other = torch.ones(n, dtype=torch.bool, device="cuda")
    other[bad] = False
    for op, x, cols in ((mg.OP_FWD, z, m), (mg.OP_FWD_RELU, z, m), (mg.OP_DGRAD, g, k)):
        runs = []
        for _ in range(2):
            out = torch.empty(n, (cols + 7) // 8 * 8, device="cuda", dtype=dtype)[:, :cols]
            mg.update(op, x[:, :k] if op != mg.OP_DGRAD else x[:, :m], w, out, n, k, m)
            runs.append(out)
            x[bad[0], 0], x[bad[1], 1], x[bad[2], 2], x[bad[3], 3] = float("inf"), float("nan"), -float("inf"), 3e38
            x[bad[3], 4] = 3e38
        assert torch.equal(runs[0][other], runs[1][other]), op
        assert op == mg.OP_FWD_RELU or not runs[1][bad[:3]].isfinite().any()


# rows: one, around a step of 16 and around slabs; columns of both operands around the tiles of 32, 64 and 128
WGRAD_SHAPES = [(1, 1, 1), (15, 3, 32), (16, 33, 33), (17, 127, 64), (130, 129, 65), (1000, 100, 127),
                (2063, 128, 128), (4096, 64, 32), (3001, 602, 41), (777, 257, 130), (40000, 16, 300)]


@pytest.mark.parametrize("n,k,m", WGRAD_SHAPES)
def test_fp32_weight_gradient_element_by_element(mg, n, k, m):
    """A dropped term and six roundings of a step's partial sum per product (as above, MFMAs that truncate
    counted twice), one rounding of the running sum per step of a slab, slabs added in 64 bits, and the
    rounding of the result."""
    gen = torch.Generator(device="cuda").manual_seed(n + k + m)
    z, g, h = (padded(n, c, torch.float32, gen) for c in (k, m, m))
    for ref in (None, h[:, :m]):
        for beta in (0.0, 1.0):
            dw = torch.full((k, (m + 3) // 4 * 4 + 4), 3.0, device="cuda")
            mg.update(mg.OP_WGRAD, z[:, :k], g[:, :m], dw[:, :m], n, k, m, relu_ref=ref, beta=beta)
            dp = g[:, :m] if ref is None else torch.where(ref > 0, g[:, :m], torch.zeros_like(g[:, :m]))
            want = z[:, :k].double().t() @ dp.double() + 3.0 * beta
            mag = z[:, :k].double().abs().t() @ dp.double().abs()
            steps = -(-min(n, 1024) // 16)
            bad = (dw[:, :m].double() - want).abs() > (mag + 3.0) * (26 + steps) * 2.0 ** -24
            assert not bad.any() and (dw[:, m:] == 3.0).all(), (int(bad.sum()), beta)


def test_fp32_weight_gradient_keeps_its_accuracy_over_many_rows(mg):
    """What the matrix cores lose by truncation does not add up over the rows: normal inputs, relative error
    below 64 roundings of 2^-25 added as a random walk (64 steps in a slab) with room for the partial sums;
    a drift of the truncation would give 2e-6 here."""
    n, k, m = 1 << 19, 128, 128
    gen = torch.Generator(device="cuda").manual_seed(2)
    z, g = (torch.randn(n, c, device="cuda", generator=gen) for c in (k, m))
    dw = torch.empty(k, m, device="cuda")
    mg.update(mg.OP_WGRAD, z, g, dw, n, k, m)
    ref = z.double().t() @ g.double()
    assert (dw.double() - ref).norm() <= 8 * 2.0 ** -24 * ref.norm()


@pytest.mark.parametrize("m", [128, 40, 16])
def test_fp32_weight_gradient_of_values_that_are_not_finite(mg, m):
    n, k = 1100, 200
    gen = torch.Generator(device="cuda").manual_seed(m)
    z = torch.rand(n, k, device="cuda", generator=gen) + 0.5
    g = torch.rand(n, m, device="cuda", generator=gen) * 0.25 + 0.25
    z[3, 5], z[40, 20], z[70, 140], z[1099, 150] = float("inf"), float("nan"), 3.4e38, -float("inf")
    dw = torch.empty(k, m, device="cuda")
    mg.update(mg.OP_WGRAD, z, g, dw, n, k, m)
    ref = (z.double().t() @ g.double()).float()
    assert torch.equal(dw.isnan(), ref.isnan()) and torch.equal(dw.isposinf(), ref.isposinf())
    assert torch.equal(dw.isneginf(), ref.isneginf())
    fin = ref.isfinite()
    assert ((dw - ref)[fin].abs() <= 1e-5 * ref[fin].abs()).all()
    # the ReLU derivative takes an infinity of the gradient out
    h = torch.ones(n, m, device="cuda")
    h[7], g[7] = -1.0, float("inf")
    mg.update(mg.OP_WGRAD, z[:, :4], g, dw[:4], n, 4, m, relu_ref=h)
    assert dw[:4].isfinite().all()


def test_fp32_weight_gradient_of_a_pitch_past_32_bit_offsets(mg):
    n, k, m, pitch = 19, 70, 40, 1 << 22
    gen = torch.Generator(device="cuda").manual_seed(5)
    z = torch.empty(n * pitch, device="cuda").view(n, pitch)[:, :k]
    z.copy_(torch.randn(n, k, device="cuda", generator=gen))
    g, h = (torch.randn(n, m, device="cuda", generator=gen) for _ in range(2))
    dw = torch.empty(k, m, device="cuda")
    mg.update(mg.OP_WGRAD, z, g, dw, n, k, m, relu_ref=h)
    check(dw, z.t(), torch.where(h > 0, g, torch.zeros_like(g)), torch.float32, n, "weight gradient")


@pytest.mark.parametrize("n,k,m,far", [(19, 70, 40, "zgh"), (33, 130, 20, "z"), (16, 20, 100, "g"), (50, 33, 129, "h"),
                                       (17, 40, 65, "gh"), (2, 5, 3, "zgh")])
def test_fp32_weight_gradient_does_not_depend_on_the_pitch(mg, n, k, m, far):
    """From 2^22 elements on rows are addressed with 64 bits: the same bits for every operand that is so far
    apart, with what is not finite, and zeros for the rows past the last step."""
    gen = torch.Generator(device="cuda").manual_seed(n)
    for bad in (False, True):
        near, wide = {}, {}
        for name, cols in (("z", k), ("g", m), ("h", m)):
            t = padded(n, cols, torch.float32, gen)[:, :cols]
            if bad and name != "h":
                t[n // 2, 0] = float("inf")
            near[name] = wide[name] = t
            if name in far:
                wide[name] = torch.empty(n * ((1 << 22) + 4), device="cuda").view(n, -1)[:, :cols]
                wide[name].copy_(t)
        for ref in (False, True):
            dw = [torch.empty(k, (m + 3) // 4 * 4, device="cuda")[:, :m] for _ in range(2)]
            for d, x in zip(dw, (near, wide)):
                mg.update(mg.OP_WGRAD, x["z"], x["g"], d, n, k, m, relu_ref=x["h"] if ref else None)
            assert torch.equal(dw[0].view(torch.int32), dw[1].view(torch.int32)), (bad, ref)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n,k,m", [(300, 40, 72), (300, 128, 256), (140, 130, 700), (300, 20, 24)])
def test_the_relu_derivative_of_nan_is_zero(mg, dtype, n, k, m):
    """1[R > 0] in every path of a masked product, next to both infinities and both zeros."""
    gen = torch.Generator(device="cuda").manual_seed(n + k + m)
    z, g, h = (padded(n, c, dtype, gen) for c in (k, m, m))
    w = torch.randn(k, m, device="cuda", generator=gen)
    special = torch.tensor([float("nan"), float("inf"), -float("inf"), 0.0, -0.0, 1e-38], device="cuda", dtype=dtype)
    at = torch.randint(0, 24, (n, m), device="cuda", generator=gen)
    h[:, :m] = torch.where(at < 6, special[at.clamp(max=5)], h[:, :m])
    if dtype == torch.bfloat16:  # a NaN of every sign and payload
        h[:, :m].view(torch.int16)[at == 6] = 0x7F81
        h[:, :m].view(torch.int16)[at == 7] = -1
    plain = torch.where(h > 0, 1.0, -1.0).to(dtype)
    out = []
    for ref in (h[:, :m], plain[:, :m]):
        dz, dw = padded(n, k, dtype, gen), torch.empty(k, m, device="cuda")
        mg.update(mg.OP_DGRAD, g[:, :m], w, dz[:, :k], n, k, m, relu_ref=ref)
        mg.update(mg.OP_WGRAD, z[:, :k], g[:, :m], dw, n, k, m, relu_ref=ref)
        out.append((dz[:, :k], dw))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


# layers whose backward pass hands the ReLU derivative on as bits: rows that fill no step or slab, several column and row
# tiles of the weight gradient, widths that are no multiple of 4 or 32, memory that dH shares; and layers that read the
# derivative twice
BITS = [(1, 128, 512, "nothing"), (31, 100, 640, "nothing"), (2500, 128, 1024, "nothing"), (700, 32, 512, "nothing"),
        (1000, 256, 512, "nothing"), (65537, 256, 259, "nothing"), (65600, 384, 601, "nothing"),
        (1000, 256, 512, "dH over Hout"), (1000, 512, 512, "dH over G"), (1000, 256, 512, "columns beside Z"),
        (1000, 384, 512, "columns beside G"), (1000, 256, 640, "columns beside Hout"),
        (700, 32, 512, "columns beside Hout")]
NO_BITS = [(31, 132, 601, "nothing"), (1000, 256, 256, "nothing"), (5000, 300, 259, "nothing"),
           (2500, 128, 1030, "nothing"), (700, 20, 512, "nothing"), (700, 32, 513, "nothing"), (3000, 128, 128, "nothing"),
           (1000, 256, 256, "dH over G"), (1000, 256, 256, "dH over Hout"), (3000, 128, 128, "dH over G"),
           (1000, 300, 256, "columns beside G")]


@pytest.mark.parametrize("n,k,m,share,bits", [(*c, True) for c in BITS] + [(*c, False) for c in NO_BITS])
@pytest.mark.parametrize("streams", [1, 2])
def test_layer_backward_is_its_two_products_and_the_aggregation(mg, n, k, m, share, bits, streams):
    pay = mg.load_library()._ZN6mixgcn13relu_bits_payElii
    pay.argtypes, pay.restype = [ctypes.c_int64, ctypes.c_int, ctypes.c_int], ctypes.c_bool
    assert pay(n, k, m) == bits
    gen = torch.Generator(device="cuda").manual_seed(n + k + m)
    ends = [torch.randint(0, n, (3 * n,), device="cuda", dtype=torch.int32, generator=gen) for _ in range(2)]
    g = mg.build_csr(*ends, n)
    mg.normalize(g)

    def features(cols, *names):
        """A buffer of its own, or one with the columns of dH before them (the pitch of G is that of Hout)."""
        extra = (k + 3) // 4 * 4 if share in [f"columns beside {x}" for x in names] else 0
        t = padded(n, extra + cols, torch.float32, gen)
        return t[:, extra:], t[:, :extra]

    (z, by_z), (hout, by_hout), (grad, by_g) = features(k, "Z"), features(m, "Hout", "G"), features(m, "Hout", "G")
    hout[:, :m].clamp_(min=0)
    hout[0, 0], hout[-1, m - 1] = float("nan"), float("inf")
    w = torch.randn(k, (m + 3) // 4 * 4, device="cuda", generator=gen)[:, :m]
    dw, want_dw = torch.empty_strided(w.shape, w.stride(), device="cuda"), torch.empty_strided(w.shape, w.stride(), device="cuda")
    want_z, want_dh = z.clone(), torch.full((n, (k + 3) // 4 * 4), 7.0, device="cuda")
    mg.update(mg.OP_WGRAD, z[:, :k], grad[:, :m], want_dw, n, k, m, relu_ref=hout[:, :m])
    mg.update(mg.OP_DGRAD, grad[:, :m], w, want_z[:, :k], n, k, m, relu_ref=hout[:, :m])
    mg.aggregate(g, want_z[:, :k], want_dh[:, :k], transpose=True)
    dh = {"nothing": torch.full_like(z, 7.0), "dH over G": grad, "dH over Hout": hout, "columns beside Z": by_z,
          "columns beside Hout": by_hout, "columns beside G": by_g}[share]
    past = dh[:, k:].clone()
    side = (torch.cuda.Stream(), torch.cuda.Stream())
    pipe = mg.Pipeline() if streams == 1 else mg.Pipeline(*side)
    torch.cuda.synchronize()
    mg.layer_bwd(g, z[:, :k], hout[:, :m], w, grad[:, :m], dw, dh[:, :k], pipe, relu=True, n_chunks=streams)
    torch.cuda.synchronize()
    same = lambda a, b: torch.equal(a.contiguous().view(torch.int32), b.contiguous().view(torch.int32))
    assert same(dw, want_dw) and same(z[:, :k], want_z[:, :k]) and same(dh[:, :k], want_dh[:, :k])
    assert same(dh[:, k:], past)
    g.free()


@pytest.mark.parametrize("k,m", [(128, 128), (100, 50), (130, 20), (300, 200)])
@pytest.mark.parametrize("n", [1, 31, 32, 33, 2079, 40001])
def test_bf16_weight_gradient_of_any_number_of_rows(mg, n, k, m):
    """The last n % 32 rows are a slab of their own; what lies past the rows and the columns is NaN.  Element by
    element: products of bf16 are exact in fp32, a slab adds at most 2048 rows in MFMAs of 16 (their sums lose less than
    2^-23 of the running sum each), the slabs are added in 64 bits and rounded once."""
    gen = torch.Generator(device="cuda").manual_seed(n + k + m)
    a, g, h = (padded(n + 40, c, torch.bfloat16, gen) for c in (k, m, m))
    for t in (a, g, h):
        t[n:] = float("nan")
    a, g, h = a[:n, :k], g[:n, :m], h[:n, :m]
    dw = torch.empty(k, (m + 3) // 4 * 4, device="cuda")[:, :m]
    for ref in (None, h):
        dp = g if ref is None else torch.where(ref > 0, g, torch.zeros_like(g))
        want, mag = a.double().t() @ dp.double(), a.double().abs().t() @ dp.double().abs()
        bound = mag * (2048 / 16 + 2) * 2.0 ** -23
        for beta in (0.0, 1.0):
            mg.update(mg.OP_WGRAD, a, g, dw, n, k, m, relu_ref=ref, beta=beta)
            assert ((dw.double() - (1 + beta) * want).abs() <= (1 + 2 * beta) * bound + 1e-30).all()


@pytest.mark.parametrize("n,k", [(5000, 128), (20003, 100), (300, 32), (5000, 48), (20003, 64), (8192, 64), (300, 33)])
def test_fp32_forward_written_over_its_features(mg, n, k):
    """Up to 128 columns a row's features are all read before its sums are written, whatever the number of rows."""
    gen = torch.Generator(device="cuda").manual_seed(n)
    z = padded(n, k, torch.float32, gen)
    w = torch.randn(k, (k + 3) // 4 * 4, device="cuda", generator=gen)[:, :k]
    out = padded(n, k, torch.float32, gen)
    mg.update(mg.OP_FWD_RELU, z[:, :k], w, out[:, :k], n, k, k)
    mg.update(mg.OP_FWD_RELU, z[:, :k], w, z[:, :k], n, k, k)
    assert torch.equal(z[:, :k], out[:, :k])


@pytest.mark.parametrize("n,k,m", [(5000, 128, 64), (20003, 100, 256), (300, 37, 47), (8192, 64, 32)])
@pytest.mark.parametrize("left", [False, True])
def test_fp32_forward_into_other_columns_of_its_buffer(mg, n, k, m, left):
    gen = torch.Generator(device="cuda").manual_seed(n)
    wide = [(c + 3) // 4 * 4 for c in (k, m)]
    both = torch.randn(n, sum(wide), device="cuda", generator=gen)
    z, c = (both[:, wide[1]:][:, :k], both[:, :m]) if left else (both[:, :k], both[:, wide[0]:][:, :m])
    w = torch.randn(k, wide[1], device="cuda", generator=gen)[:, :m]
    out, before = padded(n, m, torch.float32, gen), z.clone()
    mg.update(mg.OP_FWD, z, w, out[:, :m], n, k, m)
    mg.update(mg.OP_FWD, z, w, c, n, k, m)
    assert torch.equal(c, out[:, :m]) and torch.equal(z, before)
