"""The row products (forward and data gradient) at the edges of their kernel: 32-row tiles, reduction steps
of 128 bytes of a row, weights that stay in LDS and weights that stream through it, output tiles of 16, 32,
64 and 128 columns; what rows hold past their columns, infinities and NaN."""
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


# rows: one, around a tile and a workgroup's rows; depths: below, at and past a step, the most that keeps
# 128 columns of weights in LDS (fp32 160, bf16 256) and beyond; columns: around every tile width
SHAPES = [(1, 1, 1), (31, 3, 16), (32, 32, 17), (33, 31, 33), (255, 33, 64), (257, 64, 65), (64, 160, 128),
          (100, 161, 129), (300, 256, 127), (290, 257, 100), (520, 320, 47), (45, 602, 41), (8200, 16, 96),
          (129, 1027, 130)]


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
