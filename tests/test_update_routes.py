"""Host side of the update products: which forward products of fp32 features take the kernel with the weights in LDS, and
launches that fail."""
import ctypes

import pytest
import torch

import paper_2501_01951_amd as mg


@pytest.fixture(scope="module")
def in_lds():
    f = mg.load_library()._ZN6mixgcn20forward_rows_appliesElii  # mixgcn::forward_rows_applies(n, k, m)
    f.argtypes, f.restype = [ctypes.c_int64, ctypes.c_int, ctypes.c_int], ctypes.c_bool
    return f


# (rows, depth, columns) at which the tiles of the general kernel measured 5 to 40 % faster: shallow depths, a last step
# mostly of zeros, a last tile that few wavefronts have, no tile of the general kernel at an edge, workgroups that do not
# fit the chip at once, column tiles that leave compute units idle
@pytest.mark.parametrize("n,k,m", [
    (33_000, 16, 32), (100_000, 47, 24), (66_000, 80, 8), (135_000, 256, 16), (400_000, 256, 4), (1_500_000, 64, 32),
    (33_000, 128, 32), (4_096, 64, 32), (16_384, 256, 64), (25_600, 256, 128), (12_032, 96, 256), (270_000, 200, 47),
    (5_000, 256, 602), (16_384, 16, 128), (300, 64, 4096), (1_500, 64, 2048), (1_000, 16, 2048), (267_000, 256, 384),
    (100_000, 160, 640), (67_000, 128, 1024)])
def test_sizes_of_the_general_kernel(in_lds, n, k, m):
    assert not in_lds(n, k, m)


@pytest.mark.parametrize("n,k,m", [
    (1, 64, 1), (10_000, 256, 16), (4_096, 256, 16), (20_000, 602, 32), (100_000, 128, 16), (50_000, 256, 32),
    (262_144, 256, 16), (20_000, 256, 64), (12_000, 128, 48), (1 << 20, 256, 47), (300_000, 256, 64), (5_000, 602, 128),
    (20_000, 256, 128), (4_096, 64, 128), (5_000, 16, 128), (1_000, 64, 1500), (16_000, 16, 80), (1 << 18, 128, 256),
    (1 << 20, 256, 256), (1 << 21, 128, 1024)])
def test_sizes_with_the_weights_in_lds(in_lds, n, k, m):
    assert in_lds(n, k, m)


# (rows, input columns, output columns) at which reading the activations twice measured 2 to 6 % faster
@pytest.mark.parametrize("n,k,m", [(20_000, 300, 400), (20_000, 200, 600), (1_000_000, 48, 600), (20_000, 256, 256),
                                   (20_000, 192, 768), (1_000_000, 96, 640), (1_000_000, 128, 600)])
def test_layers_that_read_the_relu_derivative_twice(n, k, m):
    f = mg.load_library()._ZN6mixgcn13relu_bits_payElii  # mixgcn::relu_bits_pay(n, k, m)
    f.argtypes, f.restype = [ctypes.c_int64, ctypes.c_int, ctypes.c_int], ctypes.c_bool
    assert not f(n, k, m) and f(n, 128, 1024)


@pytest.mark.parametrize("dtype", [mg.F32, mg.BF16])
@pytest.mark.parametrize("k,m", [(3, 2), (64, 16), (64, 47), (256, 47), (256, 256), (602, 1024)])
def test_products_without_rows(in_lds, dtype, k, m):
    """Nothing is launched, and nothing divides by the number of tiles."""
    assert not in_lds(0, k, m)
    for op in (mg.OP_FWD, mg.OP_FWD_RELU, mg.OP_DGRAD):
        pitch = 1024
        assert mg.load_library().mixgcn_update(op, dtype, 4096, pitch, 4096, pitch, 4096, pitch, 0, k, m, None, 0,
                                               ctypes.c_float(0), None) == 0


class ReluBits(ctypes.Structure):
    _fields_ = [("p", ctypes.c_void_p), ("pitch", ctypes.c_int64)]


@pytest.mark.skipif(torch.cuda.is_available(), reason="the launches have to fail: no device")
@pytest.mark.parametrize("k,m", [(256, 256), (32, 512), (64, 512)])
@pytest.mark.parametrize("ref,bits", [(None, None), (4096, None), (4096, 4096)])
def test_a_data_gradient_that_is_not_launched_is_an_error(k, m, ref, bits):
    # mixgcn::launch_update_rows(dtype, w_is_kd_major, relu, A, lda, W, ldw, C, ldc, n, KD, MD, R, ldr, s, bits); nothing
    # reads the addresses on the host
    f = mg.load_library()._ZN6mixgcn18launch_update_rowsEibbPKvlPKflPvlliiS1_lP12ihipStream_tNS_8ReluBitsE
    i, l, v, b = ctypes.c_int, ctypes.c_int64, ctypes.c_void_p, ctypes.c_bool
    f.argtypes, f.restype = [i, b, b, v, l, v, l, v, l, l, i, i, v, l, v, ReluBits], i
    assert f(mg.F32, False, False, 4096, m, 4096, m, 4096, k, 32, m, k, ref, m, None, ReluBits(bits, 4 * k)) == -3
