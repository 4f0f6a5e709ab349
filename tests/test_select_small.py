"""The selector on problems too small to pay for the prefill kernels' launches and
pipelines, the XOR route's choice between its two kernels, and the range of the
tall tiles.  The model runs on
the host; the problems and the kernel each belongs on were measured on MI355X with
cold weights (the faster kernel by 20% or more)."""
import ctypes

import pytest

import paper_2508_19087_amd as apt


def few_token(M, N, K, p, q, unpacked=False):
    """Whether the XOR route with its launch shape open runs the few-token GEMM."""
    f = apt.lib().apt_test_few_token
    f.restype = ctypes.c_int
    return f(M, N, K, p, q, int(unpacked)) == 1


# microseconds: XOR + popcount, and the kernel a fixed part too small sent them to
@pytest.mark.parametrize("M,N,K,p,q", [
    (13, 256, 256, 2, 2),     # 2.6, 8.8
    (35, 1408, 640, 2, 4),    # 5.8, 9.9
    (148, 256, 750, 1, 2),    # 5.0, 14.4
    (106, 239, 165, 4, 2),    # 4.1, 17.9
    (207, 175, 838, 3, 4),    # 4.8, 15.4
    (263, 167, 508, 4, 1),    # 5.3, 20.2
    (55, 721, 256, 2, 2),     # 4.7, 6.6
    (52, 640, 256, 5, 3),     # 4.6, 6.4
    (37, 896, 384, 1, 1)])    # 4.5, 6.4
def test_small_problems_stay_on_xor(M, N, K, p, q):
    assert apt.select_config(M, N, K, p, q).route == apt.APT_ROUTE_XOR
    assert not few_token(M, N, K, p, q)


@pytest.mark.parametrize("M,N,K,p,q", [
    (749, 1408, 384, 4, 4),   # 12.9 on 128 x 128 tiles, 15.9
    (614, 2560, 256, 3, 3)])
def test_short_k_stays_on_small_tiles(M, N, K, p, q):
    c = apt.select_config(M, N, K, p, q)
    assert (c.route, c.bm, c.bn) == (apt.APT_ROUTE_INT8_MFMA, 128, 128)


@pytest.mark.parametrize("M,N,K,p,q", [
    (64, 11008, 4096, 4, 4), (64, 4096, 1024, 4, 4), (12, 254, 6784, 8, 8), (51, 161, 4480, 8, 4), (16, 256, 6961, 6, 6),
    (400, 1024, 8192, 4, 8)])  # 16.4, 31.0 on 128 x 128 tiles
def test_few_tokens_take_the_few_token_kernel(M, N, K, p, q):
    assert apt.select_config(M, N, K, p, q).route == apt.APT_ROUTE_XOR
    assert few_token(M, N, K, p, q)


@pytest.mark.parametrize("M,N,K,p,q", [(2048, 11008, 4096, 4, 4), (1024, 11008, 4096, 2, 2), (1024, 4096, 11008, 2, 4),
                                       (2048, 4096, 4096, 4, 4)])
def test_prefill_keeps_the_six_bit_kernel(M, N, K, p, q):
    c = apt.select_config(M, N, K, p, q)
    assert (c.route, c.bm, c.bn, c.waves_m, c.waves_n) == (apt.APT_ROUTE_INT8_MFMA, 256, 128, 4, 1)


def test_tall_tiles_only_in_a_partly_filled_round():
    """512 x 128 tiles at 8 bits up to three quarters of the compute units (192 tiles
    here); at 248 the 256 x 128 tiles are 5% faster."""
    c = apt.select_config(1024, 12288, 4096, 8, 8)
    assert (c.bm, c.bn) == (512, 128)
    for s in ((1643, 7936, 5504, 7, 7), (1608, 7936, 9600, 7, 8)):
        c = apt.select_config(*s)
        assert (c.bm, c.bn) == (256, 128)


@pytest.mark.parametrize("p,q,last", [(5, 5, 8192), (6, 6, 8192), (8, 8, 8192), (8, 4, 8192), (4, 8, 12288), (2, 8, 12288),
                                      (4, 4, 16384)])
def test_last_k_of_the_few_token_kernel(p, q, last):
    """Its operands are held for all of K: past the last K that the registers hold, a
    call of few tokens runs XOR + popcount."""
    for unpacked in (False, True):
        assert few_token(8, 4096, last, p, q, unpacked)
        assert not few_token(8, 4096, last + 1, p, q, unpacked)
