"""GPU parity of the few-token GEMM (gemm_thin.h), which the XOR route runs where
its launch shape is left open and it is the faster kernel: every operand class
and shape built, at the edges of its tiles, K groups and token tiles, from
packed activations, int8 codes and fp16 values.  int32 equals the oracle and
the forced XOR + popcount kernel bit for bit, fp16 lies within the epilogue's
tolerance, fp16 row scales are bit-exact.  Weights of 5 to 8 bits and activations of
more than 4 end at K = 8192 (12288 at up to 4 weight bits): past it the same calls
run XOR + popcount."""
import numpy as np
import pytest

import paper_2508_19087_amd as apt
import synth
from gpu_util import assert_int32_equal, dev
from oracle import oracle as ref
from test_select_small import few_token

pytestmark = pytest.mark.gpu

OPEN = apt.apt_config_t.make(apt.APT_ROUTE_XOR)
XOR = apt.apt_config_t.make(apt.APT_ROUTE_XOR, mt=1, waves_m=4, waves_n=1)


def weights(g, N, K, p):
    codes = synth.uniform_codes(g, N, K, p)
    return codes, apt.pack(dev(codes), p), synth.scales(g, N, *synth.W_SCALE_RANGE)


def check_fp16(c16, C, sa, sw, what):
    E, _ = ref.epilogue(C, sa, sw)
    assert ref.fp16_close(c16.cpu().numpy(), E).all(), what


# most of these take the few-token GEMM (some of those with more than 32 tokens, and
# the byte operands past K = 8192, run XOR + popcount); test_few_tokens_taken has
# token tiles and rows of workgroups that all do
@pytest.mark.parametrize("M,N,K", [
    (8, 4096, 128), (7, 4700, 100), (8, 4097, 513), (5, 6600, 4096), (3, 8191 // 2 * 2 + 2731, 4000),
    (8, 4111, 4097), (8, 4100, 8300), (6, 5500, 12289),        # 2, 3 and 4 K groups per wave
    (16, 2100, 700), (17, 2000, 4096), (33, 1000, 1000), (64, 520, 4100), (70, 500, 300), (130, 260, 2000)])
@pytest.mark.parametrize("p,q", [(1, 1), (2, 4), (4, 4), (3, 2), (5, 7), (8, 8), (4, 8), (8, 3)])
def test_few_tokens_packed(M, N, K, p, q):
    g = synth.rng(110, M, N, K, p, q)
    wc, w, sw = weights(g, N, K, p)
    ac = synth.uniform_codes(g, M, K, q)
    sa = synth.scales(g, M, *synth.A_SCALE_RANGE)
    a = apt.pack(dev(ac), q, activations=True)
    c32, c16 = apt.gemm(a, w, a_scale=dev(sa), w_scale=dev(sw), out_fp16=True, cfg=OPEN)
    x32, _ = apt.gemm(a, w, cfg=XOR)
    what = "%dx%dx%d W%dA%d" % (M, N, K, p, q)
    C = ref.gemm(ac, wc, p, q)
    assert_int32_equal(c32.cpu().numpy(), C, what)
    assert_int32_equal(x32.cpu().numpy(), C, what + " XOR")
    check_fp16(c16, C, sa, sw, what)


@pytest.mark.parametrize("M,N,K", [(8, 4096, 128), (7, 4700, 100), (8, 4100, 4097), (5, 6600, 4096),
                                   (8, 4097, 8320), (6, 5500, 11008), (4, 8190, 16000)])
@pytest.mark.parametrize("p,q", [(1, 1), (2, 4), (4, 4), (3, 2), (5, 7), (8, 8), (4, 8)])
def test_few_tokens_unpacked(M, N, K, p, q):
    g = synth.rng(111, M, N, K, p, q)
    wc, w, sw = weights(g, N, K, p)
    ac = synth.uniform_codes(g, M, K, q)
    sa = synth.scales(g, M, *synth.A_SCALE_RANGE)
    what = "%dx%dx%d W%dA%d" % (M, N, K, p, q)
    c32, c16, _ = apt.gemm_decode(dev(ac), q, w, a_scale=dev(sa), w_scale=dev(sw), out_fp16=True)
    C = ref.gemm(ac, wc, p, q)
    assert_int32_equal(c32.cpu().numpy(), C, what)
    check_fp16(c16, C, sa, sw, what)
    x = synth.fp16_activations(g, M, K)
    x[0, :min(K, 64)] = 0.0
    x[1] = 0.0                                     # scale 0
    x[2] *= np.float16(2.0 ** -14)                 # a subnormal scale: the long quantizer
    x[0, 5:9] = [-0.0, 2.0 ** -24, -2.0 ** -24, -0.0]
    codes, s16 = ref.quantize_fp16(x, q)
    c32, c16, sc = apt.gemm_decode(dev(x), q, w, w_scale=dev(sw), out_fp16=True)
    assert np.array_equal(sc.cpu().numpy().view(np.uint16), s16.view(np.uint16)), what
    C = ref.gemm(codes, wc, p, q)
    assert_int32_equal(c32.cpu().numpy(), C, what + " fp16")
    check_fp16(c16, C, s16, sw, what + " fp16")


@pytest.mark.parametrize("M,N,K", [(9, 4100, 4100), (32, 4100, 700), (33, 6100, 1000), (70, 3100, 300), (130, 1030, 2000),
                                   (512, 300, 1100)])
@pytest.mark.parametrize("p,q", [(2, 4), (4, 4), (5, 7), (8, 8), (4, 8), (8, 3)])
def test_few_tokens_taken(M, N, K, p, q):
    assert few_token(M, N, K, p, q)
    test_few_tokens_packed(M, N, K, p, q)


def taken_unpacked(M, N, K, p, q):
    assert few_token(M, N, K, p, q, unpacked=True)
    test_few_tokens_unpacked(M, N, K, p, q)


@pytest.mark.parametrize("K", [4096, 4000])
@pytest.mark.parametrize("p,q", [(2, 4), (4, 4), (5, 7), (8, 8), (4, 8), (8, 3)])
def test_three_tokens_unpacked(K, p, q):
    """Two waves per row, the last two with none."""
    taken_unpacked(3, 11008, K, p, q)


@pytest.mark.parametrize("N,K,p,q", [(11008, 4096, 2, 4), (11008, 4096, 4, 4), (11008, 4096, 8, 3), (16500, 2999, 4, 4),
                                     (16500, 2999, 4, 8), (16500, 2999, 8, 8), (22016, 4097, 5, 7)])
def test_two_tokens_unpacked(N, K, p, q):
    """Four waves per row."""
    assert few_token(2, N, K, p, q, unpacked=True)
    g = synth.rng(113, N, K, p, q)
    wc, w, sw = weights(g, N, K, p)
    ac, sa = synth.uniform_codes(g, 2, K, q), synth.scales(g, 2, *synth.A_SCALE_RANGE)
    x = synth.fp16_activations(g, 2, K)
    x[1, 3:] = 0.0
    codes, s16 = ref.quantize_fp16(x, q)
    for src, c, s, kw in ((ac, ac, sa, {"a_scale": dev(sa)}), (x, codes, s16, {})):
        what = "2x%dx%d W%dA%d %s" % (N, K, p, q, src.dtype)
        c32, c16, sc = apt.gemm_decode(dev(src), q, w, w_scale=dev(sw), out_fp16=True, **kw)
        C = ref.gemm(c, wc, p, q)
        assert_int32_equal(c32.cpu().numpy(), C, what)
        check_fp16(c16, C, s, sw, what)
        if sc is not None:
            assert np.array_equal(sc.cpu().numpy().view(np.uint16), s16.view(np.uint16)), what


@pytest.mark.parametrize("M", [8, 40])
@pytest.mark.parametrize("p,q", [(2, 4), (8, 8)])
def test_few_tokens_affine(M, p, q):
    prob = synth.affine_problem("few", M, 4200, 1000, p, q, synth.rng(112, M, p, q))
    a = apt.pack(dev(prob.a_codes), q, activations=True)
    w = apt.pack(dev(prob.w_codes), p)
    z = [dev(v) for v in (prob.a_scale, prob.a_zero, prob.w_scale, prob.w_zero)]
    f, c = apt.gemm_affine(a, w, *z, out_int32=True, cfg=OPEN)
    fx, cx = apt.gemm_affine(a, w, *z, out_int32=True, cfg=XOR)
    assert_int32_equal(c.cpu().numpy(), ref.gemm(prob.a_codes, prob.w_codes, p, q), "affine")
    assert_int32_equal(cx.cpu().numpy(), c.cpu().numpy(), "affine XOR")
    assert np.array_equal(f.cpu().numpy().view(np.uint16), fx.cpu().numpy().view(np.uint16))


def test_few_tokens_extreme_codes():
    """Every product at its largest magnitude, both signs (the largest sums)."""
    for p, q, K in [(4, 4, 16384), (8, 8, 8192), (2, 4, 16384)]:
        for lo_a, lo_w in [(True, True), (False, True), (False, False)]:
            val = lambda lo, b: -(1 << (b - 1)) if lo else (1 << (b - 1)) - 1  # noqa: E731
            ac = np.full((8, K), val(lo_a, q), np.int8)
            wc = np.full((4096, K), val(lo_w, p), np.int8)
            a = apt.pack(dev(ac), q, activations=True)
            c32, _ = apt.gemm(a, apt.pack(dev(wc), p), cfg=OPEN)
            want = K * (2 * val(lo_a, q) + 1) * (2 * val(lo_w, p) + 1)
            assert (c32.cpu().numpy() == want).all(), (p, q, lo_a, lo_w)
            c32, _, _ = apt.gemm_decode(dev(ac), q, apt.pack(dev(wc), p))
            assert (c32.cpu().numpy() == want).all(), (p, q, lo_a, lo_w)
