"""GPU parity of the direct-weight kernel (gemm_direct.h), which the int8 route's
256 x 128 shape with 4 x 1 waves runs on six-bit codes for operands of at most
4 bits: at the edges of its 128 x 256 tiles and chunk pairs, from packed rows,
codes and fp16 values, with every output form.  int32 equals the oracle bit for
bit and fp16 lies within the epilogue's tolerance."""
import numpy as np
import pytest

import paper_2508_19087_amd as apt
import synth
from gpu_util import assert_int32_equal, dev
from oracle import oracle as ref

pytestmark = pytest.mark.gpu

CFG = apt.apt_config_t.make(apt.APT_ROUTE_INT8_MFMA, 256, 128, 128, 4, 1, 0, 3)


@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (127, 255, 128), (128, 256, 256), (129, 257, 257), (33, 70, 640),
                                   (300, 712, 1000), (1100, 520, 385), (260, 1032, 4097)])
@pytest.mark.parametrize("p,q", [(1, 1), (2, 4), (3, 2), (4, 4), (4, 1)])
def test_direct_weights(M, N, K, p, q):
    g = synth.rng(120, M, N, K, p, q)
    wc, ac = synth.uniform_codes(g, N, K, p), synth.uniform_codes(g, M, K, q)
    sw, sa = synth.scales(g, N, *synth.W_SCALE_RANGE), synth.scales(g, M, *synth.A_SCALE_RANGE)
    w, a = apt.pack(dev(wc), p), apt.pack(dev(ac), q, activations=True)
    what = "%dx%dx%d W%dA%d" % (M, N, K, p, q)
    C = ref.gemm(ac, wc, p, q)
    E, _ = ref.epilogue(C, sa, sw)
    both32, both16 = apt.gemm(a, w, a_scale=dev(sa), w_scale=dev(sw), out_fp16=True, cfg=CFG)
    assert_int32_equal(both32.cpu().numpy(), C, what)
    assert ref.fp16_close(both16.cpu().numpy(), E).all(), what
    _, only16 = apt.gemm(a, w, out_int32=False, a_scale=dev(sa), w_scale=dev(sw), out_fp16=True, cfg=CFG)
    assert np.array_equal(only16.cpu().numpy().view(np.uint16), both16.cpu().numpy().view(np.uint16)), what
    c32, _, _ = apt.gemm_act(dev(ac), q, w, cfg=CFG)
    assert_int32_equal(c32.cpu().numpy(), C, what + " codes")
    x = synth.fp16_activations(g, M, K)
    codes, s16 = ref.quantize_fp16(x, q)
    c32, _, sc = apt.gemm_act(dev(x), q, w, cfg=CFG)
    assert_int32_equal(c32.cpu().numpy(), ref.gemm(codes, wc, p, q), what + " fp16")
    assert np.array_equal(sc.cpu().numpy().view(np.uint16), s16.view(np.uint16)), what


@pytest.mark.parametrize("M,N", [(130, 264), (64, 257)])
@pytest.mark.parametrize("p,q", [(2, 4), (4, 3)])
def test_direct_affine(M, N, p, q):
    prob = synth.affine_problem("direct", M, N, 500, p, q, synth.rng(121, M, N, p, q))
    a, w = apt.pack(dev(prob.a_codes), q, activations=True), apt.pack(dev(prob.w_codes), p)
    z = [dev(v) for v in (prob.a_scale, prob.a_zero, prob.w_scale, prob.w_zero)]
    va, vw = ref.values(prob.a_codes, q), ref.values(prob.w_codes, p)
    C = ref.matmul(va, vw)
    E, T = ref.affine_epilogue(C, ref.rowsum(va), ref.rowsum(vw), prob.K, prob.a_scale, prob.a_zero, prob.w_scale,
                               prob.w_zero)
    f1, _ = apt.gemm_affine(a, w, *z, cfg=CFG)
    f2, c = apt.gemm_affine(a, w, *z, out_int32=True, cfg=CFG)
    assert_int32_equal(c.cpu().numpy(), C, "affine")
    for f in (f1, f2):
        assert ref.fp16_affine_close(f.cpu().numpy(), E, T).all()


@pytest.mark.parametrize("p,q,K", [(4, 4, 74565), (2, 4, 372827), (4, 4, 74566)])
def test_direct_exact_at_its_bound(p, q, K):
    """Every product u_a u_w at its largest: the sum stays below 2^24 (the last
    K takes int8 operands instead)."""
    ac = np.full((2, K), (1 << (q - 1)) - 1, np.int8)
    wc = np.full((3, K), (1 << (p - 1)) - 1, np.int8)
    wc[1] = -(1 << (p - 1))
    a, w = apt.pack(dev(ac), q, activations=True), apt.pack(dev(wc), p)
    c32, _ = apt.gemm(a, w, cfg=CFG)
    top = K * ((1 << p) - 1) * ((1 << q) - 1)
    assert (c32.cpu().numpy() == np.array([top, -top, top])).all()


@pytest.mark.parametrize("grid", [0, 512])
def test_direct_stays_inside_its_workspace(grid):
    """The workspace holds the fragments alone, whatever the grid: 2000 x 1300 outputs
    whose tiles a persistent round would share, with guard bytes behind."""
    import torch
    M, N, K, p, q = 2000, 1300, 300, 4, 3
    g = synth.rng(122, M, N)
    wc, ac = synth.uniform_codes(g, N, K, p), synth.uniform_codes(g, M, K, q)
    w, a = apt.pack(dev(wc), p), apt.pack(dev(ac), q, activations=True)
    cfg = apt.apt_config_t.make(apt.APT_ROUTE_INT8_MFMA, 256, 128, 128, 4, 1, grid, 3)
    need = apt.apt_gemm_workspace_bytes(M, N, K, p, q, cfg)
    ws = torch.full((need + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    c32, _ = apt.gemm(a, w, cfg=cfg, workspace=ws[:need])
    assert_int32_equal(c32.cpu().numpy(), ref.gemm(ac, wc, p, q), "direct")
    assert (ws[need:].cpu().numpy() == 0x5A).all()
