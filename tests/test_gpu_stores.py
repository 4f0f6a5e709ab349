"""GPU parity of the output stores of the int8 route's kernels (gemm_int8.h and,
at up to 4 bits on the 256 x 128 shape with 4 x 1 waves, gemm_direct.h): blocks of
32 x 32 outputs inside the matrix and across each of its edges, rows that start
16-byte aligned (streamed) and rows that do not, outputs moved off their
allocation's alignment, each output alone and both.  int32 bit-exact, fp16 equal
to the outputs of the aligned call."""
import numpy as np
import pytest

import paper_2508_19087_amd as apt
import synth
from gpu_util import INT8_SHAPES, assert_int32_equal, dev
from oracle import oracle as ref

pytestmark = pytest.mark.gpu

K = 129


def call(a, w, sa, sw, cfg, off32, off16):
    """(int32, fp16) with the outputs `off` elements into their allocations;
    None leaves an output out."""
    import torch
    M, N = a.rows, w.rows
    c32 = torch.full((M * N + 16,), -1, dtype=torch.int32, device="cuda")
    c16 = torch.full((M * N + 16,), -1.0, dtype=torch.float16, device="cuda")
    ws = torch.empty(apt.apt_gemm_workspace_bytes(M, N, K, w.bits, a.bits, cfg), dtype=torch.uint8, device="cuda")
    p32 = None if off32 is None else c32.data_ptr() + 4 * off32
    p16 = None if off16 is None else c16.data_ptr() + 2 * off16
    st = apt.apt_gemm(M, N, K, w.bits, a.bits, a.data.data_ptr(), w.data.data_ptr(), a.rowsum.data_ptr(),
                      w.rowsum.data_ptr(), p32, sa.data_ptr(), sw.data_ptr(), p16, cfg, ws.data_ptr(), ws.numel(),
                      torch.cuda.current_stream().cuda_stream)
    assert st == apt.APT_OK, apt.status_string(st)
    out = []
    for c, off in ((c32, off32), (c16, off16)):
        if off is None:
            out.append(None)
            continue
        c = c.cpu().numpy()
        assert (c[:off] == -1).all() and (c[off + M * N:] == -1).all(), "stores outside the output"
        out.append(c[off:off + M * N].reshape(M, N))
    return out


@pytest.mark.parametrize("M,N", [(32, 32), (31, 36), (33, 64), (64, 33), (95, 131), (160, 260), (257, 290), (300, 519)])
@pytest.mark.parametrize("p,q", [(4, 4), (6, 5)])
def test_output_blocks(M, N, p, q):
    g = synth.rng(130, M, N, p, q)
    wc, ac = synth.uniform_codes(g, N, K, p), synth.uniform_codes(g, M, K, q)
    sw, sa = synth.scales(g, N, *synth.W_SCALE_RANGE), synth.scales(g, M, *synth.A_SCALE_RANGE)
    w, a = apt.pack(dev(wc), p), apt.pack(dev(ac), q, activations=True)
    dsa, dsw = dev(sa), dev(sw)
    C = ref.gemm(ac, wc, p, q)
    E, _ = ref.epilogue(C, sa, sw)
    for bm, bn, wm, wn in INT8_SHAPES:
        cfg = apt.apt_config_t.make(apt.APT_ROUTE_INT8_MFMA, bm, bn, 128, wm, wn, 0, 3)
        first = None
        for off32, off16 in ((0, 0), (0, None), (None, 0), (1, 1), (3, None), (None, 5), (4, 8)):
            what = "%dx%d W%dA%d %dx%d off %s %s" % (M, N, p, q, bm, bn, off32, off16)
            c32, c16 = call(a, w, dsa, dsw, cfg, off32, off16)
            if c32 is not None:
                assert_int32_equal(c32, C, what)
            if c16 is not None:
                assert ref.fp16_close(c16, E).all(), what
                first = c16 if first is None else first
                assert np.array_equal(c16.view(np.uint16), first.view(np.uint16)), what
