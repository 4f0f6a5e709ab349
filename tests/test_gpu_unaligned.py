"""GPU parity where rows start at any byte: K off the 16-element groups (whole
groups are one unaligned load, the group across the row's end takes byte loads)
and N off the four-column stores, with the source moved off its allocation's
alignment, for every kernel that reads rows: the packer, the fragment writer,
the fused GEMV and the few-token GEMM.  int32 bit-exact against the oracle,
fp16 within the epilogue's tolerance, fused and unfused bit-identical."""
import pytest

import paper_2508_19087_amd as apt
from test_gpu_act import check
from test_select_small import few_token

pytestmark = pytest.mark.gpu

INT8 = apt.apt_config_t.make(apt.APT_ROUTE_INT8_MFMA, 256, 128, 128, 4, 1, 0, 0)
OPEN_XOR = apt.apt_config_t.make(apt.APT_ROUTE_XOR, 0, 0, 0, 0, 0, 0, 0)


@pytest.mark.parametrize("K", [1, 15, 16, 17, 31, 33, 47, 129, 1039, 2999])
@pytest.mark.parametrize("fp16_src", [False, True])
def test_rows_at_any_byte(K, fp16_src):
    for M, N, cfg in ((1, 37, OPEN_XOR), (3, 65, OPEN_XOR), (37, 131, INT8)):
        for p, q in ((2, 4), (3, 8)):
            for offset in (0, 1, 5):
                check(M, N, K, p, q, cfg=cfg, fp16_src=fp16_src, offset=offset, seed=7,
                      what="%dx%d" % (M, N))


@pytest.mark.parametrize("K", [1, 15, 16, 17, 31, 33, 47, 129, 1039, 2999])
@pytest.mark.parametrize("fp16_src", [False, True])
def test_few_token_rows_at_any_byte(K, fp16_src):
    """The few-token GEMM, which none of the sizes above reaches."""
    for p, q in ((2, 4), (3, 8)):
        assert few_token(8, 4100, K, p, q, unpacked=True)
        for offset in (0, 1, 5):
            check(8, 4100, K, p, q, cfg=OPEN_XOR, fp16_src=fp16_src, offset=offset, seed=8, what="few tokens")
