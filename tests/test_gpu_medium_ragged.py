"""The row-adaptive kernel on one weight whose rows of C do not start on 16 bytes
(columns stored one by one) or whose rows are not whole lines: ragged N above 80
rows, where K is long enough for it, and at up to 80 with a short K."""
import pytest

import oracle
import paper_2607_04031_amd as tl
from paper_2607_04031_amd import synth
from tests._gpu import banner, dev_bf16, host_bits, host_f32, parity, parity_bf16_out

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,row_major", [(127, 130, 1288, False), (128, 1, 1288, True), (81, 2001, 1992, True),
                                             (96, 998, 1984, True), (113, 518, 1400, False), (80, 1003, 264, False),
                                             (65, 129, 72, True), (40, 32771, 200, True), (81, 1001, 1280, False)])
def test_ragged_columns(M, N, K, row_major):
    kind = tl.TL_LAYOUT_NK_ROW if row_major else tl.TL_LAYOUT_TILE
    fetch = tl.TL_FETCH_NATIVE if row_major else tl.TL_FETCH_BLOCK
    banner(f"row-adaptive ragged M={M} N={N} K={K} row_major={row_major}")
    A = synth.normal_bf16((M, K), seed=210 + M)
    W = synth.normal_bf16((N, K), seed=211, sigma=synth.W_SIGMA)
    y_ref = oracle.gemm_f64(A, W)
    Wd = dev_bf16(W) if row_major else tl.repack(dev_bf16(W), 1024, 16)
    for out in (tl.TL_OUT_F32, tl.TL_OUT_BF16):
        C = tl.gemm(dev_bf16(A), Wd, N, tl.layout(kind=kind, G=1024, block_rows=16, out_dtype=out), fetch)
        if out == tl.TL_OUT_F32:
            parity(host_f32(C), y_ref, "f32")
        else:
            parity_bf16_out(host_bits(C), y_ref, "bf16")
