"""The row-adaptive kernel on one weight, around the lines of the rule for its
non-temporal loads: one round of workgroups and one more, rows that are whole
lines and not, K split; and the ragged columns past 88 rows that stay
on the 128 x 128 kernel where there is more than one round."""
import pytest

import oracle
import paper_2607_04031_amd as tl
from paper_2607_04031_amd import synth
from tests._gpu import banner, dev_bf16, host_f32, parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("row_major", [False, True])
@pytest.mark.parametrize("M,N,K,split", [
    (65, 32768, 136, 1), (72, 32896, 192, 1), (128, 32768, 128, 1), (128, 33000, 320, 1), (88, 32771, 1288, 1),
    (89, 32771, 1288, 1), (89, 32767, 1288, 1), (97, 12288, 1024, 2), (113, 12032, 1000, 2), (81, 4096, 4088, 8),
    (128, 2048, 2056, 4), (200, 2048, 4096, 8),
])
def test_loads(M, N, K, split, row_major):
    import torch
    kind = tl.TL_LAYOUT_NK_ROW if row_major else tl.TL_LAYOUT_TILE
    fetch = tl.TL_FETCH_NATIVE if row_major else tl.TL_FETCH_BLOCK
    d = tl.layout(kind=kind, G=4096, block_rows=32)
    plan = tl.tl_gemm_plan(M, N, K, d, fetch)
    banner(f"row-adaptive loads M={M} N={N} K={K} row_major={row_major} plan={plan}")
    assert plan["split_k"] == split
    A = synth.normal_bf16((M, K), seed=480 + M)
    W = synth.normal_bf16((N, K), seed=481, sigma=synth.W_SIGMA)
    Wd = dev_bf16(W) if row_major else tl.repack(dev_bf16(W), 4096, 32)
    C = torch.full((M + 1, N), 7.0, dtype=torch.float32, device="cuda")
    tl.tl_gemm(dev_bf16(A), Wd, C, M, N, K, d, fetch)
    assert bool((C[M] == 7.0).all())
    parity(host_f32(C[:M].contiguous()), oracle.gemm_f64(A, W), "f32")
    db = tl.layout(kind=kind, G=4096, block_rows=32, out_dtype=tl.TL_OUT_BF16)
    H = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    tl.tl_gemm(dev_bf16(A), Wd, H, M, N, K, db, fetch)
    assert torch.equal(H, C[:M].to(torch.bfloat16))
