"""K splits of 128 x 128 tiles at 65 - 128 rows: the 128 x 128 kernel (short K
ranges on nearly all the CUs) and the row-adaptive kernel, around the lines of
the rule between them; partial row blocks and a partial last K step."""
import pytest

import oracle
import paper_2607_04031_amd as tl
from paper_2607_04031_amd import synth
from tests._gpu import banner, dev_bf16, host_f32, parity

pytestmark = pytest.mark.gpu


# M, N, K, K splits: 192, 190 and 188 workgroups of 16 steps and of a part of
# one; 17 steps; 96 and 97 rows; 240 and 256 workgroups below 97 rows; 8 splits
@pytest.mark.parametrize("row_major", [False, True])
@pytest.mark.parametrize("M,N,K,split", [
    (97, 12288, 1024, 2), (128, 12160, 2048, 2), (113, 12032, 1000, 2), (128, 8064, 2056, 4), (128, 12288, 2112, 2),
    (96, 12288, 1024, 2), (81, 4096, 4088, 8), (96, 6144, 3200, 5), (100, 4096, 4088, 8),
])
def test_splits(M, N, K, split, row_major):
    import torch
    kind = tl.TL_LAYOUT_NK_ROW if row_major else tl.TL_LAYOUT_TILE
    fetch = tl.TL_FETCH_NATIVE if row_major else tl.TL_FETCH_BLOCK
    d = tl.layout(kind=kind, G=4096, block_rows=32)
    plan = tl.tl_gemm_plan(M, N, K, d, fetch)
    banner(f"prefill splits M={M} N={N} K={K} row_major={row_major} plan={plan}")
    assert (plan["split_k"], plan["tile_m"], plan["tile_n"]) == (split, 128, 128)
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
