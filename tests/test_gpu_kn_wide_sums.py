"""[K][N] weights on 256-column workgroups: the edges of their tiles, splits and
steps against the oracle, and fp32 sums no further from the exact
ones than on the 64-column workgroups, which a requested tile selects.  N and K
where the two take different numbers of K splits, one and two M tiles."""
import numpy as np
import pytest

import oracle
import paper_2607_04031_amd as tl
from paper_2607_04031_amd import synth
from tests._gpu import banner, dev_bf16, host_f32, parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(32, 24576, 4096), (17, 30720, 8192), (32, 16640, 4096), (24, 10240, 8192),
                                   (32, 57344, 2048), (16, 24576, 4096), (32, 33000, 4096), (32, 22024, 4160)])
def test_error_against_64_bits(M, N, K):
    import torch
    banner(f"[K][N] sums M={M} N={N} K={K}")
    A = dev_bf16(synth.normal_bf16((M, K), seed=11))
    W = torch.randn((K, N), generator=torch.Generator(device="cuda").manual_seed(12), device="cuda").mul_(0.02).bfloat16()
    exact = torch.cat([A.double() @ W[:, n:n + 4096].double() for n in range(0, N, 4096)], dim=1)
    errors = []
    for tile_n in (0, 64):
        d = tl.layout(kind=tl.TL_LAYOUT_KN_ROW, out_dtype=tl.TL_OUT_F32, tile_n=tile_n)
        C = torch.empty((M, N), dtype=torch.float32, device="cuda")
        tl.tl_gemm(A, W, C, M, N, K, d, tl.TL_FETCH_NATIVE)
        errors.append(float((C.double() - exact).norm() / exact.norm()))
    print(f"errors: {errors[0]:.3g} {errors[1]:.3g}")
    # half a million sums and more on either side: the two norms scatter by under 1 %
    assert errors[0] <= 1.02 * errors[1]


# a last workgroup with columns past N (whole 64-column waves and part of one),
# K steps fewer than the wave pairs, sixteen splits, three splits of rows that
# are not whole lines, more tiles than CUs, one and two M tiles
@pytest.mark.parametrize("M,N,K,S", [(8, 3400, 16384, 16), (32, 3264, 18560, 16), (5, 50000, 64, 1), (17, 49200, 192, 1),
                                     (16, 33096, 3072, 3), (17, 33096, 4160, 3), (1, 102408, 128, 1), (32, 24640, 2048, 2)])
def test_edges(M, N, K, S):
    d = tl.layout(kind=tl.TL_LAYOUT_KN_ROW)
    p = tl.tl_gemm_plan(M, N, K, d, tl.TL_FETCH_NATIVE)
    banner(f"[K][N] 256-column workgroups M={M} N={N} K={K} plan={p}")
    # eight waves past 512 workgroups of 64 columns: only this plan has them
    assert (p["split_k"], p["waves"]) == (S, 8) and p["workgroups"] > 512
    A = synth.normal_bf16((M, K), seed=1400 + M)
    W = synth.normal_bf16((N, K), seed=1401, sigma=synth.W_SIGMA)
    import torch
    C = torch.empty((M, N), dtype=torch.float32, device="cuda")
    tl.tl_fetch_counter_read()
    tl.tl_gemm(dev_bf16(A), dev_bf16(np.ascontiguousarray(W.T)), C, M, N, K, d, tl.TL_FETCH_NATIVE | tl.TL_FETCH_COUNT)
    assert tl.tl_fetch_counter_read() == -(-N // 64) * 64 * K * 2       # the 64-column tiles inside N
    parity(host_f32(C), oracle.gemm_f64(A, W), f"M={M} N={N} K={K}")
