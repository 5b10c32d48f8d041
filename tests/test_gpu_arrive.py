"""K splits summed inside a decode launch (small weights): the last workgroup of
a tile to arrive adds the partials in split order, so the result equals, bit for
bit, that of tl_gemm_noalloc, which sums them in a second launch; the arrival
counters are back at zero after every call, also in a replayed graph."""
import pytest

import paper_2607_04031_amd as tl
from paper_2607_04031_amd import synth
from tests._gpu import banner, dev_bf16

pytestmark = pytest.mark.gpu

# (M, N, K, splits, bf16 out): both sides of 4096 floats of partials per tile,
# N not a multiple of 4 (element-wise sums), of 32 (a partial tile), a K split
# of one step, more than eight splits
SHAPES = [(1, 1024, 1024, 0, True), (1, 1024, 1024, 0, False), (16, 1024, 4096, 8, True), (16, 1024, 4096, 9, True),
          (3, 1001, 2048, 4, False), (5, 998, 512, 8, True), (8, 256, 16384, 16, False), (33, 96, 1024, 2, True),
          (64, 512, 4096, 1, True), (64, 512, 4096, 2, False)]


@pytest.mark.parametrize("M,N,K,S,bf16", SHAPES)
def test_equals_the_second_launch(M, N, K, S, bf16):
    import torch
    banner(f"in-launch split-K sum M={M} N={N} K={K} S={S}")
    d = tl.layout(split_k=S, out_dtype=tl.TL_OUT_BF16 if bf16 else tl.TL_OUT_F32)
    W = tl.repack(dev_bf16(synth.normal_bf16((N, K), seed=2, sigma=synth.W_SIGMA)), 4096, 32)
    dt = torch.bfloat16 if bf16 else torch.float32
    got, want = (torch.empty((M, N), dtype=dt, device="cuda") for _ in range(2))
    for seed in range(5):
        A = dev_bf16(synth.normal_bf16((M, K), seed=10 + seed))
        got.fill_(float("nan"))
        tl.tl_gemm(A, W, got, M, N, K, d)
        tl.tl_gemm_noalloc(A, W, want, M, N, K, d)
        assert torch.equal(got, want), f"call {seed}"


def test_replayed_graph():
    import torch
    banner("in-launch split-K sum, graph replays between eager calls")
    M, N, K = 4, 1024, 4096
    d = tl.layout(out_dtype=tl.TL_OUT_BF16)
    W = tl.repack(dev_bf16(synth.normal_bf16((N, K), seed=2, sigma=synth.W_SIGMA)), 4096, 32)
    A = dev_bf16(synth.normal_bf16((M, K), seed=3))
    C, E = (torch.empty((M, N), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        tl.tl_gemm(A, W, C, M, N, K, d, stream=s)
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            tl.tl_gemm(A, W, C, M, N, K, d, stream=s)
            tl.tl_gemm(A, W, C, M, N, K, d, stream=s)
        for seed in range(4):
            A.copy_(dev_bf16(synth.normal_bf16((M, K), seed=20 + seed)))
            C.zero_()
            g.replay()
            tl.tl_gemm(A, W, E, M, N, K, d, stream=s)
            s.synchronize()
            assert torch.equal(C, E), f"replay {seed}"
