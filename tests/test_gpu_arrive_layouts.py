"""K splits summed inside the launch over every layout and type that does so, by
turns on one stream with different splits, tiles and sizes: each result equals,
bit for bit, that of tl_gemm_noalloc, which sums in a second launch (which calls
take which path: tests/test_host_arrive.py)."""
import pytest

import paper_2607_04031_amd as tl
from paper_2607_04031_amd import synth
from tests._gpu import banner, dev_bf16

pytestmark = pytest.mark.gpu

# (kind, element bytes, M, N, K, splits): one and two M tiles, 8 and 16 waves,
# a ragged N (whole and element-wise sums), 2 to 16 splits
CALLS = [
    (tl.TL_LAYOUT_TILE, 2, 1, 1024, 1024, 0), (tl.TL_LAYOUT_NK_ROW, 2, 16, 1024, 4096, 8), (tl.TL_LAYOUT_KN_ROW, 2, 8, 2048, 2048, 4),
    (tl.TL_LAYOUT_TILE, 1, 4, 1024, 2048, 0), (tl.TL_LAYOUT_NK_ROW, 1, 5, 1001, 2048, 4), (tl.TL_LAYOUT_KN_ROW, 2, 17, 264, 4096, 3),
    (tl.TL_LAYOUT_NK_ROW, 2, 3, 998, 2048, 5), (tl.TL_LAYOUT_TILE, 1, 17, 256, 8192, 6), (tl.TL_LAYOUT_TILE, 2, 2, 4096, 1024, 2),
    (tl.TL_LAYOUT_KN_ROW, 2, 1, 64, 16384, 16), (tl.TL_LAYOUT_TILE, 2, 33, 96, 1024, 2),
]


def weight(kind, elem, N, K, seed):
    import torch
    if elem == 1:
        w = torch.randint(0, 120, (N, K), generator=torch.Generator().manual_seed(seed), dtype=torch.uint8).cuda()
    else:
        w = dev_bf16(synth.normal_bf16((N, K), seed=seed, sigma=synth.W_SIGMA))
    if kind == tl.TL_LAYOUT_TILE:
        return tl.repack(w, 4096, 32)
    return w.t().contiguous() if kind == tl.TL_LAYOUT_KN_ROW else w


@pytest.mark.parametrize("bf16", [False, True])
def test_by_turns_on_one_stream(bf16):
    import torch
    dt = torch.bfloat16 if bf16 else torch.float32
    calls = []
    for i, (kind, elem, M, N, K, S) in enumerate(CALLS):
        banner(f"in-launch split-K sum kind={kind} elem={elem} M={M} N={N} K={K} S={S}")
        d = tl.layout(kind=kind, elem_bytes=elem, split_k=S, out_dtype=tl.TL_OUT_BF16 if bf16 else tl.TL_OUT_F32)
        fetch = tl.TL_FETCH_BLOCK if kind == tl.TL_LAYOUT_TILE else tl.TL_FETCH_NATIVE
        args = (dev_bf16(synth.normal_bf16((M, K), seed=50 + i)), weight(kind, elem, N, K, 60 + i))
        want = torch.empty((M, N), dtype=dt, device="cuda")
        tl.tl_gemm_noalloc(*args, want, M, N, K, d, fetch)
        calls.append((args, M, N, K, d, fetch, want))
    got = [torch.empty_like(c[-1]) for c in calls]
    for turn in range(6):
        for g in got:
            g.fill_(float("nan"))
        for (args, M, N, K, d, fetch, _), g in zip(calls, got):
            tl.tl_gemm(*args, g, M, N, K, d, fetch)
        if turn == 2:
            tl.tl_fetch_counter_read()      # clears the tally, not the counters
        for c, g in zip(calls, got):
            assert torch.equal(g, c[-1]), (turn, c[1:6])
        calls, got = calls[3:] + calls[:3], got[3:] + got[:3]      # another order
