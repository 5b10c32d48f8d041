"""The row-adaptive kernel's grouped GEMMs add the same products in the same order
as the decode kernel's, which a requested tile selects: the results are equal bit
for bit, in fp32 too, whatever the number of rows of a group, the bound on it, the
configuration and the layout."""
import numpy as np
import pytest

import paper_2607_04031_amd as tl
from paper_2607_04031_amd import synth
from tests._gpu import banner, dev_bf16

pytestmark = pytest.mark.gpu


def dev_i32(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()


# groups around the 32-row blocks and the 128- and 192-row tiles, more than one
# chunk, empty ones; K below one step, of one to five (fewer than, as many as and
# more than the four sums), with a part of a step, and long; few tiles (128 x 128)
# and many (192 x 256); more than 64 and more than 256 groups.  With a bound of 129
# rows or more all of them take the row-adaptive kernel: groups with more than 64
# rows on average, or more than 600 tiles of 64 weight rows, or 64-row tiles and
# more than 32 rows
CASES = [
    ([17, 0, 1, 32] * 80, 96, 24), ([33, 64, 0, 65], 320, 64), ([128, 129, 3], 160, 136), ([192, 0, 193, 31], 128, 192),
    ([256, 255, 5], 288, 200), ([257, 16, 400], 64, 256), ([190, 40, 385], 128, 328), ([100, 250], 256, 8192),
    ([20] * 70, 800, 128), ([90, 0, 20, 193] * 33, 512, 968), ([17, 0, 3, 40] * 80, 256, 320),
]


@pytest.mark.parametrize("kind", [tl.TL_LAYOUT_TILE, tl.TL_LAYOUT_NK_ROW])
@pytest.mark.parametrize("swiglu", [False, True])
@pytest.mark.parametrize("counts,N,K", CASES)
def test_same_bits_as_the_decode_kernel(counts, N, K, swiglu, kind):
    import torch
    E, T, a_rows = len(counts), sum(counts), 60
    offsets = dev_i32(np.concatenate([[0], np.cumsum(counts)]))
    rng = np.random.default_rng(T + K)
    ids = dev_i32(rng.integers(-1, a_rows + 1, size=T))      # some outside A
    A = dev_bf16(synth.normal_bf16((a_rows, K), seed=31))
    rows_w = 2 * N if swiglu else N
    tile = kind == tl.TL_LAYOUT_TILE
    stride = tl.tl_tile_bytes(rows_w, K, 2, 1024, 16) if tile else rows_w * K * 2
    stack = torch.zeros(E * stride // 2, dtype=torch.bfloat16, device="cuda")
    distinct = [dev_bf16(synth.normal_bf16((rows_w, K), seed=400 + e, sigma=synth.W_SIGMA)) for e in range(3)]
    for e in range(E):
        part = stack[e * stride // 2:(e + 1) * stride // 2]
        if tile:
            tl.tl_repack(distinct[e % 3], part, rows_w, K, 2, 1024, 16)
        else:
            part.copy_(distinct[e % 3].flatten())
    banner(f"grouped sums {counts[:4]}x{E} N={N} K={K} swiglu={swiglu} kind={kind}")
    fn = tl.tl_gemm_grouped_swiglu if swiglu else tl.tl_gemm_grouped
    fetch = tl.TL_FETCH_BLOCK if tile else tl.TL_FETCH_NATIVE
    got = []
    for tile_m, bound in ((64, max(counts)), (0, max(counts)), (0, max(129, max(counts)))):
        C = torch.full((T, N), float("nan"), dtype=torch.float32, device="cuda")
        d = tl.layout(kind=kind, G=1024, block_rows=16, tile_m=tile_m, out_dtype=tl.TL_OUT_F32)
        fn(A, a_rows, ids, offsets, E, T, bound, stack, stride, C, N, K, d, fetch)
        got.append(C)
    assert torch.equal(got[0], got[1])
    assert torch.equal(got[0], got[2])

