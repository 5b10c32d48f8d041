"""Plans at the kernels' addressing limits (host only): sizes far past any real
weight, accepted by the library, where an offset in too few bits would wrap."""
import pytest

import paper_2607_04031_amd as tl


# The LDS decode kernel holds a lane's weight offset, over all the 32-row tiles
# of a workgroup, in 32 bits: it may be planned only where those rows are below
# 4 GB.  Both its M ranges, the two sides of the limit for the widest groups of
# tiles (7) and for 4 (whose limit the tile's own, tile_n rows below 2 GB, covers).
@pytest.mark.parametrize("M,N,K,br", [
    (17, 7168, 9586176, 32), (17, 7168, 9587200, 32), (17, 7168, 9830400, 32), (20, 7168, 11534336, 32),
    (32, 6144, 13421568, 16), (32, 5120, 14900224, 16), (32, 4096, 16776704, 32), (33, 3584, 16776704, 32),
])
def test_lds_decode_rows_below_4_gb(M, N, K, br):
    p = tl.tl_gemm_plan(M, N, K, tl.layout(block_rows=br))
    assert p["kernel"] == 1
    rows = N * p["split_k"] // p["workgroups"]          # weight rows of one workgroup
    assert rows % 32 == 0 and rows <= 224
    padded = -(-K // (2048 // br)) * (2048 // br)
    assert rows * padded * 2 < 2 ** 32, (rows, p)


def test_lds_decode_is_still_planned_below_the_limit():
    p = tl.tl_gemm_plan(17, 7168, 9586176, tl.layout())
    assert (p["workgroups"], p["split_k"], p["waves"], p["tile_n"]) == (256, 8, 8, 32)


# 192- and 320-row prefill tiles replace 256-row ones only with at least as many
# K splits, so an fp32 sum never runs over more of K than on 256-row tiles.  (A
# whole number of 256-row tiles takes no others and has the same splits.)
@pytest.mark.parametrize("M", [225, 257, 300, 321, 384, 385, 500, 577, 700, 769, 1000, 1025, 1200])
def test_prefill_tiles_keep_the_k_splits(M):
    taken = 0
    for N in (256, 1024, 2560, 4096, 5120, 8192, 10240, 14336, 24576, 28672):
        if -(-M // 256) * (N // 256) >= 256:
            continue
        for K in (512, 1024, 2048, 4096, 4160, 8192, 16384, 28672):
            p, q = (tl.tl_gemm_plan(m, N, K, tl.layout()) for m in (M, -(-M // 256) * 256))
            taken += p["tile_m"] in (192, 320)
            assert p["split_k"] >= q["split_k"], (N, K, p, q)
    assert taken


# ... nor where only the columns past the whole rounds of 256-row tiles split K
# (384 tiles: 128 left, 2 splits; 320: 64 left, 4).
@pytest.mark.parametrize("M,N,K,S", [(300, 49152, 8192, 2), (260, 40960, 8192, 4)])
def test_prefill_tiles_keep_the_remainders_k_splits(M, N, K, S):
    assert tl.tl_gemm_plan(M, N, K, tl.layout())["split_k"] >= S
