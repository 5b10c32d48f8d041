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
