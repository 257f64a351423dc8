"""Plans of products (fg_gemm_plan) on whose tile a measured rule decides; CPU, no launch."""
import pytest

from paper_2009_12263_amd import binding as fg

COL, ROW = fg.FG_COL, fg.FG_ROW


@pytest.mark.parametrize("M,N,K,la,lb,tile", [
    (752, 6032, 144, ROW, ROW, "64x64x64"), (3344, 1520, 144, ROW, ROW, "64x64x64"), (7968, 624, 176, ROW, ROW, "64x64x64"),
    (2336, 1856, 224, ROW, COL, "64x64x64"), (800, 5312, 256, COL, ROW, "64x64x64"), (8880, 3728, 400, COL, COL, "128x128x64")])
def test_short_k_is_left_to_small_tiles(M, N, K, la, lb, tile):
    """The 256x128 tile has eight waves where K is short, and is priced with their rate."""
    for variant in (fg.FG_PLAN_REAL, fg.FG_PLAN_REAL_BF16):
        assert fg.fg_gemm_plan(M, N, K, la, lb, variant=variant).endswith("_" + tile)
