"""Plans of products (fg_gemm_plan) on whose tile a measured rule decides; CPU, no launch."""
import re

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


@pytest.mark.parametrize("M,N,K,la,lb", [
    (1440, 5832, 704, ROW, COL), (1824, 5104, 832, ROW, COL), (2528, 3520, 1024, ROW, COL), (3520, 2768, 1824, ROW, COL), (5280, 1888, 1312, ROW, COL),
    (1792, 5232, 672, ROW, COL), (8128, 1464, 544, ROW, COL), (6080, 1408, 1424, COL, ROW), (4448, 2064, 1056, COL, COL), (5904, 2048, 1152, ROW, ROW),
    (3360, 2592, 4288, COL, COL), (2832, 3008, 3136, ROW, ROW), (1552, 1792, 15776, ROW, COL), (2688, 1056, 12448, ROW, COL)])
def test_no_sum_is_longer_than_before(M, N, K, la, lb):
    """Products of the deep 128x128 tile, which adds an entry up in two sums, do not go to the 256x256 tile, which has one (their error against
    64 bits was 1.38 times as large there)."""
    for variant in (fg.FG_PLAN_REAL, fg.FG_PLAN_REAL_BF16):
        assert "_256x256x64" not in fg.fg_gemm_plan(M, N, K, la, lb, variant=variant)


@pytest.mark.parametrize("variant,M,N,K,tile", [
    (fg.FG_PLAN_REAL, 8192, 6000, 256, "256x256x64"), (fg.FG_PLAN_REAL, 8192, 8192, 256, "256x128x64"), (fg.FG_PLAN_REAL, 5408, 5104, 128, "256x128x64"), (fg.FG_PLAN_REAL, 5748, 5376, 128, "256x256x64"),
    (fg.FG_PLAN_REAL, 5408, 5104, 192, "256x256x64"), (fg.FG_PLAN_REAL_BF16, 8192, 6000, 256, "256x256x64"), (fg.FG_PLAN_REAL_F16_CD, 2384, 5584, 128, "256x128x64"),
    (fg.FG_PLAN_REAL_F16_CD, 9024, 6784, 256, "256x128x64"), (fg.FG_PLAN_REAL_F16_CD, 3524, 7968, 256, "256x256x64"),
    (fg.FG_PLAN_REAL_AB_ADD, 4096, 4096, 256, "256x128x64"), (fg.FG_PLAN_REAL_AB_ADD, 4096, 4096, 320, "256x256x64")])
def test_tile_of_a_short_k(variant, M, N, K, tile):
    """The 256x128 tile in place of the 256x256 one: where C and D stream, by what decides that (keeps_real_cd), and not by M and N alone."""
    assert fg.fg_gemm_plan(M, N, K, fg.FG_COL, fg.FG_COL, variant=variant).replace("_k32", "").endswith("_" + tile)


def _scratch(M, N, plan):
    """Bytes of partial products of a plan with one workgroup per compute unit."""
    tm, tn = (int(v) for v in re.search(r"_(\d+)x(\d+)x", plan).groups())
    tiles = -(-M // tm) * -(-N // tn)
    split, tail = re.search(r"\+splitk(\d+)", plan), re.search(r"\+tailsplitk(\d+)", plan)
    return (tiles * int(split[1]) if split else tiles % 256 * int(tail[1]) if tail else 0) * tm * tn * 4


@pytest.mark.parametrize("M,N,K,la,lb,limit", [
    (6832, 3408, 12000, ROW, COL, 0), (2528, 6432, 13552, ROW, ROW, 0), (7627, 5147, 6160, ROW, ROW, 0), (8059, 5054, 7592, COL, ROW, 0),
    (2960, 6976, 5680, COL, COL, 0), (5824, 2864, 1952, ROW, COL, 0), (7436, 1060, 3736, COL, ROW, 0), (3270, 5114, 1144, ROW, COL, 0),
    (7248, 176, 9328, COL, COL, 16 << 20), (1481, 708, 12568, COL, ROW, 16 << 20), (696, 2002, 8416, ROW, COL, 16 << 20), (1056, 7835, 8024, COL, ROW, 16 << 20),
    (368, 4096, 12832, ROW, COL, 16 << 20), (1855, 746, 10848, COL, COL, 16 << 20)])
def test_no_call_needs_more_scratch_memory_than_before(M, N, K, la, lb, limit):
    """What needed none can be captured without the workspace, what fitted the static array can be made by fg_gemm_noalloc: the kernels with
    four waves and their rates change neither."""
    for variant in (fg.FG_PLAN_REAL, fg.FG_PLAN_REAL_BF16):
        assert _scratch(M, N, fg.fg_gemm_plan(M, N, K, la, lb, variant=variant)) <= limit


@pytest.mark.parametrize("M,N,la,lb,tile", [
    (1584, 29072, ROW, fg.FG_DIAG, "256x128x64"), (14488, 3552, fg.FG_DIAG, ROW, "256x128x64"), (10848, 4736, ROW, fg.FG_DIAG, "256x128x64"), (12192, 4512, fg.FG_DIAG, COL, "256x128x64"),
    (10384, 4960, COL, fg.FG_DIAG, "256x128x64"), (17816, 3032, COL, fg.FG_DIAG, "256x128x64"), (7272, 7360, fg.FG_DIAG, ROW, "256x128x64"), (3952, 12816, fg.FG_DIAG, ROW, "256x128x64")])
def test_diagonal_products_by_rates_of_their_own(M, N, la, lb, tile):
    """Their kernels have eight waves: the rates of the kernels with four are not theirs."""
    assert fg.fg_gemm_plan(M, N, M if la == fg.FG_DIAG else N, la, lb).endswith("_" + tile)
