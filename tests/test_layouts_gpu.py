"""GPU parity tests of the layout adapters of fg_gemm: diagonal operands (Section 5.2) and
planar-split complex operands (Section 5.4), against the CPU oracle."""
import itertools

import pytest

from paper_2009_12263_amd import binding as fg
from tests.parity import run_cgemm_case, run_diag_case

pytestmark = pytest.mark.gpu
LAYOUTS = [fg.FG_COL, fg.FG_ROW]


def say(msg):
    print("[case] " + msg, flush=True)


@pytest.mark.parametrize("side", ["A", "B"])
@pytest.mark.parametrize("other,ldl", list(itertools.product(LAYOUTS, LAYOUTS)))
def test_diagonal_operand_small(side, other, ldl):
    for (M, N, K) in [(256, 256, 256), (512, 384, 512), (128, 320, 256), (384, 128, 64)]:
        # rectangular diagonal operands hold min(rows, cols) entries; rows/columns beyond are zero
        say("diag %s M=%d N=%d K=%d other=%d D=%d" % (side, M, N, K, other, ldl))
        run_diag_case(M, N, K, side, other, ldl, ints=True)
    run_diag_case(512, 512, 512, side, other, ldl, alpha=0.5, beta=-1.25)


def test_diagonal_config4_4096():
    """BASELINE config 4 variant: D = diag(d) B + C, N = 4096, B column-major; every entry is
    checked against the closed form the oracle was pinned to (d_i B_ij + C_ij)."""
    say("diag A 4096 ints"); run_diag_case(4096, 4096, 4096, "A", ints=True, samples=20000)
    say("diag A 4096 floats"); run_diag_case(4096, 4096, 4096, "A", samples=20000)


@pytest.mark.parametrize("la,lb", list(itertools.product(LAYOUTS, LAYOUTS)))
def test_complex_small_all_layouts(la, lb):
    for (M, N, K) in [(64, 64, 64), (256, 128, 192), (384, 512, 128)]:
        say("cgemm ints M=%d N=%d K=%d la=%d lb=%d" % (M, N, K, la, lb))
        run_cgemm_case(M, N, K, la, lb, ints=True, pad=8)
    say("cgemm floats 512"); run_cgemm_case(512, 512, 512, la, lb, alpha=0.5, beta=2.0)
    say("cgemm row-major D"); run_cgemm_case(256, 384, 128, la, lb, ld_layout=fg.FG_ROW, ints=True)


def test_complex_config4_4096():
    """BASELINE config 4: planar complex D = A B + C at 4096^3, sampled."""
    say("cgemm 4096 floats"); run_cgemm_case(4096, 4096, 4096, samples=4096)
    say("cgemm 4096 ints"); run_cgemm_case(4096, 4096, 4096, ints=True, samples=4096)


def test_edge_tiles_diagonal_and_complex():
    """Sizes that are not multiples of any tile (K a multiple of 8) for the layout adapters."""
    for side in ("A", "B"):
        for other in LAYOUTS:
            say("diag %s edge other=%d" % (side, other))
            run_diag_case(300, 200, 264, side, other, ints=True)
            run_diag_case(70, 333, 72, side, other, fg.FG_ROW, ints=True)
    for la, lb in itertools.product(LAYOUTS, LAYOUTS):
        say("cgemm edge la=%d lb=%d" % (la, lb))
        run_cgemm_case(100, 75, 40, la, lb, ints=True, pad=8)
        run_cgemm_case(300, 513, 136, la, lb, ld_layout=fg.FG_ROW, alpha=0.5, beta=1.5)


@pytest.mark.parametrize("la,lb", list(itertools.product(LAYOUTS, LAYOUTS)))
def test_dual_numbers_all_layouts(la, lb):
    """Dual-number products (Section 5.4, eps^2 = 0) on the planar layout: exact on integers for
    every tile shape, floats within tolerance, edge tiles and a row-major result."""
    for (M, N, K) in [(64, 64, 64), (256, 128, 192), (384, 512, 128), (100, 75, 40)]:
        say("dual ints M=%d N=%d K=%d la=%d lb=%d" % (M, N, K, la, lb))
        run_cgemm_case(M, N, K, la, lb, ints=True, pad=8, dual=True)
    say("dual floats 512"); run_cgemm_case(512, 512, 512, la, lb, alpha=0.5, beta=2.0, dual=True)
    say("dual row-major D"); run_cgemm_case(300, 513, 136, la, lb, ld_layout=fg.FG_ROW, alpha=0.5, beta=1.5, dual=True)
    say("dual no C"); run_cgemm_case(256, 384, 128, la, lb, with_c=False, ints=True, dual=True)


def test_dual_4096():
    say("dual 4096 floats"); run_cgemm_case(4096, 4096, 4096, samples=4096, dual=True)
    say("dual 4096 ints"); run_cgemm_case(4096, 4096, 4096, ints=True, samples=4096, dual=True)


@pytest.mark.parametrize("la,lb", list(itertools.product(LAYOUTS, LAYOUTS)))
def test_interleaved_complex_all_layouts(la, lb):
    """Complex matrices with real and imaginary parts adjacent in memory (Section 5.4's global
    layout); the oracle is fed the same numbers in planar form, which its own pins tie to the
    interleaved form.  Exact on integers for every tile shape, edge tiles, a K tail, no C, and a
    row-major result."""
    for (M, N, K) in [(64, 64, 64), (256, 128, 192), (384, 512, 128), (100, 75, 40)]:
        say("interleaved ints M=%d N=%d K=%d la=%d lb=%d" % (M, N, K, la, lb))
        run_cgemm_case(M, N, K, la, lb, ints=True, pad=8, interleaved=True)
    say("interleaved floats 512"); run_cgemm_case(512, 512, 512, la, lb, alpha=0.5, beta=2.0, interleaved=True)
    say("interleaved row-major D"); run_cgemm_case(300, 513, 136, la, lb, ld_layout=fg.FG_ROW, alpha=0.5, beta=1.5, interleaved=True)
    say("interleaved no C"); run_cgemm_case(256, 384, 128, la, lb, with_c=False, ints=True, interleaved=True)


def test_interleaved_complex_4096():
    say("interleaved 4096 floats"); run_cgemm_case(4096, 4096, 4096, samples=4096, interleaved=True)
    say("interleaved 2048x4096x256 ints, every entry"); run_cgemm_case(2048, 4096, 256, ints=True, interleaved=True)


def test_interleaved_and_planar_matrices_are_not_mixed():
    import torch
    H = torch.zeros(2 * 64 * 64, dtype=torch.float16, device="cuda")
    F = torch.zeros(2 * 64 * 64, dtype=torch.float32, device="cuda")
    il = lambda t, d: fg.Matrix(t, fg.FG_COL, 64, dtype=d)
    kw = dict(raise_on_error=False)
    assert fg.fg_gemm(64, 64, 64, 1.0, il(H, fg.FG_CF16), il(H, fg.FG_CF16), 0.0, None, fg.Matrix(F, fg.FG_COL, 64, im=F), **kw) == fg.FG_ERR_UNSUPPORTED
    assert fg.fg_gemm(64, 64, 64, 1.0, il(H, fg.FG_CF16), fg.Matrix(H, fg.FG_COL, 64), 0.0, None, il(F, fg.FG_CF32), **kw) == fg.FG_ERR_UNSUPPORTED
    assert fg.fg_gemm(64, 64, 64, 1.0, fg.Matrix(H, fg.FG_COL, 64), fg.Matrix(H, fg.FG_COL, 64), 0.0, None, il(F, fg.FG_CF32), **kw) == fg.FG_ERR_UNSUPPORTED
    assert fg.fg_gemm(64, 64, 64, 1.0, il(H, fg.FG_CF16), il(H, fg.FG_CF16), 0.0, None, il(F, fg.FG_CF32), act=fg.FG_ACT_RELU, **kw) == fg.FG_ERR_UNSUPPORTED
    assert fg.fg_gemm(64, 64, 64, 1.0, fg.Matrix(H, fg.FG_COL, 64, im=H, dtype=fg.FG_CF16), il(H, fg.FG_CF16), 0.0, None, il(F, fg.FG_CF32), **kw) == fg.FG_ERR_LAYOUT


KINDS = [dict(), dict(dual=True), dict(interleaved=True)]
TILES = ["0", "1", "2", "3"]           # 256x128, 128x128, 64x64, 64x64 with two K groups


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("tile", TILES)
def test_cache_policies_of_complex_results(monkeypatch, kind, tile):
    """C and D of complex and dual products are kept in the caches or streamed past them: the same results on interior and edge
    tiles of every tile shape, with C and without, for columns on the lines, on half lines and off them.  Passes of 7 to
    16 MB on the lines stream up to K = 256 and are kept above; of the large ones (over 80 MB), those beside large A and B stream and those
    off the lines beside small ones are kept (test_cache_policy.py has the rule)."""
    from tests.parity import delenv, setenv
    setenv(monkeypatch, "FG_FORCE_TILE", tile)
    for M, N, K, with_c in itertools.product((256, 264, 260), (128, 133), (72, 264), (True, False)):
        say("tile %s M=%d N=%d K=%d C=%d %s" % (tile, M, N, K, with_c, kind))
        run_cgemm_case(M, N, K, ints=True, alpha=2.0, beta=-1.0, with_c=with_c, **kind)
    run_cgemm_case(133, 264, 72, fg.FG_ROW, fg.FG_ROW, fg.FG_ROW, ints=True, **kind)
    for M, N, K in ((1440, 613, 136), (1440, 613, 328), (1504, 2003, 2800), (1507, 2003, 2800), (2052, 2603, 72)):
        say("tile %s M=%d N=%d K=%d C=1 %s" % (tile, M, N, K, kind))
        run_cgemm_case(M, N, K, fg.FG_ROW, fg.FG_COL, ints=True, alpha=2.0, beta=-1.0, samples=3000, **kind)
    delenv(monkeypatch, "FG_FORCE_TILE")


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("tile", TILES)
def test_every_complex_tile_shape(monkeypatch, kind, tile):
    """Every tile of the complex, dual and interleaved kernels over all layouts: less than a tile, ragged M and N, short and
    long K with a tail, several tiles; integers, every entry exact, and floats."""
    from tests.parity import delenv, setenv
    setenv(monkeypatch, "FG_FORCE_TILE", tile)
    for la, lb in itertools.product(LAYOUTS, LAYOUTS):
        say("tile %s la=%d lb=%d %s" % (tile, la, lb, kind))
        run_cgemm_case(70, 45, 8, la, lb, ints=True, pad=8, poison=True, **kind)
        run_cgemm_case(300, 270, 136, la, lb, ints=True, pad=8, poison=True, beta=-2.0, **kind)
        run_cgemm_case(270, 131, 1032, la, lb, fg.FG_ROW, ints=True, with_c=False, **kind)
        run_cgemm_case(513, 260, 40, la, lb, ints=True, **kind)
        run_cgemm_case(261, 200, 328, la, lb, alpha=0.5, beta=2.0, **kind)
    delenv(monkeypatch, "FG_FORCE_TILE")


@pytest.mark.parametrize("kind", KINDS)
def test_two_64x64_tiles_of_complex_products_are_told_apart(monkeypatch, kind):
    """One K group and two (which share a plan name) add the same products up in different orders: on floats their results
    differ in the last bits, so one that silently ran as the other is seen.  The planner takes one up to K = 160, two above."""
    import torch
    from paper_2009_12263_amd import workloads as W
    from tests.parity import delenv, setenv
    def result(M, N, K):
        planes = 1 if kind.get("interleaved") else 2
        def mat(rows, cols, stream, dtype, code):
            n = rows * cols * (2 if planes == 1 else 1)
            t = [W.uniform_pm1(n, stream + i, device="cuda", dtype=dtype) for i in range(planes)]
            return fg.Matrix(t[0], fg.FG_COL, rows, im=t[1] if planes == 2 else None, dtype=code if planes == 1 else None)
        A, B = mat(M, K, 1, torch.float16, fg.FG_CF16), mat(K, N, 3, torch.float16, fg.FG_CF16)
        D = mat(M, N, 5, torch.float32, fg.FG_CF32)
        (fg.fg_gemm_dual if kind.get("dual") else fg.fg_gemm)(M, N, K, 1.0, A, B, 0.0, None, D)
        torch.cuda.synchronize()
        return torch.cat([D.re, D.im]) if planes == 2 else D.re
    for M, N, K, planned in ((200, 136, 96, "2"), (200, 136, 160, "2"), (200, 136, 168, "3"), (304, 200, 1032, "3")):
        got = {}
        for tile in ("2", "3"):
            setenv(monkeypatch, "FG_FORCE_TILE", tile)
            got[tile] = result(M, N, K)
        delenv(monkeypatch, "FG_FORCE_TILE")
        say("M=%d N=%d K=%d %s" % (M, N, K, kind))
        assert not torch.equal(got["2"], got["3"])
        assert torch.equal(result(M, N, K), got[planned]), (M, N, K)


@pytest.mark.parametrize("kind", [dict(), dict(dual=True), dict(interleaved=True)])
@pytest.mark.parametrize("la,lb", list(itertools.product(LAYOUTS, LAYOUTS)))
def test_k_groups_of_complex_products(monkeypatch, kind, la, lb):
    """The 64x64 tile whose two groups of waves take its K tiles in turns: fewer K tiles than groups, an odd count, a K tail in
    either group's last tile, edge tiles, several tiles per workgroup; integers, every entry exact."""
    from tests.parity import delenv, setenv
    setenv(monkeypatch, "FG_FORCE_TILE", "3")
    for K in (8, 64, 72, 136, 192, 200, 328):
        say("K groups K=%d la=%d lb=%d %s" % (K, la, lb, kind))
        run_cgemm_case(131, 70, K, la, lb, ints=True, pad=8, poison=True, **kind)
    run_cgemm_case(70, 131, 264, la, lb, fg.FG_ROW, ints=True, alpha=2.0, beta=-1.0, **kind)
    say("several tiles per workgroup"); run_cgemm_case(1290, 1100, 136, la, lb, ints=True, samples=3000, **kind)
    delenv(monkeypatch, "FG_FORCE_TILE")
    say("planner's own choice, floats"); run_cgemm_case(300, 200, 1032, la, lb, **kind)
