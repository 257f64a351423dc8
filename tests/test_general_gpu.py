"""GPU parity of the general kernel (operands the tiled kernels cannot take) at the sizes where its
pieces of eight, its K steps of 64, its two block tiles and its K split can go wrong.  Integer data
unless stated: every entry must equal the exact result."""
import itertools
import math

import pytest
import torch

from paper_2009_12263_amd import binding as fg
from paper_2009_12263_amd import workloads as W
from tests.parity import delenv, run_contract_case, run_unaligned_gemm_case, setenv

pytestmark = pytest.mark.gpu
LAYOUTS = [fg.FG_COL, fg.FG_ROW]
a, b, c, d, e, f, g = range(7)


def say(msg):
    print("[case] " + msg, flush=True)


@pytest.mark.parametrize("tile", ["2", "3"])
@pytest.mark.parametrize("la,lb", list(itertools.product(LAYOUTS, LAYOUTS)))
def test_matrix_edges(monkeypatch, tile, la, lb):
    """K around the 8 k of a piece, the 64 of a step and the 72 from which a step takes unchecked
    loads; rows around the tiles; operands of fewer than eight elements; tight and padded leading
    dimensions (a tight one puts the last piece at the very end of the operand)."""
    setenv(monkeypatch, "FG_FORCE_TILE", tile)
    for K in (1, 7, 9, 63, 65, 71, 72, 73, 127, 129, 200, 263, 521):
        for (M, N) in ((1, 1), (3, 65), (129, 7), (200, 131)):
            say("tile %s %dx%dx%d A=%d B=%d" % (tile, M, N, K, la, lb))
            run_unaligned_gemm_case(M, N, K, la, lb, pads=(0, 0, 0), offsets=(1, 0, 0))
            run_unaligned_gemm_case(M, N, K, la, lb, fg.FG_ROW, pads=(1, 3, 2), bias_dim=1, act=fg.FG_ACT_RELU, c_act=fg.FG_ACT_RELU, beta=-2.0)
    run_unaligned_gemm_case(130, 70, 77, la, lb, bf16=True, pads=(0, 1, 0))
    run_unaligned_gemm_case(130, 70, 77, la, lb, ab_add=(1.0, -2.0), pads=(0, 1, 0))


@pytest.mark.parametrize("tile,splits", [("2", 2), ("2", 5), ("3", 2), ("3", 3), ("3", 9)])
def test_matrix_k_split(monkeypatch, tile, splits):
    """Partial products over K ranges, an odd number of steps per range, empty ranges at the end."""
    setenv(monkeypatch, "FG_FORCE_TILE", tile)
    setenv(monkeypatch, "FG_FORCE_SPLIT", str(splits))
    for (M, N, K) in ((70, 45, 1001), (131, 129, 641), (65, 200, 65), (9, 5, 577)):
        for la, lb in ((fg.FG_COL, fg.FG_COL), (fg.FG_ROW, fg.FG_ROW)):
            say("tile %s split %d %dx%dx%d" % (tile, splits, M, N, K))
            run_unaligned_gemm_case(M, N, K, la, lb, bias_dim=0, act=fg.FG_ACT_RELU, beta=0.5)
            run_unaligned_gemm_case(M, N, K, la, lb, ints=False, ab_add=(0.5, -0.25))


def test_planners_own_choices():
    for (M, N, K) in ((301, 301, 6001), (17, 1025, 4099), (1531, 130, 515), (1100, 1030, 129)):
        say("%dx%dx%d floats" % (M, N, K))
        run_unaligned_gemm_case(M, N, K, fg.FG_ROW, fg.FG_COL, ints=False, pads=(0, 0, 0), offsets=(0, 0, 0))


def test_leading_dimensions_beyond_the_tiled_kernels():
    """Offsets that need 64 bits, in every matrix."""
    run_unaligned_gemm_case(3, 2, 5, fg.FG_COL, fg.FG_COL, pads=((1 << 24) + 1, (1 << 23) + 3, (1 << 22) + 1))
    run_unaligned_gemm_case(9, 3, 70, fg.FG_ROW, fg.FG_ROW, pads=((1 << 23) + 1, 1, (1 << 22) + 1))


def test_split_calls_without_allocation_and_in_a_graph():
    """The allocation-free entry point makes the same plan (bit-identical floats); a captured split
    call replays to the eager result."""
    M, N, K = 301, 99, 4101
    A = W.uniform_pm1(M * K, 1, device="cuda"); B = W.uniform_pm1(K * N, 2, device="cuda")
    Cm = W.uniform_pm1(M * N, 3, device="cuda", dtype=torch.float32)
    want, D = torch.empty_like(Cm), torch.empty_like(Cm)
    fg.fg_init()

    def call(out, **kw):
        fg.fg_gemm(M, N, K, 0.5, fg.Matrix(A, fg.FG_COL, M), fg.Matrix(B, fg.FG_COL, K), 1.0, fg.Matrix(Cm, fg.FG_COL, M), fg.Matrix(out, fg.FG_COL, M), **kw)
    call(want)
    call(D, noalloc=True)
    torch.cuda.synchronize()
    assert torch.equal(D, want)
    s, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=s):
            call(D, stream=s)
    torch.cuda.synchronize()
    for rep in range(3):
        D.fill_(float("nan"))
        call(torch.empty_like(D))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        say("replay %d" % rep)
        assert torch.equal(D, want)


def captured_nodes(stream, call):
    """Nodes of the graph that `call` leaves when it is made on a capturing stream (nothing runs)."""
    import ctypes
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
    hip = ctypes.CDLL(path)
    s, graph, n = ctypes.c_void_p(stream.cuda_stream), ctypes.c_void_p(), ctypes.c_size_t()
    assert hip.hipStreamBeginCapture(s, 2) == 0               # relaxed mode
    call()
    assert hip.hipStreamEndCapture(s, ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    return n.value


@pytest.mark.parametrize("tile,splits", [("2", 3), ("3", 5)])
@pytest.mark.parametrize("dt", [torch.float16, torch.bfloat16])
def test_split_without_scratch_memory_gives_the_same_bits(monkeypatch, tile, splits, dt):
    """Products of this kernel need no scratch memory where a call may overlap with others that the
    library does not order against it: captured calls and allocation-free calls are one kernel each, which
    adds the K ranges up itself.  The result is bit for bit that of the eager call, whose ranges go through
    the workspace, with every option (floats; an odd number of steps per range, an empty last range)."""
    setenv(monkeypatch, "FG_FORCE_TILE", tile)
    setenv(monkeypatch, "FG_FORCE_SPLIT", str(splits))
    fg.fg_init()
    s = torch.cuda.Stream()
    for (M, N, K) in ((131, 67, 1501), (65, 130, 7 * 64 + 1), (9, 5, 4 * splits * 64 - 63)):
        A = W.uniform_pm1(M * K, 1, device="cuda", dtype=dt); B = W.uniform_pm1(K * N, 2, device="cuda", dtype=dt)
        Cm = W.uniform_pm1(M * N, 3, device="cuda", dtype=torch.float32); bias = W.uniform_pm1(M + N, 4, device="cuda", dtype=torch.float32)
        for opts in (dict(), dict(C=True), dict(C=True, bias=bias, bias_dim=0, act=fg.FG_ACT_RELU, c_act=fg.FG_ACT_RELU), dict(bias=bias, bias_dim=1),
                     dict(C=True, a_add=0.5, b_add=-0.25) if dt == torch.float16 else dict(C=True, bias=bias, bias_dim=1)):
            opts = dict(opts)
            C_ = fg.Matrix(Cm, fg.FG_COL, M) if opts.pop("C", False) else None
            want, D = torch.full_like(Cm, float("nan")), torch.full_like(Cm, float("nan"))

            def call(out, **kw):
                fg.fg_gemm(M, N, K, 0.3, fg.Matrix(A, fg.FG_COL, M), fg.Matrix(B, fg.FG_ROW, N), 0.7, C_, fg.Matrix(out, fg.FG_COL, M), **opts, **kw)
            say("tile %s split %d %dx%dx%d %s" % (tile, splits, M, N, K, sorted(opts)))
            call(want)
            call(D, noalloc=True)
            torch.cuda.synchronize()
            assert torch.isfinite(want).all() and torch.equal(D, want)
            assert captured_nodes(s, lambda: call(D, stream=s)) == 1
            assert captured_nodes(s, lambda: call(D, stream=s, noalloc=True)) == 1
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.stream(s):
                with torch.cuda.graph(graph, stream=s):
                    call(D, stream=s)
            torch.cuda.synchronize()
            for rep in range(2):
                D.fill_(float("nan"))
                call(torch.empty_like(D))                     # an eager split call beside the replays
                graph.replay()
                torch.cuda.synchronize()
                assert torch.equal(D, want), "replay %d" % rep


def test_one_k_step():
    """K up to 64, the planner's own choice: matrices of more than two 64x64 tiles per unit run them with one
    group of waves, fewer tiles with two, many with the 128x128 tile; contractions always with one group."""
    for K in (1, 7, 33, 63, 64):
        for (M, N) in ((1700, 1290), (3, 33001), (130, 70)):
            say("%dx%dx%d" % (M, N, K))
            run_unaligned_gemm_case(M, N, K, fg.FG_ROW if K % 2 else fg.FG_COL, fg.FG_COL, pads=(1, 1, 1), bias_dim=1, act=fg.FG_ACT_RELU)
    run_unaligned_gemm_case(1700, 1290, 30, fg.FG_COL, fg.FG_ROW, bf16=True)
    run_unaligned_gemm_case(1700, 1290, 30, fg.FG_ROW, fg.FG_ROW, fg.FG_ROW, ints=False, ab_add=(0.5, -0.25), c_act=fg.FG_ACT_RELU)
    run_unaligned_gemm_case(5001, 4999, 3, fg.FG_COL, fg.FG_COL, pads=(0, 0, 0))
    for ext in ({a: 4, b: 4, d: 4, g: 1500}, {a: 9, b: 5, d: 64, g: 700}, {a: 66, b: 130, d: 33, g: 70}):
        for modes in (([a, d, g], [d, b, g], [a, b, g]), ([g, a, d], [g, d, b], [g, a, b]), ([d, a, g], [d, b, g], [b, a, g])):
            say("batches %s %s" % (ext, modes)); run_contract_case(ext, *modes, ints=True, beta=1.0)
    say("outer product"); run_contract_case({a: 1023, b: 1025}, [a], [b], [a, b], ints=True)


@pytest.mark.parametrize("tile", ["2", "3"])
def test_contraction_forms(monkeypatch, tile):
    """Which direction the pieces run along (rows, summed modes, element by element), leading modes
    that pieces do not divide, several modes per group, batch modes, and strides with gaps that
    hold NaN."""
    setenv(monkeypatch, "FG_FORCE_TILE", tile)
    say("rows x columns"); run_contract_case({a: 13, b: 5, c: 7, d: 11, e: 9, f: 6}, [a, e, b, f], [d, f, c, e], [a, b, c, d], ints=True, beta=1.0)
    say("both along the summed mode"); run_contract_case({a: 70, b: 131, d: 77}, [d, a], [d, b], [a, b], ints=True)
    say("along the summed mode and along columns"); run_contract_case({a: 33, b: 21, d: 13, e: 6}, [d, a, e], [b, e, d], [a, b], ints=True, beta=-1.0)
    say("along two different summed modes"); run_contract_case({a: 33, b: 140, d: 13, e: 11}, [d, e, a], [e, d, b], [a, b], ints=True)
    say("unit modes of extent 2"); run_contract_case({a: 2, b: 3, c: 65, d: 67, e: 9}, [a, c, e], [b, e, d], [a, c, b, d], ints=True)
    say("result along the second row mode"); run_contract_case({a: 9, b: 11, c: 70, d: 65}, [b, d, a], [d, c], [a, b, c], ints=True)
    for (na, nb) in ((4, 9), (11, 8), (3, 20), (70, 17)):
        say("... extents %d and %d" % (na, nb)); run_contract_case({a: na, b: nb, c: 6, d: 13}, [b, d, a], [d, c], [a, b, c], ints=True, beta=1.0)
    say("... three row modes"); run_contract_case({a: 9, b: 21, c: 6, d: 13, e: 5}, [b, d, e, a], [d, c], [a, e, b, c], ints=True, beta=1.0)
    say("... four row modes"); run_contract_case({a: 9, b: 21, c: 6, d: 13, e: 2, f: 3}, [b, d, e, a, f], [d, c], [a, e, b, f, c], ints=True)
    say("batch modes"); run_contract_case({a: 13, b: 9, d: 65, g: 3, f: 2}, [a, d, f, g], [d, b, g, f], [a, g, b, f], ints=True, beta=2.0)
    say("one row"); run_contract_case({b: 70, d: 133}, [d], [b, d], [b], ints=True)
    say("one row, one column"); run_contract_case({d: 300}, [d], [d], [], ints=True)
    say("no summed mode"); run_contract_case({a: 70, b: 133, g: 2}, [a, g], [b, g], [a, b, g], ints=True)
    say("operands of a few elements"); run_contract_case({a: 3, b: 2, d: 2}, [a, d], [d, b], [a, b], ints=True)
    ext = {a: 21, b: 67, c: 3, d: 37}
    for sA, sB in (([1, 23, 23 * 37 + 5], [1, 39]), ([2, 43, 43 * 37], [3, 113]), ([111, 1, 4441], [201, 3])):
        say("strides %s %s" % (sA, sB))
        run_contract_case(ext, [a, d, c], [d, b], [a, b, c], ints=True, beta=1.0, stridesA=sA, stridesB=sB, stridesC=[1, 23, 23 * 67 + 1], poison=True)
    say("floats"); run_contract_case({a: 37, b: 9, c: 11, d: 15, e: 27, f: 25}, [a, e, b, f], [d, f, c, e], [a, b, c, d], alpha=0.5, beta=1.5)
    delenv(monkeypatch, "FG_FORCE_TILE")


@pytest.mark.parametrize("tile", ["2", "3"])
def test_contraction_bases_inside_words_and_chunks(monkeypatch, tile):
    """Bases 1 to 7 elements into 16-byte chunks, so that pieces start inside 4-byte words for every
    combination of the operands; leading extents that are and are not multiples of eight, whose last piece ends
    with the operand; NaN right before and behind A and B."""
    setenv(monkeypatch, "FG_FORCE_TILE", tile)
    for offsets in ((1, 0, 0), (0, 1, 0), (1, 1, 1), (2, 1, 0), (3, 2, 1), (7, 5, 3)):
        for ext in ({a: 13, b: 5, c: 7, d: 11, e: 9, f: 6}, {a: 16, b: 5, c: 7, d: 24, e: 10, f: 8}):
            say("offsets %s rows x columns %s" % (offsets, ext)); run_contract_case(ext, [a, e, b, f], [d, f, c, e], [a, b, c, d], ints=True, beta=1.0, offsets=offsets)
        say("offsets %s dense 16 x 128 beside odd strides" % (offsets,)); run_contract_case({a: 16, b: 65, d: 128}, [a, d], [b, d], [a, b], ints=True, offsets=offsets)
        run_contract_case({a: 16, b: 33, c: 3, d: 128}, [a, d], [b, c, d], [a, b, c], ints=True, offsets=offsets)
        say("offsets %s along the summed mode" % (offsets,)); run_contract_case({a: 33, b: 21, d: 13, e: 6}, [d, a, e], [b, e, d], [a, b], ints=True, beta=-1.0, offsets=offsets)
        run_contract_case({a: 33, b: 21, d: 72, g: 3}, [d, a, g], [d, b, g], [b, a, g], ints=True, offsets=offsets)


@pytest.mark.parametrize("tile", ["2", "3"])
def test_contraction_spans_of_2_31_elements(monkeypatch, tile):
    """Offsets that do not fit 32 bits, between rows, between summed indices and between batches: what the
    strides do not reach is NaN."""
    setenv(monkeypatch, "FG_FORCE_TILE", tile)
    far = (1 << 31) + 6
    for name, ext, mA, sA, mB, sB, mC in (
            ("rows", {a: 21, c: 2, d: 70, b: 67}, [a, d, c], [1, 23, far + 1], [d, b], [1, 71], [a, b, c]),
            ("summed indices, A along rows", {a: 21, d: 70, e: 2, b: 67}, [a, d, e], [1, 23, far], [b, d, e], [1, 69, 69 * 70], [a, b]),
            ("summed indices, A along them", {a: 21, d: 37, e: 2, b: 67}, [d, a, e], [1, 39, far + 1], [d, b, e], [1, 39, 39 * 67], [a, b]),
            ("batches", {a: 21, d: 70, g: 2, b: 67}, [a, d, g], [1, 21, far], [b, d, g], [1, 67, 67 * 70], [a, b, g])):
        say(name)
        shape = lambda ms: [ext[m] for m in ms]
        span = lambda ms, st: 1 + sum((ext[m] - 1) * s for m, s in zip(ms, st))
        A = torch.full((span(mA, sA),), float("nan"), dtype=torch.float16, device="cuda")
        B = torch.full((span(mB, sB),), float("nan"), dtype=torch.float16, device="cuda")
        va, vb = A.as_strided(shape(mA), sA), B.as_strided(shape(mB), sB)
        va.copy_(W.small_ints(va.numel(), 1, device="cuda").view(shape(mA)))
        vb.copy_(W.small_ints(vb.numel(), 2, device="cuda").view(shape(mB)))
        sC = list(W.col_major_strides(tuple(shape(mC))))
        D = torch.full((span(mC, sC),), float("nan"), dtype=torch.float32, device="cuda")
        fg.fg_contract(mA, sA, A, mB, sB, B, mC, sC, None, D, ext)
        torch.cuda.synchronize()
        sums = [m for m in mA if m in mB and m not in mC]
        rows, cols, batch = [m for m in mC if m not in mB], [m for m in mC if m not in mA], [m for m in mC if m in mA and m in mB]
        n = lambda ms: math.prod(shape(ms))
        x = va.cpu().double().permute([mA.index(m) for m in batch + rows + sums]).reshape(n(batch), n(rows), n(sums))
        y = vb.cpu().double().permute([mB.index(m) for m in batch + sums + cols]).reshape(n(batch), n(sums), n(cols))
        order = batch + rows + cols
        want = torch.stack([x[i] @ y[i] for i in range(n(batch))]).reshape(shape(order)).permute([order.index(m) for m in mC])
        got = D.as_strided(shape(mC), sC).cpu().double()
        del A, B, va, vb
        torch.cuda.empty_cache()
        assert torch.equal(got, want), name


@pytest.mark.parametrize("tile", ["2", "3"])
def test_contraction_infinities_and_nan(monkeypatch, tile):
    """NaN and infinities inside A, B and Cin reach exactly the results they belong to, in every direction
    that pieces run along, with K tails and rounded leading modes."""
    setenv(monkeypatch, "FG_FORCE_TILE", tile)
    inf, nan = float("inf"), float("nan")
    for K in (13, 70, 133):
        M, N = 21, 67
        for mA, mB in (([a, d], [b, d]), ([d, a], [d, b]), ([d, a], [b, d]), ([a, d], [d, b])):
            say("K=%d A%s B%s" % (K, mA, mB))
            x, y, z = (W.small_ints(n, i, device="cpu").double() for i, n in ((1, M * K), (2, K * N), (3, M * N)))
            x, y, z = x.view(M, K), y.view(K, N) + 9, z.view(M, N)          # B has no zeros
            x[3, 5], x[8, K - 1], x[M - 1, 0], y[2, 6], y[K - 1, N - 1], z[0, 1] = inf, nan, -inf, inf, nan, nan
            want = x @ y + 2 * z
            ext = {a: M, b: N, d: K}
            stored = lambda t, lab, modes: (t if modes[0] != lab else t.T).contiguous().reshape(-1)      # first mode fastest
            A = stored(x, a, mA).to(torch.float16).cuda(); B = stored(y, d, mB).to(torch.float16).cuda()
            Cin = z.T.contiguous().reshape(-1).float().cuda()
            D = torch.zeros(M * N, dtype=torch.float32, device="cuda")
            st = lambda ms: [1, ext[ms[0]]]
            fg.fg_contract(mA, st(mA), A, mB, st(mB), B, [a, b], [1, M], Cin, D, ext, beta=2.0)
            torch.cuda.synchronize()
            got = D.view(N, M).T.cpu().double()
            assert torch.equal(torch.isnan(got), torch.isnan(want))
            assert torch.equal(torch.nan_to_num(got, nan=7.0), torch.nan_to_num(want, nan=7.0))


def float_result(M, N, K, la, lb, **kw):
    A = W.uniform_pm1(M * K, 1, device="cuda"); B = W.uniform_pm1(K * N, 2, device="cuda")
    D = torch.full((M * N,), float("nan"), dtype=torch.float32, device="cuda")
    fg.fg_gemm(M, N, K, 1.0, fg.Matrix(A, la, M if la == fg.FG_COL else K), fg.Matrix(B, lb, K if lb == fg.FG_COL else N), 0.0, None, fg.Matrix(D, fg.FG_COL, M), **kw)
    torch.cuda.synchronize()
    return D


def test_k_group_kernels_run(monkeypatch):
    """One K group, two that take equal runs of the K tiles (ring of two) and two that take them in turns (ring of four) add the
    same products up in different orders: on floats the three tiles differ in the last bits (plan names do not tell them
    apart), so a tile that silently ran as another one is seen; the planner's choice at 1024^3 is the ring of four, and for
    fewer than 56 tiles of twelve to fifteen K tiles, which wait for nothing, the ring of two."""
    for la, lb in itertools.product(LAYOUTS, LAYOUTS):
        got = {}
        for tile in ("3", "6", "7"):
            setenv(monkeypatch, "FG_FORCE_TILE", tile)
            got[tile] = float_result(1024, 1024, 1024, la, lb)
        delenv(monkeypatch, "FG_FORCE_TILE")
        say("A=%d B=%d" % (la, lb))
        assert not torch.equal(got["3"], got["6"]) and not torch.equal(got["3"], got["7"]) and not torch.equal(got["6"], got["7"])
        assert torch.equal(float_result(1024, 1024, 1024, la, lb), got["7"])
        for M, N, tile in ((184, 104, "6"), (64, 1728, "6"), (1024, 512, "7")):
            small = {}
            for t in ("6", "7"):
                setenv(monkeypatch, "FG_FORCE_TILE", t)
                small[t] = float_result(M, N, 864, la, lb)
            delenv(monkeypatch, "FG_FORCE_TILE")
            assert not torch.equal(small["6"], small["7"]) and torch.equal(float_result(M, N, 864, la, lb), small[tile]), (M, N)


@pytest.mark.parametrize("tile", ["6", "7", "8"])
def test_k_groups(monkeypatch, tile):
    """The tiles whose two groups of waves share their K tiles (tiled kernels): fewer K tiles than
    groups, runs that do not come out even, a K tail in the last group's last and last but one tile,
    several tiles per workgroup, K splits, and every option of the families."""
    from tests.parity import run_gemm_case
    setenv(monkeypatch, "FG_FORCE_TILE", tile)
    for la, lb in itertools.product(LAYOUTS, LAYOUTS):
        for K in (8, 64, 72, 128, 200, 264, 320, 456, 520, 568, 1032):
            say("tile %s K=%d A=%d B=%d" % (tile, K, la, lb))
            run_gemm_case(131, 70, K, la, lb, ints=True, pad=8, poison=True, bias_dim=0)
            run_gemm_case(131, 70, K, la, lb, fg.FG_ROW, ints=True, ab_add=(3.0, -1.0), c_act=fg.FG_ACT_RELU, act=fg.FG_ACT_RELU)
        run_gemm_case(200, 130, 456, la, lb, ints=True, bf16=True, pad=8)
        run_gemm_case(200, 130, 456, la, lb, ints=True, cd16=True, pad=8, bias_dim=1)
    say("several tiles per workgroup"); run_gemm_case(2100, 1400, 328, ints=True, beta=-2.0)
    for S in (2, 3, 5):
        setenv(monkeypatch, "FG_FORCE_SPLIT", str(S))
        say("tile %s split %d" % (tile, S)); run_gemm_case(131, 200, 1160, fg.FG_ROW, fg.FG_COL, ints=True, bias_dim=1, act=fg.FG_ACT_RELU, pad=8, poison=True)
        run_gemm_case(131, 200, 1160, ints=True, ab_add=(1.0, 2.0))
    delenv(monkeypatch, "FG_FORCE_SPLIT")
    delenv(monkeypatch, "FG_FORCE_TILE")
    say("planner's own choice, floats"); run_gemm_case(1024, 1024, 2048); run_gemm_case(1500, 1000, 2048, fg.FG_ROW, fg.FG_COL, bf16=True)
