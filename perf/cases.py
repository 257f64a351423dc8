"""The work that users of this library have it do, as cases that can be timed and checked.

A case is one call of a public entry point (``fg_gemm``, ``fg_gemm_dual`` or ``fg_contract``) on
operands that are already on the GPU, with the result buffer that a program keeps.  Entries are
uniform in [-1, 1), as in the workloads of ``paper_2009_12263_amd.workloads``.

Keys of a matrix case: ``M, N, K``; ``a, b, d`` the storage of A, B and C/D ("N": column-major, "T":
row-major); ``kind`` "real", "complex" (planar), "interleaved", "dual", "diag" (A diagonal);
``dtype`` of A and B; ``cd`` of C and D; ``c``: there is a C operand; ``bias`` "", "M" or "N"; ``relu``;
``add``: a constant is added to the loaded A and B and the loaded C is clamped (the paper's fusion
table); ``tight``: leading dimensions equal the extents, whatever they are (otherwise they are
rounded up to whole 16-byte chunks).  Keys of a contraction: ``spec`` (A,B->C, first mode fastest)
and ``ext``, the extents.
"""
import math

import torch

from paper_2009_12263_amd import binding as fg


def gemm(M, N, K, a="N", b="N", d="N", kind="real", dtype="f16", cd="f32", c=True, bias="", relu=False, add=False, tight=False,
         alpha=1.0, beta=1.0):
    return dict(M=M, N=N, K=K, a=a, b=b, d=d, kind=kind, dtype=dtype, cd=cd, c=c, bias=bias, relu=relu, add=add, tight=tight,
                alpha=alpha, beta=beta)


def contraction(spec, ext, beta=0.0):
    return dict(spec=spec, ext=" ".join("%s=%d" % kv for kv in sorted(ext.items())), beta=beta)


def listed():
    return [
        # the smallest call: a program with many little products, bound by the launch
        dict(gemm(256, 256, 256), name="square_256"),
        # the middle of the square sweep, rows of K on the left, columns of N on the right
        dict(gemm(1024, 1024, 1024, "T", "T"), name="square_1024_tt"),
        # a linear layer in bfloat16: activations and weights with K contiguous, row-major result, bias
        dict(gemm(2048, 2048, 2048, "T", "N", "T", dtype="bf16", c=False, bias="N"), name="linear_bf16_2048"),
        # the headline: large square product with C, the case that fills the chip
        dict(gemm(8192, 8192, 8192), name="square_8192"),
        # fused bias and ReLU on a rectangular product of one round of tiles
        dict(gemm(8192, 1024, 4096, c=False, bias="M", relu=True), name="relu_bias_8192x1024x4096"),
        # a narrow batch against a large weight matrix: bound by reading that matrix, K has to be split
        dict(gemm(128, 4096, 16384), name="skinny_128x4096x16384"),
        # sizes as data has them: nothing a multiple of anything, leading dimensions equal to the extents
        dict(gemm(1531, 1021, 2003, tight=True), name="odd_1531x1021x2003"),
        # complex product, planar storage
        dict(gemm(4096, 4096, 4096, kind="complex"), name="complex_4096"),
        # diagonal scaling of a matrix: memory traffic only
        dict(gemm(4096, 4096, 4096, kind="diag"), name="diag_4096"),
        # tensor times matrix along the middle mode
        dict(contraction("adc,db->abc", dict(a=256, b=256, c=256, d=256)), name="contract_3mode_256"),
        # two four-mode tensors, two summed modes
        dict(contraction("aebf,dfce->abcd", dict(a=64, b=64, c=64, d=64, e=64, f=64)), name="contract_4mode_64"),
        # the same with extents as a problem has them
        dict(contraction("aebf,dfce->abcd", dict(a=37, b=29, c=31, d=35, e=27, f=25)), name="contract_4mode_odd"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _sizes(rng, lo, hi, flops, k_step, per=2):
    """M, N, K spread over their logarithm, the product at most `flops`."""
    while True:
        M, N, K = (_log(rng, lo, hi) for _ in range(3))
        if rng.random() < 0.3:                      # round sizes are common
            M, N = max(64, M // 64 * 64), max(64, N // 64 * 64)
        K = max(k_step, K // k_step * k_step)
        if 1e6 < per * M * N * K <= flops:
            return M, N, K


_SPECS = ("adc,db->abc", "aebf,dfce->abcd", "bda,dc->abc", "adg,dbg->abg", "dac,db->abc", "ad,bd->ba")


def draw(rng):
    pick = lambda *xs: rng.choice(xs)  # noqa: E731
    kind = rng.random()
    if kind < 0.34:                                 # real products over the sweep's range
        M, N, K = _sizes(rng, 64, 8192, 5e11, 8)
        dtype, cd, add = pick("f16", "f16", "bf16"), "f32", False
        if dtype == "f16":
            cd, add = pick(("f32", False), ("f32", False), ("f32", True), ("f16", False))
        return gemm(M, N, K, pick("N", "T"), pick("N", "T"), pick("N", "T"), dtype=dtype, cd=cd, add=add, c=pick(True, False),
                    bias=pick("", "M", "N"), relu=pick(True, False), alpha=pick(1.0, 0.5), beta=pick(1.0, -0.5))
    if kind < 0.44:                                 # few rows or columns, long K
        small, large, K = _log(rng, 8, 512), _log(rng, 256, 8192), _log(rng, 2048, 16384) // 8 * 8
        M, N = pick((small, large), (large, small))
        return gemm(M, N, K, pick("N", "T"), pick("N", "T"), pick("N", "T"), dtype=pick("f16", "bf16"), c=pick(True, False), bias=pick("", "N"))
    if kind < 0.60:                                 # any sizes, leading dimensions equal to the extents
        M, N, K = _sizes(rng, 48, 3000, 6e9, 1)
        return gemm(M | 1, N, K | 1, pick("N", "T"), pick("N", "T"), pick("N", "T"), dtype=pick("f16", "bf16"), c=pick(True, False),
                    bias=pick("", "M"), relu=pick(True, False), tight=True)
    if kind < 0.74:                                 # complex and dual numbers
        M, N, K = _sizes(rng, 128, 4096, 5e11, 8, per=8)
        return gemm(M, N, K, pick("N", "T"), pick("N", "T"), pick("N", "T"), kind=pick("complex", "interleaved", "dual"), c=pick(True, False))
    if kind < 0.80:                                 # diagonal scaling
        M, N = _log(rng, 256, 8192), _log(rng, 256, 8192)
        K = (M + 7) // 8 * 8
        return gemm(M, N, K, "N", pick("N", "T"), pick("N", "T"), kind="diag", c=pick(True, False))
    spec = pick(*_SPECS)
    odd = kind > 0.91
    labels = sorted(set(spec) - set(",->"))
    hi = {2: 3000, 3: 2000, 4: 320, 6: 48}[min(6, len(labels) if len(labels) != 5 else 6)]
    lo = {2: 64, 3: 64, 4: 24, 6: 10}[min(6, len(labels) if len(labels) != 5 else 6)]
    while True:
        ext = {m: _log(rng, lo, hi) for m in labels}
        for m in labels:
            ext[m] = ext[m] | 1 if odd else max(8, ext[m] // 8 * 8)
        flops = 2.0 * math.prod(ext.values())
        if 1e6 < flops < (1.5e9 if odd else 1.2e11):
            return contraction(spec, ext, beta=pick(0.0, 0.0, 1.0))


def is_contraction(case):
    return "spec" in case


# ---- matrices -----------------------------------------------------------------------------------

_HALF = {"f16": torch.float16, "bf16": torch.bfloat16}
_COMPLEX = ("complex", "interleaved", "dual")


def _uniform(gen, n, dtype):
    return (torch.rand(n, generator=gen, device="cuda") * 2 - 1).to(dtype)


def _lead(extent, tight, chunk):
    return extent if tight else (extent + chunk - 1) // chunk * chunk


def _matrix(gen, rows, cols, layout, dtype, planes, tight, interleaved=False):
    """A stored matrix: its fg.Matrix and the logical rows x cols planes as views of the same memory."""
    lead, other = (rows, cols) if layout == "N" else (cols, rows)
    chunk = 1 if dtype is None else (4 if dtype == torch.float32 else 8)
    ld = _lead(lead, tight, chunk)
    lay = fg.FG_COL if layout == "N" else fg.FG_ROW
    n = ld * other
    new = (lambda k: _uniform(gen, k, dtype)) if gen is not None else (lambda k: torch.zeros(k, dtype=dtype, device="cuda"))

    def view(t):
        t = t.view(other, ld)[:, :lead]
        return t.T if layout == "N" else t
    if interleaved:
        t = new(2 * n)
        both = t.view(n, 2)
        code = fg.FG_CF32 if dtype == torch.float32 else fg.FG_CF16
        return fg.Matrix(t, lay, ld, dtype=code), [view(both[:, 0]), view(both[:, 1])]
    ts = [new(n) for _ in range(planes)]
    return fg.Matrix(ts[0], lay, ld, im=ts[1] if planes == 2 else None), [view(t) for t in ts]


def _prepare_gemm(case, gen):
    M, N, K = case["M"], case["N"], case["K"]
    half = _HALF[case["dtype"]]
    cd = torch.float16 if case["cd"] == "f16" else torch.float32
    planes = 2 if case["kind"] in _COMPLEX else 1
    il, tight = case["kind"] == "interleaved", case["tight"]
    if case["kind"] == "diag":
        t = _uniform(gen, min(M, K), half)
        A, a = fg.Matrix(t, fg.FG_DIAG, 0), [t]
    else:
        A, a = _matrix(gen, M, K, case["a"], half, planes, tight, il)
    B, b = _matrix(gen, K, N, case["b"], half, planes, tight, il)
    C, c = _matrix(gen, M, N, case["d"], cd, planes, tight, il) if case["c"] else (None, None)
    D, d = _matrix(None, M, N, case["d"], cd, planes, tight, il)
    bias = _uniform(gen, M if case["bias"] == "M" else N, torch.float32) if case["bias"] else None
    call = dict(bias=bias, bias_dim=0 if case["bias"] == "M" else 1, act=fg.FG_ACT_RELU if case["relu"] else fg.FG_ACT_NONE)
    if case["add"]:
        call.update(a_add=0.25, b_add=-0.5, c_act=fg.FG_ACT_RELU if case["c"] else fg.FG_ACT_NONE)
    return dict(size=(M, N, K), alpha=case["alpha"], beta=case["beta"], A=A, B=B, C=C, D=D, call=call, dual=case["kind"] == "dual",
                out=tuple(d) if planes == 2 else d[0], a=a, b=b, c=c, bias=bias)


def _exact_gemm(case, s):
    f8 = lambda t: t.to(torch.float64)  # noqa: E731
    b = [f8(t) for t in s["b"]]
    if case["kind"] == "diag":
        n = s["a"][0].numel()
        y = torch.zeros(case["M"], case["N"], dtype=torch.float64, device="cuda")
        y[:n] = f8(s["a"][0])[:, None] * b[0][:n]
        ys = [y]
    else:
        a = [f8(t) for t in s["a"]]
        if case["add"]:                             # formed and rounded once in binary16, as the entry point says
            a, b = [f8(s["a"][0] + 0.25)], [f8(s["b"][0] - 0.5)]
        if case["kind"] in ("complex", "interleaved"):
            ys = [a[0] @ b[0] - a[1] @ b[1], a[0] @ b[1] + a[1] @ b[0]]
        elif case["kind"] == "dual":
            ys = [a[0] @ b[0], a[0] @ b[1] + a[1] @ b[0]]
        else:
            ys = [a[0] @ b[0]]
    ys = [y * case["alpha"] for y in ys]
    if case["c"]:
        for i, y in enumerate(ys):
            c = f8(s["c"][i])
            y += case["beta"] * (c.clamp_min(0) if case["add"] else c)
    if s["bias"] is not None:
        ys[0] += f8(s["bias"])[:, None] if case["bias"] == "M" else f8(s["bias"])[None, :]
    if case["relu"]:
        ys[0].clamp_min_(0)
    return tuple(ys) if len(ys) == 2 else ys[0]


# ---- contractions -------------------------------------------------------------------------------

def _modes(case):
    ins, c = case["spec"].split("->")
    a, b = ins.split(",")
    return a, b, c, {m: int(v) for m, v in (kv.split("=") for kv in case["ext"].split())}


def _tensor(gen, modes, ext, dtype):
    """A dense tensor, first mode fastest: its memory, its strides and its logical view."""
    shape = [ext[m] for m in modes]
    n = math.prod(shape)
    t = _uniform(gen, n, dtype) if gen is not None else torch.zeros(n, dtype=dtype, device="cuda")
    strides, st = [], 1
    for e in shape:
        strides.append(st)
        st *= e
    return t, strides, t.as_strided(shape, strides)


def _prepare_contraction(case, gen):
    a, b, c, ext = _modes(case)
    A, sA, va = _tensor(gen, a, ext, torch.float16)
    B, sB, vb = _tensor(gen, b, ext, torch.float16)
    Cin, sC, vc = _tensor(gen, c, ext, torch.float32) if case["beta"] else (None, None, None)
    Cout, sC, vd = _tensor(None, c, ext, torch.float32)
    lab = lambda ms: [ord(m) for m in ms]  # noqa: E731
    args = (lab(a), sA, A, lab(b), sB, B, lab(c), sC, Cin, Cout, {ord(m): e for m, e in ext.items()})
    return dict(args=args, beta=case["beta"], out=vd, a=va, b=vb, c=vc)


def _exact_contraction(case, s):
    a, b, c, ext = _modes(case)
    batch = [m for m in c if m in a and m in b]
    rows, cols = [m for m in c if m in a and m not in b], [m for m in c if m in b and m not in a]
    sums = [m for m in a if m in b and m not in c]
    size = lambda ms: math.prod([ext[m] for m in ms])  # noqa: E731
    x = s["a"].to(torch.float64).permute([a.index(m) for m in batch + rows + sums]).reshape(size(batch), size(rows), size(sums))
    y = s["b"].to(torch.float64).permute([b.index(m) for m in batch + sums + cols]).reshape(size(batch), size(sums), size(cols))
    z = torch.stack([x[i] @ y[i] for i in range(size(batch))])
    order = batch + rows + cols
    z = z.reshape([ext[m] for m in order]).permute([order.index(m) for m in c])
    if case["beta"]:
        z = z + case["beta"] * s["c"].to(torch.float64)
    return z


# ---- the cases' interface -----------------------------------------------------------------------

def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return (_prepare_contraction if is_contraction(case) else _prepare_gemm)(case, gen)


def run(s):
    if "args" in s:
        fg.fg_contract(*s["args"], beta=s["beta"])
    else:
        M, N, K = s["size"]
        if s["dual"]:
            fg.fg_gemm_dual(M, N, K, s["alpha"], s["A"], s["B"], s["beta"], s["C"], s["D"])
        else:
            fg.fg_gemm(M, N, K, s["alpha"], s["A"], s["B"], s["beta"], s["C"], s["D"], **s["call"])
    return s["out"]


def work(case):
    if is_contraction(case):
        a, b, c, ext = _modes(case)
        size = lambda ms: math.prod([ext[m] for m in ms])  # noqa: E731
        return {"bytes": 2 * (size(a) + size(b)) + 4 * size(c) * (2 if case["beta"] else 1), "flops": 2 * math.prod(ext.values())}
    M, N, K = case["M"], case["N"], case["K"]
    planes = 2 if case["kind"] in _COMPLEX else 1
    cd = 2 if case["cd"] == "f16" else 4
    if case["kind"] == "diag":
        n = min(M, K)
        return {"bytes": 2 * n + 2 * n * N + cd * M * N * (2 if case["c"] else 1), "flops": n * N}
    per = {"complex": 8, "interleaved": 8, "dual": 6}.get(case["kind"], 2)
    return {"bytes": planes * (2 * (M * K + K * N) + cd * M * N * (2 if case["c"] else 1)), "flops": per * M * N * K}


def tolerance(case):
    """Four times the largest error against 64 bits measured over the listed and drawn cases: 8e-7
    for sums in 32 bits (K up to 16384, in whatever order), 2.1e-4 for results stored as binary16."""
    return {"rel": 1e-3} if case.get("cd") == "f16" else {"rel": 4e-6}


def exact(case, seed):
    s = prepare(case, seed)
    return (_exact_contraction if is_contraction(case) else _exact_gemm)(case, s)
