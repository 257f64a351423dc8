"""CPU test of the kernels as they were compiled: what hand-written assembly hides from the compiler is looked for in the disassembly of
the library (csrc/ as built by paper_2009_12263_amd/build.py)."""
import os
import re
import struct
import subprocess

import pytest

from paper_2009_12263_amd import build

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{name: instructions} of every kernel; an instruction is (mnemonic, operands)."""
    if not os.path.exists(build.LIB):
        build.build()
    d = tmp_path_factory.mktemp("code")
    subprocess.run([LLVM + "/llvm-objcopy", "-O", "binary", "--dump-section", ".hip_fatbin=%s" % (d / "fat"), build.LIB, os.devnull], check=True)
    data = (d / "fat").read_bytes()
    found = {}
    for at in (m.start() for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data)):
        n, = struct.unpack_from("<Q", data, at + 24)
        o = at + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, o)
            target = data[o + 24:o + 24 + length]
            o += 24 + length
            if b"gfx950" not in target or not size:
                continue
            (d / "co").write_bytes(data[at + off:at + off + size])
            text = subprocess.run([LLVM + "/llvm-objdump", "-d", "--no-show-raw-insn", str(d / "co")], check=True, stdout=subprocess.PIPE, text=True).stdout
            for line in text.splitlines():
                if line.startswith("\t"):
                    op, _, rest = line.split("//", 1)[0].strip().partition(" ")
                    code.append((op, rest.strip()))
                elif line.endswith(">:"):
                    code = found[line[line.index("<") + 1:-2]] = []
    assert len(found) > 150
    return found


def _registers(operand):
    """v[4:7] -> {("v", 4) .. ("v", 7)}"""
    m = re.fullmatch(r"\|?-?([vsa])(?:(\d+)|\[(\d+):(\d+)\])\|?", operand.strip())
    if not m:
        return set()
    lo, hi = (int(m[2]), int(m[2])) if m[2] else (int(m[3]), int(m[4]))
    return {(m[1], i) for i in range(lo, hi + 1)}


def _wait_states(op, rest):
    return int(rest) + 1 if op == "s_nop" else 1


def _too_close(code, writes, reads, least):
    """Pairs of instructions, fewer than `least` wait states apart, of which the first writes a register that the second reads."""
    out = []
    for i, (op, rest) in enumerate(code):
        need = reads(op, rest)
        if not need:
            continue
        passed, j = 0, i - 1
        while j >= 0 and passed < least:
            wrote = writes(*code[j])
            if wrote & need:
                out.append((code[j], code[i]))
                break
            passed += _wait_states(*code[j])
            j -= 1
    return out


def test_lane_exchanges_wait_for_vector_results(kernels):
    """v_permlane16_swap / v_permlane32_swap need two wait states after a vector instruction that writes what they read."""
    def writes(op, rest):
        if not op.startswith("v_") or op.startswith(("v_cmp", "v_nop")):
            return set()
        return _registers(rest.split(",")[0])

    def reads(op, rest):
        return set().union(*(_registers(r) for r in rest.split(","))) if op.startswith("v_permlane") and "swap" in op else set()
    seen = 0
    for name, code in kernels.items():
        seen += sum(op.startswith("v_permlane") for op, _ in code)
        bad = _too_close(code, writes, reads, 2)
        assert not bad, "%s: %d lane exchanges right behind the result they read, first %s" % (name, len(bad), bad[0])
    assert seen > 10000


def test_matrix_instructions_wait_for_vector_results(kernels):
    """A matrix instruction needs two wait states after another vector instruction that writes what it reads; those of the kernels with
    four waves are assembly."""
    def writes(op, rest):
        if not op.startswith("v_") or op.startswith(("v_cmp", "v_nop", "v_mfma")):
            return set()
        return {r for r in _registers(rest.split(",")[0]) if r[0] != "s"}

    def reads(op, rest):
        return set().union(*(_registers(r) for r in rest.split(",")[1:])) if op.startswith("v_mfma") else set()
    for name, code in kernels.items():
        bad = _too_close(code, writes, reads, 2)
        assert not bad, "%s: %d matrix instructions right behind the result they read, first %s" % (name, len(bad), bad[0])


def test_loads_wait_for_descriptors_that_vector_instructions_write(kernels):
    """A vector memory instruction needs five wait states after a vector instruction (the reload of a spill) that writes a scalar
    register it reads."""
    def writes(op, rest):
        return {r for r in _registers(rest.split(",")[0]) if r[0] == "s"} if op.startswith("v_") else set()

    def reads(op, rest):
        if not op.startswith(("buffer_", "global_", "flat_", "scratch_")):
            return set()
        return {r for operand in rest.split(",") for r in _registers(operand.split()[0]) if r[0] == "s"}
    seen = 0
    for name, code in kernels.items():
        seen += sum(op.startswith("buffer_") and rest.endswith(" lds") for op, rest in code)
        bad = _too_close(code, writes, reads, 5)
        assert not bad, "%s: %d accesses right behind the reload of a register they read, first %s" % (name, len(bad), bad[0])
    assert seen > 10000


def test_accumulators_belong_to_the_assembly(kernels):
    """The kernels with four waves keep their results in accumulation registers that the compiler knows nothing of (csrc/wide_loop.hpp): it
    must have no use of its own for one.  All that touches them is their clearing, once each, the matrix instructions, which add
    to what they hold, and the reads of the epilogues."""
    wide = {name: code for name, code in kernels.items() if "11gemm_kernelI" in name and "Lb1EEEEEvNT_" in name}       # TileCfg::WIDE
    assert len(wide) == 36                     # three tiles, four layouts; FP16, bfloat16 and binary16 results
    for name, code in wide.items():
        cleared, read = [], set()
        for op, rest in code:
            operands = [o.strip() for o in rest.split(",")]
            touched = [o for o in operands if any(r[0] == "a" for r in _registers(o.split()[0] if o else o))]
            if not touched:
                continue
            if op == "v_accvgpr_write_b32":
                assert operands[1] == "0", (name, op, rest)
                cleared += _registers(operands[0])
            elif op == "v_accvgpr_read_b32":
                read |= _registers(operands[1])
            else:
                assert op.startswith("v_mfma_f32_16x16x32_") and touched == [operands[0], operands[3]] and operands[0] == operands[3], (name, op, rest)
        assert sorted(cleared) == [("a", i) for i in range(len(cleared))] and len(cleared) in (128, 256), name
        assert read == set(cleared), name
