"""CPU test of the size of a descriptor (csrc/operand_window.hpp, compiled with the host compiler): over operands up to 8 GiB a masked
lane's offset is out of range, and a lane's own offset is in range exactly where the operand has a piece."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2009_12263_amd", "csrc")

PROGRAM = r"""
#include "operand_window.hpp"
#include <cstdio>
#include <initializer_list>
using namespace fg;
int main() {
    // rows, K and leading dimension of K-contiguous operands; the descriptor of the last K tile of each panel of 256 rows
    const int64_t shapes[][3] = {{320, 4194248, 4194248}, {300000, 8200, 8200}, {70000, 16392, 16448}, {256, 4000072, 4194296}, {1, 8, 8}, {300, 136, 144}, {500000, 4104, 4104}};
    for (auto &s : shapes) {
        const int64_t rows = s[0], K = s[1], ld = s[2], span = ((rows - 1) * ld + K + 7) / 8 * 8;
        for (int64_t row0 = 0; row0 < rows; row0 += 256) {
            const int64_t rest = (span - row0 * ld - (K - 1) / 64 * 64) * 2;
            const uint32_t size = window_bytes(rest);
            if ((uint64_t)kOutOfRange < size) { printf("%ld x %ld, row %ld: a masked lane is in range of %u bytes\n", (long)rows, (long)K, (long)row0, size); return 1; }
            for (int64_t r : {0, 1, 31, 127, 255}) {
                const int64_t at = r * ld * 2;
                if (at + 16 >= (1ll << 31)) continue;               // what the host refuses
                if ((at + 16 <= rest) != (at + 16 <= (int64_t)size)) { printf("%ld x %ld, row %ld + %ld\n", (long)rows, (long)K, (long)row0, (long)r); return 1; }
            }
        }
    }
    for (int64_t rest : {-(1ll << 40), -1ll, 0ll}) if (window_bytes(rest) != 0) return 1;
    for (int64_t rest : {1ll, 16ll, 0x7fffffffll}) if (window_bytes(rest) != (uint32_t)rest) return 1;
    for (int64_t rest : {0x80000000ll, 0xfffffff0ll, 0x100000000ll, 1ll << 40}) if (window_bytes(rest) != 0x7fffffffu) return 1;
    puts("ok");
}
"""


def test_masked_lanes_are_out_of_range(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout
