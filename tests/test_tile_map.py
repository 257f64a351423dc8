"""The tile that a workgroup computes (csrc/tile_map.hpp), compiled for the CPU: the form with prepared divisions gives what the plain
one does, every tile is computed once, and the divisions are exact."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2009_12263_amd", "csrc")

PROGRAM = r"""
#include "tile_map.hpp"
#include <cstdio>
#include <vector>
int main() {
    for (int m = 1; m <= 41; ++m)
        for (int n = 1; n <= 70; n += n < 20 ? 1 : 7) {
            std::vector<char> seen(m * n, 0);
            const fg::Division d = fg::tile_group(m, n);
            for (int b = 0; b < m * n; ++b) {
                int tm, tn, um, un;
                fg::block_to_tile(b, m, n, tm, tn);
                fg::block_to_tile(b, m, n, d, um, un);
                if (tm != um || tn != un || tm < 0 || tm >= m || tn < 0 || tn >= n || seen[tm + m * tn]++) { printf("%d x %d, workgroup %d\n", m, n, b); return 1; }
            }
        }
    for (int m : {1, 2, 3, 4, 5, 1000, 30000, 1 << 20})
        for (int n : {1, 3, 7, 33, 1500, 2000})
            for (long k = 0, nb = (long)m * n; k < 1000; ++k) {
                if (nb >= 1l << 31) break;
                int tm, tn, um, un;
                const int b = (int)(nb * k / 1000);
                fg::block_to_tile(b, m, n, tm, tn);
                fg::block_to_tile(b, m, n, fg::tile_group(m, n), um, un);
                if (tm != um || tn != un) { printf("%d x %d, workgroup %d\n", m, n, b); return 1; }
            }
    for (unsigned d = 1; d < 5000; ++d)
        for (unsigned x : {0u, 1u, d - 1, d, d + 1, 2 * d - 1, 1000003u, 0x7fffffffu, 0x7fffffffu - d, 0x7fffffffu / d * d, 0x7fffffffu / d * d - 1})
            if (fg::divided((int)x, fg::division_by(d)) != (int)(x / d)) { printf("%u / %u\n", x, d); return 1; }
    for (unsigned d : {65535u, 65536u, 65537u, 1u << 20, (1u << 24) + 1, 1u << 30, 0x7fffffffu})
        for (unsigned x : {0u, d - 1, d, 0x7fffffffu, 0x40000000u})
            if (fg::divided((int)x, fg::division_by(d)) != (int)(x / d)) { printf("%u / %u\n", x, d); return 1; }
    puts("ok");
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("tile_map")
    src, exe = d / "t.cpp", d / "t"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return str(exe)


def test_tiles_with_prepared_divisions(program):
    r = subprocess.run([program], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout
