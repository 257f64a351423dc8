"""CPU test of the rules that say which accesses of the matrix kernels carry the streaming policy: the header that the
library uses is compiled with the host compiler."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2009_12263_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include "cache_policy.hpp"
int main(int n, char **v) {
    auto num = [&](int i) { return (long long)strtoll(v[i], nullptr, 10); };
    (void)n;
    if (!strcmp(v[1], "once")) printf("%d\n", (int)fg::streams_once((uint64_t)num(2), num(3), num(4)));
    if (!strcmp(v[1], "real")) printf("%d\n", (int)fg::keeps_real_cd(num(2), num(3), num(4) != 0, num(5), num(6)));
    if (!strcmp(v[1], "complex")) printf("%d\n", (int)fg::keeps_complex_cd(num(2), num(3), num(4), num(5) != 0, num(6) != 0, num(7), num(8)));
    return 0;
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("cache_policy")
    (d / "t.cpp").write_text(PROGRAM)
    subprocess.check_call([cxx, "-O1", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(d / "t.cpp"), "-o", str(d / "t")])
    return lambda *args: int(subprocess.check_output([str(d / "t")] + [str(int(a)) if not isinstance(a, str) else a for a in args]))


def test_only_operands_that_no_cache_can_hold_stream(rule):
    """What the memory-side cache (256 MB) may still hold, from the call before or from the kernel that wrote it, is not
    streamed: 128 x 4096 x 16384 and 128 x 8320 x 16384 (128 and 260 MB) do not stream, 128 x 16384 x 12288 (384 MB) does, and the
    operands of test_operands_that_are_read_once do."""
    MB = 1 << 20
    for mb, streams in ((64, 0), (128, 0), (192, 0), (256, 0), (260, 0), (383, 0), (384, 1), (1187, 1)):
        assert rule("once", 4096, 16384, mb * MB) == streams, mb
    assert rule("once", 4096 + 64, 16384, 1024 * MB) == 0 and rule("once", 4096, 16384 + 32, 1024 * MB) == 0      # rows off the lines
    assert rule("once", 4096, 16448, 12296 * 16392 * 2) == 1 and rule("once", 4096, 12352, 12296 * 16392 * 2) == 1
    assert rule("once", 4096, 8256, 24648 * 8200 * 2) == 1 and rule("once", 4096, 24704, 24648 * 8200 * 2) == 1


def test_real_results_above_the_memory_side_cache_are_kept_only_off_the_half_lines(rule):
    """(M, N, K), element size of C and D, leading dimension: C and D beside small A and B are kept if their columns begin inside
    half lines, streamed if they begin on whole or half ones; without C they stream; what fits the cache is kept."""
    def keeps(M, N, K, es, ld, c=True):
        return rule("real", (M * K + K * N) * 2, M * N * es * (2 if c else 1), c, ld * es, ld * es)
    for M, ld_off, kept in ((8144, 0, 0), (8144, 16, 0), (8136, 8, 1), (8140, 4, 1), (8152, 24, 1)):
        ld = M // 32 * 32 + ld_off
        assert keeps(ld, 5000, 1040, 4, ld) == kept, ld
        assert keeps(ld, 5000, 1040, 4, ld, c=False) == 1                   # 163 MB and operands: fits
        assert keeps(ld, 9000, 1040, 4, ld, c=False) == 0
        assert keeps(ld, 5000, 9000, 4, ld) == 0                            # A and B 225 MB
    for off, kept in ((0, 0), (32, 0), (16, 1), (8, 1)):
        assert keeps(9984 + off, 9000, 400, 2, 9984 + off) == kept, off
    assert keeps(3000, 3000, 3000, 4, 3000) == 1 and keeps(8192, 8192, 8192, 4, 8192) == 0


def test_complex_results_of_short_passes_stream(rule):
    """Complex and dual results on the lines with C: kept up to 80 MB, but streamed where the whole pass is 7 to 16 MB and K at
    most 256; off the lines kept; above 80 MB kept only off the lines beside small A and B."""
    def keeps(M, N, K, ilv=0, c=True, off=0):
        ld = M + off
        return rule("complex", (M * K + K * N) * 4, M * N * 8 * (2 if c else 1), K, ilv, c, ld * (8 if ilv else 4), ld * (8 if ilv else 4))
    assert keeps(1440, 613, 136) == 0 and keeps(1216, 544, 200) == 0 and keeps(704, 810, 120, ilv=1) == 0       # 9 to 14 MB
    assert keeps(640, 256, 176, ilv=1) == 1 and keeps(320, 1024, 120) == 1                                    # 3 and 6 MB
    assert keeps(1440, 613, 136, off=8) == 1                                                                 # the same off the lines
    assert keeps(736, 395, 848, ilv=1) == 1 and keeps(2592, 200, 360, ilv=1) == 1                            # 8 and 11 MB, longer K
    assert keeps(544, 2711, 192) == 1 and keeps(1408, 2907, 160) == 1                                        # 24 and 65 MB
    assert keeps(1536, 1536, 512) == 1 and keeps(1536, 1536, 512, c=False) == 0 and keeps(1536, 1536, 512, c=False, off=4) == 1
    assert keeps(2048, 2048, 2048) == 0 and keeps(4040, 2048, 400, off=8) == 1 and keeps(896, 3562, 3832, off=4) == 0
    assert keeps(3000, 2500, 1000, ilv=1, off=0) == 0                                                        # on half lines
