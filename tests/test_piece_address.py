"""CPU test of the address arithmetic with which the general kernel fetches pieces of eight elements:
the header the kernel uses is compiled with the host compiler and run over every position of small
operands."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2009_12263_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstring>
#include "piece_address.hpp"
using namespace fg;

// An operand of `span` elements whose first one lies `lead` bytes into a word: the words that hold its elements
// are [0, words_end).  Every piece that the kernel may fetch as words reads nothing else, and gives the eight elements.
static int check(int span, unsigned lead) {
    const unsigned words_end = (lead + 2u * span + 3u) / 4u * 4u;
    unsigned char memory[1024];
    for (unsigned i = 0; i < sizeof memory; ++i) memory[i] = (unsigned char)(i * 37 + 11);
    int pieces = 0;
    for (int off = 0; off < span; ++off)
        for (int kmax = 0; off + kmax < span; ++kmax) {
            if (!piece_inside(off, kmax, span)) continue;
            for (int k = 0; k <= kmax; ++k) {
                const unsigned at = lead + 2u * (unsigned)(off + k);
                const OddPiece o = odd_piece(at);
                if (o.words % 4 || o.fifth % 4 || o.words + 16 > words_end || o.fifth + 4 > words_end) {
                    printf("span %d lead %u piece at element %d: words at byte %u, fifth at %u, the operand's words end at %u\n",
                           span, lead, off + k, o.words, o.fifth, words_end);
                    return -1;
                }
                unsigned char five[20];
                memcpy(five, memory + o.words, 16);
                memcpy(five + 16, memory + o.fifth, 4);
                if (memcmp(five + o.skew, memory + at, 16)) { printf("span %d lead %u piece at element %d: wrong elements\n", span, lead, off + k); return -1; }
                ++pieces;
            }
        }
    return pieces;
}

int main() {
    long total = 0;
    for (unsigned lead = 0; lead <= 2; lead += 2)
        for (int span = 1; span <= 72; ++span) {
            const int n = check(span, lead);
            if (n < 0) return 1;
            total += n;
        }
    // rows of 16 elements, 128 of them, at stride 16 (a 4096-byte operand): the last piece ends with the operand
    const OddPiece last = odd_piece(2u * (8 + 16 * 127));
    if (!piece_inside(8, 16 * 127, 16 * 128) || last.fifth + 4 > 4096 || last.words + 16 > 4096) { printf("last piece of 16 x 128: fifth word at byte %u of 4096\n", last.fifth); return 1; }
    printf("%ld pieces\n", total);
    return total > 0 ? 0 : 1;
}
"""


def test_pieces_read_as_words_stay_inside_the_operand(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "pieces.cpp", tmp_path / "pieces"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, str(src), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
