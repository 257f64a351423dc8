// Which accesses of the matrix kernels carry the streaming policy.  Plain integer arithmetic without HIP: a CPU test compiles
// this header.
#pragma once
#include <stdint.h>

namespace fg {

// The memory-side cache, which all XCDs share.
constexpr int64_t kMemorySideCache = 256ll << 20;

// An operand that one row (column) of tiles reads is read once, and its loads may stream: they then take no place behind the L2
// (whose hits and misses stay the same, 3.01 and 3.51 million at 128x12288x16384 either way).  But they also pass by what
// the memory-side cache holds of it, from the call before or from the kernel that wrote it, so only operands of one and a half
// times that cache's size, of which a pass finds nothing there, stream; and only rows of whole lines (a line that two K
// tiles share would be fetched twice).
// Microseconds without and with streaming, three operand sets in turn / the same one again / written by the kernel before
// (with that kernel): 128 MB (128x4096x16384) 45.4 43.6 / 34.8 45.0 / 79.0 87.9; 192 MB 63.6 56.5 / 42.2 56.2 /
// 97.0 101.7; 260 MB 96.1 77.7 / 75.7 77.3 / 185 199; 320 MB 95.9 82.8 / 91.3 85.0 / 205 219; 384 MB (128x16384x12288)
// 122 113 / 122 113 / 249 246; 1187 MB (128x151936x4096) 293 286 / 296 286 / 729 686.
inline bool streams_once(uint64_t address, int64_t ld, int64_t bytes) {
    return address % 128 == 0 && ld % 64 == 0 && 2 * bytes >= 3 * kMemorySideCache;
}

// C and D of a real product are kept in the caches (default policy) instead of streamed past the L2.  They are touched
// once and would displace the A and B panels that other workgroups re-read, so they stream, unless
//  - the whole problem fits the memory-side cache: then nothing is displaced for long (3000^3: 73.6 us against 87.4 streamed,
//    4096^3: -6 %, 5000x3000x2000: 76.7 against 103.1 back to back; equal on cache-cold operands; from 300 MB up
//    streaming wins by 4 to 9 %);
//  - there is a C, columns do not begin on half a 128-byte line, and A and B, which C and D push out of the memory-side cache, take
//    at most 112 MB: columns that share lines are fetched from memory once for each when streamed.  36 products above 256 MB,
//    kept / streamed: 0.65 to 0.94 off the half lines with A and B up to 60 MB (6692x6497x248 134.0 / 195.9), 0.92 to 1.03 above
//    (6856x7081x4064 433 / 442; 3928x6503x4240 285 / 277); on half lines 1.02 to 1.12 (8143x3710x1040 125.1 / 112.1), as on whole
//    ones (6560x7903x2584 315 / 303).  Binary16 C and D: 0.78 to 1.04 and 1.01 to 1.06.
// Sizes in bytes; ld: bytes from one column of C (D) to the next.
inline bool keeps_real_cd(int64_t ab, int64_t cd, bool has_c, int64_t ldc, int64_t ldd) {
    if (ab + cd <= kMemorySideCache) return true;
    return has_c && (ldc % 64 != 0 || ldd % 64 != 0) && ab <= (112ll << 20);
}

// The same for complex and dual products, whose planes or pairs double all of it.  Up to 80 MB in all: with C they are kept
// (1536^2 x 512 24.4 -> 21.6 us, dual 2048^2 x 512 32.0 -> 29.4), but for a pass over 7 to 16 MB with a short K whose
// columns are on the lines, which the L2s turn over faster streamed (20 products with K 32 to 216: 0.96 to 1.14 of the time kept,
// 1.04 on average, complex 1440x613x136 8.8 / 7.7; smaller ones equal within 1 %, interleaved ones up to 5 % faster kept; with K from
// 336 on 2 to 11 % faster kept); without C off the lines only (dual 1532x2368x1112 41.3 -> 34.2; on them 22.4 streamed and
// 23.6 kept, complex 2048^3, 100 MB, 77.4 and 78.4).  Above 80 MB: off the lines while A and B are small (4040x2048x400 complex 72.3 -> 62.9):
// larger ones stay in the memory-side cache only if C and D do not push them out, and the K loop waits for memory (dual 899x3562x3832,
// A and B 68 MB: 124 streamed, 156 kept).  Off the lines: planar ones off 128 bytes, interleaved ones off 64 (on half lines
// 3000x2500x1000 84.5 streamed, 88.2 kept).
// Sizes in bytes; ld: bytes from one column of a plane (of pairs, if interleaved) to the next.
inline bool keeps_complex_cd(int64_t ab, int64_t cd, int64_t K, bool interleaved, bool has_c, int64_t ldc, int64_t ldd) {
    const int64_t line = interleaved ? 64 : 128;
    const bool off = ldd % line != 0 || (has_c && ldc % line != 0);
    if (ab + cd > (80ll << 20)) return off && ab <= (32ll << 20);
    return off || (has_c && (K > 256 || ab + cd > (16ll << 20) || ab + cd < (7ll << 20)));
}

}  // namespace fg
