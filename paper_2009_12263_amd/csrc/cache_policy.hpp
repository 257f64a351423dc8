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

}  // namespace fg
