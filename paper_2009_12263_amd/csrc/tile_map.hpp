// Which tile of the output a workgroup computes.  Plain integer arithmetic without HIP: a CPU test compiles this header.
#pragma once
#include <stdint.h>

#ifndef FG_HOST_DEVICE
#ifdef __HIP__
#define FG_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define FG_HOST_DEVICE inline
#endif
#endif

namespace fg {

// Workgroups are dealt round-robin to the 8 XCDs (each with its own L2).  Give every XCD a
// contiguous run of tiles (the first tiles mod 8 XCDs one more than the others), and walk tiles in
// groups of 4 tile rows so that the workgroups resident on one XCD at a time share A row panels and
// B column panels.  (Tile counts that are not multiples of 8 used to be dealt out one by one:
// 1 to 5 % slower on ragged products.)
FG_HOST_DEVICE void block_to_tile(int bid, int tiles_m, int tiles_n, int &tm, int &tn) {
    int nb = tiles_m * tiles_n;
    const int x = bid & 7, left = nb & 7;
    int id = x * (nb >> 3) + (x < left ? x : left) + (bid >> 3);
    int gm = tiles_m >= 4 ? 4 : tiles_m;
    int per_group = gm * tiles_n;
    int group = id / per_group;
    int first_m = group * gm;
    int rows = (tiles_m - first_m) < gm ? (tiles_m - first_m) : gm;
    int within = id - group * per_group;
    tm = first_m + within % rows;
    tn = within / rows;
}

// x / d for 0 <= x < 2^31, with constants made of d >= 1 by the host: mulhi(2 x, magic) >> shift, magic = floor(2^(31 + shift) / d) + 1,
// d <= 2^shift < 2 d.  No case apart, also not d = 1: a branch would part the loads of a kernel's arguments in two.
struct Division { uint32_t magic, shift; };
inline Division division_by(uint32_t d) {
    const uint32_t shift = d <= 1 ? 0 : 32u - (uint32_t)__builtin_clz(d - 1);
    return {(uint32_t)(((1ull << (31 + shift)) / d) + 1), shift};
}
inline Division division_to_zero() { return {0, 0}; }           // what is divided is less than the divisor: no division on the host
FG_HOST_DEVICE int divided(int x, Division d) { return (int)((uint32_t)(((uint64_t)(2u * (uint32_t)x) * d.magic) >> 32) >> d.shift); }

// The same tile with the division by the tiles of a group prepared by the host (tile_group): integer divisions on the scalar unit
// are a hundred instructions in front of a workgroup's first load.  Bfloat16 2048^3 21.4 -> 20.3 us with the loader's shorter start
// (WideLoader); 1024^3 TT 8.39 -> 8.17; 256^3 in replayed graphs 4.42 -> 4.24 (4.33 with a branch for a divisor of 1).  Contractions, which divide by their modes' extents all the same, measured 1 to 5 % slower with it
// (aebf,dfce->abcd with a = c = 24, b = f = 32, d = e = 8: 19.2, 20.2 us) and keep the plain form.
inline Division tile_group(int tiles_m, int tiles_n) { return tiles_m <= 4 ? division_to_zero() : division_by((uint32_t)(4 * tiles_n)); }
FG_HOST_DEVICE void block_to_tile(int bid, int tiles_m, int tiles_n, Division per_group, int &tm, int &tn) {
    const int nb = tiles_m * tiles_n, x = bid & 7, left = nb & 7;
    const int id = x * (nb >> 3) + (x < left ? x : left) + (bid >> 3);
    const int gm = tiles_m >= 4 ? 4 : tiles_m;
    const int group = divided(id, per_group), first_m = group * gm;
    const int rows = (tiles_m - first_m) < gm ? (tiles_m - first_m) : gm, within = id - group * (gm * tiles_n);
    tn = divided(within, Division{rows == 3 ? 0xaaaaaaabu : 0x80000001u, (uint32_t)(rows - 1 - (rows >> 2))});   // 1 to 4 rows
    tm = first_m + within - tn * rows;
}

}  // namespace fg
