// Where the pieces of eight 16-bit elements of the general kernel (general_kernel.hpp) are fetched from.
// Plain integer arithmetic without HIP: a CPU test compiles this header and checks that nothing outside an
// operand is read.
#pragma once
#include <stdint.h>

#ifdef __HIP__
#define FG_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define FG_HOST_DEVICE inline
#endif

namespace fg {

// The piece `off` + (offset of any k, at most kmax) elements from the first of an operand that spans `span`
// elements ends inside the operand.
FG_HOST_DEVICE bool piece_inside(int64_t off, int64_t kmax, int64_t span) { return off + kmax + 8 <= span; }

// A piece at an even byte offset `at` from a word-aligned address, as the words that hold it: four from `words` on and a
// fifth, of which `skew` bytes are dropped in front.  A piece that starts with a word (skew 0) is whole in the
// four: there the fifth is the first of them again, because the word behind the piece may lie outside the operand.
struct OddPiece { uint32_t words, fifth, skew; };
FG_HOST_DEVICE OddPiece odd_piece(uint32_t at) {
    const uint32_t words = at & ~3u, skew = at & 2u;
    return OddPiece{words, words + 8u * skew, skew};
}

}  // namespace fg
