// Instantiations of the general kernel for real matrix products (see general_kernel.hpp): operands
// with any leading dimension, bases aligned to an element only, any K.
#include "general_kernel.hpp"
#include "kernel_table.hpp"

namespace fg {
namespace {

template <bool BF16, bool RANGES>
GeneralFn pick(bool a_kc, bool b_kc, int variant) {
    if constexpr (!RANGES)
        if (variant == GENERAL_64x64_ONE) return general_fn<64, 64, 2, 2, 1, BF16, true>(a_kc, b_kc);
    return variant == GENERAL_128x128 ? general_fn<128, 128, 4, 2, 1, BF16, true, RANGES>(a_kc, b_kc) : general_fn<64, 64, 2, 2, 2, BF16, true, RANGES>(a_kc, b_kc);
}

}  // namespace

hipError_t launch_gemm_general(const GeneralParams &p, bool a_kc, bool b_kc, bool bf16, int variant, bool ranges, hipStream_t stream) {
    const GeneralFn fn = ranges ? (bf16 ? pick<true, true>(a_kc, b_kc, variant) : pick<false, true>(a_kc, b_kc, variant))
                                : (bf16 ? pick<true, false>(a_kc, b_kc, variant) : pick<false, false>(a_kc, b_kc, variant));
    return launch_general(fn, variant, p, stream, ranges);
}

}  // namespace fg
