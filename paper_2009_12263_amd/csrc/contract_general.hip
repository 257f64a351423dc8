// Instantiations of the general kernel for tensor contractions (see general_kernel.hpp): any
// strides and extents, tensors of any size, outer products.
#include "general_kernel.hpp"
#include "kernel_table.hpp"

namespace fg {

namespace {
GeneralFn pick(bool a_kc, bool b_kc, int variant) {
    return variant == GENERAL_128x128 ? general_fn<128, 128, 4, 2, 1, false, false>(a_kc, b_kc)
         : variant == GENERAL_64x64   ? general_fn<64, 64, 2, 2, 2, false, false>(a_kc, b_kc) : general_fn<64, 64, 2, 2, 1, false, false>(a_kc, b_kc);
}
}  // namespace

hipError_t launch_contract_general(const GeneralParams &p, bool a_kc, bool b_kc, int variant, hipStream_t stream) {
    return launch_general(pick(a_kc, b_kc, variant), variant, p, stream);
}

}  // namespace fg
