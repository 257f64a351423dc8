// Kernel instantiations for planar-split complex products (Section 5.4).
#include "kernel_table.hpp"
namespace fg {
#define FG_CPLX_TILE(BM, BN, BK, ST, WGM, WGN, KG, W, TAG)                                             \
    FG_ENTRY_X(BM, BN, BK, ST, WGM, WGN, false, true, 0, 1, KG, W, "cgemm_nn_" TAG),              \
    FG_ENTRY_X(BM, BN, BK, ST, WGM, WGN, false, false, 0, 1, KG, W, "cgemm_nt_" TAG),             \
    FG_ENTRY_X(BM, BN, BK, ST, WGM, WGN, true, true, 0, 1, KG, W, "cgemm_tn_" TAG),               \
    FG_ENTRY_X(BM, BN, BK, ST, WGM, WGN, true, false, 0, 1, KG, W, "cgemm_tt_" TAG)
const KernelEntry *kernel_table_cplx() {
    static const KernelEntry t[CTILE_COUNT * 4] = {
        FG_CPLX_TILE(256, 128, 32, 2, 4, 2, 1, 1, "256x128x32"),
        FG_CPLX_TILE(128, 128, 32, 2, 2, 2, 1, 2, "128x128x32"),
        FG_CPLX_TILE(64, 64, 32, 2, 2, 2, 1, 4, "64x64x32"),
        FG_CPLX_TILE(64, 64, 64, 2, 2, 2, 2, 1, "64x64x32"),
    };
    return t;
}
}  // namespace fg
