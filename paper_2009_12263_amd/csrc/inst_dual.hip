// Kernel instantiations for planar-split dual-number products (Section 5.4: eps^2 = 0, three real products).
#include "kernel_table.hpp"
namespace fg {
#define FG_DUAL_TILE(BM, BN, BK, ST, WGM, WGN, KG, W, TAG)                                             \
    FG_ENTRY_X(BM, BN, BK, ST, WGM, WGN, false, true, 0, 2, KG, W, "dgemm_nn_" TAG),              \
    FG_ENTRY_X(BM, BN, BK, ST, WGM, WGN, false, false, 0, 2, KG, W, "dgemm_nt_" TAG),             \
    FG_ENTRY_X(BM, BN, BK, ST, WGM, WGN, true, true, 0, 2, KG, W, "dgemm_tn_" TAG),               \
    FG_ENTRY_X(BM, BN, BK, ST, WGM, WGN, true, false, 0, 2, KG, W, "dgemm_tt_" TAG)
const KernelEntry *kernel_table_dual() {
    static const KernelEntry t[CTILE_COUNT * 4] = {
        FG_DUAL_TILE(256, 128, 32, 2, 4, 2, 1, 1, "256x128x32"),
        FG_DUAL_TILE(128, 128, 32, 2, 2, 2, 1, 2, "128x128x32"),
        FG_DUAL_TILE(64, 64, 32, 2, 2, 2, 1, 4, "64x64x32"),
        FG_DUAL_TILE(64, 64, 64, 2, 2, 2, 2, 1, "64x64x32"),
    };
    return t;
}
}  // namespace fg
