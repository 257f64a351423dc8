// Registry of the compiled kernel variants.  A variant is chosen by
// (tile shape, A K-contiguous?, B K-contiguous?, strided tensor addressing?, operator).
#pragma once
#include "gemm_kernel.hpp"

namespace fg {

// TILE_128x128_DEEP: the 128x128 tile with a ring of four buffers (128 KB of LDS, one workgroup per
// compute unit), for outputs of at most one such tile per unit: a
// lone workgroup turns a K tile over too fast for a two-buffer ring to cover the memory latency.  Matrix kernels of real products: four
// waves of 64x64, one per SIMD, on 16x16x32 instructions (TileCfg::WIDE; 2048^3 bfloat16 22.4 us with eight waves of 32x64,
// which cover each other's latencies, 19.5 so).  Addition on A and B and contractions: eight waves on 32x32x16.
// TILE_256x128: matrix kernels with a ring of three buffers (144 KB).  With two, a K tile has one tile's time to
// arrive in (0.9 us), which data that comes from memory takes: 8192x1024x4096 with three operand sets in turn 82.5 -> 71.5 us
// (one set, from the memory-side cache: 69.0 -> 67.2), with C 93.5 -> 80.0, 3000^3 94.1 -> 88.4, 2329x3267x5104 127.8 -> 111.  A
// fourth does not fit.  One wave per SIMD (four of 128x64) in place of eight of 64x64: 71.5 -> 64.5.  Contractions have eight, measured 0
// to 4 % slower with three buffers (extents 192, 72, 200 over 208: 11.3, 11.7) and keep two.
// TILE_256x128_PASS, TILE_128x128_PASS: the 256x128 and the deep 128x128 tile with eight waves and 32x32x16 instructions, for products of short K
// (select_kernel).
// TILE_256x256, TILE_256x256_K32: 16x16x32 matrix instructions (TileCfg::M16), which on a chip at its power limit sustain a higher
// rate on the same data.  Plain, BF16 and binary16-result matrix kernels: one kernel under both names, with one wave per SIMD
// (TileCfg::WIDE, wide_loop.hpp; eight waves with 32x32x16 instructions, which outputs of fewer than 192 such tiles used to run on: 3000x3000x2000
// with C 71.5 -> 59.4 us, 6144x2048x4096 116 -> 98, 4096x4096x320 40.4 -> 38.8, 3072x4096x512 35.2 -> 36.3).  The A/B-addition
// kernels have eight waves, with 32x32x16 instructions (TILE_256x256) or, two layout pairs, 16x16x32 ones; contractions
// 32x32x16 ones.
// TILE_64x64_KG2, TILE_64x64_KG2_DEEP: the 64x64 tile with two groups of four waves that share its K tiles
// (TileCfg::KG), for outputs of at most two such tiles per unit: one group alone spends most of a K tile in barrier
// and LDS latency.  DEEP: rings of four, for outputs of at most one tile per unit, whose two-buffer rings wait for
// their loads (1024^2 x 4096: 34.9 us with one group, 23.9 with two, 21.4 with four groups and
// two buffers, which this form replaces, 17.8 with two groups and four buffers; 512^2 x 2048: 13.5, 12.8, 10.7; five buffers
// and one group with eight measured no faster).  The direct-to-LDS path of a unit gives 104 GB/s with all units at it
// (150 alone); this loop takes 80.
// TILE_64x128_KG2: the same with 64x128 tiles and rings of three, for outputs between one 64x64 tile per unit and one
// 128x128 tile: fewer bytes per product, and one tile per unit where the 64x64 tile needs two (1536x1024x2048: 17.5 us
// with two groups, 15.5; 1895x714x1256: 15.3, 14.0; 128x64 tiles 15.7 and 14.9).
// All three: matrix kernels of real products.
enum TileId { TILE_256x256 = 0, TILE_256x128 = 1, TILE_128x128 = 2, TILE_64x64 = 3, TILE_128x128_DEEP = 4,
              TILE_256x256_K32 = 5, TILE_64x64_KG2 = 6, TILE_64x64_KG2_DEEP = 7, TILE_64x128_KG2 = 8,
              TILE_256x128_PASS = 9, TILE_128x128_PASS = 10, TILE_COUNT = 11, DIAG_TILE_COUNT = 4 };

struct KernelEntry {
    const void *fn;           // void (*)(const GemmParams), contractions: (const ContractParams)
    const char *name;
    int bm, bn, threads, lds_bytes;
    int kg;                   // K groups: a K split hands out multiples of this many K tiles (0: no groups)
};

// Defined by the instantiation files (one per layout pair).
const KernelEntry *kernel_table_nn();   // A M-contiguous, B K-contiguous  (A 'N', B 'N')
const KernelEntry *kernel_table_nt();   // A M-contiguous, B N-contiguous  (A 'N', B 'T')
const KernelEntry *kernel_table_tn();   // A K-contiguous, B K-contiguous  (A 'T', B 'N')
const KernelEntry *kernel_table_tt();   // A K-contiguous, B N-contiguous  (A 'T', B 'T')

// The same four layout pairs with bfloat16 A and B (plain matrices only): index = tile.
const KernelEntry *kernel_table_nn_bf16();
const KernelEntry *kernel_table_nt_bf16();
const KernelEntry *kernel_table_tn_bf16();
const KernelEntry *kernel_table_tt_bf16();

// The four layout pairs with a constant added to every loaded element of A and B: index = tile.
const KernelEntry *kernel_table_nn_xf();
const KernelEntry *kernel_table_nt_xf();
const KernelEntry *kernel_table_tn_xf();
const KernelEntry *kernel_table_tt_xf();

// The four layout pairs with C and D stored as binary16 (TileCfg::CD16): index = tile.
const KernelEntry *kernel_table_nn_h16();
const KernelEntry *kernel_table_nt_h16();
const KernelEntry *kernel_table_tn_h16();
const KernelEntry *kernel_table_tt_h16();

// Diagonal operands: index tile * 4 + {0: A diag, B K-contiguous; 1: A diag, B N-contiguous;
//                                       2: B diag, A K-contiguous; 3: B diag, A M-contiguous}.
const KernelEntry *kernel_table_diag();
// Planar complex: index ctile * 4 + {nn, nt, tn, tt}; ctile 0: 256x128, 1: 128x128, 2: 64x64, 3: 64x64 with two K
// groups (TileCfg::KG), whose K tiles of 64 also fetch K-contiguous operands in whole 128-byte lines (32: 300x400x2048, TN,
// 26.6 us, 64: 21.5; one group of 32: 33.1).  The 128x128 kernels are held to 256 registers and the planar 64x64 ones to 128
// (TileCfg::WAVES), so that two and four workgroups fit a unit: left to the compiler they took 496 and 168 (interleaved
// 3000x2500x1000 on the 128x128 tile 95.0 -> 84.3 us, dual 1532x2368x1112 on the 64x64 tile 42.0 -> 38.9); the interleaved
// 64x64 kernels, 136, measured 2 to 6 % slower with 128.  Both 64x64 tiles keep the name that callers compare.
const KernelEntry *kernel_table_cplx();
// Interleaved complex (real and imaginary part adjacent in A, B, C and D): same indexing.
const KernelEntry *kernel_table_cplx_il();
// Planar dual numbers (eps^2 = 0): same indexing as the complex table.
const KernelEntry *kernel_table_dual();
enum { CTILE_64x64 = 2, CTILE_64x64_KG2 = 3, CTILE_COUNT = 4 };

// Second pass of a split-K product (splitk_reduce.hip).
hipError_t launch_splitk_reduce(const float *W, int splits, int tile_begin, int tile_count, int bm, int bn, int tiles_m,
                                int tiles_n, int M, int N, float alpha, float beta, const float *C, int64_t ldc, float *D,
                                int64_t ldd, const float *bias, int bias_dim, int act, int c_act, hipStream_t stream);

// General kernel (general_kernel.hpp): matrices with unaligned operands or a K that is not a multiple
// of 8 (gemm_general.hip), contractions the tiled kernels cannot take (contract_general.hip).  128x128
// tiles with eight 32x64 waves; 64x64 tiles whose two groups of four waves take alternate K steps; 64x64 tiles with one
// group, for products of one K step.
enum GeneralVariant { GENERAL_128x128 = 0, GENERAL_64x64 = 1, GENERAL_64x64_ONE = 2, GENERAL_COUNT = 3 };
struct GeneralParams;
// ranges: one launch whose workgroups compute the p.splits K ranges of their tiles in turn, into D.
hipError_t launch_gemm_general(const GeneralParams &p, bool a_kc, bool b_kc, bool bf16, int variant, bool ranges, hipStream_t stream);
hipError_t launch_contract_general(const GeneralParams &p, bool a_kc, bool b_kc, int variant, hipStream_t stream);

// Entry index inside one table of real kernels: three variants per tile.
enum Variant { VARIANT_MATRIX = 0, VARIANT_CONTRACT = 1, VARIANT_CONTRACT_STREAM = 2, VARIANT_COUNT = 3 };
inline int entry_index(int tile, int variant) { return tile * VARIANT_COUNT + variant; }

// real kernels with BK = 64: ring refills are spread between the MFMAs (TileCfg::SPREAD)
#define FG_CFG(BM, BN, BK, ST, WGM, WGN, AKC, BKC, STR) TileCfg<BM, BN, BK, ST, WGM, WGN, AKC, BKC, STR, 0, 0, true>
// the tiles with two K groups (64 rows; BN columns, ring of ST); BF: bfloat16 inputs, XF: addition on A and B, H: binary16 C and D
#define FG_CFG_KG(AKC, BKC, BF, XF, H, BN, ST, TURNS) TileCfg<64, BN, 64, ST, 2, 2, AKC, BKC, false, 0, 0, true, BF, XF, false, false, H, false, 2, TURNS>
#define FG_ENTRY_KG(AKC, BKC, BF, XF, H, BN, ST, TURNS, NAME)                                      \
    { (const void *)gemm_kernel<FG_CFG_KG(AKC, BKC, BF, XF, H, BN, ST, TURNS)>, NAME, 64, BN,      \
      FG_CFG_KG(AKC, BKC, BF, XF, H, BN, ST, TURNS)::NTHREADS, FG_CFG_KG(AKC, BKC, BF, XF, H, BN, ST, TURNS)::LDS_BYTES, 2 }
#define FG_EMPTY_ENTRY { nullptr, nullptr, 0, 0, 0, 0, 0 }
// the same with 16x16x32 matrix instructions and one wave per SIMD (TileCfg::M16, WIDE); BF: bfloat16 inputs, H: binary16 C and D
#define FG_CFG_K32(BM, BN, BK, ST, WGM, WGN, AKC, BKC, BF, H) TileCfg<BM, BN, BK, ST, WGM, WGN, AKC, BKC, false, 0, 0, true, BF, false, false, false, H, true, 1, false, 1, true>
#define FG_ENTRY_K32(BM, BN, BK, ST, WGM, WGN, AKC, BKC, BF, H, NAME)                              \
    { (const void *)gemm_kernel<FG_CFG_K32(BM, BN, BK, ST, WGM, WGN, AKC, BKC, BF, H)>, NAME, BM, BN,            \
      FG_CFG_K32(BM, BN, BK, ST, WGM, WGN, AKC, BKC, BF, H)::NTHREADS,                             \
      FG_CFG_K32(BM, BN, BK, ST, WGM, WGN, AKC, BKC, BF, H)::LDS_BYTES }
#define FG_ENTRY(BM, BN, BK, ST, WGM, WGN, AKC, BKC, STR, NAME)                                    \
    { (const void *)gemm_kernel<FG_CFG(BM, BN, BK, ST, WGM, WGN, AKC, BKC, STR)>, NAME, BM, BN,                  \
      FG_CFG(BM, BN, BK, ST, WGM, WGN, AKC, BKC, STR)::NTHREADS,                                   \
      FG_CFG(BM, BN, BK, ST, WGM, WGN, AKC, BKC, STR)::LDS_BYTES }

// contraction kernels whose result streams past the L2 (TileCfg::CSTREAM)
#define FG_CFG_GS(BM, BN, BK, ST, WGM, WGN, AKC, BKC) TileCfg<BM, BN, BK, ST, WGM, WGN, AKC, BKC, true, 0, 0, true, false, false, false, true>
#define FG_ENTRY_GS(BM, BN, BK, ST, WGM, WGN, AKC, BKC, NAME)                                      \
    { (const void *)gemm_kernel<FG_CFG_GS(BM, BN, BK, ST, WGM, WGN, AKC, BKC)>, NAME, BM, BN,                    \
      FG_CFG_GS(BM, BN, BK, ST, WGM, WGN, AKC, BKC)::NTHREADS,                                     \
      FG_CFG_GS(BM, BN, BK, ST, WGM, WGN, AKC, BKC)::LDS_BYTES }

#define FG_CFG_BF16(BM, BN, BK, ST, WGM, WGN, AKC, BKC) TileCfg<BM, BN, BK, ST, WGM, WGN, AKC, BKC, false, 0, 0, true, true>
#define FG_ENTRY_BF16(BM, BN, BK, ST, WGM, WGN, AKC, BKC, NAME)                                    \
    { (const void *)gemm_kernel<FG_CFG_BF16(BM, BN, BK, ST, WGM, WGN, AKC, BKC)>, NAME, BM, BN,                  \
      FG_CFG_BF16(BM, BN, BK, ST, WGM, WGN, AKC, BKC)::NTHREADS,                                   \
      FG_CFG_BF16(BM, BN, BK, ST, WGM, WGN, AKC, BKC)::LDS_BYTES }

#define FG_DEFINE_TABLE_BF16(FUNC, AKC, BKC, TAG)                                                  \
    const KernelEntry *FUNC() {                                                                    \
        static const KernelEntry t[TILE_COUNT] = {                                                 \
            FG_ENTRY_K32(256, 256, 64, 2, 2, 2, AKC, BKC, true, false, "gemm_bf16_" TAG "_256x256x64"), \
            FG_ENTRY_K32(256, 128, 64, 3, 2, 2, AKC, BKC, true, false, "gemm_bf16_" TAG "_256x128x64"), \
            FG_ENTRY_BF16(128, 128, 64, 2, 2, 2, AKC, BKC, "gemm_bf16_" TAG "_128x128x64"),        \
            FG_ENTRY_BF16(64, 64, 64, 2, 2, 2, AKC, BKC, "gemm_bf16_" TAG "_64x64x64"),            \
            FG_ENTRY_K32(128, 128, 64, 4, 2, 2, AKC, BKC, true, false, "gemm_bf16_" TAG "_128x128x64_deep"), \
            FG_ENTRY_K32(256, 256, 64, 2, 2, 2, AKC, BKC, true, false, "gemm_bf16_" TAG "_256x256x64_k32"), \
            FG_ENTRY_KG(AKC, BKC, true, false, false, 64, 2, false, "gemm_bf16_" TAG "_64x64x64"),            \
            FG_ENTRY_KG(AKC, BKC, true, false, false, 64, 4, true, "gemm_bf16_" TAG "_64x64x64"),            \
            FG_ENTRY_KG(AKC, BKC, true, false, false, 128, 3, true, "gemm_bf16_" TAG "_64x128x64"), \
            FG_ENTRY_BF16(256, 128, 64, 3, 4, 2, AKC, BKC, "gemm_bf16_" TAG "_256x128x64"),        \
            FG_ENTRY_BF16(128, 128, 64, 4, 4, 2, AKC, BKC, "gemm_bf16_" TAG "_128x128x64_deep"),   \
        };                                                                                         \
        return t;                                                                                  \
    }

#define FG_CFG_H16(BM, BN, BK, ST, WGM, WGN, AKC, BKC) TileCfg<BM, BN, BK, ST, WGM, WGN, AKC, BKC, false, 0, 0, true, false, false, false, false, true>
#define FG_ENTRY_H16(BM, BN, BK, ST, WGM, WGN, AKC, BKC, NAME)                                     \
    { (const void *)gemm_kernel<FG_CFG_H16(BM, BN, BK, ST, WGM, WGN, AKC, BKC)>, NAME, BM, BN,                   \
      FG_CFG_H16(BM, BN, BK, ST, WGM, WGN, AKC, BKC)::NTHREADS,                                    \
      FG_CFG_H16(BM, BN, BK, ST, WGM, WGN, AKC, BKC)::LDS_BYTES }

#define FG_DEFINE_TABLE_H16(FUNC, AKC, BKC, TAG)                                                   \
    const KernelEntry *FUNC() {                                                                    \
        static const KernelEntry t[TILE_COUNT] = {                                                 \
            FG_ENTRY_K32(256, 256, 64, 2, 2, 2, AKC, BKC, false, true, "gemm_h16_" TAG "_256x256x64"), \
            FG_ENTRY_K32(256, 128, 64, 3, 2, 2, AKC, BKC, false, true, "gemm_h16_" TAG "_256x128x64"), \
            FG_ENTRY_H16(128, 128, 64, 2, 2, 2, AKC, BKC, "gemm_h16_" TAG "_128x128x64"),          \
            FG_ENTRY_H16(64, 64, 64, 2, 2, 2, AKC, BKC, "gemm_h16_" TAG "_64x64x64"),              \
            FG_ENTRY_K32(128, 128, 64, 4, 2, 2, AKC, BKC, false, true, "gemm_h16_" TAG "_128x128x64_deep"), \
            FG_ENTRY_K32(256, 256, 64, 2, 2, 2, AKC, BKC, false, true, "gemm_h16_" TAG "_256x256x64_k32"), \
            FG_ENTRY_KG(AKC, BKC, false, false, true, 64, 2, false, "gemm_h16_" TAG "_64x64x64"),             \
            FG_ENTRY_KG(AKC, BKC, false, false, true, 64, 4, true, "gemm_h16_" TAG "_64x64x64"),             \
            FG_ENTRY_KG(AKC, BKC, false, false, true, 128, 3, true, "gemm_h16_" TAG "_64x128x64"), \
            FG_ENTRY_H16(256, 128, 64, 3, 4, 2, AKC, BKC, "gemm_h16_" TAG "_256x128x64"),          \
            FG_ENTRY_H16(128, 128, 64, 4, 4, 2, AKC, BKC, "gemm_h16_" TAG "_128x128x64_deep"),     \
        };                                                                                         \
        return t;                                                                                  \
    }

#define FG_CFG_XF(BM, BN, BK, ST, WGM, WGN, AKC, BKC) TileCfg<BM, BN, BK, ST, WGM, WGN, AKC, BKC, false, 0, 0, true, false, true>
#define FG_ENTRY_XF(BM, BN, BK, ST, WGM, WGN, AKC, BKC, NAME)                                      \
    { (const void *)gemm_kernel<FG_CFG_XF(BM, BN, BK, ST, WGM, WGN, AKC, BKC)>, NAME, BM, BN,                    \
      FG_CFG_XF(BM, BN, BK, ST, WGM, WGN, AKC, BKC)::NTHREADS,                                     \
      FG_CFG_XF(BM, BN, BK, ST, WGM, WGN, AKC, BKC)::LDS_BYTES }

// The 256x256 tile of that family on 16x16x32 matrix instructions, for the two layout pairs on
// which it measured faster than the 32x32x16 kernel (A and B contiguous along different
// directions: -3.5 % and -1.5 % run time on 8192^3; the other two pairs 0 and +3 %).
template <bool AKC, bool BKC>
inline KernelEntry xf_k32_entry(const char *name) {
    if constexpr (AKC != BKC) {
        using Cfg = TileCfg<256, 256, 64, 2, 2, 4, AKC, BKC, false, 0, 0, true, false, true, false, false, false, true>;
        return { (const void *)gemm_kernel<Cfg>, name, 256, 256, Cfg::NTHREADS, Cfg::LDS_BYTES };
    } else {
        return FG_EMPTY_ENTRY;
    }
}

#define FG_DEFINE_TABLE_XF(FUNC, AKC, BKC, TAG)                                                    \
    const KernelEntry *FUNC() {                                                                    \
        static const KernelEntry t[TILE_COUNT] = {                                                 \
            FG_ENTRY_XF(256, 256, 64, 2, 2, 4, AKC, BKC, "gemm_abadd_" TAG "_256x256x64"),         \
            FG_ENTRY_XF(256, 128, 64, 3, 4, 2, AKC, BKC, "gemm_abadd_" TAG "_256x128x64"),         \
            FG_ENTRY_XF(128, 128, 64, 2, 2, 2, AKC, BKC, "gemm_abadd_" TAG "_128x128x64"),         \
            FG_ENTRY_XF(64, 64, 64, 2, 2, 2, AKC, BKC, "gemm_abadd_" TAG "_64x64x64"),             \
            FG_ENTRY_XF(128, 128, 64, 4, 4, 2, AKC, BKC, "gemm_abadd_" TAG "_128x128x64_deep"),    \
            xf_k32_entry<AKC, BKC>("gemm_abadd_" TAG "_256x256x64_k32"),                           \
            FG_ENTRY_KG(AKC, BKC, false, true, false, 64, 2, false, "gemm_abadd_" TAG "_64x64x64"),           \
            FG_ENTRY_KG(AKC, BKC, false, true, false, 64, 4, true, "gemm_abadd_" TAG "_64x64x64"),           \
            FG_ENTRY_KG(AKC, BKC, false, true, false, 128, 3, true, "gemm_abadd_" TAG "_64x128x64"), \
            FG_EMPTY_ENTRY, FG_EMPTY_ENTRY,                                                        \
        };                                                                                         \
        return t;                                                                                  \
    }

// KG: K groups (in turns), W: TileCfg::WAVES
#define FG_CFG_IL(BM, BN, BK, ST, WGM, WGN, AKC, BKC, KG, W) TileCfg<BM, BN, BK, ST, WGM, WGN, AKC, BKC, false, 0, 1, false, false, false, true, false, false, false, KG, (KG > 1), W>
#define FG_ENTRY_IL(BM, BN, BK, ST, WGM, WGN, AKC, BKC, KG, W, NAME)                               \
    { (const void *)gemm_kernel<FG_CFG_IL(BM, BN, BK, ST, WGM, WGN, AKC, BKC, KG, W)>, NAME, BM, BN,             \
      FG_CFG_IL(BM, BN, BK, ST, WGM, WGN, AKC, BKC, KG, W)::NTHREADS,                              \
      FG_CFG_IL(BM, BN, BK, ST, WGM, WGN, AKC, BKC, KG, W)::LDS_BYTES }

#define FG_CFG_X(BM, BN, BK, ST, WGM, WGN, AKC, BKC, DG, CX, KG, W) TileCfg<BM, BN, BK, ST, WGM, WGN, AKC, BKC, false, DG, CX, false, false, false, false, false, false, false, KG, (KG > 1), W>
#define FG_ENTRY_X(BM, BN, BK, ST, WGM, WGN, AKC, BKC, DG, CX, KG, W, NAME)                         \
    { (const void *)gemm_kernel<FG_CFG_X(BM, BN, BK, ST, WGM, WGN, AKC, BKC, DG, CX, KG, W)>, NAME, BM, BN,     \
      FG_CFG_X(BM, BN, BK, ST, WGM, WGN, AKC, BKC, DG, CX, KG, W)::NTHREADS,                       \
      FG_CFG_X(BM, BN, BK, ST, WGM, WGN, AKC, BKC, DG, CX, KG, W)::LDS_BYTES }

#define FG_DEFINE_TABLE(FUNC, AKC, BKC, TAG)                                                       \
    const KernelEntry *FUNC() {                                                                    \
        static const KernelEntry t[TILE_COUNT * VARIANT_COUNT] = {                                 \
            FG_ENTRY_K32(256, 256, 64, 2, 2, 2, AKC, BKC, false, false, "gemm_" TAG "_256x256x64"), \
            FG_ENTRY(256, 256, 64, 2, 2, 4, AKC, BKC, true, "gett_" TAG "_256x256x64"),            \
            FG_ENTRY_GS(256, 256, 64, 2, 2, 4, AKC, BKC, "gett_stream_" TAG "_256x256x64"),        \
            FG_ENTRY_K32(256, 128, 64, 3, 2, 2, AKC, BKC, false, false, "gemm_" TAG "_256x128x64"), \
            FG_ENTRY(256, 128, 64, 2, 4, 2, AKC, BKC, true, "gett_" TAG "_256x128x64"),            \
            FG_ENTRY_GS(256, 128, 64, 2, 4, 2, AKC, BKC, "gett_stream_" TAG "_256x128x64"),        \
            FG_ENTRY(128, 128, 64, 2, 2, 2, AKC, BKC, false, "gemm_" TAG "_128x128x64"),           \
            FG_ENTRY(128, 128, 64, 2, 2, 2, AKC, BKC, true, "gett_" TAG "_128x128x64"),            \
            FG_ENTRY_GS(128, 128, 64, 2, 2, 2, AKC, BKC, "gett_stream_" TAG "_128x128x64"),        \
            FG_ENTRY(64, 64, 64, 2, 2, 2, AKC, BKC, false, "gemm_" TAG "_64x64x64"),               \
            FG_ENTRY(64, 64, 64, 2, 2, 2, AKC, BKC, true, "gett_" TAG "_64x64x64"),                \
            FG_ENTRY_GS(64, 64, 64, 2, 2, 2, AKC, BKC, "gett_stream_" TAG "_64x64x64"),            \
            FG_ENTRY_K32(128, 128, 64, 4, 2, 2, AKC, BKC, false, false, "gemm_" TAG "_128x128x64_deep"), \
            FG_ENTRY(128, 128, 64, 4, 4, 2, AKC, BKC, true, "gett_" TAG "_128x128x64_deep"),       \
            FG_ENTRY_GS(128, 128, 64, 4, 4, 2, AKC, BKC, "gett_stream_" TAG "_128x128x64_deep"),   \
            FG_ENTRY_K32(256, 256, 64, 2, 2, 2, AKC, BKC, false, false, "gemm_" TAG "_256x256x64_k32"), \
            FG_EMPTY_ENTRY, FG_EMPTY_ENTRY,                                                        \
            FG_ENTRY_KG(AKC, BKC, false, false, false, 64, 2, false, "gemm_" TAG "_64x64x64"), FG_EMPTY_ENTRY, FG_EMPTY_ENTRY, \
            FG_ENTRY_KG(AKC, BKC, false, false, false, 64, 4, true, "gemm_" TAG "_64x64x64"), FG_EMPTY_ENTRY, FG_EMPTY_ENTRY, \
            FG_ENTRY_KG(AKC, BKC, false, false, false, 128, 3, true, "gemm_" TAG "_64x128x64"), FG_EMPTY_ENTRY, FG_EMPTY_ENTRY, \
            FG_ENTRY(256, 128, 64, 3, 4, 2, AKC, BKC, false, "gemm_" TAG "_256x128x64"), FG_EMPTY_ENTRY, FG_EMPTY_ENTRY, \
            FG_ENTRY(128, 128, 64, 4, 4, 2, AKC, BKC, false, "gemm_" TAG "_128x128x64_deep"), FG_EMPTY_ENTRY, FG_EMPTY_ENTRY, \
        };                                                                                         \
        return t;                                                                                  \
    }

}  // namespace fg
