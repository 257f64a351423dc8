// C ABI of libflexgemm.so: argument validation, the "params" choice (Section 4.2.1: which block
// tile and kernel variant serve a problem) and the launch.  All arithmetic of the method runs in
// the kernels of gemm_kernel.hpp; this file only describes problems to them.
#include "../../include/flexgemm.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>

#include "cache_policy.hpp"
#include "general_kernel.hpp"
#include "kernel_table.hpp"

namespace {

thread_local char g_err[512] = "";

fg_status fail(fg_status st, const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return st;
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
bool aligned_to(const void *p, unsigned bytes) { return (reinterpret_cast<uintptr_t>(p) & (bytes - 1)) == 0; }

// Requirements of the tiled kernels that the general kernel does not have (16-byte aligned bases,
// leading dimensions in whole 16-byte chunks, K a multiple of 8).  A call that misses one of them
// is noted here while it is validated; plain real products then run on the general kernel, every
// other kind of product fails with the noted status and message.
struct Relaxed { fg_status status; char msg[256]; };
thread_local Relaxed g_relaxed = {FG_OK, ""};

void note_relaxed(fg_status st, const char *fmt, ...) {
    if (g_relaxed.status != FG_OK) return;          // keep the first
    g_relaxed.status = st;
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_relaxed.msg, sizeof g_relaxed.msg, fmt, ap);
    va_end(ap);
}

constexpr int kNumCU = 256;   // MI355X: 8 XCDs x 32 compute units

// Tuning overrides of the planner, from the environment: FG_FORCE_TILE=0..10 picks a tile shape (0..3
// for the four tiles of the complex and dual kernels)
// (5: the 256x256 tile by its k32 name, another kernel than 0 for addition on A and B only; 6, 7: the 64x64 tile with two K
// groups and rings of two or four buffers, 8: the 64x128 tile with two, 9 and 10: the 256x128 and the deep 128x128 tile with eight waves), FG_FORCE_SPLIT=n a split of K
// for every tile, FG_FORCE_TAIL=n a split of K for the tiles of the last round (1: never).  Read
// when the library is loaded and again by fg_reload_tuning(), not on every call.
std::atomic<int> g_force_tile{-1}, g_force_split{0}, g_force_tail{0};

void read_tuning_from_environment() {
    const char *t = getenv("FG_FORCE_TILE"), *s = getenv("FG_FORCE_SPLIT"), *l = getenv("FG_FORCE_TAIL");
    g_force_tile.store(t ? atoi(t) : -1);
    g_force_split.store(s ? atoi(s) : 0);
    g_force_tail.store(l ? atoi(l) : 0);
}
struct TuningAtLoad { TuningAtLoad() { read_tuning_from_environment(); } } g_tuning_at_load;

// ---- description of one GEMM after normalisation to "column-major D" ------------------------
struct Problem {
    int64_t M, N, K;
    const void *A, *A_im, *B, *B_im;
    bool a_kc, b_kc;         // operand is K-contiguous
    bool a_diag, b_diag;
    int64_t lda, ldb;
    const float *C, *C_im;
    float *D, *D_im;
    int64_t ldc, ldd;
    const float *bias;
    int bias_dim, act;
    float alpha, beta;
    bool cplx;               // two planes per operand: complex, or dual when `dual` is set
    bool dual;
    bool bf16;               // A and B hold bfloat16
    int c_act;               // activation on loaded C
    uint16_t a_add, b_add;   // FP16 bit patterns of the addends on loaded A and B; ab_add: in use
    bool ab_add;
    bool ilv;                // complex matrices in interleaved storage
    bool general;            // operands miss a requirement of the tiled kernels: use the general kernel
    bool cd16;               // C and D hold binary16 (converted when loaded / stored)
};

// What to launch for a normalised problem: block tile, and into how many K ranges the product is
// split (1: one pass; more: partial products into the workspace, then the reduction pass).
// tail_splits > 1: the tiles that fill whole rounds of the persistent grid are computed in one
// pass, and only the tiles of the last, partly filled round are split over K.
struct Plan { int tile; int splits; int tail_splits; };

constexpr int64_t kWorkspaceBytes = 64ll << 20;    // split-K partial products, per device
constexpr int64_t kStaticScratchBytes = 16ll << 20;   // those of the allocation-free entry point

const fg::KernelEntry *table_h16_for(bool a_kc, bool b_kc) {
    if (!a_kc && b_kc) return fg::kernel_table_nn_h16();
    if (!a_kc && !b_kc) return fg::kernel_table_nt_h16();
    if (a_kc && b_kc) return fg::kernel_table_tn_h16();
    return fg::kernel_table_tt_h16();
}

const fg::KernelEntry *table_for(bool a_kc, bool b_kc) {
    if (!a_kc && b_kc) return fg::kernel_table_nn();
    if (!a_kc && !b_kc) return fg::kernel_table_nt();
    if (a_kc && b_kc) return fg::kernel_table_tn();
    return fg::kernel_table_tt();
}

// The params heuristic (Section 4.2.1 picks the largest tile that fits shared memory; here every
// tile fits, so the question is which shape, and which split of K, finishes first).  Estimated
// time = rounds x (time of one workgroup on its share of K + the time of its epilogue) + the cost
// of the reduction pass if K is split.  A round = as many workgroups as there are slots, 256 compute
// units x workgroups of that shape per unit, the last one with those that it has; a workgroup's rate is a measured fraction of what a
// compute unit sustains with the 256x256 tile (about 4.7 TFLOP/s), one set for workgroups that
// share a unit and one for a workgroup that has a unit to itself.  Edge tiles are predicated, so
// a tile need not divide the problem.  K is split only when the output has too few tiles to fill
// the GPU and K is long (may_split: plain real products).
// k32: the kernel family has a 256x256 kernel named for its 16x16x32 matrix instructions (TILE_256x256_K32).  It is not a candidate
// of its own.  k32 == 2: it replaces the 256x256 tile
// when that one is chosen and the output has such a tile for at least three quarters of the
// compute units (addition on A and B, whose two 256x256 kernels differ: measured +1 to +5 % from 192 tiles up, K from 1024
// to 8192; equal at 176 tiles, -1 to -6 % at 160 and fewer: a partly busy chip is not at its power limit; in the other
// families both entries are one kernel).  k32 == 1: only when forced (A and B both M/N-contiguous).
// allow_groups: the family has the tiles with K groups.  The rates, the cost of a split and the prices of rows off the
// lines are fitted to the times of replayed graphs of every tile and split forced over 190 products (64x64x32768 to
// 4876x7518x2448): the choice by them alone is on average 1.7 % slower than the fastest (5 % with the rates before the larger
// rings), at most 42 % (6708x5150x96), and over 16 % only with K up to 224; held to what plan_product promises, 3.4 % (4.7 %).
// Since then the rates of the two large tiles went up with their K loops (1 -> 1.12, 0.88 -> 0.95): 2 of the 190 products take another
// plan, and 572 of 60000 random ones, 266 of which at 0.93 of the time by the rates before, 0.76 to 1.14.
constexpr int kTileM[fg::TILE_COUNT] = {256, 256, 128, 64, 128, 256, 64, 64, 64, 256, 128};
constexpr int kTileN[fg::TILE_COUNT] = {256, 128, 128, 64, 128, 256, 64, 64, 128, 128, 128};
constexpr int kTilesPerCU[fg::TILE_COUNT] = {1, 1, 2, 4, 1, 1, 2, 1, 1, 1, 1};
constexpr int kSplits[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64}, kSplitCount = sizeof kSplits / sizeof *kSplits;
struct Rates {
    double shared[fg::TILE_COUNT], alone[fg::TILE_COUNT];
    double round_fixed, cu_cd_bw, reduce_launch, reduce_bw;
    // A piece of 64 elements lies on two 128-byte lines where its row does not begin on one, and a line costs a unit's
    // fill path the same whole or in part (64x64 tiles fetched with rows 5936 bytes apart: 54 GB/s per unit, 4096
    // apart 128): what the K loop takes longer for each of A and B whose rows are off the lines.
    double off_line[fg::TILE_COUNT];
    bool last_round;         // the last, partly filled round is priced with the workgroups that it has
    // K groups and sets of accumulators per group, which share a workgroup's sum over K (TileCfg::KG, ACC_SETS)
    int groups[fg::TILE_COUNT] = {1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1}, sets[fg::TILE_COUNT] = {1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1};
};
// Sets of the 256x128 tile: it has two, but is counted with the one of eight waves.  With two the limit on sums (plan_product) admits it in
// place of the 256x256 tile's twice as many ranges, which is slower (29 products 1.03, 8784x160x16016 90.4 and 122.6 us).
constexpr Rates kRates = {{1.12, 0.95, 0.732, 0.596, 0.74, 1, 0.373, 0.367, 0.384},
                          {1.12, 0.95, 0.527, 0.169, 0.74, 1, 0.233, 0.367, 0.384},
                          2.07e-6, 26.8e9, 6.92e-6, 8.7e12,
                          {0, 0.022, 0, 0.0446, 0.0395, 0, 0.09, 0.142, 0.098}, true,
                          {1, 1, 1, 1, 1, 1, 2, 2, 2, 1, 1}, {1, 1, 1, 1, 2, 1, 2, 2, 2, 1, 2}};
// K up to 512, with C 768, where the 256x128 tile has eight waves (select_kernel): its rate with those.  At the one above it took products
// from the smaller tiles that these are faster on (47 random ones with K up to 256 from the 64x64 tile, which takes 0.84 of the time, at best
// 0.74, 752x6032x144 with C 13.3 -> 9.8 us; 16 from the 128x128 tile, 0.92, with C and K from 512 to 768 on it 0.87 to 0.97; 7 go to the 256x256
// tile, 0.98).
constexpr Rates kRatesShort = {{1.12, 0.88, 0.732, 0.596, 0.74, 1, 0.373, 0.367, 0.384},
                               {1.12, 0.88, 0.527, 0.169, 0.74, 1, 0.233, 0.367, 0.384},
                               2.07e-6, 26.8e9, 6.92e-6, 8.7e12,
                               {0, 0.022, 0, 0.0446, 0.0395, 0, 0.09, 0.142, 0.098}, true,
                               {1, 1, 1, 1, 1, 1, 2, 2, 2, 1, 1}, {1, 1, 1, 1, 2, 1, 2, 2, 2, 1, 2}};
// Addition on A and B and diagonal operands, whose kernels of the large tiles have eight waves (170 diagonal products above 256 MB took the 256x256
// tile by the rates above, at 1.085 of the time, 11888x2800 with A diagonal 78.7 and 96.1 us); what all real products were priced with
// before there were others (see plan_product).
constexpr Rates kRatesAdd = {{1, 0.88, 0.732, 0.596, 0.74, 1, 0.373, 0.367, 0.384},
                             {1, 0.88, 0.527, 0.169, 0.74, 1, 0.233, 0.367, 0.384},
                             2.07e-6, 26.8e9, 6.92e-6, 8.7e12,
                             {0, 0.022, 0, 0.0446, 0.0395, 0, 0.09, 0.142, 0.098}, true,
                             {1, 1, 1, 1, 1, 1, 2, 2, 2, 1, 1}, {1, 1, 1, 1, 2, 1, 2, 2, 2, 1, 2}};
using fg::TileCfg;
static_assert(FG_CFG_K32(256, 256, 64, 2, 2, 2, false, true, false, false)::ACC_SETS == 1 && FG_CFG_K32(256, 128, 64, 3, 2, 2, false, true, false, false)::ACC_SETS == 2 &&
              FG_CFG(256, 128, 64, 3, 4, 2, false, true, false)::ACC_SETS == 1 && FG_CFG_K32(128, 128, 64, 4, 2, 2, false, true, false, false)::ACC_SETS == 2 &&
              FG_CFG(128, 128, 64, 4, 4, 2, false, true, false)::ACC_SETS == 2 && FG_CFG_KG(false, true, false, false, false, 64, 2, false)::ACC_SETS == 2 &&
              FG_CFG_KG(false, true, false, false, false, 64, 4, true)::ACC_SETS == 2 && FG_CFG_KG(false, true, false, false, false, 128, 3, true)::ACC_SETS == 2, "Rates::sets");
// Binary16 C and D with K from 512 on: a tile's C and D at three quarters of the bytes (they are half, in lines that are accessed
// all the same), rows off the lines priced for the tiles without K groups (these products cannot be split, and were priced
// without), and the 64x64 tile at its former shared rate.  216 random products: 0.6 % slower than the fastest tile on average, over 5 % for
// 11 (without all that 2.4 % and 39: 3817x2363x1944 66.8 -> 53.2 us, 6308x2574x1016 77.1 -> 56.7, 1600x5376x768 with C 32.6 -> 27.8).
// With a price on the K groups too, long narrow products leave the 64x128 tile for the deep 128x128 one, which has half as many workgroups
// (8799x66x14168 94.7 and 175.3 us; 19 of 19 slower).  A shorter K keeps the rates above: these chose tiles 17 to 44 % slower there.
constexpr Rates kRates16 = {{1, 0.88, 0.732, 0.40, 0.74, 1, 0.373, 0.367, 0.384},
                            {1, 0.88, 0.527, 0.169, 0.74, 1, 0.233, 0.367, 0.384},
                            2.07e-6, 26.8e9 * 4 / 3, 6.92e-6, 8.7e12,
                            {0, 0.022, 0, 0.0446, 0.0395, 0, 0, 0, 0}, true,
                            {1, 1, 1, 1, 1, 1, 2, 2, 2, 1, 1}, {1, 1, 1, 1, 2, 1, 2, 2, 2, 1, 2}};
// The rates that decided what a call needs scratch memory for before the 64x64 tile had K groups
// (see plan_product).
constexpr Rates kPromisedRates = {{1.0, 0.8, 0.73, 0.45, 0.57, 1.0, 0, 0, 0}, {1.0, 0.8, 0.43, 0.17, 0.57, 1.0, 0, 0, 0}, 2e-6, 25e9, 6e-6, 3e12, {}, false};
// The rates of the planner before the larger rings (four K groups as tile 7, no 64x128 tile): see plan_product.
constexpr Rates kFormerRates = {{1.0, 0.8, 0.73, 0.40, 0.645, 1.0, 0.35, 0.29, 0}, {1.0, 0.8, 0.43, 0.135, 0.645, 1.0, 0.27, 0.29, 0}, 1.6e-6, 27e9, 12.3e-6, 7.2e12,
                                {0, 0, 0, 0, 0, 0, 0.1, 0.1, 0}, false, {1, 1, 1, 1, 1, 1, 2, 4, 1, 1, 1}};
// Contractions have neither K groups nor splits, which the rates above were fitted with: over 320 contractions those
// picked the fastest tile to within 2.4 % on average and 44 % at most (192 x 960 rows and columns over 2560: 33.8 us
// with the deep 128x128 tile, 23.6 with the 64x64 tile), these to within 0.5 % and 43 %, and no tile slower than
// either those or the promised rates pick (176 batches of 120 x 112 over 320: 11.6 us, 17.2 by the promised rates).
constexpr Rates kContractRates = {{1.0, 0.8, 0.73, 0.394, 0.57, 1.0, 0, 0, 0}, {1.0, 0.8, 0.43, 0.17, 0.57, 1.0, 0, 0, 0}, 1.8e-6, 25e9, 0, 1, {}, false};

// What an estimate takes from the rates alone, seconds; index n: n + 1 workgroups share a compute unit.  A call makes up to
// four searches (the former planners' too, see plan_product), which bounds the host's part of a small or split
// product; so they have no divisions left in them and skip a tile that cannot win: 256^3
// 0.20 -> 0.14 us on the host (2.7 GHz Xeon), 128x4096x16384 2.3 -> 1.05; 1024^3, which used to ask one planner, 0.44 and 0.45.
struct Prices {
    bool has[fg::TILE_COUNT];
    double k_tile[fg::TILE_COUNT][4], epilogue[fg::TILE_COUNT][4];      // of a K tile, and of the rest of a workgroup
    double unit_k_tile[fg::TILE_COUNT];                                 // a K tile's share of a unit's time, at the least
    double off_line[fg::TILE_COUNT], reduce_launch, reduce_byte;
    bool last_round;
    int8_t group_shift[fg::TILE_COUNT], set_shift[fg::TILE_COUNT];
};
constexpr int log2_of(int x) { return x == 1 ? 0 : 1 + log2_of(x / 2); }
constexpr Prices priced(const Rates &r) {
    constexpr double cu_flops = 4.7e12;
    Prices p{};
    for (int t = 0; t < fg::TILE_COUNT; ++t) {
        p.has[t] = r.shared[t] != 0 && t != fg::TILE_256x256_K32;
        p.off_line[t] = r.off_line[t];
        p.group_shift[t] = (int8_t)log2_of(r.groups[t]);
        p.set_shift[t] = (int8_t)log2_of(r.sets[t]);
        for (int n = 0; n < kTilesPerCU[t] && p.has[t]; ++n) {
            // workgroups that share a compute unit at a time: a unit's rate grows linearly from the
            // lone-workgroup rate to the rate with every slot taken, and is divided among them
            const double unit = kTilesPerCU[t] == 1 ? r.alone[t] : r.alone[t] + (r.shared[t] - r.alone[t]) * n / (kTilesPerCU[t] - 1);
            p.k_tile[t][n] = 2.0 * kTileM[t] * kTileN[t] * 64 / (cu_flops * unit / (n + 1));
            // the C read and D write of a tile stream at what one compute unit gets of the memory
            // bandwidth, divided among the workgroups that share the unit
            p.epilogue[t][n] = r.round_fixed + (n + 1) * 8.0 * kTileM[t] * kTileN[t] / r.cu_cd_bw;
            const double share = p.k_tile[t][n] / (n + 1);
            if (n == 0 || share < p.unit_k_tile[t]) p.unit_k_tile[t] = share;
        }
    }
    p.reduce_launch = r.reduce_launch;
    p.reduce_byte = 1 / r.reduce_bw;
    p.last_round = r.last_round;
    return p;
}
constexpr Prices kPrices = priced(kRates), kPricesShort = priced(kRatesShort), kPrices16 = priced(kRates16), kPricesAdd = priced(kRatesAdd), kContractPrices = priced(kContractRates);
constexpr Prices kPromisedPrices = priced(kPromisedRates), kFormerPrices = priced(kFormerRates);

// The K ranges that a product may be split into: at least four K tiles (256 k) each.
struct KRanges {
    int32_t nk;                       // K tiles (every real kernel has BK = 64)
    int n = 0;
    int32_t share[kSplitCount];       // K tiles of one of kSplits[i] ranges, i < n
    explicit KRanges(int64_t K) : nk((int32_t)((K + 63) / 64)) {
        // divided by multiplication: nk is below 2^25, so (2^40 / S, rounded up) is off by less than 2^25 / 2^40
        do { share[n] = (int32_t)(((uint64_t)(nk + kSplits[n] - 1) * kInverse.of[n]) >> 40); ++n; } while (n < kSplitCount && nk >= 4 * kSplits[n]);
    }
    struct Inverse { uint64_t of[kSplitCount]; };
    static constexpr Inverse inverses() {
        Inverse v{};
        for (int i = 0; i < kSplitCount; ++i) v.of[i] = ((1ull << 40) + kSplits[i] - 1) / kSplits[i];
        return v;
    }
    static const Inverse kInverse;
};
constexpr KRanges::Inverse KRanges::kInverse = KRanges::inverses();

struct Shifts { int m[fg::TILE_COUNT], n[fg::TILE_COUNT], slots[fg::TILE_COUNT], cu; };
constexpr Shifts shifts_of_tiles() {
    Shifts s{};
    s.cu = log2_of(kNumCU);
    for (int t = 0; t < fg::TILE_COUNT; ++t) {
        s.m[t] = log2_of(kTileM[t]);
        s.n[t] = log2_of(kTileN[t]);
        s.slots[t] = s.cu + log2_of(kTilesPerCU[t]);
    }
    return s;
}
constexpr Shifts kShifts = shifts_of_tiles();
static_assert(1 << kShifts.cu == kNumCU, "the searches shift instead of dividing");

// How many additions follow one another in an entry of a plan of S ranges of `share` K tiles: four matrix instructions to a K
// tile in one accumulator, and the partial products of the ranges.  The error against 64 bits goes with the square root: with T products
// in all, the rounding of T / n sums of n adds T * n, that of adding them up T * (T / n).
int32_t sum_length(const Prices &prices, int tile, int S, int32_t share) {
    const int g = prices.group_shift[tile];
    return (((share + (1 << g) - 1) >> g) * 4 >> prices.set_shift[tile]) + S;
}

// longest: no plan whose sums are longer (sum_length).
Plan choose_plan(int64_t M, int64_t N, const KRanges &ranges, bool may_split, bool allow_smallest, int64_t batches,
                 bool allow_deep, int k32, bool allow_groups, int64_t scratch_bytes, const Prices &prices, int straddling = 0, int32_t longest = INT32_MAX) {
    constexpr double tail_launch = 6e-6, tail_bw = 3e12;      // the leftover tiles' reduction follows a full round
    // tuning overrides (see read_tuning_from_environment)
    int force_tile = -1;
    const int force_split = g_force_split.load(std::memory_order_relaxed), force_tail = g_force_tail.load(std::memory_order_relaxed);
    bool force_k32 = false, forced_plain = false;
    {
        int t = g_force_tile.load(std::memory_order_relaxed);
        if (t == fg::TILE_256x256_K32) { t = fg::TILE_256x256; force_k32 = true; }
        else forced_plain = (t == fg::TILE_256x256);
        if (t == fg::TILE_256x128_PASS) t = fg::TILE_256x128;
        if (t == fg::TILE_128x128_PASS) t = fg::TILE_128x128_DEEP;
        if (t >= 0 && t < fg::TILE_COUNT) force_tile = t;
    }
    const int32_t nk = ranges.nk;
    Plan best{0, 1, 1}, large_tail{0, 1, 1};
    constexpr double never = 1e300;
    double best_cost = never, large_tail_cost = never;
    for (int t = 0; t < fg::TILE_COUNT; ++t) {
        if (force_tile >= 0 && t != force_tile) continue;
        if (t == fg::TILE_64x64 && !allow_smallest) continue;
        if (t == fg::TILE_128x128_DEEP && !allow_deep) continue;
        if (!prices.has[t] || (t >= fg::TILE_64x64_KG2 && !allow_groups)) continue;
        const int slot_shift = kShifts.slots[t];
        const int64_t tiles = ((M + kTileM[t] - 1) >> kShifts.m[t]) * ((N + kTileN[t] - 1) >> kShifts.n[t]) * batches;
        const int64_t slots = 1ll << slot_shift;
        const int64_t slot_bytes = (int64_t)kTileM[t] * kTileN[t] * 4;
        // no plan of this tile can take less than its K tiles at the best rate
        if (force_tail < 2 && (double)tiles * nk * prices.unit_k_tile[t] * (1.0 / kNumCU) >= best_cost) continue;
        const double lines = 1 + prices.off_line[t] * straddling;
        auto share_time = [&](int64_t wgs, int S, int32_t share) {     // one workgroup on its share of K, plus its epilogue
            int64_t n = wgs <= kNumCU ? 0 : (wgs - 1) >> kShifts.cu;         // (no workgroups at all: the plan query of an empty result)
            if (n >= kTilesPerCU[t]) n = kTilesPerCU[t] - 1;
            return prices.k_tile[t][n] * share * (S == 1 || prices.last_round ? lines : 1) + prices.epilogue[t][n];
        };
        // K groups: at least four K tiles for each, or their reduction costs more than they save (256^3:
        // 4.5 us on the GPU with one group, 4.8 with two; 519x736x320: 5.1, 5.5); the larger rings, which take longer to
        // fill, from six on.  With fewer than 56 workgroups the ring of four buffers takes eight: with few at the memory
        // the ring of two does not wait (47 products of fewer tiles and twelve to fifteen K tiles 3 to 12 % faster with it, 184x9x864
        // 6.9 -> 6.1 us, 52 to 57 tiles even, from 60 on 1 to 13 % slower, 4291x17x912 7.2 and 8.1; split ranges of that length: 20
        // products of 4 to 48 workgroups up to 21 % faster with the ring of two, 30x284x3768 9.9 -> 8.4, with more 2 to 9 % slower).
        const int32_t least = t < fg::TILE_64x64_KG2 || force_tile >= 0 ? 0 : t == fg::TILE_64x64_KG2 ? 8 : prices.last_round ? 12 : 16;
        auto least_of = [&](int S) { return t == fg::TILE_64x64_KG2_DEEP && force_tile < 0 && prices.last_round && tiles * S < 56 ? 16 : least; };
        auto consider = [&](int S, int tail, int32_t share, double cost) {
            if (cost >= best_cost || nk < least_of(S) * S * tail || sum_length(prices, t, S, share) > longest) return;
            best = Plan{t, S, tail};
            best_cost = cost;
        };
        // (a) every tile split S ways (S = 1: the plain launch)
        auto split_all = [&](int S, int32_t share) {
            const int64_t wgs = tiles * S;
            const int64_t whole = wgs >> slot_shift, last = wgs & (slots - 1);
            double cost = prices.last_round && last > 0 ? (whole > 0 ? (double)whole * share_time(slots, S, share) : 0.0) + share_time(last, S, share)
                                                        : (double)(whole + (last > 0)) * share_time(wgs, S, share);
            if (S > 1) cost += prices.reduce_launch + (2.0 * S + 2.0) * (double)(tiles * slot_bytes) * prices.reduce_byte;
            consider(S, 1, share, cost);
        };
        if (force_split >= 1) {                                   // one candidate: the forced split, if it is possible
            const bool legal = force_split == 1 || (may_split && force_split <= nk && tiles * force_split * slot_bytes <= scratch_bytes);
            const int S = legal ? force_split : 1;
            split_all(S, (nk + S - 1) / S);
            continue;
        }
        for (int i = 0; i < ranges.n; ++i) {
            if (i > 0 && (!may_split || tiles * kSplits[i] * slot_bytes > scratch_bytes)) break;
            // The rates of the plain 64x64 tile were fitted to whole products.  Split, it is overrated: 60 plans that it won take 0.90 of its
            // time on the tiles with K groups or the deep 128x128 one (157x4293x12808 75.7 -> 56.4 us, 5219x11x14856 43.7 -> 36.6; two are 3
            // and 5 % slower), so it is left to ranges that are too short for K groups.
            if (i > 0 && t == fg::TILE_64x64 && allow_groups && prices.last_round && nk >= 8 * kSplits[i]) continue;
            split_all(kSplits[i], ranges.share[i]);
        }
        // (b) whole rounds in one pass, the tiles of the last, partly filled round split over K
        const int64_t rest = tiles & (slots - 1), full = tiles - rest;
        if (!may_split || full == 0 || rest == 0 || force_tail == 1) continue;
        if (force_tail > 1) {
            if (force_tail <= nk && rest * force_tail * slot_bytes <= scratch_bytes) consider(1, force_tail, nk, 0.0);
            continue;
        }
        const double in_front = (double)(full >> slot_shift) * share_time(full, 1, nk) + 2e-6 + tail_launch;
        for (int i = 1; i < ranges.n; ++i) {
            const int S = kSplits[i];
            if (rest * S > slots || rest * S * slot_bytes > scratch_bytes) break;
            const double cost = in_front + share_time(rest * S, S, ranges.share[i]) + (2.0 * S + 2.0) * (double)(rest * slot_bytes) * (1 / tail_bw);
            consider(1, S, nk, cost);
            if (t == fg::TILE_256x256 && sum_length(prices, t, 1, nk) <= longest && cost < large_tail_cost) {
                large_tail = Plan{t, 1, S};
                large_tail_cost = cost;
            }
        }
    }
    // Of two plans with whole rounds in front of a split tail, the 256x256 tile's runs 4 % faster than the 256x128 tile's whose
    // estimate is up to 9 % lower (36 such products, 0.885 to 1.006: 6318x2901x3304 174.0 -> 153.9 us, 4361x3946x5016 with C 245.5 -> 233.3,
    // 8000x2240x4352 175.4 and 176.5).
    if (prices.last_round && force_tile < 0 && force_split < 1 && best.tile == fg::TILE_256x128 && best.tail_splits > 1 &&
        large_tail_cost <= 1.09 * best_cost)
        best = large_tail;
    if (best.tile == fg::TILE_256x256 && k32 > 0 && !forced_plain) {
        const int64_t tiles = ((M + 255) / 256) * ((N + 255) / 256) * batches;
        if (force_k32 || (k32 == 2 && tiles >= kNumCU * 3 / 4)) best.tile = fg::TILE_256x256_K32;
    }
    return best;
}

// Scratch bytes that a plan's partial products take.
int64_t scratch_need(const Plan &plan, int64_t M, int64_t N) {
    if (plan.splits <= 1 && plan.tail_splits <= 1) return 0;
    const int t = plan.tile;
    const int64_t tiles = ((M + kTileM[t] - 1) >> kShifts.m[t]) * ((N + kTileN[t] - 1) >> kShifts.n[t]);
    const int64_t tile_bytes = (int64_t)kTileM[t] * kTileN[t] * 4;
    return (plan.splits > 1 ? tiles * plan.splits : (tiles & ((1ll << kShifts.slots[t]) - 1)) * plan.tail_splits) * tile_bytes;
}

// The most that a product with this need may take: none, the static array, the workspace.
int64_t scratch_class(int64_t bytes) { return bytes == 0 ? 0 : bytes <= kStaticScratchBytes ? kStaticScratchBytes : kWorkspaceBytes; }

// What the planner before the larger rings chose (kFormerRates, four K groups as tile 7, itself held to the scratch classes of
// kPromisedRates), as far as calls still depend on it.
struct Former { int64_t scratch; int32_t longest; };
Former former_plan(int64_t M, int64_t N, int64_t K, const KRanges &ranges, bool may_split, int k32, int straddling) {
    int64_t promised = 0;
    if (may_split) promised = scratch_class(scratch_need(choose_plan(M, N, ranges, true, true, 1, true, k32, false, kWorkspaceBytes, kPromisedPrices), M, N));
    // (the best plan within the promised class; rows off the lines counted in long K loops only, and only for a split)
    auto plan_of = [&](int lines) { return choose_plan(M, N, ranges, promised > 0, true, 1, true, k32, true, promised, kFormerPrices, lines); };
    const int lines = promised > 0 && K > 3904 ? straddling : 0;
    Plan former = plan_of(lines);
    if (lines > 0 && former.splits == 1 && former.tail_splits == 1) former = plan_of(0);
    const int32_t share = (ranges.nk + former.splits - 1) / former.splits;
    return Former{scratch_class(scratch_need(former, M, N)), sum_length(kFormerPrices, former.tile, former.splits, share)};
}

// Plan of a real product without a diagonal operand.  Two things that the former planner chose hold still:
// - Which scratch memory a call needs is part of what it promises: a call that needed none can be captured before the
//   workspace exists and beside others, one whose partial products fit the static array can be made without allocation.  So no plan
//   leaves the class (none, static array, workspace) of the former one (6 % of random shapes).
// - No sum is longer (sum_length): fewer partial sums of a long K (0.7 % of random shapes) had an error against 64 bits 19 % larger on
//   average, 408x8792x12960 4.2e-7 -> 7.2e-7, and were 6 % slower than by the former plan; held to it 48 of them are 3 % faster
//   with an error 8 % smaller.  Twice as many ranges as before, whose partial products are added up one after the other (9 % of
//   random shapes, small outputs with a long K), had one 3 to 20 % larger; those are as fast as before on average (0.88 to 1.16), 22 % more exact.
// The former plan's own tile and split are always among the candidates (the larger ring with two groups of two sums in place of
// the four groups).  Products of fewer than eight K tiles have neither splits nor groups and need not ask.  Costs about 1 us on the host.
// Both hold as well against the rates before the kernels with four waves (kRatesAdd).  These left to the deep 128x128 tile, with two sums
// to an entry, what would run on the 256x256 tile's one now: 34 such products had an error against 64 bits 1.38 times as
// large, 3360x2592x4288 2.82e-7 -> 4.23e-7; and 81 of 60000 random products would need scratch memory where they needed none, or more than
// the static array (2960x6976x5680, 696x2002x8416).  Only a plan with that tile or with a split has to ask.
Plan plan_product(int64_t M, int64_t N, int64_t K, bool may_split, int k32, int straddling, const Prices &prices) {
    const KRanges ranges(K);
    const bool forced = g_force_split.load(std::memory_order_relaxed) >= 1 || g_force_tail.load(std::memory_order_relaxed) > 1 ||
                        g_force_tile.load(std::memory_order_relaxed) >= 0;
    if (forced) return choose_plan(M, N, ranges, may_split, true, 1, true, k32, true, kWorkspaceBytes, prices, straddling);
    const Former former = ranges.n == 1 ? Former{may_split ? kWorkspaceBytes : 0, INT32_MAX} : former_plan(M, N, K, ranges, may_split, k32, straddling);
    auto plan_of = [&](const Prices &by, int64_t scratch, int32_t longest) {
        return choose_plan(M, N, ranges, scratch > 0, true, 1, true, k32, true, scratch, by, straddling, longest);
    };
    const Plan plan = plan_of(prices, former.scratch, former.longest);
    const bool large = plan.tile == fg::TILE_256x256 || plan.tile == fg::TILE_256x256_K32, split = plan.splits > 1 || plan.tail_splits > 1;
    if ((!large && !split) || (&prices != &kPrices && &prices != &kPricesShort)) return plan;
    const Plan before = plan_of(kPricesAdd, former.scratch, former.longest);
    auto sum_of = [&](const Plan &p) { return sum_length(kPricesAdd, p.tile, p.splits, (ranges.nk + p.splits - 1) / p.splits); };
    const int64_t allowed = scratch_class(scratch_need(before, M, N));
    if (scratch_need(plan, M, N) <= allowed && (!large || sum_of(plan) <= sum_of(before))) return plan;
    return plan_of(prices, allowed, std::min(former.longest, sum_of(before)));
}

// Tile of the complex and dual kernels (256x128, 128x128 with two workgroups per unit, 64x64 with
// four, 64x64 with K groups with one): the one with the smallest estimated time.  Whole rounds run with every slot of a unit
// taken, the workgroups of the last, partly filled round share a unit with fewer others; a
// workgroup's rate is a fraction of what a unit sustains with the 256x128 tile.  Over 130 random products (K 8 to 3000) the choice is
// 0.7 % slower than the fastest tile on average, over 5 % for nine (2.1 % and 18 without the rules on K).
// A K up to 128 makes the product a pass over C and D, which four small workgroups per unit overlap best (complex
// 986x5218x88 with C: 23.4 us with the 64x64 tile, 31.5 and 33.9 with the larger ones; dual 2141x1751x8 12.5, 16.6, 18.4; of 79
// such products the 64x64 tile is more than 2 % slower than another in five, at most 14 %, 6528x2560x24).
// The 64x64 tile with two K groups: one tile per unit and K steps for both groups, 1024^3 22.4 -> 15.9 us against the tile with
// one group, 500x700x3000 interleaved 53.5 -> 33.5, and sums half as long: the error against 64 bits is 0.73 to 0.78 of one group's.
// For that it is taken from K = 168 on, though up to 216 the second group costs planar operands 3 to 14 % (195x702x176 5.6, 6.1; around
// 250 it is even, interleaved ones gain from 216 on; 42 products); from 136 to 160 it costs 8 to 18 %, in a second round it does not
// pay (1300x1300x800 21.8, 26.4; 1536^2 x 512 21.5, 29.7).
int choose_ctile(int64_t M, int64_t N, int64_t K) {
    static const int bm[fg::CTILE_COUNT] = {256, 128, 64, 64};
    static const int bn[fg::CTILE_COUNT] = {128, 128, 64, 64};
    static const int per_cu[fg::CTILE_COUNT] = {1, 2, 4, 1};
    static const double rate_shared[fg::CTILE_COUNT] = {1.0, 0.94, 0.72, 0.7};
    static const double rate_alone[fg::CTILE_COUNT] = {1.0, 0.74, 0.45, 0.7};
    const int forced = g_force_tile.load(std::memory_order_relaxed);      // tuning override, 0..3 here
    if (forced >= 0 && forced < fg::CTILE_COUNT) return forced;
    if (K <= 128) return fg::CTILE_64x64;
    int best = 0;
    double best_cost = -1;
    for (int t = 0; t < fg::CTILE_COUNT; ++t) {
        const int64_t tiles = ((M + bm[t] - 1) / bm[t]) * ((N + bn[t] - 1) / bn[t]);
        const int64_t slots = (int64_t)kNumCU * per_cu[t];
        if (t == fg::CTILE_64x64_KG2 && (tiles > slots || K <= 160)) continue;
        auto tile_time = [&](int64_t sharing) {     // one tile, `sharing` workgroups on its unit
            const double unit = per_cu[t] == 1 ? rate_alone[t]
                              : rate_alone[t] + (rate_shared[t] - rate_alone[t]) * (double)(sharing - 1) / (per_cu[t] - 1);
            return (double)bm[t] * bn[t] * (double)sharing / unit;
        };
        const int64_t full = tiles / slots, rest = tiles - full * slots;
        double cost = (double)full * tile_time(per_cu[t]);
        if (rest > 0) cost += tile_time((rest + kNumCU - 1) / kNumCU);
        // More than a round of small tiles with a long K: they fall behind the estimate (the next larger tile, of 22 products:
        // K 144 to 504 0.87 to 1.01 as fast, from 512 on 1.04 to 1.39 but for interleaved ones up to K = 1000, 0.93 to 0.99;
        // dual 2701x3001x1504 141 us, 126 on the 128x128 tile, 1617x3113x904 60.1 and 43.3)
        if (t == fg::CTILE_64x64 && tiles > slots && K >= 512) cost *= 1.29;
        if (best_cost < 0 || cost < best_cost) { best = t; best_cost = cost; }
    }
    return best;
}

// Whether C and D stay in the caches (GemmParams::cd_cached).  (The plan query has neither a C nor leading dimensions.)
bool keeps_cd(const Problem &q) {
    const int64_t ab = (q.M * q.K + q.K * q.N) * 2, cd = q.M * q.N * (q.cd16 ? 2 : 4) * (q.C ? 2 : 1), elem = q.ilv ? 8 : q.cd16 ? 2 : 4;
    return q.cplx ? fg::keeps_complex_cd(2 * ab, 2 * cd, q.K, q.ilv, q.C != nullptr, q.ldc * elem, q.ldd * elem)
                  : fg::keeps_real_cd(ab, cd, q.C != nullptr, q.ldc * elem, q.ldd * elem);
}

// Kernel variant for a normalised problem.
const fg::KernelEntry *select_kernel(const Problem &q, Plan *plan_out = nullptr) {
    if (plan_out) *plan_out = Plan{0, 1, 1};
    if (q.cplx) {
        const int t = choose_ctile(q.M, q.N, q.K);
        if (t < 0) return nullptr;
        const int v = (q.a_kc ? 2 : 0) + (q.b_kc ? 0 : 1);     // nn, nt, tn, tt
        if (q.ilv) return &fg::kernel_table_cplx_il()[t * 4 + v];
        return &(q.dual ? fg::kernel_table_dual() : fg::kernel_table_cplx())[t * 4 + v];
    }
    const bool may_split = plan_out && !q.a_diag && !q.b_diag && !q.cd16;   // the reduction pass writes FP32
    const int k32 = (q.a_diag || q.b_diag) ? 0 : q.ab_add ? (q.a_kc != q.b_kc ? 2 : 0) : ((q.a_kc || q.b_kc) ? 2 : 1);
    // Rows off a line: by the extents (a row is whole 16-byte pieces), so that the plan query, which knows no leading
    // dimensions, says the same.  Rows that begin on half a line are not counted: 8192x243 over 4256, both K-contiguous,
    // 33.8 us in one pass, 41.7 split in two; 443x4534 33.8, and 35.4.
    auto off_line = [](int64_t extent) { return (extent + 7) / 8 % 4 != 0; };
    const bool long16 = q.cd16 && q.K >= 512;               // (see kRates16)
    const int off = (int)off_line(q.a_kc ? q.K : q.M) + (int)off_line(q.b_kc ? q.K : q.N);
    auto product = [&](bool split, const Prices &prices) { return plan_product(q.M, q.N, q.K, split, k32, may_split || long16 ? off : 0, prices); };
    Plan plan = q.a_diag || q.b_diag ? choose_plan(q.M, q.N, KRanges(q.K), false, true, 1, false, 0, false, 0, kPricesAdd)      // (eight waves)
                                     : product(may_split, long16 ? kPrices16 : q.ab_add ? kPricesAdd : q.K <= 512 ? kPricesShort : kPrices);
    // With C the 256x128 tile has eight waves up to K = 768 (below).  Only a plan of one pass is made again, for one pass: whether a product
    // is split does not depend on C, which the plan query does not know.
    if (q.C && !q.cd16 && !q.ab_add && q.K > 512 && q.K <= 768 && plan.tile == fg::TILE_256x128 && plan.splits == 1 && plan.tail_splits == 1)
        plan = product(false, kPricesShort);
    int tile = plan.tile;
    // A product with a diagonal operand is bound by its memory traffic (one pass over the dense
    // operand, C and D; a tile row only meets the K tiles on the diagonal).  While all of it fits the
    // 256 MB memory-side cache, the smallest tile, four workgroups per unit at different points
    // between their loads and their stores, measured fastest (4096^2: 26.6 us against 29.6 us with
    // the 256x256 tile, 8192 x 1024: 14.8 against 17.0); beyond that size its short pieces cost
    // more in memory than they gain (8192^2: 180 us against 135 us), and the estimate above decides.
    if ((q.a_diag || q.b_diag) && g_force_tile.load(std::memory_order_relaxed) < 0 && q.M * q.N * 10 <= (256ll << 20))
        tile = fg::TILE_64x64;
    const int forced = g_force_tile.load(std::memory_order_relaxed);
    // A short K makes a product a pass over C and D, on which eight waves and the 256x128 tile (TILE_256x128_PASS) can be faster than the
    // 256x256 tile that the estimate picks.  Time on the former by that on the latter, 340 products:
    // - K up to 128, 0.81 to 1.04, 0.93 on average (5408x5104x16 23.7 and 26.3 us); but with a C that stays in the caches 1.01 to 1.08 (5104x5344x96
    //   50.1 and 46.5), binary16 0.9, and without one off the half lines 0.93 to 1.1 (5748x5376x128 35.7 and 32.5; by M, see off_line), binary16 0.85;
    // - K up to 256 where C and D stream, 0.78 to 1.0 (6336x5824x256 with C 73.5 and 92.1), and binary16 results without C of more than 64 MB,
    //   0.72 to 1.02 (smaller ones 1.0 to 1.1); others 0.91 to 1.37 (4260x6688x256 48.6 and 35.6);
    // - K up to 768 with a C, where C and D stream, 0.78 to 1.0 (10272x4704x512 108.8 and 139.0, 3104x11680x768 109.9 and 123.0); binary16 up to 512
    //   0.91 to 1.02, from 640 on 1.01 to 1.08; others 0.93 to 1.28 (binary16 6240x6704x512 94 and 78).
    // Addition on A and B, whose 256x256 kernels have eight waves too: K up to 256 with one of the operands K-contiguous.
    if ((tile == fg::TILE_256x256 || tile == fg::TILE_256x256_K32) && !q.a_diag && !q.b_diag && forced < 0 && plan.splits == 1 && plan.tail_splits == 1) {
        const bool streams = !keeps_cd(q), large16 = q.cd16 && !q.C && q.M * q.N * 2 > (64ll << 20);
        const int64_t longest = q.ab_add ? (k32 > 0 ? 256 : 0) : streams ? (!q.C ? 256 : q.cd16 ? 512 : 768) : large16 ? 256 : q.cd16 || (!q.C && q.M % 16 == 0) ? 128 : 0;
        if (q.K <= longest) tile = fg::TILE_256x128;
    }
    if (!q.ab_add && !q.a_diag && !q.b_diag) {
        // Short K, where loading, multiplying and storing hardly overlap within a tile: eight waves on the 256x128 tile (2560^2 x 128 with
        // C 14.9 us with four, 12.9 with eight, 8192x1024x128 without 11.3 and 10.7, at K = 512 18.6 and 17.7, 16.0 and 17.1; at 768
        // 21.0 and 20.9, 18.9 and 20.7; binary16 results with C 19.3 and 18.3, 22.1 and 21.9; 1000: 23.7, 24.2, 25.4, 26.4).  Binary16 results
        // without C, whose stores are exchanged into lines first, up to 1024 (K 520 to 800 0.935 of the time of four, 42 products, 4088x1184x576
        // 14.7 -> 12.9; up to 1024 0.967, 21; forced, from 1152 on 0.96 to 1.03).
        const int64_t pass_k = q.C ? 768 : q.cd16 ? 1024 : 512;
        if (tile == fg::TILE_256x128 && (forced == fg::TILE_256x128_PASS || (forced < 0 && q.K <= pass_k))) tile = fg::TILE_256x128_PASS;
        // The same on the deep 128x128 tile (2048^2 x 128 with C 11.8 us with four waves, 10.4 with eight, 960x4096x256 without 9.5 and 8.7, 1304x2200x512
        // 13.0 and 12.4, 2000^2 x 760 17.1 and 16.6; 768: 15.8 and 16.0, 1536x2048x1024 12.8 and 14.0); a little longer where a last K tile
        // hangs over, which four waves load first and by itself (1536x2048x1000: 15.9 and 15.4, 16.1 and 16.0; 2000^2 x 2024: 28.1 and 29.3), and for
        // binary16 results with both operands off the lines, whose fills a second wave per SIMD covers better (K 1024 to 2560 0.965 of the time of
        // four, 78 products; up to 4096 0.99; FP32 results 0.93 to 1.1, 0.99 on average).
        const bool short_k = q.K <= 768 || (q.K < 1024 && q.K % 64 != 0) || (q.cd16 && off == 2 && q.K <= 2560);
        if (tile == fg::TILE_128x128_DEEP && (forced == fg::TILE_128x128_PASS || (forced < 0 && short_k && plan.splits == 1))) tile = fg::TILE_128x128_PASS;
    }
    if (plan_out) { *plan_out = plan; plan_out->tile = tile; }
    if (q.a_diag) return &fg::kernel_table_diag()[tile * 4 + (q.b_kc ? 0 : 1)];
    if (q.b_diag) return &fg::kernel_table_diag()[tile * 4 + (q.a_kc ? 2 : 3)];
    if (q.ab_add) {
        const fg::KernelEntry *t = !q.a_kc ? (q.b_kc ? fg::kernel_table_nn_xf() : fg::kernel_table_nt_xf())
                                           : (q.b_kc ? fg::kernel_table_tn_xf() : fg::kernel_table_tt_xf());
        return &t[tile];
    }
    if (q.cd16) return &table_h16_for(q.a_kc, q.b_kc)[tile];
    if (q.bf16) {
        const fg::KernelEntry *t = !q.a_kc ? (q.b_kc ? fg::kernel_table_nn_bf16() : fg::kernel_table_nt_bf16())
                                           : (q.b_kc ? fg::kernel_table_tn_bf16() : fg::kernel_table_tt_bf16());
        return &t[tile];
    }
    return &table_for(q.a_kc, q.b_kc)[fg::entry_index(tile, fg::VARIANT_MATRIX)];
}

// Once per (kernel, device): raise the dynamic LDS limit and ask how many workgroups of this
// kernel fit on a compute unit.
fg_status prepare(const fg::KernelEntry &k, int dev, int &per_cu) {
    static std::mutex m;
    static struct { const void *fn; int dev; int per_cu; } done[512];
    static int n_done = 0;
    std::lock_guard<std::mutex> lock(m);
    per_cu = 0;
    for (int i = 0; i < n_done; ++i)
        if (done[i].fn == k.fn && done[i].dev == dev) per_cu = done[i].per_cu;
    if (per_cu == 0) {
        hipError_t e = hipFuncSetAttribute(k.fn, hipFuncAttributeMaxDynamicSharedMemorySize, k.lds_bytes);
        if (e != hipSuccess) return fail(FG_ERR_LAUNCH, "hipFuncSetAttribute(%s): %s", k.name, hipGetErrorString(e));
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k.fn, k.threads, (size_t)k.lds_bytes);
        if (e != hipSuccess || per_cu < 1) return fail(FG_ERR_LAUNCH, "occupancy query for %s failed: %s", k.name, hipGetErrorString(e));
        if (n_done < 512) { done[n_done].fn = k.fn; done[n_done].dev = dev; done[n_done].per_cu = per_cu; ++n_done; }
    }
    return FG_OK;
}

// Split-K workspace: two allocations of kWorkspaceBytes per device, made by fg_init() or by the
// first call that splits K, and kept until the process ends.  One belongs to the default (null)
// stream, whose calls are ordered by it and need nothing else: an event behind each costs a call 4 us
// (one kernel after another on a stream: 2.9 us each, 6.8 with an event in between).  Every other
// stream uses the other one: calls on one stream are ordered anyway; a call on another stream than
// the previous user's first waits (on the device, not on the host) for the event that user recorded
// after its reduction pass, so that calls on different streams cannot overwrite each other's partial
// products.  So no call touches a stream but its own: on the default stream an operation from elsewhere
// would wait for the work of every blocking stream, and break a capture that one of them is under.
// A stream that is being captured into a graph takes no part in this (events recorded
// into a graph order nothing outside it): captured split-K calls must be ordered by the caller,
// and the workspace must exist before the capture starts (fg_init()).
struct Workspace {
    float *ptr = nullptr;                // of every stream but the default one
    float *of_default = nullptr;         // of the default stream; null: there was no memory for it, and that stream shares ptr
    hipEvent_t last_use = nullptr;       // recorded after the most recent split-K call's reduction pass in ptr
    hipStream_t last_stream = nullptr;
    bool used = false;
};
std::mutex g_ws_mutex;
Workspace g_ws[64];

bool stream_is_capturing(hipStream_t stream) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &st) != hipSuccess) { (void)hipGetLastError(); return false; }
    return st != hipStreamCaptureStatusNone;
}

// Must be called with g_ws_mutex held.
fg_status workspace_locked(int dev, hipStream_t stream, bool may_allocate, Workspace **out) {
    if (dev < 0 || dev >= 64) return fail(FG_ERR_LAUNCH, "device index %d out of range", dev);
    Workspace &w = g_ws[dev];
    if (!w.ptr) {
        if (!may_allocate || stream_is_capturing(stream))
            return fail(FG_ERR_UNSUPPORTED, "this call splits K and needs the library's workspace, which cannot be allocated while the "
                                            "stream is being captured: call fg_init() on this device before the capture");
        void *ptr = nullptr;
        hipError_t e = hipMalloc(&ptr, (size_t)kWorkspaceBytes);
        if (e != hipSuccess) return fail(FG_ERR_LAUNCH, "hipMalloc of the split-K workspace failed: %s", hipGetErrorString(e));
        e = hipEventCreateWithFlags(&w.last_use, hipEventDisableTiming);
        if (e != hipSuccess) { (void)hipFree(ptr); return fail(FG_ERR_LAUNCH, "hipEventCreate for the split-K workspace failed: %s", hipGetErrorString(e)); }
        w.ptr = (float *)ptr;
        if (hipMalloc(&ptr, (size_t)kWorkspaceBytes) == hipSuccess) w.of_default = (float *)ptr;
        else (void)hipGetLastError();
    }
    *out = &w;
    return FG_OK;
}

// The allocation-free entry point keeps its partial products in this array instead: part of the
// library's device image, so each GPU the library runs on holds one copy until the process ends.
// Host code never uses the symbol itself as an address: g_static_scratch[dev] is the array's
// device address on GPU `dev`, asked for once per device with that device current.
static __device__ __align__(256) float scratch[kStaticScratchBytes / 4];
float *g_static_scratch[64];

fg_status static_scratch(int dev, float **out) {
    static std::mutex m;
    if (dev < 0 || dev >= 64) return fail(FG_ERR_LAUNCH, "device index %d out of range", dev);
    std::lock_guard<std::mutex> lock(m);
    if (!g_static_scratch[dev]) {
        float *ptr = nullptr;
        hipError_t e = hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) return fail(FG_ERR_LAUNCH, "hipGetSymbolAddress of the static scratch array failed: %s", hipGetErrorString(e));
        g_static_scratch[dev] = ptr;
    }
    *out = g_static_scratch[dev];
    return FG_OK;
}

// The scratch memory of one split call: the workspace (ordered against its previous user on another
// stream, held until release) or the static array of the allocation-free entry point.
struct Scratch {
    float *ptr = nullptr;
    Workspace *guard = nullptr;          // set when the library orders the use
    bool by_stream = false;              // ... by the stream alone: release() has nothing to record
    std::unique_lock<std::mutex> lock{g_ws_mutex, std::defer_lock};

    fg_status acquire(bool static_only, int dev, hipStream_t stream) {
        if (static_only) return static_scratch(dev, &ptr);
        lock.lock();
        if (fg_status st = workspace_locked(dev, stream, true, &guard)) return st;
        by_stream = stream == nullptr && guard->of_default;
        ptr = by_stream ? guard->of_default : guard->ptr;
        if (by_stream) return FG_OK;                           // (this stream cannot be captured)
        if (stream_is_capturing(stream)) guard = nullptr;      // a captured call is ordered by its graph's caller
        else if (guard->used && (guard->last_stream != stream || stream == hipStreamPerThread)) {      // (one handle, a stream for each thread)
            hipError_t e = hipStreamWaitEvent(stream, guard->last_use, 0);
            if (e != hipSuccess) return fail(FG_ERR_LAUNCH, "hipStreamWaitEvent on the workspace's last use failed: %s", hipGetErrorString(e));
        }
        return FG_OK;
    }
    // The workspace where the library orders its use (not on a capturing stream), for callers that can do
    // without: no error is left behind.
    bool try_acquire(int dev, hipStream_t stream) {
        char kept[sizeof g_err];
        memcpy(kept, g_err, sizeof kept);
        const fg_status st = acquire(false, dev, stream);
        if (st == FG_OK && guard) return true;
        if (st != FG_OK) {
            memcpy(g_err, kept, sizeof kept);
            (void)hipGetLastError();
        }
        guard = nullptr;
        lock.unlock();
        return false;
    }
    fg_status release(hipStream_t stream) {
        if (!guard || by_stream) return FG_OK;
        hipError_t e = hipEventRecord(guard->last_use, stream);
        if (e != hipSuccess) return fail(FG_ERR_LAUNCH, "hipEventRecord after the split-K reduction failed: %s", hipGetErrorString(e));
        guard->last_stream = stream;
        guard->used = true;
        return FG_OK;
    }
};

// p: the parameters of kernel k, whose size the runtime takes from the kernel; the divisions by its tile counts are filled in.
fg_status launch(const fg::KernelEntry &k, fg::GemmParams &p, hipStream_t stream, int batches = 1) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return fail(FG_ERR_LAUNCH, "no HIP device is current");
    int per_cu = 0;
    if (fg_status st = prepare(k, dev, per_cu)) return st;
    // Persistent workgroups: as many as the GPU holds at once; each walks tiles b, b + grid, ...
    const int ntiles = p.tile_count > 0 ? p.tile_count * (p.splits > 1 ? p.splits : 1) : p.tiles_m * p.tiles_n * batches;
    const int resident = per_cu * kNumCU;
    dim3 grid((unsigned)(ntiles < resident ? ntiles : resident)), block((unsigned)k.threads);
    p.by_count = p.splits > 1 ? fg::division_by((uint32_t)p.tile_count) : fg::division_to_zero();
    p.by_group = fg::tile_group(p.tiles_m, p.tiles_n);
    void *args[] = {&p};
    hipError_t e = hipLaunchKernel(k.fn, grid, block, args, (size_t)k.lds_bytes, stream);
    if (e != hipSuccess) { (void)hipGetLastError(); return fail(FG_ERR_LAUNCH, "launch of %s failed: %s", k.name, hipGetErrorString(e)); }
    return FG_OK;
}

fg_status check_sizes(int64_t M, int64_t N, int64_t K) {
    if (M < 0 || N < 0 || K < 0) return fail(FG_ERR_SHAPE, "negative size M=%lld N=%lld K=%lld", (long long)M, (long long)N, (long long)K);
    if (K % 8) note_relaxed(FG_ERR_UNSUPPORTED, "K must be a multiple of 8 (got %lld)", (long long)K);
    if (M > (1 << 30) || N > (1 << 30) || K > (1 << 30)) return fail(FG_ERR_UNSUPPORTED, "sizes above 2^30 are not supported");
    return FG_OK;
}

fg_status check_input_matrix(const char *name, const fg_matrix *X, int64_t rows, int64_t cols) {
    if (!X) return fail(FG_ERR_NULL, "%s is NULL", name);
    if (X->dtype != FG_F16 && X->dtype != FG_BF16 && X->dtype != FG_CF16) return fail(FG_ERR_LAYOUT, "%s must be FG_F16, FG_BF16 or FG_CF16", name);
    if (X->dtype == FG_CF16 && (X->im || X->layout == FG_DIAG)) return fail(FG_ERR_LAYOUT, "%s: an interleaved complex matrix has no `im` plane and is not diagonal", name);
    if (X->layout != FG_COL && X->layout != FG_ROW && X->layout != FG_DIAG) return fail(FG_ERR_LAYOUT, "%s: layout %d is not valid for an input", name, X->layout);
    if (rows > 0 && cols > 0) {
        if (!X->re) return fail(FG_ERR_NULL, "%s->re is NULL", name);
        if (!aligned_to(X->re, 2) || (X->im && !aligned_to(X->im, 2))) return fail(FG_ERR_ALIGN, "%s: element pointers must be aligned to an element", name);
        if (!aligned16(X->re) || (X->im && !aligned16(X->im))) note_relaxed(FG_ERR_ALIGN, "%s: element pointers must be 16-byte aligned", name);
        if (X->layout != FG_DIAG) {
            int64_t need = X->layout == FG_COL ? rows : cols;
            if (X->ld < need) return fail(FG_ERR_SHAPE, "%s: ld=%lld is smaller than %lld", name, (long long)X->ld, (long long)need);
            if (X->ld % 8) note_relaxed(FG_ERR_ALIGN, "%s: ld=%lld must be a multiple of 8", name, (long long)X->ld);
        }
    }
    return FG_OK;
}

fg_status check_output_matrix(const char *name, const fg_matrix *X, int64_t rows, int64_t cols, bool need_im) {
    if (X->dtype != FG_F32 && X->dtype != FG_CF32 && X->dtype != FG_F16) return fail(FG_ERR_LAYOUT, "%s must be FG_F32, FG_F16 or FG_CF32", name);
    if (X->dtype == FG_F16) {
        // stored as binary16: the kernels access it element by element, so any ld and any
        // element-aligned pointer will do
        if (X->im) return fail(FG_ERR_UNSUPPORTED, "%s: binary16 storage is for real matrices", name);
        if (X->layout != FG_COL && X->layout != FG_ROW) return fail(FG_ERR_LAYOUT, "%s: layout %d is not valid here", name, X->layout);
        if (rows > 0 && cols > 0) {
            if (!X->re) return fail(FG_ERR_NULL, "%s->re is NULL", name);
            if (!aligned_to(X->re, 2)) return fail(FG_ERR_ALIGN, "%s: element pointers must be aligned to an element", name);
            const int64_t need = X->layout == FG_COL ? rows : cols;
            if (X->ld < need) return fail(FG_ERR_SHAPE, "%s: ld=%lld is smaller than %lld", name, (long long)X->ld, (long long)need);
        }
        return FG_OK;
    }
    if (X->dtype == FG_CF32) {
        if (X->im) return fail(FG_ERR_LAYOUT, "%s: an interleaved complex matrix has no `im` plane", name);
        need_im = false;
        if (X->ld >= (1ll << 22)) return fail(FG_ERR_UNSUPPORTED, "%s: ld of an interleaved complex matrix must be below 2^22", name);
    }
    if (X->layout != FG_COL && X->layout != FG_ROW) return fail(FG_ERR_LAYOUT, "%s: layout %d is not valid here", name, X->layout);
    if (rows > 0 && cols > 0) {
        if (!X->re) return fail(FG_ERR_NULL, "%s->re is NULL", name);
        if (need_im && !X->im) return fail(FG_ERR_NULL, "%s->im is NULL but the product is complex", name);
        if (!aligned_to(X->re, 4) || (X->im && !aligned_to(X->im, 4))) return fail(FG_ERR_ALIGN, "%s: element pointers must be aligned to an element", name);
        if (!aligned16(X->re) || (X->im && !aligned16(X->im))) note_relaxed(FG_ERR_ALIGN, "%s: element pointers must be 16-byte aligned", name);
        int64_t need = X->layout == FG_COL ? rows : cols;
        if (X->ld < need) return fail(FG_ERR_SHAPE, "%s: ld=%lld is smaller than %lld", name, (long long)X->ld, (long long)need);
        if (X->ld % 4) note_relaxed(FG_ERR_ALIGN, "%s: ld=%lld must be a multiple of 4", name, (long long)X->ld);
    }
    return FG_OK;
}

// Validate an fg_gemm call and normalise it so that D is column-major: a row-major D is the
// column-major D^T = op(B)^T op(A)^T, i.e. the same kernel with the operands exchanged.
fg_status normalise(int64_t M, int64_t N, int64_t K, float alpha, const fg_matrix *A, const fg_matrix *B,
                    float beta, const fg_matrix *C, const fg_matrix *D, const fg_epilogue *ep, bool dual,
                    const fg_load_transforms *lt, Problem &q) {
    g_relaxed.status = FG_OK;
    if (fg_status st = check_sizes(M, N, K)) return st;
    if (fg_status st = check_input_matrix("A", A, M, K)) return st;
    if (fg_status st = check_input_matrix("B", B, K, N)) return st;
    if (!D) return fail(FG_ERR_NULL, "D is NULL");
    if (A->dtype != B->dtype) return fail(FG_ERR_UNSUPPORTED, "A and B must have the same element type");
    const bool bf16 = A->dtype == FG_BF16;
    const bool ilv = A->dtype == FG_CF16;
    if (ilv && (D->dtype != FG_CF32 || (C && C->layout != FG_ZERO && C->re && C->dtype != FG_CF32)))
        return fail(FG_ERR_UNSUPPORTED, "interleaved complex A and B need interleaved complex (FG_CF32) C and D");
    if (!ilv && (D->dtype == FG_CF32 || (C && C->dtype == FG_CF32 && C->layout != FG_ZERO && C->re)))
        return fail(FG_ERR_UNSUPPORTED, "FG_CF32 C and D need FG_CF16 A and B");
    if (ilv && (dual || lt)) return fail(FG_ERR_UNSUPPORTED, "interleaved complex products take no transforms and are not dual");
    const bool cplx = ilv || (A->im != nullptr) || (B->im != nullptr);
    if (dual && !cplx) return fail(FG_ERR_NULL, "a dual-number product needs the dual planes (im) of A and B");
    if (bf16 && (cplx || A->layout == FG_DIAG || B->layout == FG_DIAG))
        return fail(FG_ERR_UNSUPPORTED, "FG_BF16 operands are supported for real, non-diagonal matrices only");
    if (fg_status st = check_output_matrix("D", D, M, N, cplx)) return st;
    const bool cd16 = D->dtype == FG_F16;
    if (cd16 && (cplx || bf16 || A->layout == FG_DIAG || B->layout == FG_DIAG))
        return fail(FG_ERR_UNSUPPORTED, "FG_F16 C and D are supported for real FG_F16 products in FG_COL or FG_ROW layout");
    const bool has_c = C && C->layout != FG_ZERO && C->re != nullptr;
    if (C && C->layout != FG_ZERO && !C->re && M > 0 && N > 0) return fail(FG_ERR_NULL, "C->re is NULL (pass C == NULL or FG_ZERO for no C term)");
    if (has_c) {
        if (fg_status st = check_output_matrix("C", C, M, N, cplx)) return st;
        if (C->layout != D->layout) return fail(FG_ERR_LAYOUT, "C and D must have the same layout");
        if ((C->dtype == FG_F16) != cd16) return fail(FG_ERR_UNSUPPORTED, "C and D must have the same element type");
    }
    if (A->layout == FG_DIAG && B->layout == FG_DIAG) return fail(FG_ERR_UNSUPPORTED, "at most one of A and B may be diagonal");
    const bool has_ep = ep && (ep->bias || ep->act != FG_ACT_NONE);
    if (ep) {
        if (ep->act != FG_ACT_NONE && ep->act != FG_ACT_RELU) return fail(FG_ERR_LAYOUT, "unknown activation %d", ep->act);
        if (ep->bias && ep->bias_dim != 0 && ep->bias_dim != 1) return fail(FG_ERR_LAYOUT, "bias_dim must be 0 or 1");
        if (ep->bias && !aligned_to(ep->bias, 4)) return fail(FG_ERR_ALIGN, "bias must be aligned to an element");
    }
    if (cplx && has_ep) return fail(FG_ERR_UNSUPPORTED, "bias and activation are not defined for complex or dual products");
    if (cplx && !ilv && (!A->im || !B->im)) return fail(FG_ERR_UNSUPPORTED, "complex and dual products need the second plane of both A and B");
    if (cplx && (A->layout == FG_DIAG || B->layout == FG_DIAG)) return fail(FG_ERR_UNSUPPORTED, "complex or dual diagonal operands are not supported");

    // transforms on loaded elements
    uint16_t a_add = 0, b_add = 0;
    int c_act = FG_ACT_NONE;
    if (lt) {
        if (lt->c_act != FG_ACT_NONE && lt->c_act != FG_ACT_RELU) return fail(FG_ERR_LAYOUT, "unknown activation %d on C", lt->c_act);
        if (!(lt->a_add == lt->a_add) || !(lt->b_add == lt->b_add)) return fail(FG_ERR_SHAPE, "a_add or b_add is NaN");
        const _Float16 ha = (_Float16)lt->a_add, hb = (_Float16)lt->b_add;     // round to nearest even
        memcpy(&a_add, &ha, 2); memcpy(&b_add, &hb, 2);
        if ((a_add & 0x7fff) == 0) a_add = 0;                                   // -0 adds nothing either
        if ((b_add & 0x7fff) == 0) b_add = 0;
        c_act = lt->c_act;
    }
    const bool ab_add = a_add != 0 || b_add != 0;
    if (ab_add && (cplx || bf16 || cd16 || A->layout == FG_DIAG || B->layout == FG_DIAG))
        return fail(FG_ERR_UNSUPPORTED, "an addition on A and B needs real FG_F16 operands in FG_COL or FG_ROW layout and FP32 C and D");
    if (c_act != FG_ACT_NONE && cplx) return fail(FG_ERR_UNSUPPORTED, "an activation on C is not defined for complex or dual products");

    const bool swap = (D->layout == FG_ROW);
    q.cplx = cplx;
    q.cd16 = cd16;
    q.ilv = ilv;
    q.c_act = c_act;
    q.ab_add = ab_add;
    q.a_add = swap ? b_add : a_add;
    q.b_add = swap ? a_add : b_add;
    q.dual = dual;
    q.bf16 = bf16;
    q.alpha = alpha;
    // beta == 0: C is validated but never read (the BLAS convention), so that D may alias an
    // uninitialised C without its NaNs or infinities reaching the result as 0 * x
    const bool use_c = has_c && beta != 0.f;
    q.beta = use_c ? beta : 0.f;
    q.C = use_c ? (const float *)C->re : nullptr;
    q.C_im = use_c ? (const float *)C->im : nullptr;
    q.ldc = use_c ? C->ld : 0;
    q.D = (float *)D->re;
    q.D_im = (float *)D->im;
    q.ldd = D->ld;
    q.bias = (ep && ep->bias) ? ep->bias : nullptr;
    q.bias_dim = ep ? ep->bias_dim : 0;
    q.act = ep ? ep->act : FG_ACT_NONE;
    if (!swap) {
        q.M = M; q.N = N; q.K = K;
        q.A = A->re; q.A_im = A->im; q.lda = A->ld; q.a_diag = A->layout == FG_DIAG; q.a_kc = (A->layout == FG_ROW);
        q.B = B->re; q.B_im = B->im; q.ldb = B->ld; q.b_diag = B->layout == FG_DIAG; q.b_kc = (B->layout == FG_COL);
    } else {
        // D^T (N x M, column-major) = B^T (N x K) . A^T (K x M)
        q.M = N; q.N = M; q.K = K;
        q.A = B->re; q.A_im = B->im; q.lda = B->ld; q.a_diag = B->layout == FG_DIAG; q.a_kc = (B->layout == FG_COL);
        q.B = A->re; q.B_im = A->im; q.ldb = A->ld; q.b_diag = A->layout == FG_DIAG; q.b_kc = (A->layout == FG_ROW);
        q.bias_dim = 1 - q.bias_dim;
    }
    if (q.a_diag) q.a_kc = true;     // a diagonal operand is synthesised K-contiguous in LDS
    if (q.b_diag) q.b_kc = true;
    q.general = false;
    if (g_relaxed.status != FG_OK) {
        if (cplx || q.a_diag || q.b_diag) return fail(g_relaxed.status, "%s (complex, dual and diagonal products have no general kernel)", g_relaxed.msg);
        if (cd16) return fail(g_relaxed.status, "%s (products with FG_F16 C and D have no general kernel)", g_relaxed.msg);
        q.general = true;
    }
    return FG_OK;
}


// ---- general kernel (general_kernel.hpp) --------------------------------------------------------------

// Block tile and K ranges of a product on the general kernel: the smallest estimated time.  Measured
// with one workgroup per compute unit and little less per workgroup with two: a K step of 64
// takes 0.9 us with the 128x128 tile, two steps (one per wave group) 0.7 us with the 64x64 tile, a
// workgroup's start and stores 1 us (64x64) or 2; a split adds a launch and the reduction pass (5 us and its
// traffic).  Against every tile and split forced over 13 shapes from 195x65x2500 to 4095x4097x4099 the
// choice is the fastest or within 8 %: 1531x1021x2003 28.0 us (128x128: 35.7), 4095x4097x4099 244 us
// (64x64: 367), 301x301x6001 split in ten 18 us (one pass: 37).
// The partial products of a split are kept to 16 MiB of the workspace.
//
// K up to 64 is one step.  The 64x64 tile's second wave group would have nothing to multiply, yet take half of
// the LDS, an exchange and its waves' slots, so that few tiles run side by side: contractions (many
// small batches above all) and matrices of more than two tiles per unit have a form with one group and one
// buffer.  Two groups -> one: 65536 batches of 4x4x4 780 -> 337 us (378 with the element-wise kernel of before), 8192 of
// 16x16x9 97 -> 45 (59), matrices 3001x2999x3 25 -> 16 (26).  With fewer tiles the second group's threads help to
// load and store: 301x299x50 5.4 us with two, 6.4 with one.  Where the 128x128 tile begins was read from both
// forced on 58 calls (4x4x4 to 5001x4999x3, where it takes 38.5 us): contractions pay more per small tile.
struct GeneralPlan { int variant, bm, bn, splits; };
GeneralPlan choose_general(int64_t M, int64_t N, int64_t K, int64_t batches, bool matrix) {
    static const int edge[] = {128, 64}, groups[] = {1, 2};           // GENERAL_128x128, GENERAL_64x64
    static const double round_us[] = {0.9, 0.7}, fixed_us[] = {2, 1};
    static const int split_options[] = {1, 2, 3, 4, 6, 8, 10, 12, 16, 24, 32, 48, 64};
    const int64_t nk = (K + 63) / 64;
    const int ft = g_force_tile.load(std::memory_order_relaxed), fs = g_force_split.load(std::memory_order_relaxed);
    if (nk <= 1) {
        const int64_t small = ((M + 63) / 64) * ((N + 63) / 64) * batches, large = ((M + 127) / 128) * ((N + 127) / 128) * batches;
        const double small_us = 5 + (matrix ? 1.47 : 2.0) * (small > kNumCU ? (double)small / kNumCU : 1.0);
        const double large_us = 6.5 + 4.6 * (double)((large + kNumCU - 1) / kNumCU);
        if (ft == fg::TILE_128x128 || (ft != fg::TILE_64x64 && large_us < small_us)) return GeneralPlan{fg::GENERAL_128x128, 128, 128, 1};
        return GeneralPlan{matrix && small <= 2 * kNumCU ? fg::GENERAL_64x64 : fg::GENERAL_64x64_ONE, 64, 64, 1};
    }
    GeneralPlan best{fg::GENERAL_64x64, 64, 64, 1};
    double best_cost = -1;
    for (int v = fg::GENERAL_128x128; v <= fg::GENERAL_64x64; ++v) {
        if (ft == fg::TILE_128x128 && v != fg::GENERAL_128x128) continue;
        if (ft == fg::TILE_64x64 && v != fg::GENERAL_64x64) continue;
        const int64_t tiles = ((M + edge[v] - 1) / edge[v]) * ((N + edge[v] - 1) / edge[v]) * batches;
        const double tile_bytes = 4.0 * edge[v] * edge[v];
        for (int S : split_options) {
            if (fs >= 1) { if (S != 1) break; S = fs; }
            if (S > 1 && (!matrix || S > nk || (fs < 1 && nk / S < 4) || (double)tiles * S * tile_bytes > kStaticScratchBytes)) {
                if (fs < 1) break;
                S = 1;
            }
            const int64_t steps = (nk + S - 1) / S, load = (tiles * S + kNumCU - 1) / kNumCU;
            double cost = (double)load * ((double)((steps + groups[v] - 1) / groups[v]) * round_us[v] + fixed_us[v]);
            if (S > 1) cost += 5 + (2.0 * S + 2) * (double)tiles * tile_bytes / 3e6;
            if (best_cost < 0 || cost < best_cost) { best = GeneralPlan{v, edge[v], edge[v], S}; best_cost = cost; }
        }
    }
    return best;
}

fg_status general_gemm(const Problem &q, bool static_only, hipStream_t stream) {
    fg::GeneralParams f;
    memset(&f, 0, sizeof f);
    GeneralPlan plan = choose_general(q.M, q.N, q.K, 1, true);
    f.M = (int32_t)q.M; f.N = (int32_t)q.N; f.K = (int32_t)q.K;
    f.A = (const uint16_t *)q.A; f.B = (const uint16_t *)q.B;
    f.a_rs = q.a_kc ? q.lda : 1; f.a_ks = q.a_kc ? 1 : q.lda;
    f.b_rs = q.b_kc ? q.ldb : 1; f.b_ks = q.b_kc ? 1 : q.ldb;
    f.a_span = (q.M - 1) * f.a_rs + (q.K - 1) * f.a_ks + 1; f.b_span = (q.N - 1) * f.b_rs + (q.K - 1) * f.b_ks + 1;
    f.C = q.C; f.D = q.D; f.ldc = q.ldc; f.ldd = q.ldd;
    f.bias = q.bias; f.bias_dim = q.bias_dim; f.act = q.act; f.c_act = q.c_act;
    f.alpha = q.alpha; f.beta = q.beta;
    f.a_add2 = (uint32_t)q.a_add * 0x10001u; f.b_add2 = (uint32_t)q.b_add * 0x10001u; f.ab_add = q.ab_add;
    f.batches = 1; f.splits = 1;
    const int64_t tiles_m = (q.M + plan.bm - 1) / plan.bm, tiles_n = (q.N + plan.bn - 1) / plan.bn;
    if (tiles_m * tiles_n >= (1ll << 31)) return fail(FG_ERR_UNSUPPORTED, "too many tiles");
    f.tiles_m = (int32_t)tiles_m; f.tiles_n = (int32_t)tiles_n;
    const int tiles = (int)(tiles_m * tiles_n);
    // The K ranges of a split go side by side through the workspace, or one after another in a single
    // launch without scratch memory: same bits.  The second way serves every call that may overlap with
    // others on the GPU without being ordered against them -- on a stream under capture and through the
    // allocation-free entry point -- because products of this kind never shared memory before they were
    // split, and calls that cannot have the workspace.  It is slower (301x301x6001: 58 us against 13,
    // 1450 with the element-wise kernel that served these calls before).
    Scratch scratch;
    bool side_by_side = false;
    if (plan.splits > 1) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) return fail(FG_ERR_LAUNCH, "no HIP device is current");
        side_by_side = !static_only && scratch.try_acquire(dev, stream);
        f.splits = plan.splits;
        f.split_kt = (int32_t)(((q.K + 63) / 64 + plan.splits - 1) / plan.splits);
    }
    if (side_by_side) {
        fg::GeneralParams part = f;
        part.D = scratch.ptr;
        hipError_t e = fg::launch_gemm_general(part, q.a_kc, q.b_kc, q.bf16, plan.variant, false, stream);
        if (e == hipSuccess)
            e = fg::launch_splitk_reduce(scratch.ptr, plan.splits, 0, tiles, plan.bm, plan.bn, f.tiles_m, f.tiles_n, f.M, f.N, q.alpha, q.beta,
                                         q.C, q.ldc, q.D, q.ldd, q.bias, q.bias_dim, q.act, q.c_act, stream);
        if (e != hipSuccess) return fail(FG_ERR_LAUNCH, "launch of the general kernel failed: %s", hipGetErrorString(e));
        return scratch.release(stream);
    }
    hipError_t e = fg::launch_gemm_general(f, q.a_kc, q.b_kc, q.bf16, plan.variant, plan.splits > 1, stream);
    if (e != hipSuccess) return fail(FG_ERR_LAUNCH, "launch of the general kernel failed: %s", hipGetErrorString(e));
    return FG_OK;
}

// ---- tensor contraction -> GEMM description (Section 5.5) -----------------------------------------
// Modes shared by A and C become GEMM rows (M), modes shared by B and C columns (N), modes
// shared by A and B the summed index (K).  Inside a merged index the first mode is the fastest
// (the (ba) -> m convention of the paper's layout listing).  No data moves: the kernel computes
// element offsets from these groups while it loads tiles and stores results.
struct Contraction {
    bool general;            // a requirement of the tiled kernels is missed: use the general kernel
    char why_general[160];
    int64_t M, N, K, batches;
    fg::ModeGroup a_b, b_b, c_b;
    const void *A, *B;
    bool a_kc, b_kc;
    fg::ModeGroup a_m, a_k, b_n, b_k, c_m, c_n;
    // general kernel only: true extents of the leading modes, element strides inside a piece, elements
    // each operand spans
    int32_t m_ext0, n_ext0, k_ext0, m_hi;
    int64_t a_es, b_es, a_span, b_span, a_kmax, b_kmax;
};

struct TensorView { int32_t n; const int32_t *modes; const int64_t *strides; };

int find_mode(const TensorView &t, int32_t label) {
    for (int i = 0; i < t.n; ++i) if (t.modes[i] == label) return i;
    return -1;
}

fg_status plan_contraction(int32_t nA, const int32_t *modesA, const int64_t *stridesA, const void *A,
                           int32_t nB, const int32_t *modesB, const int64_t *stridesB, const void *B,
                           int32_t nC, const int32_t *modesC, const int64_t *stridesC, const float *Cin, float *Cout,
                           int32_t n_modes, const int32_t *labels, const int64_t *extents, Contraction &c) {
    (void)Cin;
    if (nA < 0 || nB < 0 || nC < 0 || n_modes < 0) return fail(FG_ERR_SHAPE, "negative mode count");
    if ((nA && (!modesA || !stridesA)) || (nB && (!modesB || !stridesB)) || (nC && (!modesC || !stridesC)) || (n_modes && (!labels || !extents)))
        return fail(FG_ERR_NULL, "a mode, stride, label or extent array is NULL");
    if (nA > 12 || nB > 12 || nC > 12 || n_modes > 24) return fail(FG_ERR_UNSUPPORTED, "too many modes");
    TensorView ta{nA, modesA, stridesA}, tb{nB, modesB, stridesB}, tc{nC, modesC, stridesC};
    auto extent_of = [&](int32_t label, int64_t &e) {
        for (int i = 0; i < n_modes; ++i) if (labels[i] == label) { e = extents[i]; return true; }
        return false;
    };
    for (int i = 0; i < n_modes; ++i) {
        if (extents[i] < 0) return fail(FG_ERR_SHAPE, "mode %d has a negative extent", labels[i]);
        for (int j = i + 1; j < n_modes; ++j) if (labels[i] == labels[j]) return fail(FG_ERR_MODES, "mode label %d is listed twice", labels[i]);
    }
    const TensorView *views[3] = {&ta, &tb, &tc};
    const char *names = "ABC";
    for (int v = 0; v < 3; ++v)
        for (int i = 0; i < views[v]->n; ++i) {
            int64_t e;
            if (!extent_of(views[v]->modes[i], e)) return fail(FG_ERR_MODES, "%c uses mode %d, which has no extent", names[v], views[v]->modes[i]);
            for (int j = i + 1; j < views[v]->n; ++j)
                if (views[v]->modes[i] == views[v]->modes[j]) return fail(FG_ERR_MODES, "%c lists mode %d twice (trace modes are not supported)", names[v], views[v]->modes[i]);
        }
    // every used label must sit in exactly two tensors
    bool any_zero = false;
    for (int i = 0; i < n_modes; ++i) {
        int cnt = (find_mode(ta, labels[i]) >= 0) + (find_mode(tb, labels[i]) >= 0) + (find_mode(tc, labels[i]) >= 0);
        if (cnt == 0) continue;
        if (cnt == 1) return fail(FG_ERR_MODES, "mode %d appears in only one of A, B, C (no reduction or broadcast modes)", labels[i]);
        if (extents[i] == 0) any_zero = true;
    }
    c.M = c.N = 0; c.K = 0; c.batches = 1;
    c.general = false; c.why_general[0] = 0;
    if (any_zero) return FG_OK;               // an empty tensor: nothing to compute
    if (!A || !B || !Cout) return fail(FG_ERR_NULL, "A, B or Cout is NULL");
    if (!aligned_to(A, 2) || !aligned_to(B, 2) || !aligned_to(Cout, 4) || (Cin && !aligned_to(Cin, 4)))
        return fail(FG_ERR_ALIGN, "tensor base pointers must be aligned to an element");
    // A description that misses a requirement of the tiled kernels is computed by the general
    // kernel; the first reason is kept for fg_contract_plan.
    auto need_general = [&](const char *fmt, int x = 0, int y = 0) {
        if (!c.general) { c.general = true; snprintf(c.why_general, sizeof c.why_general, fmt, x, y); }
    };
    if (!aligned16(A) || !aligned16(B) || !aligned16(Cout) || (Cin && !aligned16(Cin))) need_general("a tensor base pointer is not 16-byte aligned");

    // Lanes of the result run along GEMM rows, so C's unit-stride mode should be a row mode:
    // exchange the roles of A and B when it belongs to B only.
    int c_unit = -1;
    for (int i = 0; i < nC; ++i) { int64_t e; extent_of(modesC[i], e); if (stridesC[i] == 1 && e > 1) { c_unit = modesC[i]; break; } }
    if (c_unit >= 0 && find_mode(tb, c_unit) >= 0 && find_mode(ta, c_unit) < 0) { TensorView t = ta; ta = tb; tb = t; const void *q = A; A = B; B = q; }
    c.A = A; c.B = B;
    auto in_a = [&](int32_t l) { return find_mode(ta, l) >= 0; };
    auto in_b = [&](int32_t l) { return find_mode(tb, l) >= 0; };
    auto in_c = [&](int32_t l) { return find_mode(tc, l) >= 0; };
    auto is_row = [&](int32_t l) { return in_a(l) && in_c(l) && !in_b(l); };
    auto is_col = [&](int32_t l) { return in_b(l) && in_c(l) && !in_a(l); };
    auto is_sum = [&](int32_t l) { return in_a(l) && in_b(l) && !in_c(l); };
    auto is_batch = [&](int32_t l) { return in_a(l) && in_b(l) && in_c(l); };

    auto unit_mode = [&](const TensorView &t) {
        int best = -1;
        for (int i = 0; i < t.n; ++i) {
            int64_t e; extent_of(t.modes[i], e);
            if (t.strides[i] == 1 && e % 8 == 0 && e > 0 && !is_batch(t.modes[i])) { best = t.modes[i]; break; }
        }
        return best;
    };
    int ua = unit_mode(ta), ub = unit_mode(tb);
    if (ua < 0 || ub < 0) need_general("A or B has no row, column or summed mode with stride 1 and an extent that is a multiple of 8");
    c.a_kc = ua >= 0 && is_sum(ua);           // A's contiguous mode is summed over
    c.b_kc = ub >= 0 && is_sum(ub);
    if (c.a_kc && c.b_kc && ua != ub) need_general("A and B are contiguous along different summed modes (%d and %d)", ua, ub);

    // order of the modes inside each merged index
    int32_t m_modes[16], n_modes_[16], k_modes[16], b_modes[16];
    int nm = 0, nn = 0, nkk = 0, nb = 0;
    auto push_unique = [](int32_t *arr, int &n, int32_t label) { for (int i = 0; i < n; ++i) if (arr[i] == label) return; arr[n++] = label; };
    if (!c.a_kc && ua >= 0) push_unique(m_modes, nm, ua);
    else if (c_unit >= 0 && is_row(c_unit)) push_unique(m_modes, nm, c_unit);
    for (int i = 0; i < tc.n; ++i) if (is_row(tc.modes[i])) push_unique(m_modes, nm, tc.modes[i]);
    if (!c.b_kc && ub >= 0) push_unique(n_modes_, nn, ub);
    for (int i = 0; i < tc.n; ++i) if (is_col(tc.modes[i])) push_unique(n_modes_, nn, tc.modes[i]);
    if (c.a_kc) push_unique(k_modes, nkk, ua);
    else if (c.b_kc) push_unique(k_modes, nkk, ub);
    for (int i = 0; i < ta.n; ++i) if (is_sum(ta.modes[i])) push_unique(k_modes, nkk, ta.modes[i]);
    for (int i = 0; i < tc.n; ++i) if (is_batch(tc.modes[i])) push_unique(b_modes, nb, tc.modes[i]);
    if (nm > fg::kMaxGroupModes || nn > fg::kMaxGroupModes || nkk > fg::kMaxGroupModes || nb > fg::kMaxGroupModes)
        return fail(FG_ERR_UNSUPPORTED, "at most %d modes per merged index", fg::kMaxGroupModes);
    if (nkk == 0) need_general("no summed mode (an outer product)");

    // Modes of extent 1 carry no index and are dropped.  For the others the kernel divides by the
    // extent with a multiply-high: with 2^s < e <= 2^(s+1) and magic = floor(2^(32+s)/e) + 1,
    // floor(idx / e) == (idx * magic) >> (32 + s) for every 0 <= idx < 2^31.
    auto set_mode = [](fg::ModeGroup &g, int k, int64_t e, int64_t stride) {
        uint32_t sh = 0;
        while ((2ull << sh) < (uint64_t)e) ++sh;              // 2^sh < e <= 2^(sh+1)
        g.extent[k] = (int32_t)e;
        g.stride[k] = stride;
        g.shift[k] = sh;
        g.magic[k] = (uint32_t)(((1ull << (32 + sh)) / (uint64_t)e) + 1);
    };
    auto fill = [&](fg::ModeGroup &g, const int32_t *modes, int n, const TensorView &t, int64_t &total, bool round_first = false) {
        g.n = 0; total = 1;
        for (int i = 0; i < n; ++i) {
            int64_t e; extent_of(modes[i], e);
            if (i == 0 && round_first && e > 1) e = (e + 7) / 8 * 8;
            total *= e;
            if (e == 1) continue;
            set_mode(g, g.n++, e, t.strides[find_mode(t, modes[i])]);
        }
        for (int i = g.n; i < fg::kMaxGroupModes; ++i) { g.extent[i] = 2; g.stride[i] = 0; g.magic[i] = 0; g.shift[i] = 0; }
    };
    int64_t t1, t2;
    fill(c.a_m, m_modes, nm, ta, c.M); fill(c.c_m, m_modes, nm, tc, t1);
    fill(c.b_n, n_modes_, nn, tb, c.N); fill(c.c_n, n_modes_, nn, tc, t2);
    fill(c.a_k, k_modes, nkk, ta, c.K); fill(c.b_k, k_modes, nkk, tb, t1);
    fill(c.a_b, b_modes, nb, ta, c.batches); fill(c.b_b, b_modes, nb, tb, t1); fill(c.c_b, b_modes, nb, tc, t2);
    if (nb == 0) c.batches = 1;
    if (nm == 0) c.M = 1;
    if (nn == 0) c.N = 1;

    for (int i = 0; i < ta.n; ++i) if (ta.strides[i] < 0) return fail(FG_ERR_UNSUPPORTED, "negative strides are not supported");
    for (int i = 0; i < tb.n; ++i) if (tb.strides[i] < 0) return fail(FG_ERR_UNSUPPORTED, "negative strides are not supported");
    for (int i = 0; i < tc.n; ++i) if (tc.strides[i] < 0) return fail(FG_ERR_UNSUPPORTED, "negative strides are not supported");
    auto span = [&](const TensorView &t) {
        int64_t sp = 1;
        for (int i = 0; i < t.n; ++i) { int64_t e; extent_of(t.modes[i], e); sp += (e - 1) * t.strides[i]; }
        return sp;
    };
    if (!c.general) {
        if ((c.a_kc || c.b_kc) && c.a_k.n > 0 && c.a_k.extent[0] % 8) need_general("the leading summed mode (%d) is contiguous in A or B and its extent is not a multiple of 8", k_modes[0]);
        if (c.a_kc && c.a_k.n > 0 && c.a_k.stride[0] != 1) need_general("the leading summed mode is not contiguous in A");
        if (c.b_kc && c.b_k.n > 0 && c.b_k.stride[0] != 1) need_general("the leading summed mode (%d) is contiguous in A but not in B", k_modes[0]);
        if ((c.a_kc || c.b_kc) && c.a_k.n == 0) need_general("the contiguous summed mode has extent 1");
        if (!c.a_kc && (c.a_m.n == 0 || c.a_m.stride[0] != 1 || c.a_m.extent[0] % 8)) need_general("A's contiguous row mode must have an extent that is a multiple of 8");
        if (!c.b_kc && (c.b_n.n == 0 || c.b_n.stride[0] != 1 || c.b_n.extent[0] % 8)) need_general("B's contiguous column mode must have an extent that is a multiple of 8");
        // The tiled kernels fetch 16-byte pieces along the contiguous mode: every other stride of A
        // and B must keep those pieces 16-byte aligned.
        auto strides_ok = [](const fg::ModeGroup &g, int first) {
            for (int t = first; t < g.n; ++t) if (g.stride[t] % 8) return false;
            return true;
        };
        if (!strides_ok(c.a_m, c.a_kc ? 0 : 1) || !strides_ok(c.a_k, c.a_kc ? 1 : 0) || !strides_ok(c.a_b, 0))
            need_general("a stride of A other than its contiguous mode's is not a multiple of 8 elements");
        if (!strides_ok(c.b_n, c.b_kc ? 0 : 1) || !strides_ok(c.b_k, c.b_kc ? 1 : 0) || !strides_ok(c.b_b, 0))
            need_general("a stride of B other than its contiguous mode's is not a multiple of 8 elements");
        // the tiled kernels address A, B and C with 32-bit byte offsets inside a 2 GiB window
        if (span(ta) * 2 >= (1ll << 31) || span(tb) * 2 >= (1ll << 31) || span(tc) * 4 >= (1ll << 31)) need_general("A, B or C spans 2 GiB or more");
    }
    if (!c.general) {
        if (c.a_k.n == 0) {
            // every summed mode has extent 1: one K step whose k = 0 alone is loaded
            c.a_k.n = c.b_k.n = 1;
            c.a_k.extent[0] = c.b_k.extent[0] = 1;
            c.a_k.stride[0] = c.b_k.stride[0] = 0;
        }
        // K steps of 64 walk the leading summed mode; when its extent is not a multiple of 64 the
        // last step of each pass is zero-filled, so the tiled kernels see that extent rounded up
        c.K = c.K / c.a_k.extent[0] * ((c.a_k.extent[0] + 63) / 64 * 64);
    }
    if (c.M > (1 << 30) || c.N > (1 << 30) || c.K > (1 << 30) || c.batches > (1 << 20)) return fail(FG_ERR_UNSUPPORTED, "merged extents above 2^30 (2^20 for batch modes) are not supported");
    if (c.general) {
        // Groups for the general kernel, whose threads fetch pieces of eight elements along one mode
        // of each operand: the mode with stride 1, as one load per piece.  A unit-stride mode
        // shorter than 5 would fill its pieces badly, and pieces along the summed modes can follow one mode
        // only; such an operand is fetched element by element along its longest row or column mode.
        auto extent = [&](int32_t label) { int64_t e = 1; extent_of(label, e); return e; };
        auto unit_any = [&](const TensorView &t) {
            for (int i = 0; i < t.n; ++i)
                if (t.strides[i] == 1 && extent(t.modes[i]) >= 5 && !is_batch(t.modes[i])) return (int)t.modes[i];
            return -1;
        };
        auto longest = [&](const int32_t *modes, int n) {
            int best = -1;
            for (int i = 0; i < n; ++i) if (best < 0 || extent(modes[i]) > extent(best)) best = modes[i];
            return best;
        };
        auto to_front = [](int32_t *modes, int n, int32_t label) {
            for (int i = 0; i < n; ++i)
                if (modes[i] == label) { for (; i > 0; --i) modes[i] = modes[i - 1]; modes[0] = label; return; }
        };
        int la = unit_any(ta), lb = unit_any(tb);
        bool have_a = la >= 0, have_b = lb >= 0;
        c.a_kc = have_a && is_sum(la); c.b_kc = have_b && is_sum(lb);
        if (c.a_kc && c.b_kc && la != lb) {
            if (span(ta) >= span(tb)) { c.b_kc = false; have_b = false; }
            else { c.a_kc = false; have_a = false; }
        }
        if (!have_a) la = longest(m_modes, nm);
        if (!have_b) lb = longest(n_modes_, nn);
        if (c_unit >= 0) to_front(m_modes, nm, c_unit);
        if (!c.a_kc) to_front(m_modes, nm, la);
        if (!c.b_kc) to_front(n_modes_, nn, lb);
        if (c.a_kc) to_front(k_modes, nkk, la);
        else if (c.b_kc) to_front(k_modes, nkk, lb);
        const bool k_pad = c.a_kc || c.b_kc;
        int64_t padded;
        fill(c.a_m, m_modes, nm, ta, c.M, !c.a_kc); fill(c.c_m, m_modes, nm, tc, padded, !c.a_kc);
        fill(c.b_n, n_modes_, nn, tb, c.N, !c.b_kc); fill(c.c_n, n_modes_, nn, tc, padded, !c.b_kc);
        fill(c.a_k, k_modes, nkk, ta, c.K, k_pad); fill(c.b_k, k_modes, nkk, tb, padded, k_pad);
        // true extent of a group's leading mode, and its stride in the operand; a group without modes has one index
        auto lead = [&](fg::ModeGroup &g, fg::ModeGroup &other, bool rounded, int label, int64_t &total, int32_t &ext0) {
            if (g.n == 0 && rounded) {           // one row (or column): a piece with one element
                g.n = other.n = 1;
                set_mode(g, 0, 8, 0);
                set_mode(other, 0, 8, 0);
                total = 8; ext0 = 1;
            } else {
                ext0 = rounded ? (int32_t)extent(label) : g.extent[0];
            }
        };
        lead(c.a_m, c.c_m, !c.a_kc, la, c.M, c.m_ext0);
        lead(c.b_n, c.c_n, !c.b_kc, lb, c.N, c.n_ext0);
        lead(c.a_k, c.b_k, k_pad, c.a_kc ? la : lb, c.K, c.k_ext0);
        // The result contiguous along another row mode than A: rows in A's order would put the 64 lanes
        // of a store (and of a read of Cin) on 64 different lines.  The leading mode is split into
        // its pieces of eight and the rest, which goes last, so that a tile holds eight rows of it for each of
        // several values of the result's contiguous mode and a store touches a quarter of the lines.
        // A is then read in separate pieces, which pays while K is not long against N: D_abc = A_bda B_dc
        // with (a, b, c, d) = (111, 99, 301, 65) 30.0 -> 23.2 us (49.1 -> 26.4 with Cin, which doubles the
        // scattered accesses), (63, 31, 511, 373) 16.2 -> 16.2 (20.3 -> 17.4), (211, 55, 65, 201) 15.6 -> 17.9
        // (23.5 -> 19.4), (99, 201, 33, 501) 17.8 -> 28.2 (21.0 -> 29.2).  Drawn from these four: elsewhere the line may
        // lie differently.  (A Cin that beta == 0 leaves unread counts as one; at (99, 201, 100, 301) that is the better
        // side, 20.6 against 23.6 us.)
        c.m_hi = 0;
        if (have_a && c.K <= (Cin ? 4 * c.N : c.N * 3 / 2) && !c.a_kc && c_unit >= 0 && c_unit != la && is_row(c_unit) && extent(c_unit) >= 4 && c.a_m.n >= 2 && c.a_m.n < fg::kMaxGroupModes && c.a_m.extent[0] > 8) {
            const int hi = c.a_m.n;
            for (fg::ModeGroup *g : {&c.a_m, &c.c_m}) {
                set_mode(*g, hi, g->extent[0] / 8, 8 * g->stride[0]);
                set_mode(*g, 0, 8, g->stride[0]);
                g->n = hi + 1;
            }
            c.m_hi = hi;
        }
        auto stride_of = [&](const TensorView &t, int label, bool pseudo) { const int i = pseudo ? -1 : find_mode(t, label); return i < 0 ? (int64_t)1 : t.strides[i]; };
        c.a_es = stride_of(ta, la, nm == 0 && !c.a_kc); c.b_es = stride_of(tb, lb, nn == 0 && !c.b_kc);
        c.a_span = span(ta); c.b_span = span(tb);
        c.a_kmax = c.b_kmax = 0;
        for (int i = 0; i < nkk; ++i) {
            c.a_kmax += (extent(k_modes[i]) - 1) * ta.strides[find_mode(ta, k_modes[i])];
            c.b_kmax += (extent(k_modes[i]) - 1) * tb.strides[find_mode(tb, k_modes[i])];
        }
    }
    return FG_OK;
}

}  // namespace

extern "C" {

const char *fg_last_error(void) { return g_err; }

int32_t fg_version(void) { return 100; }   // 0.1.0

fg_status fg_init(void) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return fail(FG_ERR_LAUNCH, "no HIP device is current");
    struct { const fg::KernelEntry *t; int n; } tables[] = {
        {fg::kernel_table_nn(), fg::TILE_COUNT * fg::VARIANT_COUNT}, {fg::kernel_table_nt(), fg::TILE_COUNT * fg::VARIANT_COUNT},
        {fg::kernel_table_tn(), fg::TILE_COUNT * fg::VARIANT_COUNT}, {fg::kernel_table_tt(), fg::TILE_COUNT * fg::VARIANT_COUNT},
        {fg::kernel_table_nn_bf16(), fg::TILE_COUNT}, {fg::kernel_table_nt_bf16(), fg::TILE_COUNT},
        {fg::kernel_table_tn_bf16(), fg::TILE_COUNT}, {fg::kernel_table_tt_bf16(), fg::TILE_COUNT},
        {fg::kernel_table_nn_xf(), fg::TILE_COUNT}, {fg::kernel_table_nt_xf(), fg::TILE_COUNT},
        {fg::kernel_table_tn_xf(), fg::TILE_COUNT}, {fg::kernel_table_tt_xf(), fg::TILE_COUNT},
        {fg::kernel_table_nn_h16(), fg::TILE_COUNT}, {fg::kernel_table_nt_h16(), fg::TILE_COUNT},
        {fg::kernel_table_tn_h16(), fg::TILE_COUNT}, {fg::kernel_table_tt_h16(), fg::TILE_COUNT},
        {fg::kernel_table_diag(), fg::DIAG_TILE_COUNT * 4},
        {fg::kernel_table_cplx(), fg::CTILE_COUNT * 4}, {fg::kernel_table_dual(), fg::CTILE_COUNT * 4},
        {fg::kernel_table_cplx_il(), fg::CTILE_COUNT * 4},
    };
    for (auto &tb : tables)
        for (int i = 0; i < tb.n; ++i) {
            int per_cu = 0;
            if (!tb.t[i].fn) continue;          // a variant that is not built for this tile
            if (fg_status st = prepare(tb.t[i], dev, per_cu)) return st;
        }
    float *st = nullptr;
    if (fg_status s2 = static_scratch(dev, &st)) return s2;
    std::lock_guard<std::mutex> lock(g_ws_mutex);
    Workspace *w = nullptr;
    return workspace_locked(dev, nullptr, true, &w);
}

// static_only: the allocation-free entry point.  Same plan as the ordinary call; partial products
// of a K split go to the static scratch array (FG_ERR_UNSUPPORTED if they do not fit), and nothing
// on this path allocates, frees or creates anything.
static fg_status gemm_impl(int64_t M, int64_t N, int64_t K, float alpha, const fg_matrix *A, const fg_matrix *B,
                           float beta, const fg_matrix *C, const fg_matrix *D, const fg_epilogue *ep, bool dual,
                           const fg_load_transforms *lt, void *hip_stream, bool static_only = false) {
    Problem q;
    if (fg_status st = normalise(M, N, K, alpha, A, B, beta, C, D, ep, dual, lt, q)) return st;
    if (q.M == 0 || q.N == 0) return FG_OK;
    if (q.general) return general_gemm(q, static_only, (hipStream_t)hip_stream);
    Plan plan{0, 1, 1};
    const fg::KernelEntry *kp = select_kernel(q, &plan);
    if (!kp) return fail(FG_ERR_UNSUPPORTED, "no kernel for M=%lld, N=%lld", (long long)q.M, (long long)q.N);
    const fg::KernelEntry &k = *kp;

    fg::GemmParams p;
    memset(&p, 0, sizeof p);
    p.M = (int32_t)q.M; p.N = (int32_t)q.N; p.K = (int32_t)q.K;
    p.tiles_m = (int32_t)((q.M + k.bm - 1) / k.bm); p.tiles_n = (int32_t)((q.N + k.bn - 1) / k.bn);
    p.A = (const _Float16 *)q.A; p.B = (const _Float16 *)q.B;
    p.A_im = (const _Float16 *)q.A_im; p.B_im = (const _Float16 *)q.B_im;
    p.a_rs = q.a_kc ? q.lda : 1; p.a_ks = q.a_kc ? 1 : q.lda;
    p.b_rs = q.b_kc ? q.ldb : 1; p.b_ks = q.b_kc ? 1 : q.ldb;
    // stored span of each operand, rounded up to whole 16-byte chunks (see TileLoader::begin)
    auto span8 = [](bool kc, int64_t rows, int64_t k, int64_t ld) { int64_t s = kc ? (rows - 1) * ld + k : (k - 1) * ld + rows; return (s + 7) / 8 * 8; };
    p.a_span = q.K > 0 ? span8(q.a_kc, q.M, q.K, q.lda) : 0;
    p.b_span = q.K > 0 ? span8(q.b_kc, q.N, q.K, q.ldb) : 0;
    // A and B may be of any size; what must fit 32 bits is the byte offset a lane forms inside one
    // block panel at one K step (up to 256 rows by 64 k) and the advance from one K step to the next.
    const int64_t ab_elem_bytes = q.ilv ? 4 : 2;
    auto reach = [&](bool kc, int64_t ld) { return (kc ? 255 * ld + 64 : 64 * ld + 256) * ab_elem_bytes; };
    if ((!q.a_diag && reach(q.a_kc, q.lda) >= (1ll << 31)) || (!q.b_diag && reach(q.b_kc, q.ldb) >= (1ll << 31)))
        return fail(FG_ERR_UNSUPPORTED, "leading dimension of A or B too large (row-of-K operands: below 2^22 elements, others below 2^24)");
    const int64_t cd_limit = q.ilv ? (1ll << 20) : (1ll << 21);
    if (q.ldc >= cd_limit || q.ldd >= cd_limit) return fail(FG_ERR_UNSUPPORTED, "leading dimension of C or D must be below 2^21 elements (2^20 interleaved)");
    p.C = q.C; p.D = q.D; p.C_im = q.C_im; p.D_im = q.D_im; p.ldc = q.ldc; p.ldd = q.ldd;
    p.bias = q.bias; p.bias_dim = q.bias_dim; p.act = q.act; p.has_c = q.C != nullptr;
    p.c_act = q.c_act;
    p.a_add2 = (uint32_t)q.a_add * 0x10001u; p.b_add2 = (uint32_t)q.b_add * 0x10001u;
    p.alpha = q.alpha; p.beta = q.beta;
    const int64_t tiles64 = (int64_t)p.tiles_m * p.tiles_n;
    if (tiles64 >= (1ll << 31) / 64) return fail(FG_ERR_UNSUPPORTED, "too many tiles");
    const int tiles = (int)tiles64;
    p.tile_begin = 0; p.tile_count = tiles; p.splits = 1;
    p.cd_cached = keeps_cd(q);
    p.rotate = (p.tiles_m == 1 && q.b_kc) || (p.tiles_n == 1 && q.a_kc);
    p.once = p.tiles_m == 1 && fg::streams_once((uintptr_t)q.B, q.ldb, q.N * q.K * 2) ? 1
           : p.tiles_n == 1 && fg::streams_once((uintptr_t)q.A, q.lda, q.M * q.K * 2) ? 2 : 0;
    hipStream_t stream = (hipStream_t)hip_stream;
    if (plan.splits <= 1 && plan.tail_splits <= 1) return launch(k, p, stream);

    // Split K for all tiles, or for the tiles of the last round only: partial products into the
    // workspace, then the reduction pass that also applies alpha, beta.C, bias and the activations.
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return fail(FG_ERR_LAUNCH, "no HIP device is current");
    int S = plan.splits, first = 0, count = tiles;
    if (plan.tail_splits > 1) {
        int per_cu = 0;
        if (fg_status st = prepare(k, dev, per_cu)) return st;
        const int slots = per_cu * kNumCU;
        first = tiles / slots * slots; count = tiles - first; S = plan.tail_splits;
        if (first == 0 || count == 0 || (int64_t)count * S * k.bm * k.bn * 4 > kWorkspaceBytes) S = 1;
    }
    if (S == 1) return launch(k, p, stream);
    const int64_t need = (int64_t)count * S * k.bm * k.bn * 4;
    if (static_only && need > kStaticScratchBytes)
        return fail(FG_ERR_UNSUPPORTED, "this problem is computed as %d partial products over K, which need %lld bytes of scratch memory; the "
                                        "static scratch array of the allocation-free entry point holds %lld (use fg_gemm_ex)",
                    S, (long long)need, (long long)kStaticScratchBytes);
    Scratch scratch;
    if (fg_status st = scratch.acquire(static_only, dev, stream)) return st;
    if (first > 0) {
        fg::GemmParams head = p;
        head.tile_count = first;
        if (fg_status st = launch(k, head, stream)) return st;
    }
    const int64_t nk = (q.K + 63) / 64;
    fg::GemmParams part = p;
    part.tile_begin = first; part.tile_count = count;
    part.splits = S;
    const int64_t kg = k.kg > 1 ? k.kg : 1;          // K groups share a range
    part.split_kt = (int32_t)(((nk + S - 1) / S + kg - 1) / kg * kg);
    part.D = scratch.ptr;
    part.C = nullptr; part.has_c = 0; part.bias = nullptr; part.act = 0; part.c_act = 0; part.alpha = 1.f; part.beta = 0.f;
    if (fg_status st = launch(k, part, stream)) return st;
    hipError_t e = fg::launch_splitk_reduce(scratch.ptr, S, first, count, k.bm, k.bn, p.tiles_m, p.tiles_n, (int)q.M, (int)q.N, q.alpha, q.beta,
                                            q.C, q.ldc, q.D, q.ldd, q.bias, q.bias_dim, q.act, q.c_act, stream);
    if (e != hipSuccess) return fail(FG_ERR_LAUNCH, "launch of the split-K reduction failed: %s", hipGetErrorString(e));
    return scratch.release(stream);
}

fg_status fg_gemm(int64_t M, int64_t N, int64_t K, float alpha, const fg_matrix *A, const fg_matrix *B,
                  float beta, const fg_matrix *C, const fg_matrix *D, const fg_epilogue *ep, void *hip_stream) {
    return gemm_impl(M, N, K, alpha, A, B, beta, C, D, ep, false, nullptr, hip_stream);
}

fg_status fg_gemm_ex(int64_t M, int64_t N, int64_t K, float alpha, const fg_matrix *A, const fg_matrix *B,
                     float beta, const fg_matrix *C, const fg_matrix *D, const fg_epilogue *ep,
                     const fg_load_transforms *lt, void *hip_stream) {
    return gemm_impl(M, N, K, alpha, A, B, beta, C, D, ep, false, lt, hip_stream);
}

fg_status fg_gemm_noalloc(int64_t M, int64_t N, int64_t K, float alpha, const fg_matrix *A, const fg_matrix *B,
                          float beta, const fg_matrix *C, const fg_matrix *D, const fg_epilogue *ep,
                          const fg_load_transforms *lt, void *hip_stream) {
    return gemm_impl(M, N, K, alpha, A, B, beta, C, D, ep, false, lt, hip_stream, true);
}

void fg_reload_tuning(void) { read_tuning_from_environment(); }

fg_status fg_gemm_dual(int64_t M, int64_t N, int64_t K, float alpha, const fg_matrix *A, const fg_matrix *B,
                       float beta, const fg_matrix *C, const fg_matrix *D, void *hip_stream) {
    return gemm_impl(M, N, K, alpha, A, B, beta, C, D, nullptr, true, nullptr, hip_stream);
}

fg_status fg_gemm_plan(int64_t M, int64_t N, int64_t K, int32_t layoutA, int32_t layoutB, int32_t layoutD,
                       int32_t variant, char *buf, int32_t buf_len) {
    if (!buf || buf_len <= 0) return fail(FG_ERR_NULL, "buf is NULL or empty");
    buf[0] = 0;
    g_relaxed.status = FG_OK;
    if (fg_status st = check_sizes(M, N, K)) return st;
    auto ok_in = [](int32_t l) { return l == FG_COL || l == FG_ROW || l == FG_DIAG; };
    if (!ok_in(layoutA) || !ok_in(layoutB) || (layoutD != FG_COL && layoutD != FG_ROW))
        return fail(FG_ERR_LAYOUT, "plan query: A, B take FG_COL / FG_ROW / FG_DIAG, D takes FG_COL / FG_ROW");
    if (layoutA == FG_DIAG && layoutB == FG_DIAG) return fail(FG_ERR_UNSUPPORTED, "at most one of A and B may be diagonal");
    if (variant < FG_PLAN_REAL || variant > FG_PLAN_REAL_AB_ADD) return fail(FG_ERR_LAYOUT, "plan query: unknown variant %d", variant);
    if (variant != FG_PLAN_REAL && (layoutA == FG_DIAG || layoutB == FG_DIAG))
        return fail(FG_ERR_UNSUPPORTED, "diagonal operands are supported for real FG_F16 products only");
    Problem q;
    memset(&q, 0, sizeof q);
    q.cplx = variant == FG_PLAN_COMPLEX || variant == FG_PLAN_DUAL || variant == FG_PLAN_COMPLEX_INTERLEAVED;
    q.ilv = variant == FG_PLAN_COMPLEX_INTERLEAVED;
    q.dual = variant == FG_PLAN_DUAL;
    q.bf16 = variant == FG_PLAN_REAL_BF16;
    q.cd16 = variant == FG_PLAN_REAL_F16_CD;
    q.ab_add = variant == FG_PLAN_REAL_AB_ADD;
    if (layoutD == FG_COL) {
        q.M = M; q.N = N;
        q.a_diag = layoutA == FG_DIAG; q.b_diag = layoutB == FG_DIAG;
        q.a_kc = layoutA == FG_ROW || q.a_diag; q.b_kc = layoutB == FG_COL || q.b_diag;
    } else {
        q.M = N; q.N = M;
        q.a_diag = layoutB == FG_DIAG; q.b_diag = layoutA == FG_DIAG;
        q.a_kc = layoutB == FG_COL || q.a_diag; q.b_kc = layoutA == FG_ROW || q.b_diag;
    }
    q.K = K;
    if (g_relaxed.status != FG_OK) {
        // K is not a multiple of 8 (alignment is not known to this query)
        if (q.cplx || q.a_diag || q.b_diag || q.cd16) return fail(g_relaxed.status, "%s (complex, dual, diagonal and FG_F16-result products have no general kernel)", g_relaxed.msg);
        const GeneralPlan plan = choose_general(q.M, q.N, q.K, 1, true);
        char split[24] = "";
        if (plan.splits > 1) snprintf(split, sizeof split, "+splitk%d", plan.splits);
        // the 64x64 tile keeps the name that callers compare (its K step is 64 now)
        snprintf(buf, (size_t)buf_len, "gemm_general_%s%s", plan.bm == 128 ? "128x128x64" : "64x64x32", split);
        return FG_OK;
    }
    Plan plan{0, 1, 1};
    const fg::KernelEntry *k = select_kernel(q, &plan);
    if (!k) return fail(FG_ERR_UNSUPPORTED, "no kernel for the problem");
    if (plan.splits > 1) snprintf(buf, (size_t)buf_len, "%s+splitk%d", k->name, plan.splits);
    else if (plan.tail_splits > 1) snprintf(buf, (size_t)buf_len, "%s+tailsplitk%d", k->name, plan.tail_splits);
    else snprintf(buf, (size_t)buf_len, "%s", k->name);
    return FG_OK;
}

// Kernel for a planned contraction (tiled kernels only): tile shape, streaming variant, row order.
static const fg::KernelEntry *select_contract_kernel(const Contraction &c, const float *Cin, const float *Cout, int *perm_z_out) {
    // A result that is not contiguous along the leading row mode is stored in short pieces; the
    // smallest tile makes them shorter still (measured on the paper's D_abc = A_bda B_dc).
    const bool rows_contiguous = c.c_m.n == 0 || c.c_m.stride[0] == 1;
    const int tile = choose_plan(c.M, c.N, KRanges(c.K), false, rows_contiguous || c.M < 128 || c.N < 128, c.batches, true, 0, false, 0, kContractPrices).tile;
    // The result streams past the L2 only if every store of 32 consecutive rows is one whole,
    // aligned 128-byte line: leading row mode contiguous with an extent that is a multiple of 32,
    // every other stride of C and its base a multiple of 32 elements.
    auto whole_lines = [](const fg::ModeGroup &g, int first) {
        for (int t = first; t < g.n; ++t) if (g.stride[t] % 32) return false;
        return true;
    };
    const bool c_stream = c.c_m.n > 0 && c.c_m.stride[0] == 1 && c.c_m.extent[0] % 32 == 0 && whole_lines(c.c_m, 1) &&
                          whole_lines(c.c_n, 0) && whole_lines(c.c_b, 0) && (uintptr_t)Cout % 128 == 0 &&
                          (!Cin || (uintptr_t)Cin % 128 == 0);
    const fg::KernelEntry &k = table_for(c.a_kc, c.b_kc)[fg::entry_index(tile, c_stream ? fg::VARIANT_CONTRACT_STREAM : fg::VARIANT_CONTRACT)];
    // Row order inside a tile (tile_row in the kernel): when A is contiguous along its leading row
    // mode but C along the next one, and the leading mode is short enough that a tile spans at
    // least four values of the next, let every accumulator hold 8 x 4 of (leading, next).
    *perm_z_out = 1;
    if (k.fn && !c.a_kc && c.c_m.n >= 2 && c.c_m.stride[1] == 1) {
        const int e0 = c.a_m.extent[0];
        if (e0 % 8 == 0 && k.bm % e0 == 0 && k.bm / e0 >= 4) *perm_z_out = k.bm / e0;
    }
    return k.fn ? &k : nullptr;
}

fg_status fg_contract(int32_t nA, const int32_t *modesA, const int64_t *stridesA, const void *A,
                      int32_t nB, const int32_t *modesB, const int64_t *stridesB, const void *B,
                      int32_t nC, const int32_t *modesC, const int64_t *stridesC, const float *Cin, float *Cout,
                      int32_t n_modes, const int32_t *mode_labels, const int64_t *mode_extents,
                      float alpha, float beta, void *hip_stream) {
    Contraction c;
    if (fg_status st = plan_contraction(nA, modesA, stridesA, A, nB, modesB, stridesB, B, nC, modesC, stridesC,
                                        Cin, Cout, n_modes, mode_labels, mode_extents, c))
        return st;
    if (c.M == 0 || c.N == 0) return FG_OK;
    const bool use_c = Cin != nullptr && beta != 0.f;        // beta == 0: Cin is never read
    if (c.general) {
        fg::GeneralParams f;
        memset(&f, 0, sizeof f);
        const GeneralPlan plan = choose_general(c.M, c.N, c.K, c.batches, false);
        f.M = (int32_t)c.M; f.N = (int32_t)c.N; f.K = (int32_t)c.K; f.batches = (int32_t)c.batches; f.splits = 1;
        f.A = (const uint16_t *)c.A; f.B = (const uint16_t *)c.B;
        f.a_kmax = c.a_kmax; f.b_kmax = c.b_kmax; f.k_modes = c.a_k.n > 0 ? c.a_k.n : 1; f.small = c.a_span < (1ll << 31) && c.b_span < (1ll << 31);
        f.a_span = c.a_span; f.b_span = c.b_span; f.a_es = c.a_es; f.b_es = c.b_es;
        f.C = use_c ? Cin : nullptr; f.D = Cout;
        f.a_m = c.a_m; f.a_k = c.a_k; f.b_n = c.b_n; f.b_k = c.b_k; f.c_m = c.c_m; f.c_n = c.c_n;
        f.a_b = c.a_b; f.b_b = c.b_b; f.c_b = c.c_b;
        f.m_ext0 = c.m_ext0; f.n_ext0 = c.n_ext0; f.k_ext0 = c.k_ext0; f.m_hi = c.m_hi;
        f.alpha = alpha; f.beta = use_c ? beta : 0.f;
        auto odd_strides = [](const fg::ModeGroup &g) { for (int t = 0; t < g.n; ++t) if (g.stride[t] % 2 && g.stride[t] != 1) return true; return false; };
        f.odd = ((!c.a_kc && c.m_ext0 < 64) || (!c.b_kc && c.n_ext0 < 64)) && ((uintptr_t)f.A % 4 != 0 || (uintptr_t)f.B % 4 != 0 || odd_strides(f.a_m) || odd_strides(f.a_k) || odd_strides(f.a_b) ||
                odd_strides(f.b_n) || odd_strides(f.b_k) || odd_strides(f.b_b));
        const int64_t tiles_m = (c.M + plan.bm - 1) / plan.bm, tiles_n = (c.N + plan.bn - 1) / plan.bn;
        if (tiles_m * tiles_n * c.batches >= (1ll << 31)) return fail(FG_ERR_UNSUPPORTED, "too many tiles");
        f.tiles_m = (int32_t)tiles_m; f.tiles_n = (int32_t)tiles_n;
        hipError_t e = fg::launch_contract_general(f, c.a_kc, c.b_kc, plan.variant, (hipStream_t)hip_stream);
        if (e != hipSuccess) return fail(FG_ERR_LAUNCH, "launch of the general contraction kernel failed: %s", hipGetErrorString(e));
        return FG_OK;
    }
    int perm_z = 1;
    const fg::KernelEntry *kp = select_contract_kernel(c, Cin, Cout, &perm_z);
    if (!kp) return fail(FG_ERR_UNSUPPORTED, "internal: no contraction kernel for this tile");
    const fg::KernelEntry &k = *kp;
    fg::ContractParams p;
    memset((void *)&p, 0, sizeof p);
    p.M = (int32_t)c.M; p.N = (int32_t)c.N; p.K = (int32_t)c.K;
    p.tiles_m = (int32_t)((c.M + k.bm - 1) / k.bm); p.tiles_n = (int32_t)((c.N + k.bn - 1) / k.bn);
    p.A = (const _Float16 *)c.A; p.B = (const _Float16 *)c.B;
    p.C = use_c ? Cin : nullptr; p.D = Cout;
    p.has_c = use_c;
    p.alpha = alpha; p.beta = use_c ? beta : 0.f;
    p.a_m = c.a_m; p.a_k = c.a_k; p.b_n = c.b_n; p.b_k = c.b_k; p.c_m = c.c_m; p.c_n = c.c_n;
    p.a_b = c.a_b; p.b_b = c.b_b; p.c_b = c.c_b; p.batches = (int32_t)c.batches;
    if ((int64_t)p.tiles_m * p.tiles_n * c.batches >= (1ll << 31)) return fail(FG_ERR_UNSUPPORTED, "too many tiles");
    p.perm_z = perm_z;
    return launch(k, p, (hipStream_t)hip_stream, p.batches);
}

fg_status fg_contract_plan(int32_t nA, const int32_t *modesA, const int64_t *stridesA, const void *A,
                           int32_t nB, const int32_t *modesB, const int64_t *stridesB, const void *B,
                           int32_t nC, const int32_t *modesC, const int64_t *stridesC, const float *Cin, float *Cout,
                           int32_t n_modes, const int32_t *mode_labels, const int64_t *mode_extents,
                           char *buf, int32_t buf_len) {
    if (!buf || buf_len <= 0) return fail(FG_ERR_NULL, "buf is NULL or empty");
    buf[0] = 0;
    Contraction c;
    if (fg_status st = plan_contraction(nA, modesA, stridesA, A, nB, modesB, stridesB, B, nC, modesC, stridesC,
                                        Cin, Cout, n_modes, mode_labels, mode_extents, c))
        return st;
    if (c.M == 0 || c.N == 0) { snprintf(buf, (size_t)buf_len, "nothing to compute"); return FG_OK; }
    if (c.general) {
        const GeneralPlan plan = choose_general(c.M, c.N, c.K, c.batches, false);
        snprintf(buf, (size_t)buf_len, "gett_general_64x64x32 (%s; %dx%d tiles)", c.why_general, plan.bm, plan.bn);
        return FG_OK;
    }
    int perm_z = 1;
    const fg::KernelEntry *k = select_contract_kernel(c, Cin, Cout, &perm_z);
    if (!k) return fail(FG_ERR_UNSUPPORTED, "internal: no contraction kernel for this tile");
    snprintf(buf, (size_t)buf_len, "%s", k->name);
    return FG_OK;
}

}  // extern "C"
