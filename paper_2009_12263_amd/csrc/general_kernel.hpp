// General matrix-unit kernel: operands that miss the alignment the direct-to-LDS kernels of
// gemm_kernel.hpp need.  Matrices with any leading dimension, bases aligned to an element only and
// any K; contractions with any strides and extents, tensors of any size and outer products.
//
// The direct-to-LDS loads of the tiled kernels move aligned 16-byte pieces.  Here a tile passes
// through registers instead: each thread fetches pieces of eight elements along one direction of
// the operand (an unaligned 16-byte load where the eight lie side by side in memory, eight 2-byte
// loads where they do not or where the piece would reach past the operand), clears what lies
// beyond K, and writes the piece to the place in LDS where a direct load of the tiled kernels would
// have put it, so that fragment reads and matrix instructions are theirs.  Pieces of K step t+2 are
// in flight while step t is multiplied and step t+1 waits in LDS.
//
// What bounds it: the vector-memory path of a compute unit.  A 16-byte load per lane that starts at
// an odd element costs 52 cache accesses per wave, one at an even element 22, an aligned one 15
// (TCP_TOTAL_CACHE_ACCESSES per vector load at 1531x1021x2003, where both operands start odd: 51.8; at 1530x1018x2003
// and 1536x1024x2003, whose A starts even or aligned and whose B is odd: 36.9 and 33.2; 27.9, 26.2 and 23.7 us;
// the direct-to-LDS kernels take 20 to 22 us for 1536x1024x2048).  What costs is the lines rather than the accesses: pieces that
// lie across two lines are filled at 54 GB/s per unit, others at 104, and with fewer accesses (the fifth word of an odd piece from
// the neighbouring lane) the product takes as long (28.9 us).  1531x1021x2003: 449 us with the element-wise FP32
// kernel that served these operands before.
// 4095x4097x4099: 244 us, 563 TFLOP/s.
#pragma once
#include "kernel_table.hpp"
#include "piece_address.hpp"

namespace fg {

struct GeneralParams {
    int32_t M, N, K;                  // merged extents as they are walked (see the *_ext0 below)
    int32_t tiles_m, tiles_n;
    int32_t splits, split_kt;         // as in GemmParams: split-K writes raw partial tiles to D
    int32_t items;                    // tiles x K ranges x batches
    const uint16_t *A, *B;
    int64_t a_span, b_span;           // elements from the base to one past the last stored one
    const float *C;
    float *D;
    int64_t ldc, ldd;                 // matrices: (m, n) at m + n*ld
    float alpha, beta;
    // matrices: element (row, k) at row*rs + k*ks, one of them 1
    int64_t a_rs, a_ks, b_rs, b_ks;
    const float *bias;
    int32_t bias_dim, act, c_act;
    int32_t ab_add;                   // the FP16 addends of fg_load_transforms, as two packed halves
    uint32_t a_add2, b_add2;
    // Contractions: mode groups.  Pieces of eight run along the leading mode of an operand's rows (or,
    // A_KC / B_KC, of the summed modes): its extent in the groups is rounded up to a multiple of 8
    // so that no piece straddles two values of the next mode, and *_ext0 is the true extent.
    ModeGroup a_m, a_k, b_n, b_k, c_m, c_n, a_b, b_b, c_b;
    int32_t m_ext0, n_ext0, k_ext0;
    int32_t m_hi;                     // nonzero: the rows' leading mode is split, mode 0 of the groups are its
                                      // pieces' elements and mode m_hi counts the pieces
    int64_t a_es, b_es;               // element stride inside a piece
    int64_t a_kmax, b_kmax;           // largest offset of a k in A and in B
    int32_t batches;
    int32_t k_modes;                  // modes of a_k that count (at least 1)
    int32_t odd;                      // fetch INSIDE_ODD (see FetchMode) where the kernel has it
    int32_t small;                    // A and B span less than 2^31 elements, i.e. 32-bit byte offsets reach all of them
};

// Eight 16-bit elements that may start at any element: one 16-byte load (the target runs with
// unaligned access enabled; measured no slower than an aligned one to within 5 %).
struct __attribute__((packed, aligned(2))) Piece { uint32_t w[4]; };
__device__ __forceinline__ u32x4 load_piece(const uint16_t *p) {
    const Piece v = *(const Piece *)p;
    return u32x4{v.w[0], v.w[1], v.w[2], v.w[3]};
}
// The four words from a word-aligned address on.
__device__ __forceinline__ u32x4 load_words(const char *p) {
    typedef uint32_t u32x4_word __attribute__((ext_vector_type(4), aligned(4)));
    return *(const u32x4_word *)p;
}
// The first `count` of eight elements es apart, zeros behind them.  What does not exist is read
// from element 0 instead and cleared, so that the loads carry no branches.
__device__ __forceinline__ u32x4 load_elements(const uint16_t *base, int64_t off, int64_t es, int count) {
    uint32_t e[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) e[i] = base[i < count ? off + i * es : 0];
    u32x4 v;
#pragma unroll
    for (int w = 0; w < 4; ++w) v[w] = (2 * w < count ? e[2 * w] : 0u) | (2 * w + 1 < count ? e[2 * w + 1] << 16 : 0u);
    return v;
}
// Keep the first `count` of eight elements.
__device__ __forceinline__ u32x4 keep_first(u32x4 v, int count) {
#pragma unroll
    for (int w = 0; w < 4; ++w) v[w] &= count >= 2 * w + 2 ? 0xffffffffu : count == 2 * w + 1 ? 0xffffu : 0u;
    return v;
}
// Elements n .. 7 moved to the front (0 <= n <= 7; what follows them is arbitrary).
__device__ __forceinline__ u32x4 drop_first(u32x4 v, int n) {
    if (n & 4) { v[0] = v[2]; v[1] = v[3]; }
    if (n & 2) { v[0] = v[1]; v[1] = v[2]; v[2] = v[3]; }
    if (n & 1) { v[0] = (v[0] >> 16) | (v[1] << 16); v[1] = (v[1] >> 16) | (v[2] << 16); v[2] = (v[2] >> 16) | (v[3] << 16); v[3] >>= 16; }
    return v;
}

// Offsets of the 64 k of a K step of a contraction, filled in by one wave two steps ahead.
struct KTable {
    int64_t a[64], b[64];    // element offset of k in A and in B
    int32_t left[64];        // how many k from this one on are stored side by side in the leading mode (0..8; 0: beyond K)
};

// How the pieces of a K step are fetched.  INSIDE: 16-byte loads, known to lie inside the operand.
// CLAMP: a piece that would reach past the operand's last element is loaded from its last eight
// elements and moved into place when it is committed (nothing outside the operand is read, and no
// branch stands between the load and its use: with one, every step waited for its own loads,
// 33 against 28 us at 1531x1021x2003).  GATHER: eight element loads per piece, for operands without
// a unit stride and for those of fewer than eight elements.
// INSIDE_ODD: INSIDE for operands with pieces that start in the middle of a 4-byte word: the five words
// that hold the piece are loaded (a word-aligned 16-byte load and a 4-byte one, see odd_piece, which the cache serves several
// lanes of at a time; a 16-byte load in the middle of words goes lane by lane) and shifted by 16 bits
// when committed.  Contractions on 64x64 tiles whose rows or columns come in runs shorter than the tile
// (37x29x31x35 over 27x25: 21.3 -> 19.0 us, D_abc = A_bda B_dc with 63, 31, 511, 373: 14.1 -> 13.0);
// with longer runs, on the larger tile and for matrices it measured 2 to 20 % slower.
enum FetchMode { FETCH_INSIDE, FETCH_CLAMP, FETCH_GATHER, FETCH_INSIDE_ODD };
constexpr bool is_inside(int mode) { return mode == FETCH_INSIDE || mode == FETCH_INSIDE_ODD; }

// Index along a group's leading mode; hi: the mode that counts its pieces of eight, 0 if it is not split.
__device__ __forceinline__ int leading_index(const ModeGroup &g, int idx, int hi) {
    int lead = 0;
#pragma unroll
    for (int t = 0; t < kMaxGroupModes; ++t) {
        const int q = (int)(__umulhi((uint32_t)idx, g.magic[t]) >> g.shift[t]);
        const int digit = idx - q * g.extent[t];
        if (t == 0) lead = digit;
        else if (t == hi) lead += 8 * digit;
        idx = q;
    }
    return lead;
}

template <int R, bool KC, int NT, bool PLAIN>
struct PieceLoader {
    static constexpr int CH = R * 8 / NT;            // pieces per thread and K step
    static constexpr int PER_ROW = KC ? 8 : R / 8;   // pieces per LDS row
    static constexpr int STEP = NT / PER_ROW;        // LDS rows between a thread's pieces
    static_assert(R * 8 % NT == 0 && STEP % 16 == 0, "all pieces of a thread sit at the same logical position of their LDS rows");
    int64_t off[KC ? CH : 1];    // offset of the pieces' rows (KC: rows r + s*STEP, MC: one piece of eight rows)
    int pos;                     // KC: k of the pieces inside a step; MC: k-row of the first one
    int rows;                    // MC: how many of the eight rows exist
    u32x4 stage[2][CH];             // the pieces of two K steps in flight
    int left[2][KC ? 1 : CH];       // elements of the staged pieces that are below K (MC: 0 or 8)
    int shift[2][CH];               // CLAMP: how many elements before its place a piece was loaded
    uint32_t fifth[2][CH];          // INSIDE_ODD: the word after the staged four, if the piece reaches into it
    int skew[2][CH];                // INSIDE_ODD: bytes to drop in front (0 or 2)

    __device__ __forceinline__ void init(const ModeGroup &rg, int ext0, int hi, int64_t rs, int row0, int rdim, int tid) {
        if constexpr (KC) {
            const int r = tid / 8;
            pos = ((tid % 8) ^ kc_swz<64>(r)) * 8;
#pragma unroll
            for (int s = 0; s < CH; ++s) {
                // rows past the last one repeat it: they only reach results that are not stored
                int m = row0 + r + s * STEP;
                m = m < rdim ? m : rdim - 1;
                if constexpr (PLAIN) off[s] = (int64_t)m * rs + pos;
                else off[s] = group_offset(rg, m);
            }
        } else {
            pos = tid / PER_ROW;
            const int c = (tid % PER_ROW) ^ (mc_swz<R>(pos) << 2) ^ mc_piece<R>(pos);
            int m = row0 + c * 8;
            const int last = (rdim - 1) & ~7;
            m = m < last ? m : last;
            if constexpr (PLAIN) {
                off[0] = m;
                rows = rdim - m;
            } else {
                off[0] = group_offset(rg, m);
                rows = ext0 - leading_index(rg, m, hi);
            }
        }
    }
    // one piece, `off` elements from base (the operand's first element in the CLAMP and GATHER modes)
    template <int MODE>
    __device__ __forceinline__ void request(int slot, int s, const uint16_t *base, int64_t at, int64_t span, int64_t es, int count) {
        if constexpr (MODE == FETCH_INSIDE) {
            stage[slot][s] = load_piece(base + at);
        } else if constexpr (MODE == FETCH_CLAMP) {
            const int64_t over = at + 8 - span;
            shift[slot][s] = over > 0 ? (over < 8 ? (int)over : 7) : 0;   // from 8 on no element exists
            stage[slot][s] = load_piece(base + (over > 0 ? span - 8 : at));
        } else {
            stage[slot][s] = load_elements(base, at, es, count);
        }
    }
    // Matrices: request K step kt (INSIDE: 72 or more k are left, so that even the piece at the end of the
    // last column or row of the step is followed by a whole one).
    template <int MODE>
    __device__ __forceinline__ void fetch_plain(int slot, const uint16_t *base, int64_t span, int64_t ks, int kt, int K) {
        const int k0 = kt * 64;
        if constexpr (KC) {
            const int n = K - (k0 + pos);
            if constexpr (!is_inside(MODE)) left[slot][0] = n < 0 ? 0 : n > 8 ? 8 : n;
#pragma unroll
            for (int s = 0; s < CH; ++s) request<MODE>(slot, s, base, off[s] + k0, span, 1, left[slot][0]);
        } else {
            const int64_t mine = off[0] + (int64_t)pos * ks, step = (int64_t)k0 * ks;
#pragma unroll
            for (int s = 0; s < CH; ++s) {
                if constexpr (!is_inside(MODE)) left[slot][s] = k0 + pos + s * STEP < K ? 8 : 0;
                request<MODE>(slot, s, base, mine + (step + s * STEP * ks), span, 1, left[slot][s] ? rows : 0);
            }
        }
    }
    // Contractions: request the K step whose offsets stand in koff, kleft.  INSIDE (the wave's pieces
    // lie inside the operand whatever k is, and its offsets fit 32 bits): `whole` steps, of which every
    // k is below K, need no kleft.
    template <int MODE>
    __device__ __forceinline__ void fetch_strided(int slot, const uint16_t *base, int64_t span, int64_t es, bool whole, const int64_t *koff, const int32_t *kleft) {
        if constexpr (is_inside(MODE)) {
            auto piece = [&](int s, int64_t at_row, int64_t at_k) {
                const uint32_t at = ((uint32_t)at_row + (uint32_t)at_k) * 2u;
                const char *q = (const char *)base;
                if constexpr (MODE == FETCH_INSIDE) {
                    stage[slot][s] = load_piece((const uint16_t *)(q + at));
                } else {
                    const uint32_t base_skew = (uint32_t)(uintptr_t)q & 2u;    // uniform
                    q -= base_skew;
                    const OddPiece o = odd_piece(at + base_skew);
                    skew[slot][s] = (int)o.skew;
                    stage[slot][s] = load_words(q + o.words);
                    fifth[slot][s] = *(const uint32_t *)(q + o.fifth);
                }
            };
            if (!whole) {
#pragma unroll
                for (int s = 0; s < (KC ? 1 : CH); ++s) left[slot][s] = KC ? kleft[pos] : kleft[pos + s * STEP] ? 8 : 0;
            }
#pragma unroll
            for (int s = 0; s < CH; ++s) piece(s, off[KC ? s : 0], KC ? koff[pos] : koff[pos + s * STEP]);
        } else if constexpr (KC) {
            left[slot][0] = kleft[pos];
            const int64_t k = koff[pos];
#pragma unroll
            for (int s = 0; s < CH; ++s) request<MODE>(slot, s, base, off[s] + k, span, es, left[slot][0]);
        } else {
#pragma unroll
            for (int s = 0; s < CH; ++s) {
                left[slot][s] = kleft[pos + s * STEP] ? 8 : 0;
                request<MODE>(slot, s, base, off[0] + koff[pos + s * STEP], span, es, left[slot][s] ? rows : 0);
            }
        }
    }
    // no piece of this thread reaches past the operand, kmax being the largest offset of a k
    __device__ __forceinline__ bool always_inside(int64_t kmax, int64_t span) const {
        bool ok = true;
#pragma unroll
        for (int s = 0; s < (KC ? CH : 1); ++s) ok = ok && piece_inside(off[s], kmax, span);
        return ok;
    }
    // Write the staged pieces to LDS; `whole`: every k of the step is below K.
    template <int MODE>
    __device__ __forceinline__ void commit(int slot, FG_LDS char *tile, int tid, bool whole, bool add, uint32_t addend) {
        bool moved = false;
        if constexpr (MODE == FETCH_CLAMP) {
            int any = 0;
#pragma unroll
            for (int s = 0; s < CH; ++s) any |= shift[slot][s];
            moved = __builtin_amdgcn_ballot_w64(any != 0) != 0;
        }
#pragma unroll
        for (int s = 0; s < CH; ++s) {
            u32x4 v = stage[slot][s];
            if constexpr (MODE == FETCH_INSIDE_ODD) {
                const uint32_t sh = (uint32_t)skew[slot][s], last = fifth[slot][s];
                v = u32x4{__builtin_amdgcn_alignbyte(v[1], v[0], sh), __builtin_amdgcn_alignbyte(v[2], v[1], sh),
                          __builtin_amdgcn_alignbyte(v[3], v[2], sh), __builtin_amdgcn_alignbyte(last, v[3], sh)};
            }
            if (moved) v = drop_first(v, shift[slot][s]);
            if (add) v = __builtin_bit_cast(u32x4, add8(__builtin_bit_cast(half8, v), addend));
            if ((!is_inside(MODE) || !PLAIN) && !whole) v = keep_first(v, left[slot][KC ? 0 : s]);
            *(FG_LDS u32x4 *)(tile + (s * NT + tid) * 16) = v;
        }
    }
};

// Result of a product whose K was split, from the sum of its partial products (c, bias: used if there is
// one).  Each operation is spelt out as in the reduction pass (splitk_reduce.hip), so that a tile whose ranges
// are added up here has that pass's bits.
__device__ __forceinline__ float split_value(float sum, float alpha, bool has_c, float beta, float c, bool has_bias, float bias) {
#pragma clang fp contract(off)
    float y = alpha * sum;
    if (has_c) y = __builtin_fmaf(beta, c, y);
    if (has_bias) y = y + bias;
    return y;
}

// KG groups of WGM x WGN waves share a BM x BN tile: group g multiplies the K steps kt0 + g, kt0 + g +
// KG, ... into accumulators of its own, from LDS buffers of its own, and the groups' results are
// added up through LDS at the end, each group finishing 1/KG of the registers.
// ONE (the 64x64 tile with one group): products of one K step, which need no second buffer and no prefetch.
// RANGES (matrices): a workgroup computes the K ranges of its tile one after another and adds them up as
// the reduction pass would.  It needs no scratch memory and gives the bits of the split product.
template <int BM, int BN, int WGM, int WGN, int KG, bool A_KC, bool B_KC, bool BF16, bool PLAIN, bool RANGES = false>
__global__ __launch_bounds__(64 * WGM * WGN * KG) void general_kernel(const GeneralParams p) {
    constexpr int NW = WGM * WGN, NT = 64 * NW, WTM = BM / WGM, WTN = BN / WGN, TI = WTM / 32, TJ = WTN / 32;
    constexpr bool ONE = KG == 1 && BM == 64;
    constexpr int BUFFERS = ONE ? 1 : 2;
    constexpr int A_BYTES = BM * 128, B_BYTES = BN * 128, GROUP_BYTES = BUFFERS * (A_BYTES + B_BYTES);
    constexpr int RR = 16 / KG;                         // registers of each 32x32 block that a group finishes
    static_assert((PLAIN && !ONE) || !RANGES, "contractions and products of one K step are not split");
    static_assert(KG == 1 || KG * NW * TI * TJ * 16 * 64 * 4 <= KG * GROUP_BYTES, "the exchange of the groups' results fits the K loop's buffers");
    __shared__ __attribute__((aligned(1024))) char smem_generic[KG * GROUP_BYTES];
    __shared__ KTable ktab[PLAIN ? 1 : KG][PLAIN || ONE ? 1 : 4];
    const int lane = threadIdx.x & 63;
    const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int group = wave_all / NW, wave = wave_all - group * NW, tid = wave * 64 + lane;
    const int wm = wave % WGM, wn = wave / WGM;
    FG_LDS char *smem = (FG_LDS char *)smem_generic;
    FG_LDS char *lds_a = smem + group * GROUP_BYTES, *lds_b = lds_a + BUFFERS * A_BYTES;

    // work item -> (K range or batch index, tile)
    const int tiles = p.tiles_m * p.tiles_n;
    const int64_t item64 = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    if (item64 >= p.items) return;
    const int item = (int)item64;
    int outer = item / tiles, tm, tn;
    block_to_tile(item - outer * tiles, p.tiles_m, p.tiles_n, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;
    int split = 0, batch = 0;
    if constexpr (PLAIN) split = outer;
    else { split = outer / p.batches; batch = outer - split * p.batches; }
    const int nk_all = (p.K + 63) / 64;
    typename std::conditional<RANGES, int, const int>::type kt0 = p.splits > 1 ? split * p.split_kt : 0;
    int kt1 = p.splits > 1 ? kt0 + p.split_kt : nk_all;
    if (kt1 > nk_all) kt1 = nk_all;

    const uint16_t *A = p.A, *B = p.B;
    int64_t a_span = p.a_span, b_span = p.b_span;
    if constexpr (!PLAIN) {
        const int64_t oa = group_offset(p.a_b, batch), ob = group_offset(p.b_b, batch);
        A += oa; B += ob; a_span -= oa; b_span -= ob;
    }
    PieceLoader<BM, A_KC, NT, PLAIN> la;
    PieceLoader<BN, B_KC, NT, PLAIN> lb;
    la.init(p.a_m, p.m_ext0, p.m_hi, p.a_rs, m0, p.M, tid);
    lb.init(p.b_n, p.n_ext0, 0, p.b_rs, n0, p.N, tid);
    FragReader<BM, 64, A_KC, TI> fa;
    FragReader<BN, 64, B_KC, TJ> fb;
    fa.init(wm * WTM, lane);
    fb.init(wn * WTN, lane);

    // step i of this group is K step kt(i)
    auto kt = [&](int i) { return kt0 + group + KG * i; };
    auto fill_table = [&](int i) {                      // one wave: lane <-> k of the step
        if constexpr (!PLAIN) {
            KTable &t = ktab[group][i & 3];
            const int k = kt(i) * 64 + lane;
            // 32-bit arithmetic where the operands allow it, and no further than the summed modes go: one
            // wave computes while the others wait for it at the step's barrier
            int lead, idx = k;
            int64_t oa = 0, ob = 0;
            uint32_t oa32 = 0, ob32 = 0;
            for (int m = 0; m < p.k_modes; ++m) {
                const int q = (int)(__umulhi((uint32_t)idx, p.a_k.magic[m]) >> p.a_k.shift[m]);
                const int digit = idx - q * p.a_k.extent[m];
                if (m == 0) lead = digit;
                if (p.small) {
                    oa32 += (uint32_t)digit * (uint32_t)p.a_k.stride[m];
                    ob32 += (uint32_t)digit * (uint32_t)p.b_k.stride[m];
                } else {
                    oa += digit * p.a_k.stride[m];
                    ob += digit * p.b_k.stride[m];
                }
                idx = q;
            }
            const int rest = p.k_ext0 - lead;
            const bool ok = k < p.K && rest > 0;
            t.left[lane] = ok ? (rest < 8 ? rest : 8) : 0;
            t.a[lane] = ok ? (p.small ? (int64_t)oa32 : oa) : 0;
            t.b[lane] = ok ? (p.small ? (int64_t)ob32 : ob) : 0;
        }
    };
    // every k of step i is below K (contractions whose leading summed mode is rounded up have k to clear in every step)
    auto whole_step = [&](int i) { return (PLAIN || p.k_ext0 == p.a_k.extent[0]) && kt(i) * 64 + 64 <= p.K; };
    auto fetch = [&](auto mode_tag, int i, int slot) {
        constexpr int MODE = decltype(mode_tag)::value;
        if constexpr (PLAIN) {
            la.template fetch_plain<MODE>(slot, A, a_span, p.a_ks, kt(i), p.K);
            lb.template fetch_plain<MODE>(slot, B, b_span, p.b_ks, kt(i), p.K);
        } else {
            const KTable &t = ktab[group][i & 3];
            const bool whole = whole_step(i);
            la.template fetch_strided<MODE>(slot, A, a_span, p.a_es, whole, t.a, t.left);
            lb.template fetch_strided<MODE>(slot, B, b_span, p.b_es, whole, t.b, t.left);
        }
    };
    auto commit = [&](auto mode_tag, int i, int slot) {
        constexpr int MODE = decltype(mode_tag)::value;
        const bool whole = whole_step(i);
        const bool add = PLAIN && !BF16 && p.ab_add;
        la.template commit<MODE>(slot, lds_a + slot * A_BYTES, tid, whole, add, p.a_add2);
        lb.template commit<MODE>(slot, lds_b + slot * B_BYTES, tid, whole, add, p.b_add2);
    };
    auto publish = [&] {                                // LDS writes of all waves visible; loads stay in flight
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    floatx16 acc[TI][TJ];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // The K loop.  EDGE: mode of the steps that may reach past the operands.  Every group runs the
    // same number of steps (barriers); a group's last one may be empty.
    auto k_loop = [&](auto edge_tag) {
        constexpr std::integral_constant<int, FETCH_INSIDE> INSIDE{};
        const int steps = (kt1 - kt0 + KG - 1) / KG;
        if (kt(0) < kt1) fetch(edge_tag, 0, 0);
        if constexpr (!ONE) { if (kt(1) < kt1) fetch(edge_tag, 1, 1); }
        if (kt(0) < kt1) commit(edge_tag, 0, 0);
        if constexpr (!ONE) { if (kt(2) < kt1) fetch(edge_tag, 2, 0); }
        publish();
        auto step = [&](auto mode_tag, int i, auto cur_tag) {      // step i, from LDS buffer `cur`
            constexpr int cur = decltype(cur_tag)::value, nxt = cur ^ 1;
            constexpr bool STEADY = PLAIN && is_inside(decltype(mode_tag)::value);
            // the buffer of step i+1 was last read in step i-1, before the barrier that ended it
            if constexpr (!ONE) {
                if (STEADY || kt(i + 1) < kt1) commit(mode_tag, i + 1, nxt);
                if (STEADY || kt(i + 3) < kt1) fetch(mode_tag, i + 3, nxt);
            }
            if (STEADY || kt(i) < kt1) {
                FG_LDS const char *ta = lds_a + cur * A_BYTES, *tb = lds_b + cur * B_BYTES;
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
                    half8 af[TI], bf[TJ];
#pragma unroll
                    for (int j = 0; j < TJ; ++j) bf[j] = fb.read(tb, j, ks);
#pragma unroll
                    for (int m = 0; m < TI; ++m) af[m] = fa.read(ta, m, ks);
#pragma unroll
                    for (int m = 0; m < TI; ++m)
#pragma unroll
                        for (int j = 0; j < TJ; ++j) acc[m][j] = mfma<BF16>(bf[j], af[m], acc[m][j]);
                }
            }
            if constexpr (ONE) return;
            // offsets of step i+4: their slot was last read for step i
            if constexpr (!PLAIN) { if (wave == i % NW) fill_table(i + 4); }
            publish();
        };
        if constexpr (ONE) {
            step(edge_tag, 0, std::integral_constant<int, 0>{});
            return;
        }
        int i = 0;
        if constexpr (PLAIN && decltype(edge_tag)::value == FETCH_CLAMP) {
            // while the fetches of both steps lie inside the operands and inside this work item's K
            // range, for the last group as for the first
            const int k_end = kt1 * 64 + 8 < p.K ? kt1 * 64 + 8 : p.K;
            for (; (kt0 + KG - 1 + KG * (i + 4)) * 64 + 72 <= k_end; i += 2) {
                step(INSIDE, i, std::integral_constant<int, 0>{});
                step(INSIDE, i + 1, std::integral_constant<int, 1>{});
            }
        }
        for (; i < steps; i += 2) {
            step(edge_tag, i, std::integral_constant<int, 0>{});
            if (i + 1 < steps) step(edge_tag, i + 1, std::integral_constant<int, 1>{});
        }
    };
    float y[TI][TJ][RR];                                // the groups' results (below)
    [[maybe_unused]] float total[TI][TJ][RR] = {};      // RANGES: their sum over the K ranges
    for (;;) {                                          // once, RANGES: once per K range
        if (kt0 < kt1) {
            if constexpr (!PLAIN) {
                for (int i = wave; i < (ONE ? 1 : 4); i += NW) fill_table(i);
                publish();
            }
            const bool pieces = (PLAIN || (p.a_es == 1 && p.b_es == 1)) && a_span >= 8 && b_span >= 8;
            // (contractions: the waves of a workgroup may take different loops, which have the same barriers)
            const bool inside = !PLAIN && pieces && p.small &&
                                __builtin_amdgcn_ballot_w64(!(la.always_inside(p.a_kmax, a_span) && lb.always_inside(p.b_kmax, b_span))) == 0;
            constexpr std::integral_constant<int, FETCH_INSIDE> INSIDE{};
            constexpr std::integral_constant<int, FETCH_INSIDE_ODD> INSIDE_ODD{};
            constexpr std::integral_constant<int, FETCH_CLAMP> CLAMP{};
            constexpr std::integral_constant<int, FETCH_GATHER> GATHER{};
            if constexpr (PLAIN) {
                if (!pieces) k_loop(GATHER);
                else k_loop(CLAMP);
            } else {
                constexpr bool SHORT_RUNS = !(A_KC && B_KC) && BM == 64;
                if (SHORT_RUNS && inside && p.odd) { if constexpr (SHORT_RUNS) k_loop(INSIDE_ODD); }
                else if (inside) k_loop(INSIDE);
                else if (pieces) k_loop(CLAMP);
                else k_loop(GATHER);
            }
        }

        // ---- register r0 + r of block (i, j) ends up in y[i][j][r] of group r0 / RR ----
        const int r0 = group * RR;
        if constexpr (KG == 1) {
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int j = 0; j < TJ; ++j)
#pragma unroll
                    for (int r = 0; r < RR; ++r) y[i][j][r] = acc[i][j][r];
        } else {
            FG_LDS float *ex = (FG_LDS float *)smem;
            auto at = [&](int from, int i, int j, int r) { return (((from * NW + wave) * TI * TJ + i * TJ + j) * 16 + r) * 64 + lane; };
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int j = 0; j < TJ; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) ex[at(group, i, j, r)] = acc[i][j][r];
            publish();
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int j = 0; j < TJ; ++j)
#pragma unroll
                    for (int r = 0; r < RR; ++r) {
                        float v = ex[at(0, i, j, r0 + r)];
#pragma unroll
                        for (int g = 1; g < KG; ++g) v += ex[at(g, i, j, r0 + r)];
                        y[i][j][r] = v;
                    }
        }
        if constexpr (!RANGES) {
            break;
        } else {
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int j = 0; j < TJ; ++j)
#pragma unroll
                    for (int r = 0; r < RR; ++r) total[i][j][r] += y[i][j][r];
            if (++split == p.splits) break;
            kt0 += p.split_kt;
            kt1 = kt0 + p.split_kt < nk_all ? kt0 + p.split_kt : nk_all;
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int j = 0; j < TJ; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
            publish();                                  // the exchange has been read: the next range may overwrite it
        }
    }
    if constexpr (RANGES) {
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j)
#pragma unroll
                for (int r = 0; r < RR; ++r) y[i][j][r] = total[i][j][r];
    }

    // ---- lane l, register r of block (i, j) holds row l % 32, column 8 (r/4) + 4 (l/32) + r % 4 ----
    const int r0 = group * RR, lm = lane & 31, lh = lane >> 5;
    const int mb = m0 + wm * WTM + lm, nb = n0 + wn * WTN + 4 * lh;
    auto col_of = [&](int r) { return 8 * ((r0 + r) >> 2) + ((r0 + r) & 3); };      // RR is a multiple of 4: uniform part + constant
    if (!RANGES && p.splits > 1) {
        // raw partial tile into workspace slot `item`, tile-local coordinates
        float *w = p.D + (int64_t)item * (BM * BN) + (wm * WTM + lm) + (wn * WTN + 4 * lh) * BM;
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j)
#pragma unroll
                for (int r = 0; r < RR; ++r) w[32 * i + (32 * j + col_of(r)) * BM] = y[i][j][r];
        return;
    }
    const float floor_v = p.act == 1 ? 0.f : -__builtin_inff(), floor_c = p.c_act == 1 ? 0.f : -__builtin_inff();
    const bool pass_v = p.act != 1, pass_c = p.c_act != 1;
    if constexpr (PLAIN) {
        const bool bias_m_on = p.bias && p.bias_dim == 0, bias_n_on = p.bias && p.bias_dim != 0;
#pragma unroll
        for (int i = 0; i < TI; ++i) {
            const int m = mb + 32 * i;
            if (m >= p.M) continue;
            const float bias_mi = bias_m_on ? p.bias[m] : 0.f;
#pragma unroll
            for (int j = 0; j < TJ; ++j) {
                const int n1 = nb + 32 * j;
                float cv[RR];
                if (p.C) {
                    // every C value is requested before the first result is stored; columns past N read column n1's
                    const float *c = p.C + m + (int64_t)(n1 < p.N ? n1 : 0) * p.ldc;
#pragma unroll
                    for (int r = 0; r < RR; ++r) cv[r] = c[(n1 + col_of(r) < p.N ? col_of(r) : 0) * p.ldc];
                }
                float *d = p.D + m + (int64_t)n1 * p.ldd;
#pragma unroll
                for (int r = 0; r < RR; ++r) {
                    const int n = n1 + col_of(r);
                    if (n >= p.N) continue;
                    const float bias = bias_n_on ? p.bias[n] : bias_mi;
                    float v;
                    if constexpr (RANGES) {
                        v = split_value(y[i][j][r], p.alpha, p.C, p.beta, p.C ? act_clamp(cv[r], floor_c, pass_c) : 0.f, p.bias, bias);
                    } else {
                        v = p.alpha * y[i][j][r] + bias;
                        if (p.C) v += p.beta * act_clamp(cv[r], floor_c, pass_c);
                    }
                    d[col_of(r) * p.ldd] = act_clamp(v, floor_v, pass_v);
                }
            }
        }
    } else {
        // mixed-radix offsets: rows per lane; columns decomposed by the lane that holds column l % 32
        // and fetched from there.  Rows and columns that do not exist have offset -1.
        auto offset_of = [&](const ModeGroup &g, int idx, int extent, int ext0, int hi) -> int64_t {
            return (idx < extent && leading_index(g, idx, hi) < ext0) ? group_offset(g, idx) : -1;
        };
        // read again here rather than kept in scalar registers through the K loop
        const GeneralParams ep = load_param<GeneralParams>(0);
        const int64_t base = group_offset(ep.c_b, batch);
        int64_t row[TI];
#pragma unroll
        for (int i = 0; i < TI; ++i) row[i] = offset_of(ep.c_m, mb + 32 * i, p.M, p.m_ext0, p.m_hi);
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
            const int64_t mine = offset_of(ep.c_n, n0 + wn * WTN + 32 * j + lm, p.N, p.n_ext0, 0);
            const int lo = (int)(uint32_t)mine, hi = (int)(uint32_t)((uint64_t)mine >> 32);
            int64_t col[RR];
#pragma unroll
            for (int r = 0; r < RR; ++r) {
                const int from = (col_of(r) + 4 * lh) * 4;
                const uint32_t l2 = (uint32_t)__builtin_amdgcn_ds_bpermute(from, lo), h2 = (uint32_t)__builtin_amdgcn_ds_bpermute(from, hi);
                col[r] = (int64_t)(((uint64_t)h2 << 32) | l2);
            }
#pragma unroll
            for (int i = 0; i < TI; ++i) {
                float cv[RR];
                if (p.C) {
                    // all are requested before the first store; what does not exist reads element 0
#pragma unroll
                    for (int r = 0; r < RR; ++r) cv[r] = p.C[(col[r] | row[i]) < 0 ? 0 : base + row[i] + col[r]];
                }
#pragma unroll
                for (int r = 0; r < RR; ++r) {
                    if ((col[r] | row[i]) < 0) continue;
                    float v = p.alpha * y[i][j][r];
                    if (p.C) v += p.beta * cv[r];
                    p.D[base + row[i] + col[r]] = v;
                }
            }
        }
    }
}

// One workgroup per work item, in rows of at most 2^22 (a grid dimension holds 2^32 threads).
// ranges: fn computes all K ranges of a tile.
inline hipError_t launch_general(void (*fn)(const GeneralParams), int variant, GeneralParams p, hipStream_t stream, bool ranges = false) {
    if (variant == GENERAL_64x64_ONE && p.K > 64) return hipErrorInvalidValue;
    const int64_t items = (int64_t)p.tiles_m * p.tiles_n * (ranges ? 1 : p.splits) * p.batches;
    const unsigned per_row = (unsigned)(items < (1 << 22) ? items : (1 << 22));
    p.items = (int32_t)items;
    hipLaunchKernelGGL(fn, dim3(per_row, (unsigned)((items + per_row - 1) / per_row)), dim3(variant == GENERAL_64x64_ONE ? 256 : 512), 0, stream, p);
    return hipGetLastError();
}

typedef void (*GeneralFn)(const GeneralParams);
template <int BM, int BN, int WGM, int WGN, int KG, bool BF16, bool PLAIN, bool RANGES = false>
GeneralFn general_fn(bool a_kc, bool b_kc) {
    return a_kc ? (b_kc ? general_kernel<BM, BN, WGM, WGN, KG, true, true, BF16, PLAIN, RANGES> : general_kernel<BM, BN, WGM, WGN, KG, true, false, BF16, PLAIN, RANGES>)
                : (b_kc ? general_kernel<BM, BN, WGM, WGN, KG, false, true, BF16, PLAIN, RANGES> : general_kernel<BM, BN, WGM, WGN, KG, false, false, BF16, PLAIN, RANGES>);
}

}  // namespace fg
