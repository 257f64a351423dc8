// K loop of the matrix kernels with one wave per SIMD (TileCfg::WIDE), included by gemm_kernel.hpp.
//
// Four waves share a block tile, each with a quarter of it: a 256x256 tile is 128x128 results per wave, whose accumulators
// are all 256 accumulation registers.  Per matrix instruction that is two thirds of the fragment reads of eight waves
// with 128x64 each (16 KB instead of 24 per 64 instructions), and every other instruction of a K tile is needed half as often.
// The price: no second wave covers what a wave waits for, so the loop is written as one straight line of slots, a
// matrix instruction each (16 cycles), with at most a fragment read and a direct load beside it:
//   * what a K tile costs besides is kept to 58 scalar (16 write m0, 18 copy a descriptor's words) and up to 9 vector instructions per
//     wave and 128 matrix instructions (the loaders of the other kernels take 62 and 34 per 64): descriptors are advanced in place, m0 is written by one addition with the
//     matrix instruction as the wait between it and its use, and there is no branch but one per K tile.  A taken branch, or the
//     twenty scalar instructions of a descriptor computed in one go, stall the matrix unit (8192^3 on zeros, a branch
//     around the masking of a last K tile in every K tile: 704 us, without it 660);
//   * a last K tile that hangs over the end of K is multiplied first, its loads masked outside the loop;
//   * direct loads are spread evenly over the K tile (sixteen in a row: 782 us, every second slot 736, every third 706);
//   * A has a ring of one buffer more than B where that is what fits (256x256: three and two, all 160 KB): A's tile
//     kt + 2 is requested in the first half of K tile kt and B's in the second, so that requests go out all the time
//     and have between 1.0 and 1.9 K tiles to land (rings of two: 660 us, this one 552).
// Together, 8192^3 with C on random operands: 893 -> 806 us (TN), 902 -> 815 (NN), 911 -> 814 (NT), 898 -> 815 (TT), against eight
// waves with two buffers; 4096^3 with three operand sets in turn 134 -> 122 (with the planner's other changes 117).
#pragma once

namespace fg {

template <int N> using ic = std::integral_constant<int, N>;

// compile-time loop: f(ic<0>{}) .. f(ic<N - 1>{})
template <class F, int... I>
__device__ __forceinline__ void static_for_seq(F &&f, std::integer_sequence<int, I...>) { (f(ic<I>{}), ...); }
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f) { static_for_seq(f, std::make_integer_sequence<int, N>{}); }

// ---- accumulators ---------------------------------------------------------------------------------
// The accumulators live in accumulation registers that are named in the assembly and known to nobody else: as variables the
// compiler copied them about between the K tiles and spilled (564 registers).  Fragment (i, j) of set s holds registers
// 4 ((s FI + i) FJ + j) .. + 3.  own_acc() marks all of them as written, so that the compiler keeps nothing of its
// own in one across it.  That leaves what lives between two of them; that nothing but this assembly touches an accumulation register is
// checked in the compiled kernels (tests/test_compiled_kernels.py).
#define FG_ACC10(d) "a" #d "0", "a" #d "1", "a" #d "2", "a" #d "3", "a" #d "4", "a" #d "5", "a" #d "6", "a" #d "7", "a" #d "8", "a" #d "9"
#define FG_ACC_ALL                                                                                                                      \
    "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", FG_ACC10(1), FG_ACC10(2), FG_ACC10(3), FG_ACC10(4), FG_ACC10(5),        \
    FG_ACC10(6), FG_ACC10(7), FG_ACC10(8), FG_ACC10(9), FG_ACC10(10), FG_ACC10(11), FG_ACC10(12), FG_ACC10(13), FG_ACC10(14),           \
    FG_ACC10(15), FG_ACC10(16), FG_ACC10(17), FG_ACC10(18), FG_ACC10(19), FG_ACC10(20), FG_ACC10(21), FG_ACC10(22), FG_ACC10(23),       \
    FG_ACC10(24), "a250", "a251", "a252", "a253", "a254", "a255"
__device__ __forceinline__ void own_acc() { asm volatile("" ::: FG_ACC_ALL); }
// Registers R .. R + 3.  The two wait states are those that a lane exchange of the results needs; the compiler, which does not
// see vector instructions in the assembly, would not add them.
template <int R>
__device__ __forceinline__ floatx4 acc_get() {
    float x0, x1, x2, x3;
    asm volatile("v_accvgpr_read_b32 %0, a[%4]\n\tv_accvgpr_read_b32 %1, a[%5]\n\tv_accvgpr_read_b32 %2, a[%6]\n\tv_accvgpr_read_b32 %3, a[%7]\n\ts_nop 1"
                 : "=v"(x0), "=v"(x1), "=v"(x2), "=v"(x3) : "n"(R), "n"(R + 1), "n"(R + 2), "n"(R + 3));
    return floatx4{x0, x1, x2, x3};
}
template <int R>
__device__ __forceinline__ void acc_zero() { asm volatile("v_accvgpr_write_b32 a[%0], 0" ::"n"(R)); }
// accumulator R .. R + 3 += a . b
template <bool BF16, int R>
__device__ __forceinline__ void mfma_acc(half8 a, half8 b) {
    if constexpr (BF16) asm volatile("v_mfma_f32_16x16x32_bf16 a[%0:%1], %2, %3, a[%0:%1]" ::"n"(R), "n"(R + 3), "v"(a), "v"(b));
    else asm volatile("v_mfma_f32_16x16x32_f16 a[%0:%1], %2, %3, a[%0:%1]" ::"n"(R), "n"(R + 3), "v"(a), "v"(b));
}
// the same, and a direct load to LDS address lds + OFF: the matrix instruction stands between the write of m0 and its use
// (STREAM: the load carries the streaming policy)
#define FG_MFMA_LOAD(TYPE, POLICY)                                                                                                      \
    asm volatile("s_add_u32 m0, %6, %7\n\tv_mfma_f32_16x16x32_" TYPE " a[%0:%1], %2, %3, a[%0:%1]\n\tbuffer_load_dwordx4 %4, %5, 0 offen" POLICY " lds" \
                 ::"n"(R), "n"(R + 3), "v"(a), "v"(b), "v"(voff), "s"(rsrc), "s"(lds), "n"(OFF) : "memory", "m0", "scc")
template <bool BF16, bool STREAM, int R, int OFF>
__device__ __forceinline__ void mfma_acc_load(half8 a, half8 b, u32x4 rsrc, uint32_t lds, uint32_t voff) {
    if constexpr (BF16 && STREAM) FG_MFMA_LOAD("bf16", " nt");
    else if constexpr (BF16) FG_MFMA_LOAD("bf16", "");
    else if constexpr (STREAM) FG_MFMA_LOAD("f16", " nt");
    else FG_MFMA_LOAD("f16", "");
}
#undef FG_MFMA_LOAD

// ---- loader -----------------------------------------------------------------------------------------
// One operand of a plain matrix, R rows x 64 k per K tile, in the LDS layout of TileLoader (16-row fragments); a wave
// fetches SLABS pieces of 1 KB.  The descriptor is advanced in place.  Its size, the bytes from the current K tile
// to the end of the operand, is counted in 64 bits (negative past the end).
template <int R, bool KC>
struct WideLoader {
    static constexpr int SLABS = R / 32;
    uint32_t voff[SLABS];
    u32x4 rsrc;
    uint32_t step, rest_lo;        // bytes per K tile; from the current K tile to the end of the operand
    int32_t rest_hi;
    uint32_t turn_lo, turn_hi;     // from the last K tile of a range walked in a circle to the first: (1 - its length) steps

    // K tile kt is the next one; more: there is such a tile to load (circle: length of the range, see GemmParams::rotate)
    __device__ __forceinline__ void at(const _Float16 *ptr, int row0, int64_t rs, int64_t ks, int64_t span, int kt, bool more, int circle) {
        const int64_t first = (int64_t)row0 * rs + 64 * ks * kt, rest = (span - first) * 2;
        step = (uint32_t)(128 * ks);
        point(ptr + first, rest, more);
        const int64_t turn = -(int64_t)(circle - 1) * step;
        turn_lo = (uint32_t)turn;
        turn_hi = (uint32_t)(turn >> 32);
    }
    __device__ __forceinline__ void point(const void *p, int64_t rest, bool more) {
        rest_lo = (uint32_t)rest;
        rest_hi = (int32_t)(rest >> 32);
        rsrc = make_rsrc(p, more ? window_bytes(rest) : 0u);
    }
    // the loader `tiles` K tiles further on (back, if negative), for one K tile
    __device__ __forceinline__ WideLoader moved(int tiles) const {
        WideLoader o = *this;
        const int64_t by = (int64_t)tiles * (int64_t)step;
        o.point((const char *)(((uint64_t)rsrc[1] << 32) | rsrc[0]) + by, (int64_t)(((uint64_t)(uint32_t)rest_hi << 32) | rest_lo) - by, true);
        return o;
    }
    // Which bits of a slab's chunk index differ from slab 0's: the swizzles are XORs of bits of the LDS row, and a wave's slabs begin at
    // a multiple of 16 rows.  So a lane's offset in slab s is that of slab 0 with these bits flipped, plus as many rows.
    static constexpr int SLAB_ROWS = KC ? 8 : 512 / R;
    static constexpr int flips(int s) {
        const int row = s * SLAB_ROWS;
        return KC ? (row / 2) & 7 : ((R == 64 ? (row >> 1) & 1 : row & 3) << 2) ^ (((row >> 3) & 1) << 1);
    }
    static_assert(SLABS * SLAB_ROWS % 16 == 0, "");
    __device__ __forceinline__ void init(int wave, int lane, int64_t rs, int64_t ks) {
        const uint32_t pitch = (uint32_t)(KC ? rs : ks) * 2u;             // bytes from one LDS row's source to the next
        constexpr int CH = KC ? 8 : R / 8;
        const int row = lane / CH;                                        // of the first slab's
        const int c = KC ? (lane & 7) ^ (lane >> 4) : (lane % CH) ^ (mc_swz<R>(row) << 2) ^ (((row >> 3) & 1) << 1);
        const uint32_t first = (uint32_t)(wave * (SLABS * SLAB_ROWS) + row) * pitch;
#pragma unroll
        for (int s = 0; s < SLABS; ++s) voff[s] = first + (uint32_t)((c ^ flips(s)) * 16) + (uint32_t)(s * SLAB_ROWS) * pitch;
    }
    // KC: which chunk of eight k of its row a lane fetches
    __device__ __forceinline__ int chunk(int s, int lane) const { return (lane & 7) ^ (lane >> 4) ^ flips(s); }
    // On to the next K tile, from the end of the range to its start if left == turn (ROTATE).  more: how many K tiles are still to be
    // requested; without one the loads fetch nothing.  No lane is masked here, so the size may be larger than that of
    // window_bytes.  Written out: the compiler would do it on the vector unit and move the descriptor there.
    template <bool ROTATE>
    __device__ __forceinline__ void next_base(int left, int turn) {
        uint32_t lo = rsrc[0], hi = rsrc[1];
        if constexpr (ROTATE) {
            uint32_t by_lo, by_hi;
            asm volatile("s_cmp_eq_u32 %6, %7\n\ts_cselect_b32 %2, %8, %10\n\ts_cselect_b32 %3, %9, 0\n\t"
                         "s_add_u32 %0, %0, %2\n\ts_addc_u32 %1, %1, %3\n\ts_sub_u32 %4, %4, %2\n\ts_subb_u32 %5, %5, %3"
                         : "+s"(lo), "+s"(hi), "=&s"(by_lo), "=&s"(by_hi), "+s"(rest_lo), "+s"(rest_hi)
                         : "s"(left), "s"(turn), "s"(turn_lo), "s"(turn_hi), "s"(step) : "scc");
        } else {
            asm volatile("s_add_u32 %0, %0, %4\n\ts_addc_u32 %1, %1, 0\n\ts_sub_u32 %2, %2, %4\n\ts_subb_u32 %3, %3, 0"
                         : "+s"(lo), "+s"(hi), "+s"(rest_lo), "+s"(rest_hi) : "s"(step) : "scc");
        }
        rsrc[0] = lo;
        rsrc[1] = hi;
    }
    __device__ __forceinline__ void next_size(int more) {
        uint32_t n;
        asm volatile("s_cmp_gt_i32 %1, 0\n\ts_cselect_b32 %0, -16, %2\n\ts_cmp_lt_i32 %1, 0\n\ts_cselect_b32 %0, 0, %0\n\t"
                     "s_cmp_gt_i32 %3, 0\n\ts_cselect_b32 %0, %0, 0"
                     : "=&s"(n) : "s"(rest_hi), "s"(rest_lo), "s"(more) : "scc");
        rsrc[2] = n;
    }
    // All of a K tile at once.  klim < 64: only the first klim k exist (M/N-contiguous: what lies beyond K lies beyond the operand).
    template <bool STREAM>
    __device__ __forceinline__ void issue(uint32_t lds) const {
#pragma unroll
        for (int s = 0; s < SLABS; ++s) load16_to_lds<STREAM>(rsrc, lds + s * 1024u, voff[s]);
    }
    __device__ __forceinline__ void issue(uint32_t lds, bool stream) const {
        if (stream) issue<true>(lds);
        else issue<false>(lds);
    }
    __device__ __forceinline__ void issue_part(uint32_t lds, int klim, int lane) const {
#pragma unroll
        for (int s = 0; s < SLABS; ++s) load16_to_lds(rsrc, lds + s * 1024u, KC && chunk(s, lane) * 8 >= klim ? kOutOfRange : voff[s]);
    }
};

// ---- the loop ---------------------------------------------------------------------------------------
// K tile kt lies in A's buffer kt % RA and B's buffer kt % RB.  It is two slices of 32 k, FI x FJ slots each:
//   first slice:  fragments of the second slice are read; A's tile kt + RA - 1 is requested (its buffer was retired by the
//                 barrier of tile kt - 1);
//   second slice: after the barrier at slot BAR, which publishes tile kt + 1 and retires tile kt, the first
//                 fragments of tile kt + 1 are read, and B's tile kt + RB is requested.
// ONCE: GemmParams::once.  turn: where in its range of K the walk began (GemmParams::rotate).
template <class Cfg, int ONCE, class LA, class LB, class FA, class FB>
__device__ __forceinline__ void k_loop_wide(LA &la, LB &lb, const FA &fa, const FB &fb, FG_LDS char *lds_a, FG_LDS char *lds_b, int wave, int nkt,
                                            [[maybe_unused]] int turn) {
    constexpr int TI = Cfg::FI, TJ = Cfg::FJ, SLOTS = TI * TJ, NR = TI + TJ, RA = Cfg::RING_A, RB = Cfg::STAGES;
    constexpr int NA = LA::SLABS, NB = LB::SLABS, SET2 = Cfg::ACC_SETS == 2 ? 4 * SLOTS : 0;
    // where the reads and loads of a slice stand (every third slot a read, with 64 of them)
    constexpr int BAR = SLOTS / 8, LOAD_A = SLOTS * 7 / 8 / NA, LOAD_B = SLOTS * 5 / 8 / NB;
    constexpr auto read_at = [](int n, int first) { return first + n * (SLOTS * 3 / 4) / NR; };
    constexpr int READ_1 = BAR + 2, NEXT_A = 2 + (NA - 1) * LOAD_A, SIZE_A = NEXT_A + 1;
    // Loads still in flight when tile kt + 1 must have landed: those requested after the younger of A's and B's tile kt + 1.
    constexpr int YOUNGER = RA == RB ? (RA - 2) * (NA + NB) : (RB - 1) * NA + (RB - 2) * NB;
    static_assert((RA == RB || RA == RB + 1) && RB >= 2 && YOUNGER <= 63 && LOAD_A >= 1 && LOAD_B >= 1, "");
    half8 a[2][TI], b[2][TJ];
    // read n of a slice: what the first row of slots needs comes first
    auto read = [&](auto set_tag, FG_LDS const char *ta, FG_LDS const char *tb, int ks, int n) {
        constexpr int set = set_tag;
        if (n == 0) a[set][0] = fa.read(ta, 0, ks);
        else if (n <= TJ) b[set][n - 1] = fb.read(tb, n - 1, ks);
        else a[set][n - TJ] = fa.read(ta, n - TJ, ks);
    };
    const uint32_t to_a = (uint32_t)(uintptr_t)lds_a + (uint32_t)wave * (NA * 1024u), to_b = (uint32_t)(uintptr_t)lds_b + (uint32_t)wave * (NB * 1024u);
#pragma unroll
    for (int n = 0; n < NR; ++n) read(ic<0>{}, lds_a, lds_b, 0, n);
    int left = nkt;
    auto body = [&](auto a_tag, auto b_tag) {
        constexpr int ca = a_tag, cb = b_tag;
        FG_LDS const char *ta = lds_a + ca * Cfg::A_TILE_BYTES, *tb = lds_b + cb * Cfg::B_TILE_BYTES;
        FG_LDS const char *na = lds_a + (ca + 1) % RA * Cfg::A_TILE_BYTES, *nb = lds_b + (cb + 1) % RB * Cfg::B_TILE_BYTES;
        own_acc();
        __builtin_amdgcn_sched_barrier(0);
        static_for<SLOTS>([&](auto s_tag) {
            constexpr int s = s_tag, i = s / TJ, j = s % TJ, l = (s - 1) / LOAD_A;
            if constexpr (s >= 1 && (s - 1) % LOAD_A == 0 && l < NA)
                mfma_acc_load<Cfg::BF16, ONCE == 2, 4 * s, (ca + RA - 1) % RA * Cfg::A_TILE_BYTES + l * 1024>(b[0][j], a[0][i], la.rsrc, to_a, la.voff[l]);
            else
                mfma_acc<Cfg::BF16, 4 * s>(b[0][j], a[0][i]);
            if constexpr (s == NEXT_A) la.template next_base<Cfg::ROTATE>(left, turn + RA);
            if constexpr (s == SIZE_A) la.next_size(left - RA);
#pragma unroll
            for (int n = 0; n < NR; ++n)
                if (s == read_at(n, 0)) read(ic<1>{}, ta, tb, 1, n);
            __builtin_amdgcn_sched_barrier(0);
        });
        static_for<SLOTS>([&](auto s_tag) {
            constexpr int s = s_tag, i = s / TJ, j = s % TJ, l = (s - BAR) / LOAD_B;
            if constexpr (s == BAR) {
                wait_tile<YOUNGER>();
                __builtin_amdgcn_s_barrier();
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (s >= BAR && (s - BAR) % LOAD_B == 0 && l < NB)
                mfma_acc_load<Cfg::BF16, ONCE == 1, 4 * s + SET2, cb * Cfg::B_TILE_BYTES + l * 1024>(b[1][j], a[1][i], lb.rsrc, to_b, lb.voff[l]);
            else
                mfma_acc<Cfg::BF16, 4 * s + SET2>(b[1][j], a[1][i]);
            if constexpr (s == BAR + 1 + (NB - 1) * LOAD_B) lb.template next_base<Cfg::ROTATE>(left, turn + RB + 1);
            if constexpr (s == BAR + 2 + (NB - 1) * LOAD_B) lb.next_size(left - RB - 1);
#pragma unroll
            for (int n = 0; n < NR; ++n)
                if (s == read_at(n, READ_1)) read(ic<0>{}, na, nb, 0, n);
            __builtin_amdgcn_sched_barrier(0);
        });
        return --left == 0;
    };
    static_assert(BAR + 2 + (NB - 1) * LOAD_B < SLOTS && SIZE_A < SLOTS && read_at(NR - 1, READ_1) < SLOTS, "");
    // unrolled over both rings
    if constexpr (RA == 3 && RB == 2) {
        for (;;) {
            if (body(ic<0>{}, ic<0>{})) break;
            if (body(ic<1>{}, ic<1>{})) break;
            if (body(ic<2>{}, ic<0>{})) break;
            if (body(ic<0>{}, ic<1>{})) break;
            if (body(ic<1>{}, ic<0>{})) break;
            if (body(ic<2>{}, ic<1>{})) break;
        }
    } else if constexpr (RA == 3 && RB == 3) {
        for (;;) {
            if (body(ic<0>{}, ic<0>{})) break;
            if (body(ic<1>{}, ic<1>{})) break;
            if (body(ic<2>{}, ic<2>{})) break;
        }
    } else {
        static_assert(RA == 4 && RB == 4, "");
        for (;;) {
            if (body(ic<0>{}, ic<0>{})) break;
            if (body(ic<1>{}, ic<1>{})) break;
            if (body(ic<2>{}, ic<2>{})) break;
            if (body(ic<3>{}, ic<3>{})) break;
        }
    }
    // the last matrix instructions write their results this long after they were issued; no load stays behind
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(0)\n\ts_nop 15\n\ts_nop 15" ::: "memory");
    own_acc();
    __builtin_amdgcn_sched_barrier(0);
}

// ---- epilogue ----------------------------------------------------------------------------------------
// Result (i, j) of a wave, both sets added up.
template <class Cfg, int i, int j>
__device__ __forceinline__ floatx4 acc_sum() {
    constexpr int R = (i * Cfg::FJ + j) * 4;
    if constexpr (Cfg::ACC_SETS == 2) return acc_get<R>() + acc_get<R + 4 * Cfg::FI * Cfg::FJ>();
    else return acc_get<R>();
}
// The 32x32 block (i, j) of a wave's results in the layout of TileCfg::acc_col / ACC_LH (see gather_block).
template <class Cfg, int i, int j>
__device__ __forceinline__ floatx16 gather_wide() {
    floatx16 out;
    static_for<2>([&](auto nj) {
        const floatx4 x = acc_sum<Cfg, 2 * i, 2 * j + nj>(), y = acc_sum<Cfg, 2 * i + 1, 2 * j + nj>();
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const auto s = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, (float)x[r]), __builtin_bit_cast(unsigned, (float)y[r]), false, false);
            const unsigned s0 = s[0], s1 = s[1];
            out[8 * nj + r] = __builtin_bit_cast(float, s0);
            out[8 * nj + 4 + r] = __builtin_bit_cast(float, s1);
        }
    });
    return out;
}

// epilogue() for these kernels: the same arithmetic and the same batches of sixteen values with C requested two batches ahead,
// for inner and edge tiles alike (with the accumulators out of the way there are registers enough for the masks).
// Binary16 C and D of inner tiles: two accumulators at a time, exchanged into whole lines (see epilogue).
template <class Cfg, bool HAS_C, bool CACHED>
__device__ __forceinline__ void epilogue_wide(const GemmParams &p, int m_base, int n_base, int lane) {
    constexpr int kPolicy = CACHED ? 0 : stream_policy<Cfg>();
    constexpr bool H = Cfg::CD16;
    constexpr int ES = H ? 2 : 4, NB = Cfg::TI * Cfg::TJ, AHEAD = CACHED ? 2 : 3;
    own_acc();
    const int lm = lane & 31, lh = lane >> 5;
    const bool bias_m_on = p.bias && p.bias_dim == 0, bias_n_on = p.bias && p.bias_dim != 0;
    // The larger of a value and the floor: the instruction gives the other operand for a NaN, so that 0 makes it the ReLU of act_clamp (a NaN
    // becomes 0) and NaN lets everything through.  One instruction in place of three.  Not as assembly: the compiler would not know it for a
    // vector instruction and leave out the two wait states that a lane exchange of its result needs.
    const float floor_v = p.act == 1 ? 0.f : __builtin_nanf("");
    auto act = [](float v, float floor) { return __builtin_fmaxf(v, floor); };
    const int ldc_b = (int)p.ldc * ES, ldd_b = (int)p.ldd * ES;
    const char *Cb = (const char *)p.C, *Db = (const char *)p.D;
    __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char *>(HAS_C ? Cb + (m_base + (int64_t)n_base * p.ldc) * ES : Db), 0, 0x7fffffff, 0x00020000);
    __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(Db + (m_base + (int64_t)n_base * p.ldd) * ES), 0, 0x7fffffff, 0x00020000);
    const int m_left = p.M - m_base - lm, n_last = p.N - 1 - n_base - Cfg::ACC_LH * lh;       // rows left from this lane's first on, last column
    float bias_m[Cfg::TI];
#pragma unroll
    for (int i = 0; i < Cfg::TI; ++i) bias_m[i] = bias_m_on && 32 * i < m_left ? p.bias[m_base + 32 * i + lm] : 0.f;
    auto run = [&](auto edge_tag) {
        constexpr bool EDGE = decltype(edge_tag)::value, PAIR = H && !EDGE;
        // value e of batch b: block (i, j), register r.  PAIR: registers 8 (jj & 1) .. + 7 of blocks (2 ip, j) and (2 ip + 1, j) in turn
        // Order of the batches: down the rows of a block column where C and D are cached (the scalar offsets of the columns serve all of
        // them; 4096^3 with C 115.1 us, 118.7 along the rows), along them where they stream (8192^3 787.5, 795.8).
        constexpr int I = PAIR ? Cfg::TI / 2 : Cfg::TI;
        // batch b is block row ii, block column (PAIR: half) jj
        constexpr int J = NB / I;
        constexpr auto ii = [](int b) { return CACHED ? b % I : b / J; };
        constexpr auto jj = [](int b) { return CACHED ? b / I : b % J; };
        constexpr auto col_of = [=](int b, int e) { return PAIR ? 32 * (jj(b) / 2) + Cfg::acc_col(8 * (jj(b) & 1) + e / 2) + (e & 1) * Cfg::ACC_LH
                                                              : 32 * jj(b) + Cfg::acc_col(e); };
        constexpr auto row_of = [=](int b) { return (PAIR ? 64 : 32) * ii(b); };
        const uint32_t voff_c = (uint32_t)(PAIR ? lane * ES : (lm + Cfg::ACC_LH * lh * (int)p.ldc) * ES);
        const uint32_t voff_d = (uint32_t)(PAIR ? lane * ES : (lm + Cfg::ACC_LH * lh * (int)p.ldd) * ES);
        // where value e of batch b is: out of range if its row or column does not exist (the sign of a difference, merged
        // into the offset: as compare results the masks of all columns would be kept and spilled)
        auto place = [&](uint32_t voff, int b, int e) -> uint32_t {
            if constexpr (!EDGE) return voff;
            const uint32_t v = row_of(b) < m_left ? voff : kOutOfRange;
            return v | ((uint32_t)(n_last - col_of(b, e)) & kOutOfRange);
        };
        auto exchange = [](float &x, float &y) {            // upper half of x <-> lower half of y
            const auto s = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, y), false, false);
            const unsigned s0 = s[0], s1 = s[1];
            x = __builtin_bit_cast(float, s0);
            y = __builtin_bit_cast(float, s1);
        };
        float cv[AHEAD + 1][16];
        auto load_c = [&](int b) {
            if constexpr (HAS_C) {
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    cv[b % (AHEAD + 1)][e] = load_cd<H, kPolicy>(rc, place(voff_c, b, e) + row_of(b) * ES, col_of(b, e) * ldc_b);
            }
        };
#pragma unroll
        for (int b = 0; b < AHEAD && b < NB; ++b) load_c(b);
        static_for<NB>([&](auto b_tag) {
            constexpr int b = b_tag;
            if constexpr (b + AHEAD < NB) load_c(b + AHEAD);
            constexpr int j = PAIR ? jj(b) / 2 : jj(b);
            float bn[PAIR ? 8 : 16];
            constexpr int R = PAIR ? 8 : 16, r0 = PAIR ? 8 * (jj(b) & 1) : 0;
            if (bias_n_on) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int col = 32 * j + Cfg::acc_col(r0 + r);
                    bn[r] = p.bias[n_base + Cfg::ACC_LH * lh + (EDGE && col > n_last ? (n_last < 0 ? -(n_base + Cfg::ACC_LH * lh) : n_last) : col)];
                }
            }
            // The activation of C is a comparison: a loaded value can be a signalling NaN, and the larger of that and 0 is a NaN.
            if constexpr (HAS_C) {
                if (p.c_act == 1) {
#pragma unroll
                    for (int e = 0; e < 16; ++e) cv[b % (AHEAD + 1)][e] = cv[b % (AHEAD + 1)][e] > 0.f ? cv[b % (AHEAD + 1)][e] : 0.f;
                }
            }
            float y[16];
            if constexpr (PAIR) {
                constexpr int ip = ii(b);
                const floatx16 acc0 = gather_wide<Cfg, 2 * ip, j>(), acc1 = gather_wide<Cfg, 2 * ip + 1, j>();
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    float v0 = p.alpha * acc0[r0 + r] + (bias_n_on ? bn[r] : bias_m[2 * ip]);
                    float v1 = p.alpha * acc1[r0 + r] + (bias_n_on ? bn[r] : bias_m[2 * ip + 1]);
                    if constexpr (HAS_C) {
                        float c0 = cv[b % (AHEAD + 1)][2 * r], c1 = cv[b % (AHEAD + 1)][2 * r + 1];
                        exchange(c0, c1);
                        v0 += p.beta * c0;
                        v1 += p.beta * c1;
                    }
                    v0 = act(v0, floor_v);
                    v1 = act(v1, floor_v);
                    exchange(v0, v1);
                    y[2 * r] = v0;
                    y[2 * r + 1] = v1;
                }
            } else {
                constexpr int i = ii(b);
                const floatx16 acc = gather_wide<Cfg, i, j>();
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    float v = p.alpha * acc[r] + (bias_n_on ? bn[r] : bias_m[i]);
                    if constexpr (HAS_C) v += p.beta * cv[b % (AHEAD + 1)][r];
                    y[r] = act(v, floor_v);
                }
            }
#pragma unroll
            for (int e = 0; e < 16; ++e)
                store_cd<H, kPolicy>(y[e], rd, place(voff_d, b, e) + row_of(b) * ES, col_of(b, e) * ldd_b);
            __builtin_amdgcn_sched_barrier(0);
            own_acc();
        });
    };
    if (m_base + Cfg::WTM <= p.M && n_base + Cfg::WTN <= p.N) run(std::false_type{});
    else run(std::true_type{});
}

}  // namespace fg
