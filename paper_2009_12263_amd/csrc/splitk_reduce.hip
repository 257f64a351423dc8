// Second pass of a split-K product: D = act(alpha * sum_s W_s + beta * c_act(C) + bias) on the
// tiles tile_begin .. tile_begin + tile_count - 1, where slot s * tile_count + t of the workspace
// holds the raw BM x BN partial product (column-major, leading dimension BM) that K range s
// contributed to tile tile_begin + t.  The paper names this use of the epilogue (a reduction
// across workgroups) in Section 4.2.5.  The partials are added in ascending s, so the result does
// not depend on how the first pass was scheduled.
#include "kernel_table.hpp"

namespace fg {
namespace {

// One thread per 4 consecutive rows of one column of one tile: 16-byte reads of the partials,
// lanes along M.  Bound by the latency of those reads: up to eight are requested before the first
// is added (the additions stay in ascending order of s).
// VEC: C and D in 16-byte accesses (the host has checked pointers and leading dimensions).
constexpr int kAhead = 8;
template <bool VEC>
__global__ __launch_bounds__(256) void splitk_reduce(const float *W, int splits, int tile_begin, int tile_count, int bm, int bn,
                                                     int tiles_m, int tiles_n, int M, int N, float alpha, float beta,
                                                     const float *C, int64_t ldc, float *D, int64_t ldd, const float *bias,
                                                     int bias_dim, int act, int c_act) {
#pragma clang fp contract(off)                  // the operations of split_value, one by one
    const int per_tile = (bm / 4) * bn;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)per_tile * tile_count) return;
    const int t = (int)(idx / per_tile);
    const int e = (int)(idx - (int64_t)t * per_tile);
    const int col = e / (bm / 4), row = (e - col * (bm / 4)) * 4;
    int tm, tn;
    block_to_tile(tile_begin + t, tiles_m, tiles_n, tm, tn);
    const int m = tm * bm + row, n = tn * bn + col;
    if (m >= M || n >= N) return;
    const int valid = M - m < 4 ? M - m : 4;
    const int64_t slot_elems = (int64_t)bm * bn;
    const float *w = W + (int64_t)t * slot_elems + row + (int64_t)col * bm;
    float cv[4] = {0.f, 0.f, 0.f, 0.f};
    const bool whole = VEC && valid == 4;
    if (C) {
        const float *c = C + m + (int64_t)n * ldc;
        if (whole) { const float4 v = *(const float4 *)c; cv[0] = v.x; cv[1] = v.y; cv[2] = v.z; cv[3] = v.w; }
        else for (int q = 0; q < valid; ++q) cv[q] = c[q];
    }
    float sum[4] = {0.f, 0.f, 0.f, 0.f};
    const int64_t step = (int64_t)tile_count * slot_elems;
    for (int s0 = 0; s0 < splits; s0 += kAhead) {
        float4 v[kAhead];
#pragma unroll
        for (int s = 0; s < kAhead; ++s)            // slots past the last one read it again and are not added
            v[s] = *(const float4 *)(w + (int64_t)(s0 + s < splits ? s0 + s : splits - 1) * step);   // 16-byte aligned: bm % 4 == 0
#pragma unroll
        for (int s = 0; s < kAhead; ++s)
            if (s0 + s < splits) { sum[0] += v[s].x; sum[1] += v[s].y; sum[2] += v[s].z; sum[3] += v[s].w; }
    }
    const float floor_v = act == 1 ? 0.f : -__builtin_inff();
    const float floor_c = c_act == 1 ? 0.f : -__builtin_inff();
    const bool act_none = act != 1, c_act_none = c_act != 1;
    float y[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        y[q] = alpha * sum[q];
        if (C) y[q] = __builtin_fmaf(beta, act_clamp(cv[q], floor_c, c_act_none), y[q]);
        if (bias) y[q] += bias[bias_dim == 0 ? (q < valid ? m + q : m) : n];
        y[q] = act_clamp(y[q], floor_v, act_none);
    }
    float *d = D + m + (int64_t)n * ldd;
    if (whole) *(float4 *)d = make_float4(y[0], y[1], y[2], y[3]);
    else
        for (int q = 0; q < 4; ++q)
            if (q < valid) d[q] = y[q];
}

}  // namespace

hipError_t launch_splitk_reduce(const float *W, int splits, int tile_begin, int tile_count, int bm, int bn, int tiles_m,
                                int tiles_n, int M, int N, float alpha, float beta, const float *C, int64_t ldc, float *D,
                                int64_t ldd, const float *bias, int bias_dim, int act, int c_act, hipStream_t stream) {
    const int64_t work = (int64_t)(bm / 4) * bn * tile_count;
    const unsigned blocks = (unsigned)((work + 255) / 256);
    auto vec = [](const void *p, int64_t ld) { return (uintptr_t)p % 16 == 0 && ld % 4 == 0; };
    hipLaunchKernelGGL((vec(D, ldd) && (!C || vec(C, ldc)) ? splitk_reduce<true> : splitk_reduce<false>), dim3(blocks), dim3(256), 0, stream, W, splits, tile_begin, tile_count, bm, bn, tiles_m,
                       tiles_n, M, N, alpha, beta, C, ldc, D, ldd, bias, bias_dim, act, c_act);
    return hipGetLastError();
}

}  // namespace fg
