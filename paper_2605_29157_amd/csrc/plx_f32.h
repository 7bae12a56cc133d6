// What the fp32 kernels share: generic_f32.hip (fp32 matrix instructions: every call) and prefill_f32.hip (bf16 thirds:
// large prefill launches at d = 64).
#pragma once
#include "plx_device.h"
#include "plx_kernels.h"

namespace plx {

constexpr int kF32Waves = 4, kF32Threads = 64 * kF32Waves;

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

struct F32Forward {
    const float *q, *r, *k, *v;
    float *o;
    const int32_t *seq_lens;
    // columns: index x = 16 * block + c of `heads` groups per sequence -> query row x / gcols of query
    // head group * gcols + x % gcols, which reads key head group * gcols / G
    int32_t B, Hq, G, heads, gcols, n_cols, n_blocks, Tq, Lk, d, S;
    int64_t qs[3], rs[3], ks[3], vs[3], os[3];
    float scale;
    int32_t use_r;
    int32_t tail;  // rows are the last Tq positions: row t sees the keys before len - (Tq - 1 - t)
    int32_t window;
    const int32_t *block_table;
    int32_t page_size, table_stride, num_pages;
    float *ws;                // S > 1: split records [b][hq][t][s] of (2 d + 4) floats
    float *vbar, *row_stats;  // row cache of the backward pass, or NULL
};

// Workgroups of a pass of prefill_f32.hip over n columns (query rows or keys) of B x H heads, and where that pass
// pays: from two workgroups on every one of the 256 compute units on, and over tiles (32 columns, 64 of the other side at a
// time) that are mostly full. fp32 instruction / thirds, us, forward and backward:
//   workgroups, causal: 512 31.0 / 26.6 and 76.4 / 66.8 (4 x 8 heads x 500 rows), 19.0 / 16.9 and 47.3 / 42.2 (8 x 8 x 256);
//     384 26.5 / 24.6 and 63.4 / 62.9; 256 21.9 / 24.4 and 50.5 / 59.4 (a workgroup's chain of tiles is four times as long)
//   16 x 8 heads, causal: 128 rows 13.5 / 12.2 and 32.6 / 29.4, 129 16.6 / 17.3 and 38.6 / 44.2, 176 21.5 / 21.4 and 50.6 /
//     53.8, 192 23.1 / 21.7 and 54.9 / 52.3, 224 28.5 / 24.7 and 68.0 / 61.4, 257 35.9 / 33.7 and 88.5 / 83.9; 16 x 16 heads, 208
//     rows 45.4 / 45.1 and 108 / 117; not causal: 144 rows 23.7 / 24.6 and 56.8 / 61.3, 160 27.4 / 24.4 and 65.5 / 62.3
//   128 rows, more keys: 140 14.8 / 14.9 and 35.8 / 38.0, 200 19.7 / 18.0 and 49.4 / 47.5, 600 51.4 / 38.3 and 137 / 108
//   sliding windows, 4 x 8 heads x 1024 rows: 16 18.1 / 19.9 and 40.6 / 46.9, 64 25.4 / 25.2 and 62.5 / 61.6, 96 28.8 / 25.8 and
//     67.7 / 61.7; 16 x 16 x 300: 64 51.1 / 51.6 and 121 / 124, 128 63.6 / 60.1 and 154 / 150
constexpr int kF32ThirdsD = 64, kF32ThirdsColumns = 32, kF32ThirdsMinBlocks = 512, kF32ThirdsMinRows = 128, kF32ThirdsMinWindow = 96;
inline int64_t f32_thirds_blocks(int n, int B, int H) {
    return (int64_t)((n + kF32ThirdsColumns - 1) / kF32ThirdsColumns) * B * H;
}
inline bool f32_thirds_pay(int d, int rows, int keys, bool causal, int window, int64_t blocks) {
    if (d != kF32ThirdsD || blocks < kF32ThirdsMinBlocks || rows < kF32ThirdsMinRows || keys < kF32ThirdsMinRows) return false;
    if (window > 0 && window < kF32ThirdsMinWindow) return false;
    auto fills = [](int n) { return n >= 224 || n % 64 == 0 || n % 64 >= 56; };
    const int seen = causal ? keys - rows / 2 : keys;  // by a row, on average
    return (keys >= 160 && seen >= 112) || (fills(rows) && fills(keys));
}
hipError_t launch_forward_thirds(const PrefillParams &p, hipStream_t stream);
hipError_t launch_bwd_rows_thirds(const PrefillBwdParams &p, hipStream_t stream);
hipError_t launch_bwd_cols_thirds(const PrefillBwdParams &p, hipStream_t stream);

// A key a column does not see must not reach it, also where the key's row holds infinities or NaN
// (0 * inf). Blocks that some column sees only in part are checked for that ...
template <int DP>
__device__ __forceinline__ bool f32_not_finite(const f32x4 (&a)[4][DP / 64]) {
    float chk = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int m = 0; m < DP / 64; ++m)
#pragma unroll
            for (int i = 0; i < 4; ++i) chk = fmaf(a[r][m][i], 0.f, chk);
    return __any(chk != 0.f);
}
// ... and where a value is not finite it is taken out of the operand (a zero), after what it does to the
// columns that see its key (bit r of `seen`: key 4 g + r) has been added: sums of products of finite
// numbers that overflow where +inf (up) or -inf (down) reaches a column, and both where a NaN does or a
// zero weight meets an infinity. (The common path pays for this one in registers: with the keys added one
// by one in a loop it spilled 150 to 290 of them at d = 256 and up to 35 at d = 128.)
template <int DP, int SETS>
__device__ __forceinline__ void f32_take_out_not_finite(f32x4 (&a)[4][DP / 64], const f32x4 *const (&p)[SETS],
                                                        unsigned seen, f32x4 (*const (&acc)[SETS])[DP / 16]) {
    constexpr float kBig = 3.0e38f, kInf = -kNegInf;
#pragma unroll
    for (int n = 0; n < DP / 16; ++n) {
#pragma unroll
        for (int i = 0; i < SETS; ++i)
#pragma unroll
            for (int sign = 1; sign >= -1; sign -= 2) {  // what goes up, then what goes down
                f32x4 sum = {0.f, 0.f, 0.f, 0.f};
                asm volatile("" : "+v"(seen));  // (few registers rather than few instructions)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float x = a[r][n >> 2][n & 3], w = (float)sign * (*p[i])[r];
                    const bool sees = (seen >> r) & 1;
                    sum = mfma_f32(!(x < kInf) ? kBig : 0.f, sees && !(w < 0.f) ? kBig : 0.f, sum);
                    sum = mfma_f32(!(x > kNegInf) ? kBig : 0.f, sees && !(w > 0.f) ? kBig : 0.f, sum);
                }
                (*acc[i])[n] += (float)sign * sum;
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float x = a[r][n >> 2][n & 3];
            a[r][n >> 2][n & 3] = fabsf(x) < kInf ? x : 0.f;
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Adds up two sets of N accumulators per lane over the first `live` waves (already on one scale; the
// others hold zeros): waves 2, 3 hand theirs to waves 0, 1, then wave 1 to wave 0, which holds the
// result. buf: [2][2 N * 64] f32x4.
template <int N>
__device__ __forceinline__ void f32_sum_waves(f32x4 (&a)[N], f32x4 (&b)[N], f32x4 *buf, int w, int lane, int live) {
#pragma unroll
    for (int step = 2; step > 0; step >>= 1) {
        if (live <= step) continue;  // (uniform over the workgroup)
        __syncthreads();
        if (w >= step && w < min(2 * step, live)) {
            f32x4 *to = buf + (w - step) * 2 * N * 64 + lane;
#pragma unroll
            for (int n = 0; n < N; ++n) to[n * 64] = a[n], to[(N + n) * 64] = b[n];
        }
        __syncthreads();
        if (w < step && w + step < live) {
            const f32x4 *from = buf + w * 2 * N * 64 + lane;
#pragma unroll
            for (int n = 0; n < N; ++n) a[n] += from[n * 64], b[n] += from[(N + n) * 64];
        }
    }
}

// Linear workgroup number of a grid that f32_grid made (row blocks slowest, so that all heads'
// heavy blocks come first, and the workgroups of a head stay on one XCD where 8 divides the heads)
static inline dim3 f32_grid(int64_t total) {
    const int64_t gx = total < (1 << 20) ? total : (1 << 20);
    return dim3((unsigned)gx, (unsigned)((total + gx - 1) / gx));
}
__device__ __forceinline__ int64_t f32_block_id() { return (int64_t)blockIdx.y * gridDim.x + blockIdx.x; }

}  // namespace plx
