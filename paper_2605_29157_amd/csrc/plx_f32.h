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

// Linear workgroup number of a grid that f32_grid made (row blocks slowest, so that all heads'
// heavy blocks come first, and the workgroups of a head stay on one XCD where 8 divides the heads)
static inline dim3 f32_grid(int64_t total) {
    const int64_t gx = total < (1 << 20) ? total : (1 << 20);
    return dim3((unsigned)gx, (unsigned)((total + gx - 1) / gx));
}
__device__ __forceinline__ int64_t f32_block_id() { return (int64_t)blockIdx.y * gridDim.x + blockIdx.x; }

}  // namespace plx
