// Block mask -> the lists that the block-sparse kernels walk (index bookkeeping of the sparsity
// patterns of the paper's Sec. 5, no arithmetic).
//
// A line is a row block (entries: its listed key tiles) or a key block of two key tiles (entries:
// 4 * row block + flags); lines are independent but for where their entries go. Up to kOneLaunchCells (and
// kOneLaunchLines) one launch does all: every workgroup counts the cells in front of its lines. Above, one launch
// counts and a second places: every workgroup adds up the counts in front of its lines itself
// (reads that the L2 holds) instead of a third launch scanning them. With many lines (kScanLines) those
// reads, quadratic in the number of lines, would cost more than the launch, and the scan is made. What
// bounds it otherwise is the launches, one or two; the host never learns the number of entries, so nothing waits for the GPU. Built from
// tensor operations instead (a scan, a compaction whose size the host reads back, casts: 40 launches
// and three waits per training step), the lists took 310 us of a 537 us step over 2 sequences x
// 2048 rows, 16 heads, a quarter of the cells; with these kernels the whole step took 220 us.
#include "plx_device.h"
#include "plx_kernels.h"

namespace plx {

namespace {
constexpr int kLinesPerGroup = 4;  // one wave each
constexpr int kScanThreads = 1024, kScanPerThread = 4;
// Lines of one kind from which the counts are scanned in a launch of their own. Row and key lists, us
// for two launches / three: 4096 lines in all 13.9 / -, 8192 + 8192 lines 19.1 / 16.6 (32 row blocks a
// list) and 23.6 / 20.8 (128), 32768 + 32768 130 / 71 (128) and 284 / 241 (512).
constexpr int64_t kScanLines = 8192;
// Cells up to which one launch does it, every workgroup counting what is in front of its lines from the mask itself:
// work quadratic in the cells, against a launch. Two launches / one in a replayed graph, us, row lists alone and with key
// lists: 16 x 32 cells 4.4 / 2.7 and 4.7 / 3.2; 64 x 128 5.2 / 4.1 and 5.0 / 5.0; 16 lists of 16 x 32 4.6 / 3.9 and
// 5.1 / 5.0; 16 of 32 x 64 4.9 / 7.2 and 5.7 / 9.6. (On a stream two launches cost another gap and their host time.)
// And lines: each four of them count. In a trace with 1 us a gap, 8192 lists of one cell (16384 lines with the key lists)
// 16.1 (a scan) / 18.8, 4096 of 1 x 2 (8192) 11.3 / 9.3, one list of 8192 x 1 65 / 47.
constexpr int64_t kOneLaunchCells = 8192, kOneLaunchLines = 12288;

// Entry n of a line: 0 = not listed, else 1 + the value that goes into the list.
struct LineReader {
    const uint8_t *cells;
    int64_t step;
    int n, second;  // second: bytes from a cell to its neighbour tile (0: row line, -1: none exists)
    __device__ LineReader(const BlockListParams &p, int64_t line) {
        const int64_t row_lines = (int64_t)p.lists * p.n_row_blocks;
        if (line < row_lines) {
            cells = p.mask + line * p.n_tiles, step = 1, n = p.n_tiles, second = 0;
        } else {
            const int n_cb = (p.n_tiles + 1) / 2;
            const int64_t l = line - row_lines, list = l / n_cb;
            const int tile = 2 * (int)(l % n_cb);
            cells = p.mask + list * p.n_row_blocks * p.n_tiles + tile;
            step = p.n_tiles, n = p.n_row_blocks, second = tile + 1 < p.n_tiles ? 1 : -1;
        }
    }
    __device__ int entry(int i) const {
        if (i >= n) return 0;
        const uint8_t *at = cells + i * step;
        if (second == 0) return *at ? 1 + i : 0;
        const int flags = (at[0] ? 1 : 0) | (second > 0 && at[1] ? 2 : 0);
        return flags ? 1 + 4 * i + flags : 0;
    }
};

__device__ __forceinline__ int count_line(const BlockListParams &p, int64_t line, int lane) {
    const LineReader in(p, line);
    int count = 0;
    for (int i = lane; i - lane < in.n; i += 64) count += __popcll(__ballot(in.entry(i) != 0));
    return count;
}
__device__ __forceinline__ void place_line(const BlockListParams &p, int64_t line, int32_t *idx, int at, int lane) {
    const LineReader in(p, line);
    for (int i = lane; i - lane < in.n; i += 64) {
        const int x = in.entry(i);
        const unsigned long long hits = __ballot(x != 0);
        if (x != 0) idx[at + __popcll(hits & ((1ull << lane) - 1ull))] = x - 1;
        at += __popcll(hits);
    }
}

__device__ __forceinline__ int64_t line_total(const BlockListParams &p) {
    const int64_t rows = (int64_t)p.lists * p.n_row_blocks;
    return p.col_ptr ? rows + (int64_t)p.lists * ((p.n_tiles + 1) / 2) : rows;
}

__global__ __launch_bounds__(64 * kLinesPerGroup) void block_list_count_kernel(BlockListParams p) {
    const int64_t line = (int64_t)blockIdx.x * kLinesPerGroup + (threadIdx.x >> 6);
    if (line >= line_total(p)) return;
    const int lane = threadIdx.x & 63, count = count_line(p, line, lane);
    if (lane == 0) p.counts[line] = count;
}

// Few cells and lines (so their indices fit 32 bits)
__global__ __launch_bounds__(64 * kLinesPerGroup) void block_list_kernel(BlockListParams p) {
    __shared__ int before[kLinesPerGroup], own[kLinesPerGroup];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t total = line_total(p), rows = (int64_t)p.lists * p.n_row_blocks;
    const int64_t line0 = (int64_t)blockIdx.x * kLinesPerGroup, line = line0 + w;
    const int n_cb = (p.n_tiles + 1) / 2;
    int mine = 0;  // entries in front of the workgroup's first line, of its kind: this thread's cells
    if (line0 < rows) {
        const int n = (int)line0 * p.n_tiles;
#pragma unroll 4
        for (int i = threadIdx.x; i < n; i += 64 * kLinesPerGroup) mine += p.mask[i] != 0;
    } else {
        const int l = (int)(line0 - rows), list = l / n_cb, cb0 = l % n_cb, row0 = list * p.n_row_blocks;
        const int n = (row0 + p.n_row_blocks) * n_cb;
#pragma unroll 4
        for (int i = threadIdx.x; i < n; i += 64 * kLinesPerGroup) {
            const int row = i / n_cb, cb = i - row * n_cb;
            const uint8_t *at = p.mask + row * p.n_tiles + 2 * cb;
            const bool hit = (at[0] | at[2 * cb + 1 < p.n_tiles ? 1 : 0]) != 0;
            mine += hit && (row < row0 || cb < cb0);
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mine += __shfl_xor(mine, off, 64);
    const int count = line < total ? count_line(p, line, lane) : 0;
    if (lane == 0) before[w] = mine, own[w] = count;
    __syncthreads();
    if (line >= total) return;
    const bool row_line = line < rows;
    int at = 0;
#pragma unroll
    for (int i = 0; i < kLinesPerGroup; ++i) {
        if (row_line == (line0 < rows)) at += before[i];  // (a workgroup may hold the last row line and the first key line)
        if (i < w && (line0 + i < rows) == row_line) at += own[i];
    }
    const int64_t e = row_line ? line : line - rows;
    int32_t *ptr = row_line ? p.row_ptr : p.col_ptr;
    if (lane == 0) {
        ptr[e] = at;
        if (line + 1 == (row_line ? rows : total)) ptr[e + 1] = at + count;
        p.counts[line] = count;
    }
    place_line(p, line, row_line ? p.tile_idx : p.col_idx, at, lane);
}

// Many lines: workgroup 0 turns the counts of the row lines into row_ptr, workgroup 1 those of the key
// lines into col_ptr.
__global__ __launch_bounds__(kScanThreads) void block_list_scan_kernel(BlockListParams p) {
    __shared__ int wave_sum[kScanThreads / 64];
    const int64_t rows = (int64_t)p.lists * p.n_row_blocks;
    const int64_t n = blockIdx.x == 0 ? rows : line_total(p) - rows;
    const int32_t *counts = p.counts + (blockIdx.x == 0 ? 0 : rows);
    int32_t *ptr = blockIdx.x == 0 ? p.row_ptr : p.col_ptr;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int before = 0;  // entries in front of this round's lines
    for (int64_t first = 0; first < n; first += kScanThreads * kScanPerThread) {
        const int64_t at = first + threadIdx.x * kScanPerThread;
        int c[kScanPerThread], mine = 0;
#pragma unroll
        for (int i = 0; i < kScanPerThread; ++i) c[i] = at + i < n ? counts[at + i] : 0, mine += c[i];
        int upto = mine;  // inclusive over the wave
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int x = __shfl_up(upto, off, 64);
            if (lane >= off) upto += x;
        }
        __syncthreads();  // (the last round's sums have been read)
        if (lane == 63) wave_sum[w] = upto;
        __syncthreads();
        int start = before + upto - mine, all = 0;
#pragma unroll
        for (int i = 0; i < kScanThreads / 64; ++i) {
            if (i < w) start += wave_sum[i];
            all += wave_sum[i];
        }
#pragma unroll
        for (int i = 0; i < kScanPerThread; ++i) {
            if (at + i < n) ptr[at + i] = start;
            start += c[i];
        }
        before += all;
    }
    if (threadIdx.x == 0) ptr[n] = before;
}

template <bool SCANNED>
__global__ __launch_bounds__(64 * kLinesPerGroup) void block_list_place_kernel(BlockListParams p) {
    __shared__ int part[kLinesPerGroup];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t total = line_total(p), rows = (int64_t)p.lists * p.n_row_blocks;
    const int64_t line0 = (int64_t)blockIdx.x * kLinesPerGroup, line = line0 + w;
    const bool row_line = line < rows;
    int32_t *ptr = row_line ? p.row_ptr : p.col_ptr;
    int32_t *idx = row_line ? p.tile_idx : p.col_idx;
    const int64_t e = row_line ? line : line - rows;
    int at = 0;
    if constexpr (SCANNED) {
        if (line >= total) return;
        at = ptr[e];
    } else {
        // entries in front of the workgroup's first line, of its kind (row lines and key lines are separate
        // lists; a workgroup may hold the last of one and the first of the other)
        const int64_t kind0 = line0 < rows ? 0 : rows;
        int before = 0;
        for (int64_t i = kind0 + threadIdx.x; i < line0; i += 64 * kLinesPerGroup) before += p.counts[i];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) before += __shfl_xor(before, off, 64);
        if (lane == 0) part[w] = before;
        __syncthreads();
        if (line >= total) return;
        if (row_line == (line0 < rows))
            for (int i = 0; i < kLinesPerGroup; ++i) at += part[i];
        for (int64_t i = row_line ? line0 : (line0 > rows ? line0 : rows); i < line; ++i) at += p.counts[i];
        if (lane == 0) {
            ptr[e] = at;
            if (line + 1 == (row_line ? rows : total)) ptr[e + 1] = at + p.counts[line];
        }
    }
    place_line(p, line, idx, at, lane);
}
}  // namespace

hipError_t launch_block_lists(const BlockListParams &p, hipStream_t stream) {
    const int64_t lines = (int64_t)p.lists * p.n_row_blocks + (p.col_ptr ? (int64_t)p.lists * ((p.n_tiles + 1) / 2) : 0);
    const int64_t groups = (lines + kLinesPerGroup - 1) / kLinesPerGroup;
    if (groups > (1 << 23)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)groups), block(64 * kLinesPerGroup);
    if ((int64_t)p.lists * p.n_row_blocks * p.n_tiles <= kOneLaunchCells && lines <= kOneLaunchLines) {
        hipLaunchKernelGGL(block_list_kernel, grid, block, 0, stream, p);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(block_list_count_kernel, grid, block, 0, stream, p);
    if (hipError_t err = hipGetLastError()) return err;
    const int64_t row_lines = (int64_t)p.lists * p.n_row_blocks;
    if (row_lines < kScanLines && lines - row_lines < kScanLines) {
        hipLaunchKernelGGL(block_list_place_kernel<false>, grid, block, 0, stream, p);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(block_list_scan_kernel, dim3(p.col_ptr ? 2 : 1), dim3(kScanThreads), 0, stream, p);
    if (hipError_t err = hipGetLastError()) return err;
    hipLaunchKernelGGL(block_list_place_kernel<true>, grid, block, 0, stream, p);
    return hipGetLastError();
}

}  // namespace plx
