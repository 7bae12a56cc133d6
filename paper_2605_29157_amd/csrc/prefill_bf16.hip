// Causal / full Parallax prefill forward for bf16 on gfx950.
//
// What it computes: Algorithm 1 of the paper (Sec. 3.3) -- for a block of query rows, one pass
// over key tiles with the running state (m, d1, d2, O1, O2); S1 = Q K^T * scale (masked),
// S2 = R K^T (unscaled), P1 = exp2(S1 - m), P2 = P1 * S2, O1 += P1 V, O2 += P2 V; closing
// formula O1/d1 * (1 + d2/d1) - O2/d1. Causal: key j allowed iff j <= i (Sec. 3.1); with more
// keys than query rows the rows are the last positions of the sequence, j <= i + (Tk - T).
//
// Layout for CDNA4:
//   * one workgroup = 4 waves of 32 query rows. d = 128: one wave per SIMD, so a wave may use the whole 512-register
//     budget: O1^T, O2^T and the Q, R fragments live in the accumulation registers for the whole
//     pass -- an MFMA can take its B operand from there -- and the vector registers hold scores,
//     P and LDS fragments. d = 64: 256 registers and half of the LDS, two workgroups per compute unit, as the
//     element-wise work takes as long as the matrix work there and one wave's runs under the other's
//     matrix instructions (64 rows per wave, one workgroup per unit, before: 32 heads, 4 x 4096 rows 520 -> 503 us,
//     3 x 1111 54 -> 42, 4 x 2048 with a window of 512 127 -> 88; 2 x 1024 over 16384 keys, whose workgroups all walk
//     hundreds of tiles, 478 -> 489);
//   * every global read is a direct global -> LDS load of whole rows (global_load_lds_dwordx4:
//     no staging registers, no LDS write instructions): the wave's own Q and R rows once, then
//     K/V tiles of 64 keys into a three-stage ring, fetched two tiles ahead, one load per MFMA
//     slot of the pipeline. Rows are padded, not swizzled, so that every operand address is a
//     per-lane base plus a constant; one workgroup barrier per tile;
//   * scores are produced transposed with v_mfma_f32_32x32x16_bf16, S^T = K Q^T: each K
//     fragment read from LDS feeds two MFMAs (the q branch and the r branch). In the S^T
//     accumulator a lane owns ONE query row (column) and 16 of the 32 keys, so softmax
//     statistics are per lane, S1 and S2 of a (row, key) pair share lane and register, and the
//     accumulator registers are already the B operand of O^T += V^T P^T (V^T fragments come
//     from transposing LDS reads);
//   * key blocks of 32 are software-pipelined in slots of one MFMA plus its share of vector
//     work: the score MFMAs of block i+1 run under the exp arithmetic of block i, the PV MFMAs
//     of block i under the exp arithmetic of block i+1;
//   * row sums d1, d2: per-lane fp32 adds in tiles every row sees completely; in diagonal /
//     tail tiles MFMAs against a matrix of ones, i.e. sums of exactly the bf16 operands that
//     enter O1 / O2, so that rows with very few keys come out exact (row 0 returns v_0).
//
// The running max m of Algorithm 1 only has to keep exp2 in range: ANY per-row reference gives
// the same O after the final division. The fast pass therefore fixes m to the row maximum over
// the first key block and never rescales O1/O2 (no vector-ALU work on the 128 accumulator
// registers inside the loop). If a later score exceeds that reference by more than ~2^7 in the
// exp2 domain the sums overflow to inf/NaN; this is detected at the end of the pass and the
// workgroup redoes its rows with the textbook online update (max, alpha rescale) -- slower, and
// in practice never taken for attention logits, but it keeps the softmax safe for every input.
#include <algorithm>
#include <type_traits>

#include "plx_device.h"
#include "plx_kernels.h"
#include "plx_lds_dma.h"
#include "plx_mfma_asm.h"

namespace plx {

constexpr int kBC = 64;   // keys per LDS tile
constexpr int kKB = 32;   // keys per inner block (one MFMA row block)

// Key ranges of a row block that sees `keys` keys: as few ranges of at most max_tiles tiles as will do,
// of equal length up to the last
struct PrefillRanges {
    int count, tiles;
    __host__ __device__ PrefillRanges(int keys, int max_tiles) {
        const int all = (keys + kBC - 1) / kBC;
        count = (all + max_tiles - 1) / max_tiles;
        tiles = (all + count - 1) / count;
        count = (all + tiles - 1) / tiles;  // (no empty range at the end)
    }
};
// Split records of 32 rows: O1, O2 (2 * 32 * D floats) and five row scalars
__host__ __device__ constexpr int64_t prefill_record_floats(int d) { return 64 * (int64_t)d + 5 * 32; }

// Keeps two score blocks where they are up to this point.
__device__ __forceinline__ void keep_blocks(const f32x16 &a, const f32x16 &b) { asm volatile("" ::"v"(a), "v"(b)); }

// SPLIT: a row block with many key tiles is cut into key ranges of at most p.split_tiles tiles, each a
// workgroup of its own that writes unnormalised records instead of output rows (the split-KV form of
// App. C, merged by prefill_combine_kernel) -- for launches with fewer row blocks than compute units.
// PREP: RMSNorm + RoPE on the wave's Q and R rows in their LDS landing zones, before the MFMA
// fragments are read (the operations the paper's language-model runs put in front of the attention
// call: Sec. 5 experiment setup and the backbone appendix; same formulas and order of operations as
// norm_rope.hip, the rotation taken from a table of (cos, sin) per position and pair).
// PAIR: 64 rows per workgroup. Waves w and w ^ 2 share 32 rows, each takes one 32-key half of every tile, and they add
// their sums up at the end: half the chain for twice the workgroups, for launches that wait for their longest one.
template <int D, bool USE_R, bool CAUSAL, bool WINDOW, bool STATS = false, bool SPARSE = false, bool PREP = false,
          bool SPLIT = false, bool PAIR = false>
__global__ __launch_bounds__(256, D == 64 ? 2 : 1) void prefill_bf16_kernel(PrefillParams p) {
    static_assert(!PREP || (USE_R && !WINDOW && !STATS && !SPARSE), "q / rho preparation: dense forward only");
    static_assert(!SPLIT || (!WINDOW && !SPARSE && !PREP), "key ranges: dense forward only");
    constexpr int WROWS = 32;  // query rows per wave
    constexpr int kBR = PAIR ? 2 * WROWS : 4 * WROWS;  // query rows per workgroup
    static_assert(!PAIR || (CAUSAL && !SPARSE && !SPLIT), "two waves to 32 rows: dense causal forward");
    static_assert(CAUSAL || !WINDOW, "a sliding window needs the rows' positions");
    static_assert(!STATS || USE_R, "the row cache is written for the backward pass only");
    static_assert(!SPARSE || !WINDOW, "block-sparse: its own tile iterator, no window");
    constexpr int CPR = D / 8;            // 16-byte chunks per row
    constexpr int KSTEPS = D / 16;        // k-steps of the score contraction
    constexpr int NDB = D / 32;           // 32-wide blocks of output dimensions
    constexpr int STAGES = 3;  // LDS ring; tiles are fetched STAGES - 1 ahead
    constexpr int kDist = STAGES - 1;
    // K rows are padded by one 16-byte chunk (16 consecutive rows, same chunk -> 16 different
    // bank groups), V rows by four chunks (the 4 consecutive rows of a transposing read land in
    // 4 different 64-byte bank groups). Tiles are filled by direct global->LDS loads: one
    // wave-wide instruction writes 64 consecutive chunks, so each lane fetches the global chunk
    // that belongs at its LDS position (padding positions re-fetch a neighbour), and both tiles
    // are rounded up to NDMA * 4 * 64 chunks.
    constexpr int KROW = CPR + 1, VROW = CPR + 4;  // row strides in chunks
    // Every wave fills a contiguous quarter of each tile: 16 * KROW chunks of K (CPR / 4 full
    // 64-lane loads and one 16-lane load), 16 * VROW chunks of V (CPR / 4 + 1 full loads).
    constexpr int K_WAVE_CHUNKS = 16 * KROW, V_WAVE_CHUNKS = 16 * VROW;
    constexpr int NDMA_K = CPR / 4 + 1, NDMA_V = CPR / 4 + 1;
    static_assert(K_WAVE_CHUNKS == 64 * (NDMA_K - 1) + 16 && V_WAVE_CHUNKS == 64 * NDMA_V, "split");
    constexpr int K_CHUNKS = kBC * KROW, V_CHUNKS = kBC * VROW;
    constexpr int kTileLoads = NDMA_K + NDMA_V;  // per wave and tile
    constexpr int STAGE_CHUNKS = K_CHUNKS + V_CHUNKS;

    // Behind the ring: one padded WROWS x D tile per wave. It receives the wave's Q rows at the
    // start and stages its output rows at the end. The R rows land in ring stage 2.
    constexpr int WAVE_TILE_CHUNKS = WROWS * KROW;
    // TWO (d = 64): two workgroups per compute unit. For its half of the LDS the Q zone starts in
    // the end of stage 2 that the R rows leave free: the tile loads do not reach it before the
    // fragments are in registers, and outputs are staged behind a barrier.
    constexpr bool TWO = D == 64;
    constexpr int QZONE = STAGES * STAGE_CHUNKS - (TWO ? STAGE_CHUNKS - 4 * WAVE_TILE_CHUNKS : 0);
    static_assert(STAGES >= 3 && 4 * WAVE_TILE_CHUNKS <= STAGE_CHUNKS, "R rows land in ring stage 2");
    constexpr int RZONE = 2 * STAGE_CHUNKS;
    constexpr int LDS_CHUNKS = QZONE + 4 * WAVE_TILE_CHUNKS;
    static_assert(LDS_CHUNKS * 16 <= (TWO ? 80 : 160) * 1024, "LDS of one compute unit");
    __shared__ u32x4 lds[LDS_CHUNKS];  // [stage][K tile | V tile], Q (, R)

    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int col = lane & 31;  // MFMA column: query row within the wave's 32 rows
    const int h = lane >> 5;    // half-wave

    // ---- work item: heavy row blocks first; blocks of one (batch, kv head) share an XCD ----
    const int T = p.T, G = p.G;  // query rows
    const int nrb = (T + kBR - 1) / kBR;
    const int pairs = p.B * p.Hkv;
    int rbi, pair, hg;  // (SPLIT: rbi numbers the (row block, key range) items of a head)
    {
        const int id = blockIdx.x;
        if (pairs % 8 == 0) {
            const int x = id & 7, j = id >> 3;
            const int per = (pairs / 8) * G;
            rbi = j / per;
            const int rem = j - rbi * per;
            pair = (rem / G) * 8 + x;
            hg = rem % G;
        } else {
            const int per = pairs * G;
            rbi = id / per;
            const int rem = id - rbi * per;
            pair = rem / G;
            hg = rem % G;
        }
    }
    const int item = rbi;
    int n_ranges = 1, range = 0, range_tiles = 0;
    if constexpr (SPLIT) {  // (few row blocks: the host splits launches smaller than the chip)
        rbi = 0, range = item;
        for (;; ++rbi) {
            const PrefillRanges r(CAUSAL ? min(p.Tk, (nrb - rbi) * kBR + (p.Tk - T)) : p.Tk, p.split_tiles);
            n_ranges = r.count, range_tiles = r.tiles;
            if (range < n_ranges || rbi == nrb - 1) break;
            range -= n_ranges;
        }
    }
    const int rb = CAUSAL ? nrb - 1 - rbi : rbi;
    // Sliding window: row i sees the keys i + off - window + 1 .. i + off. The key tiles before
    // the first key of the workgroup's first row are skipped by moving the K / V base; from
    // here on key positions, Tk and off are relative to that first tile.
    // (SPLIT skips the tiles before its key range the same way.)
    const int kt_skip = WINDOW  ? max(rb * kBR + (p.Tk - T) - p.window + 1, 0) / kBC
                        : SPLIT ? range * range_tiles
                                : 0;
    const int Tk = p.Tk - kt_skip * kBC;  // keys
    const int Tv = SPLIT ? min(Tk, range_tiles * kBC) : Tk;  // keys this workgroup looks at
    const int off = Tk - T;               // causal: row i sits at key position i + off
    const int b = pair / p.Hkv, hk = pair - b * p.Hkv;
    const int hq = hk * G + hg;

    const int half = PAIR ? w >> 1 : 0;  // PAIR: this wave's half of every tile
    const int row0 = rb * kBR + (PAIR ? w & 1 : w) * WROWS;  // first query row of this wave
    // this lane's query row (may be >= T)
    const int my_row = row0 + col;

    // ---- Q / R rows of this wave: global -> LDS, whole rows (a lane fetching its own MFMA
    // fragments straight from global memory would touch 64 different rows per instruction).
    // Padded like a K tile; nobody else reads them, so no barrier is needed for them. Q lands
    // behind the ring, R in ring stage 2, which the tile loads do not reach before the first
    // loop iteration -- by then the fragments are in registers -- or behind the Q zone.
    constexpr int NDMA_Q = (WAVE_TILE_CHUNKS + 63) / 64;  // full loads (+ one 32-lane load)
    constexpr int Q_LAST_LANES = WAVE_TILE_CHUNKS - 64 * (NDMA_Q - 1);
    static_assert(Q_LAST_LANES == 32 || Q_LAST_LANES == 64, "split");
    // PREP: a wave-wide pass covers 64 / CPR rows (one 16-byte chunk = 4 pairs per lane); the
    // weights of this lane's chunk and the table entries of its rows are requested first of all,
    // so that they are there when the rows have landed.
    constexpr int PREP_RPI = 64 / CPR, PREP_NIT = WROWS / PREP_RPI;
    f32x4 prep_gq[2], prep_gr[2], prep_tab[PREP ? PREP_NIT : 1][2];
    if constexpr (PREP) {
        const int lr = lane % CPR, lrow = lane / CPR;
        prep_gq[0] = *(const f32x4 *)(p.prep.gamma_q + 8 * lr), prep_gq[1] = *(const f32x4 *)(p.prep.gamma_q + 8 * lr + 4);
        prep_gr[0] = *(const f32x4 *)(p.prep.gamma_r + 8 * lr), prep_gr[1] = *(const f32x4 *)(p.prep.gamma_r + 8 * lr + 4);
        if (p.prep.table != nullptr) {  // workgroup-uniform
            const int base = p.prep.pos0 ? p.prep.pos0[b] : 0;
#pragma unroll
            for (int it = 0; it < PREP_NIT; ++it) {
                const int grow = min(row0 + it * PREP_RPI + lrow, T - 1);
                const int64_t pos = min(max(base + grow, 0), p.prep.n_pos - 1);
                const float *e = p.prep.table + (pos * (D / 2) + 4 * lr) * 2;
                prep_tab[it][0] = *(const f32x4 *)e, prep_tab[it][1] = *(const f32x4 *)(e + 4);
            }
        }
    }
    const uint32_t lds_base = lds_byte_address(lds);
    {
        const __bf16 *qhead = (const __bf16 *)p.q + b * p.qs[0] + hq * p.qs[1];
        const __bf16 *rhead = (const __bf16 *)p.r + b * p.rs[0] + hq * p.rs[1];
        const uint32_t dq = lds_base + (uint32_t)(QZONE + w * WAVE_TILE_CHUNKS) * 16u;
        const uint32_t dr = lds_base + (uint32_t)(RZONE + w * WAVE_TILE_CHUNKS) * 16u;
#pragma unroll
        for (int i = 0; i < NDMA_Q; ++i) {
            const int c = 64 * i + lane;  // lanes >= 32 of a half last load: unused
            const int64_t grow = min(row0 + min(c / KROW, WROWS - 1), T - 1);
            const int pos = min(c % KROW, CPR - 1);
            const __bf16 *sq = qhead + grow * p.qs[2] + pos * 8;
            const __bf16 *sr = rhead + grow * p.rs[2] + pos * 8;
            if (i == NDMA_Q - 1 && Q_LAST_LANES == 32) {
                tile_load16<32>(sq, dq + 1024u * i);
                if constexpr (USE_R) tile_load16<32>(sr, dr + 1024u * i);
            } else {
                tile_load16<64>(sq, dq + 1024u * i);
                if constexpr (USE_R) tile_load16<64>(sr, dr + 1024u * i);
            }
        }
    }
    u32x4 qf[KSTEPS], rf[KSTEPS];
    // SPLIT: the first 32 keys of the sequence as MFMA operands (row col, chunk 2 * ks + h), for the
    // reference; they travel with the wave's own rows.
    u32x4 k_ref[SPLIT ? KSTEPS : 1];
    if constexpr (SPLIT) {
        const __bf16 *krow = (const __bf16 *)p.k + b * p.ks[0] + hk * p.ks[1] + (int64_t)min(col, p.Tk - 1) * p.ks[2];
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) k_ref[ks] = *(const u32x4 *)(krow + (2 * ks + h) * 8);
    }

    const __bf16 *kbase = (const __bf16 *)p.k + b * p.ks[0] + hk * p.ks[1] + (int64_t)kt_skip * kBC * p.ks[2];
    const __bf16 *vbase = (const __bf16 *)p.v + b * p.vs[0] + hk * p.vs[1] + (int64_t)kt_skip * kBC * p.vs[2];

    const int key_end = CAUSAL ? min(Tv, (rb + 1) * kBR + off) : Tv;  // keys this workgroup may need
    // Block-sparse: the workgroup visits only the key tiles its row block lists (ascending tile
    // indices, caller's arrays); the ring position i and the key tile tile_at(i) then differ.
    // Entries are clamped to existing tiles, listed tiles past the causal limit are dropped.
    // (read through the constant address space: uniform, never written while the kernel runs, so the
    // reads are scalar loads that the tile loads in flight do not hold up)
    using const_i32 = const __attribute__((address_space(4))) int32_t;
    const_i32 *tile_list = nullptr;
    int n_list = 0;
    if constexpr (SPARSE) {
        const int sb = p.sparse_batch > 1 ? b : 0, sh = p.sparse_heads > 1 ? hq : 0;
        const int64_t e = ((int64_t)sb * p.sparse_heads + sh) * nrb + rb;
        const_i32 *row_ptr = (const_i32 *)(uintptr_t)p.sparse_row_ptr;
        const int first = row_ptr[e];
        tile_list = (const_i32 *)(uintptr_t)p.sparse_tile_idx + first;
        n_list = max(row_ptr[e + 1] - first, 0);
    }
    // number of leading list entries whose first key lies below `bound` (binary search: the list ascends)
    auto list_count = [&](int bound) __attribute__((always_inline)) {
        int lo = 0, hi = n_list;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if ((int64_t)max(tile_list[mid], 0) * kBC < bound)
                lo = mid + 1;
            else
                hi = mid;
        }
        return lo;
    };
    // all 64 keys of these leading entries exist and are visible to every row of the workgroup
    const int vis_end = CAUSAL ? min(rb * kBR + off + 1, Tk) : Tk;
    const int n_list_full = SPARSE ? list_count(vis_end - kBC + 1) : 0;
    if constexpr (SPARSE) n_list = list_count(key_end);
    // a row block that lists nothing runs one tile with every key masked: sums of zero, zeros out
    const bool no_tiles = SPARSE && n_list == 0;
    auto tile_at = [&](int i) __attribute__((always_inline)) {
        if constexpr (SPARSE)
            return no_tiles ? 0 : min(max(tile_list[min(i, n_list - 1)], 0), (Tk - 1) / kBC);
        else
            return i;
    };
    int n_tiles_ = SPARSE ? max(n_list, 1) : (key_end + kBC - 1) / kBC;
    // (block-sparse: the count is handed over as an opaque value. Knowing it is at least 1, the
    // compiler merges the pipeline prologue into the first loop iteration, and that one long
    // region needs more registers than the file holds.)
    if constexpr (SPARSE) asm volatile("" : "+s"(n_tiles_));
    const int n_tiles = n_tiles_;
    // leading tiles whose keys all exist and are visible to every row of the workgroup, less two
    // so that the tile prefetched two ahead inside that loop is always a complete one
    // (block-sparse: leading list entries; the entry prefetched two ahead is then not the last
    // one, the only one that may be the partial tile)
    const int n_full = SPARSE ? max(0, min(n_list_full, n_list - kDist))
                              : max(0, min(CAUSAL ? min((rb * kBR + off + 1) / kBC, Tv / kBC) : Tv / kBC, Tk / kBC - kDist));
    // sliding window: first key this lane's row sees, and the leading tiles that hold a key
    // some row of the workgroup does not see (its last row starts latest)
    int row_lo;
    row_lo = WINDOW ? my_row + off - p.window + 1 : 0;
    const int n_left = WINDOW ? min(n_tiles, max(rb * kBR + kBR + off - p.window + kBC - 1, 0) / kBC) : 0;

    // ---- global -> LDS tile loads (no staging registers, no LDS write instructions) --------
    // Load instruction i of wave w fills LDS chunks [64*(w + 4i), +64) of a tile; lane l owns
    // chunk g = 64*(w + 4i) + l = (row, pos) in the padded row-major layout.
    auto k_src = [&](int i, int &row, int &pos) __attribute__((always_inline)) {
        const int c = K_WAVE_CHUNKS * w + 64 * i + lane;  // lanes >= 16 of the last load: unused
        row = min(c / KROW, kBC - 1);
        pos = min(c % KROW, CPR - 1);
    };
    auto v_src = [&](int i, int &row, int &pos) __attribute__((always_inline)) {
        const int c = V_WAVE_CHUNKS * w + 64 * i + lane;
        row = c / VROW;
        pos = min(c % VROW, CPR - 1);
    };
    uint32_t koff[NDMA_K], voff[NDMA_V];  // byte offsets inside a tile whose 64 rows all exist
#pragma unroll
    for (int i = 0; i < NDMA_K; ++i) {
        int row, pos;
        k_src(i, row, pos);
        koff[i] = (uint32_t)(row * p.ks[2] + pos * 8) * 2u;
    }
#pragma unroll
    for (int i = 0; i < NDMA_V; ++i) {
        int row, pos;
        v_src(i, row, pos);
        voff[i] = (uint32_t)(row * p.vs[2] + pos * 8) * 2u;
    }
    const int64_t k_tile_bytes = (int64_t)(kBC * 2) * p.ks[2], v_tile_bytes = (int64_t)(kBC * 2) * p.vs[2];
    // LDS byte addresses of this wave's first K / V load of a stage
    auto stage_k_addr = [&](int stage) __attribute__((always_inline)) {
        return lds_base + (uint32_t)(stage * STAGE_CHUNKS + K_WAVE_CHUNKS * w) * 16u;
    };
    auto stage_v_addr = [&](int stage) __attribute__((always_inline)) {
        return lds_base + (uint32_t)(stage * STAGE_CHUNKS + K_CHUNKS + V_WAVE_CHUNKS * w) * 16u;
    };
    // load i of the tile at (tk, tv) into (dk, dv); tile rows all exist
    auto k_load = [&](int i, const char *tk, uint32_t dk) __attribute__((always_inline)) {
        if (i == NDMA_K - 1)
            tile_load16_uniform<true>(koff[i], tk, dk + 1024u * i);
        else
            tile_load16_uniform<false>(koff[i], tk, dk + 1024u * i);
    };
    auto v_load = [&](int i, const char *tv, uint32_t dv) __attribute__((always_inline)) {
        tile_load16_uniform<false>(voff[i], tv, dv + 1024u * i);
    };
    // tile kt with all 64 rows < T: uniform tile base + the precomputed lane offsets
    auto dma_full_tile = [&](int kt, int stage) __attribute__((always_inline)) {
        const char *tk = (const char *)kbase + kt * k_tile_bytes;
        const char *tv = (const char *)vbase + kt * v_tile_bytes;
#pragma unroll
        for (int i = 0; i < NDMA_K; ++i) k_load(i, tk, stage_k_addr(stage));
#pragma unroll
        for (int i = 0; i < NDMA_V; ++i) v_load(i, tv, stage_v_addr(stage));
    };
    // The steady-state loop spreads the loads of one tile over the MFMA slots of a pipeline step
    // (a block of 2 * NDMA loads at the top of an iteration would leave the matrix pipe idle
    // while they issue); these name the tile being fetched.
    const char *dma_tk = nullptr, *dma_tv = nullptr;
    uint32_t dma_dk = 0, dma_dv = 0;
    // any tile: rows past the last key re-read that key's row (finite data, masked where it matters)
    auto dma_tile = [&](int kt, int stage) __attribute__((always_inline)) {
        const uint32_t dk = stage_k_addr(stage), dv = stage_v_addr(stage);
#pragma unroll
        for (int i = 0; i < NDMA_K; ++i) {
            int row, pos;
            k_src(i, row, pos);
            const __bf16 *sk = kbase + (int64_t)min(kt * kBC + row, Tk - 1) * p.ks[2] + pos * 8;
            if (i == NDMA_K - 1)
                tile_load16<16>(sk, dk + 1024u * i);
            else
                tile_load16<64>(sk, dk + 1024u * i);
        }
#pragma unroll
        for (int i = 0; i < NDMA_V; ++i) {
            int row, pos;
            v_src(i, row, pos);
            const __bf16 *sv = vbase + (int64_t)min(kt * kBC + row, Tk - 1) * p.vs[2] + pos * 8;
            tile_load16<64>(sv, dv + 1024u * i);
        }
    };

    // S1^T, S2^T (32 keys x 32 rows) of key block kb of the tile in `stage`
    auto scores = [&](int stage, int kb, f32x16 &s1, f32x16 &s2) __attribute__((always_inline)) {
        const u32x4 *tk = lds + stage * STAGE_CHUNKS + col * KROW + h;
#pragma unroll
        for (int r = 0; r < 16; ++r) s1[r] = s2[r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) {
            const u32x4 kf = tk[kb * kKB * KROW + 2 * ks];
            s1 = mfma32(kf, qf[ks], s1);
            if constexpr (USE_R) s2 = mfma32(kf, rf[ks], s2);
        }
    };

    // accumulator register r of an S^T block <-> key key_base + 8*(r/4) + 4*h + r%4
    auto key_ok = [&](int key_base, int r) __attribute__((always_inline)) {
        const int key = key_base + 8 * (r >> 2) + 4 * h + (r & 3);
        return key < Tv && (!CAUSAL || key <= my_row + off) && (!WINDOW || key >= row_lo) && !no_tiles;
    };

    // d1 / d2 are accumulated by MFMAs as well: Ones(32 x 16 keys) x P^T gives a block whose
    // every row is the column sum of the bf16-ROUNDED P over the keys, i.e. the row sums of
    // Algorithm 1 taken over exactly the numbers that enter O1 / O2 -- the effective attention
    // weights then sum to one exactly, and no vector-ALU work is spent on the sums (a dot-product
    // instruction would share the matrix pipeline and stall it; measured). One accumulator block
    // serves both sums: the A operand of the P1 sum is one in rows 0..15 and
    // zero below, that of the P2 sum the other way round, so rows 0..15 of the block hold d1
    // (register 0 of every lane) and rows 16..31 hold d2 (register 8).
    // Only the masked tiles take these MFMAs; the tiles every row sees completely add the
    // unrounded fp32 values on the vector ALU.
    // TWO: no registers for that block and its constants; the masked tiles add the rounded operands with
    // dot-product instructions against (1, 1) instead, per lane like vsum below (rsum).
    constexpr bool MFMA_SUMS = !TWO;
    float m_ref;
    f32x16 o1[NDB], o2[NDB], dacc;
    float rsum1 = {}, rsum2 = {};                // !MFMA_SUMS: sums of rounded operands, this lane's keys
    float vsum1[2] = {}, vsum2[2] = {};          // per-lane partial row sums (this lane's keys)
    // Row cache only: fp32 sums of the UNROUNDED P1, P2 over the masked tiles as well. The backward
    // pass recomputes p and u in fp32 and forms 1 + ubar - u, which is 1 for a row with one key only
    // if ubar carries no bf16 rounding of P2; the output keeps the sums of the rounded operands.
    float msum1[2] = {}, msum2[2] = {};
    m_ref = kNegInf;
    const uint32_t one_top = col < 16 ? 0x3f803f80u : 0u, one_bot = col < 16 ? 0u : 0x3f803f80u;
    const u32x4 ones_top = {one_top, one_top, one_top, one_top}, ones_bot = {one_bot, one_bot, one_bot, one_bot};
    const float scale_log2 = p.scale * kLog2e;  // >= 0 (checked by the host)
    // What multiplies S1 in front of the exponential. PREP: the 1 / rms of
    // the row's RMSNorm is a per-row scalar, so it is not applied to the q elements but rides on
    // this factor (and that of rho on the final O2, d2, which are linear in S2): r_gain.
    float row_scale, r_gain;
    row_scale = scale_log2, r_gain = 1.f;

    // adds the bf16 values of a packed MFMA operand (this lane's 8 keys) to acc: one dot product
    // against (1, 1) per packed pair. Written as assembly: through the builtin, viewing a dword of
    // an integer vector as a bf16 pair is miscompiled by this toolchain (all four dot products
    // read the same register).
    auto add_rounded = [&](const u32x4 &pb, float &acc) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) asm("v_dot2c_f32_bf16_e32 %0, 0x3f803f80, %1" : "+v"(acc) : "v"(pb[e]));
    };

    // P1 = exp2(S1*scale - m_ref), P2 = P1*S2 for one key block, left as packed bf16 MFMA
    // operands (two groups of 16 keys).
    auto probs = [&](auto masked_tag, int key_base, f32x16 &s1, f32x16 &s2, u32x4(&pb1)[2],
                     u32x4(&pb2)[2]) __attribute__((always_inline)) {
        constexpr bool MASKED = decltype(masked_tag)::value;
        const float neg_m = m_ref == kNegInf ? 0.f : -m_ref;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float p1 = fast_exp2(fmaf(s1[r], row_scale, neg_m));
            if constexpr (MASKED) p1 = key_ok(key_base, r) ? p1 : 0.f;
            s1[r] = p1;
            // s2 is finite (rows past the last key re-read it) and P1 = 0 where masked
            if constexpr (USE_R) s2[r] = p1 * s2[r];
            if constexpr (STATS) {
                msum1[r & 1] += s1[r];
                msum2[r & 1] += s2[r];
            }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            // B operand k-element e <-> register 8j+e <-> key 16j + 8*(e/4) + 4h + e%4
            pb1[j] = u32x4{pack_bf16(s1[8 * j + 0], s1[8 * j + 1]), pack_bf16(s1[8 * j + 2], s1[8 * j + 3]),
                              pack_bf16(s1[8 * j + 4], s1[8 * j + 5]), pack_bf16(s1[8 * j + 6], s1[8 * j + 7])};
            if constexpr (USE_R)
                pb2[j] = u32x4{pack_bf16(s2[8 * j + 0], s2[8 * j + 1]), pack_bf16(s2[8 * j + 2], s2[8 * j + 3]),
                                  pack_bf16(s2[8 * j + 4], s2[8 * j + 5]), pack_bf16(s2[8 * j + 6], s2[8 * j + 7])};
        }
    };

    // O1^T += V^T P1^T, O2^T += V^T P2^T for key block kb of the tile in `stage`.
    // A operand: row = dimension 32n + col, k-elements = the 8 keys of the B operand, fetched by
    // two transposing LDS reads (keys 16j+4h..+3 and 16j+8+4h..+3).
    const int tr_row = 4 * h + ((lane & 15) >> 2);
    const int tr_half = (lane & 1) * 4;
    const int tr_chunk = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
    const int tr_lane_off = (tr_row * VROW + tr_chunk) * 8 + tr_half;  // in bf16 elements
    auto accumulate = [&](int stage, int kb, const u32x4(&pb1)[2], const u32x4(&pb2)[2]) __attribute__((always_inline)) {
        const unsigned short *tv16 =
            (const unsigned short *)(lds + stage * STAGE_CHUNKS + K_CHUNKS) + tr_lane_off;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int n = 0; n < NDB; ++n) {
                const int off = ((kb * kKB + 16 * j) * VROW + 4 * n) * 8;
                const u32x2 lo = lds_read_tr16(tv16 + off);
                const u32x2 hi = lds_read_tr16(tv16 + off + 8 * VROW * 8);
                const u32x4 vt = {lo[0], lo[1], hi[0], hi[1]};
                o1[n] = mfma32(vt, pb1[j], o1[n]);
                if constexpr (USE_R) o2[n] = mfma32(vt, pb2[j], o2[n]);
            }
#pragma unroll
        for (int j = 0; j < 2; ++j)
            if constexpr (MFMA_SUMS) {
                dacc = mfma32(ones_top, pb1[j], dacc);
                if constexpr (USE_R) dacc = mfma32(ones_bot, pb2[j], dacc);
            } else {
                add_rounded(pb1[j], rsum1);
                if constexpr (USE_R) add_rounded(pb2[j], rsum2);
            }
    };

    auto zero_state = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            if constexpr (MFMA_SUMS) dacc[r] = 0.f;
#pragma unroll
            for (int n = 0; n < NDB; ++n) {
                o1[n][r] = 0.f;
                o2[n][r] = 0.f;
            }
        }
        rsum1 = rsum2 = 0.f;
    };

    // does this wave see any key of the block starting at key_base?
    auto block_visible = [&](int key_base) __attribute__((always_inline)) {
        return key_base < Tv && (!CAUSAL || key_base <= row0 + WROWS - 1 + off) &&
               (!WINDOW || key_base + kKB > row0 + off - p.window + 1);
    };

    u32x4 pb1[2], pb2[2];
    pb2[0] = pb2[1] = u32x4{0u, 0u, 0u, 0u};

    // One step of the software pipeline over fully visible key blocks, written as slots of ONE
    // MFMA each followed by its share of vector-ALU work (measured on this chip: a wave can
    // issue about four vector instructions in the shadow of a 32x32x16 MFMA):
    //   phase 1 : score MFMAs of the NEXT block (S1 and S2 alternate), while the vector ALU
    //             turns the upper 16 keys of the CURRENT block into P1 / P2 (bf16 operands);
    //   phase 2 : PV and row-sum MFMAs of the CURRENT block, while the vector ALU already turns
    //             the lower 16 keys of the NEXT block into its P1 / P2.
    // Every fragment slot issues the LDS read of the fragment needed kLookAhead fragments later
    // ([K of next block | V^T of current block | K of the block after]). The scheduling fences
    // keep this order.
    constexpr int kLookAhead = 3;  // fragments read ahead of their MFMAs
    static_assert(2 * NDB == KSTEPS, "as many V^T fragments as K fragments per key block");
    u32x4 kf[KSTEPS], vt[KSTEPS];
    auto k_block_ptr = [&](int stage, int kb) __attribute__((always_inline)) {
        return (const u32x4 *)(lds + stage * STAGE_CHUNKS + col * KROW + h + kb * kKB * KROW);
    };
    auto v_block_ptr = [&](int stage, int kb) __attribute__((always_inline)) {
        return (const unsigned short *)(lds + stage * STAGE_CHUNKS + K_CHUNKS) + tr_lane_off +
               kb * kKB * VROW * 8;
    };
    auto load_kfrag = [&](const u32x4 *tk_block, int ks) __attribute__((always_inline)) {
        kf[ks] = tk_block[2 * ks];
    };
    auto load_vfrag = [&](const unsigned short *tv_block, int f) __attribute__((always_inline)) {
        const int j = f / NDB, n = f % NDB;  // key group of 16, dim block of 32
        const int off = (16 * j * VROW + 4 * n) * 8;
        const u32x2 lo = lds_read_tr16(tv_block + off);
        const u32x2 hi = lds_read_tr16(tv_block + off + 8 * VROW * 8);
        vt[f] = u32x4{lo[0], lo[1], hi[0], hi[1]};
    };
    auto prefetch = [&](int frag, const u32x4 *tk_next, const unsigned short *tv_cur,
                        const u32x4 *tk_after) __attribute__((always_inline)) {
        const int f = frag + kLookAhead;
        if (f < KSTEPS)
            load_kfrag(tk_next, f);
        else if (f < 2 * KSTEPS)
            load_vfrag(tv_cur, f - KSTEPS);
        else if constexpr (!PAIR)  // (PAIR: the block after is in a tile that has not landed yet)
            load_kfrag(tk_after, f - 2 * KSTEPS);
    };
    // exp / P2 of the 8 score registers [r0, r0+8) of a block, spread over the MFMA slots of a
    // phase as three separate stages (scale-and-shift, exp2, times S2) in consecutive slots: a
    // slot then holds independent instructions only, so the single wave of the SIMD never
    // waits on the latency of its own previous vector instruction.
    // With MASKED, `lim` is this lane's largest allowed key offset inside the block (its 4*h
    // already subtracted) and, with a sliding window, `lo` its smallest: register r holds key
    // offset 8*(r/4) + r%4.
    // last key this lane's row may see
    int row_lim;
    row_lim = no_tiles ? -1 : (CAUSAL ? min(my_row + off, Tv - 1) : Tv - 1);
    // The 8 chains (register r0 + u) of a phase, one after the other.
    auto exp_stages = [&](auto masked_tag, auto sums_tag, f32x16 &s1, f32x16 &s2, int r0, int slot,
                          int slot0, int n_slots, const float &neg_m, const int &lim, const int &lo,
                          float(&acc1)[2], float(&acc2)[2]) __attribute__((always_inline)) {
        constexpr bool MASKED = decltype(masked_tag)::value;
        constexpr bool SUMS = decltype(sums_tag)::value;  // a fourth stage adds P1, P2 to acc1, acc2
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int r = r0 + u;
            // stages in slots first, first+1, first+2 (, first+3); none before slot0, none in
            // the last two
            const int first = slot0 + u * (n_slots - (SUMS ? 5 : 4) - slot0) / 8;
            if constexpr (SUMS)
                if (slot == first + 3) {
                    acc1[u & 1] += s1[r];
                    if constexpr (USE_R) acc2[u & 1] += s2[r];
                }
            if (slot == first) s1[r] = fmaf(s1[r], row_scale, neg_m);
            if (slot == first + 1) {
                const float p1 = fast_exp2(s1[r]);
                const int key_off = 8 * (r >> 2) + (r & 3);
                const bool seen = !MASKED || (key_off <= lim && (!WINDOW || key_off >= lo));
                s1[r] = seen ? p1 : 0.f;
            }
            // P2: S2 is finite (rows past the last key re-read it) and P1 = 0 where masked
            if constexpr (USE_R)
                if (slot == first + 2) s2[r] = s1[r] * s2[r];
        }
    };
    auto pack_group = [&](const f32x16 &s, int j) __attribute__((always_inline)) {
        return u32x4{pack_bf16(s[8 * j + 0], s[8 * j + 1]), pack_bf16(s[8 * j + 2], s[8 * j + 3]),
                     pack_bf16(s[8 * j + 4], s[8 * j + 5]), pack_bf16(s[8 * j + 6], s[8 * j + 7])};
    };
    auto pipeline_step = [&](auto masked_tag, auto dma_tag, int key_base_cur, int key_base_next, const u32x4 *tk_next,
                             const unsigned short *tv_cur, const u32x4 *tk_after, f32x16 &sc1,
                             f32x16 &sc2, f32x16 &sn1, f32x16 &sn2) __attribute__((always_inline)) {
        int lim_cur, lim_next, lo_cur, lo_next;  // current block, next block
        float neg_m;
        lim_cur = row_lim - key_base_cur - 4 * h;
        lim_next = row_lim - key_base_next - 4 * h;
        lo_cur = row_lo - key_base_cur - 4 * h;
        lo_next = row_lo - key_base_next - 4 * h;
        neg_m = -m_ref;
        constexpr int SLOTS1 = 2 * KSTEPS;               // phase 1: one slot per score MFMA
        constexpr bool DMA = decltype(dma_tag)::value;  // this step also fetches tile (dma_tk, dma_tv)
        constexpr bool MASKED = decltype(masked_tag)::value;
        // Row sums of the CURRENT block belong to this step. Masked steps (a row may see only a
        // few keys, so the sums must be those of the rounded operands exactly): two MFMAs against
        // ones per key group. Unmasked steps: vector adds of the fp32 values,
        // which stay in the score registers until the next step -- upper key group behind its
        // exp stages in phase 1, lower key group (finished by the previous step) during phase 2.
        constexpr bool SUMS = !MASKED;
        constexpr int PV = 2 * NDB;                      // PV MFMAs per key group
        constexpr int GROUP2 = PV + (!SUMS && MFMA_SUMS ? 2 : 0);  // phase 2, per key group: PV (+ row sums)
        constexpr int SLOTS2 = 2 * GROUP2;
        // (row cache: masked steps add the fp32 values as well, to sums of their own)
        constexpr bool ADDS = SUMS || STATS;
        const std::integral_constant<bool, ADDS> sums_tag{};
        float(&acc1)[2] = SUMS ? vsum1 : msum1;
        float(&acc2)[2] = SUMS ? vsum2 : msum2;
        static_assert(NDMA_K <= KSTEPS && NDMA_V <= GROUP2, "one tile load per odd slot");
        u32x4 nb1, nb2;  // lower key group of the next block as operands
        nb1 = nb2 = u32x4{0u, 0u, 0u, 0u};
        // ---- phase 1: scores of the next block | upper key group of the current block ------
        // slot = (k-step, S1 | S2): a K fragment serves two MFMAs in a row
#pragma unroll
        for (int sl = 0; sl < SLOTS1; ++sl) {
            const int ks = sl / 2;
            if (sl % 2 == 0) {
                if (ks == 0)
                    mfma32_scores_first<MASKED, !TWO>(sn1, kf[ks], qf[ks]);
                else
                    mfma32_scores<MASKED, !TWO>(sn1, kf[ks], qf[ks]);
                prefetch(ks, tk_next, tv_cur, tk_after);
            } else if constexpr (USE_R) {
                if (ks == 0)
                    mfma32_scores_first<MASKED, !TWO>(sn2, kf[ks], rf[ks]);
                else
                    mfma32_scores<MASKED, !TWO>(sn2, kf[ks], rf[ks]);
            }
            if constexpr (DMA)
                if (sl % 2 == 1 && sl / 2 < NDMA_K) k_load(sl / 2, dma_tk, dma_dk);
            exp_stages(masked_tag, sums_tag, sc1, sc2, 8, sl, 0, SLOTS1, neg_m, lim_cur, lo_cur, acc1, acc2);
            // upper key group -> operands, in the last two slots
            if (sl == SLOTS1 - 2) pb1[1] = pack_group(sc1, 1);
            if (sl == SLOTS1 - 1) {
                if constexpr (USE_R) pb2[1] = pack_group(sc2, 1);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // ---- phase 2: PV + row sums of the current block | lower key group of the next block
        // The scores just issued are first read in slot 1, i.e. behind the PV MFMAs of slots 0
        // and 1. A wave issues in order and an MFMA is only accepted once the matrix pipe has
        // room, so by then the last score MFMA has retired: no wait states needed.
#pragma unroll
        for (int sl = 0; sl < SLOTS2; ++sl) {
            const int j = sl / GROUP2, t = sl % GROUP2;
            if (t < PV) {
                const int n = t / 2, f = j * NDB + n;
                if (t % 2 == 0) {
                    o1[n] = mfma32(vt[f], pb1[j], o1[n]);
                    prefetch(KSTEPS + f, tk_next, tv_cur, tk_after);
                } else if constexpr (USE_R) {
                    o2[n] = mfma32(vt[f], pb2[j], o2[n]);
                }
            } else if constexpr (MFMA_SUMS) {
                if ((t - PV) % 2 == 0)
                    dacc = mfma32(ones_top, pb1[j], dacc);
                else if constexpr (USE_R)
                    dacc = mfma32(ones_bot, pb2[j], dacc);
            }
            if constexpr (!SUMS && !MFMA_SUMS) {  // rounded operands of key group j, one operand per slot
                if (t < 2) {
                    if (t % 2 == 0)
                        add_rounded(pb1[j], rsum1);
                    else if constexpr (USE_R)
                        add_rounded(pb2[j], rsum2);
                }
            }
            if constexpr (DMA)
                if (sl % 2 == 1 && sl / 2 < NDMA_V) v_load(sl / 2, dma_tv, dma_dv);
            exp_stages(masked_tag, std::false_type{}, sn1, sn2, 0, sl, 1, SLOTS2, neg_m, lim_next, lo_next, acc1,
                       acc2);
            if constexpr (ADDS) {
                constexpr int PER = SLOTS2 / 8;  // lower key group of the current block
                if (sl % PER == 0 && sl / PER < 8) {
                    const int r = sl / PER;
                    acc1[r & 1] += sc1[r];
                    if constexpr (USE_R) acc2[r & 1] += sc2[r];
                }
            }
            if (sl == SLOTS2 - 2) nb1 = pack_group(sn1, 0);
            if (sl == SLOTS2 - 1) {
                if constexpr (USE_R) nb2 = pack_group(sn2, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        pb1[0] = nb1;
        pb2[0] = nb2;
    };

    // =========================== fast pass: fixed reference ================================
    // Ring invariant at the top of iteration kt: tiles kt and (after the barrier) kt+1 are in
    // stages kt % 3 and (kt+1) % 3 and visible to all waves. The barrier (every wave first waits
    // for its own tile loads) also proves that nobody reads tile kt-1 any more, whose stage then
    // receives tile kt+2: each tile load has a whole iteration to land.
    // load n of the first two tiles (tile 0 first, K before V), for issuing them one at a time
    auto initial_load = [&](int n) __attribute__((always_inline)) {
        const int t = n / kTileLoads, i = n % kTileLoads;
        if (Tk >= kDist * kBC) {  // workgroup-uniform: whole tiles, uniform base + lane offsets
            if (i < NDMA_K)
                k_load(i, (const char *)kbase + t * k_tile_bytes, stage_k_addr(t));
            else
                v_load(i - NDMA_K, (const char *)vbase + t * v_tile_bytes, stage_v_addr(t));
        } else {
            int row, pos;
            if (i < NDMA_K) {
                k_src(i, row, pos);
                const __bf16 *sk = kbase + (int64_t)min(t * kBC + row, Tk - 1) * p.ks[2] + pos * 8;
                if (i == NDMA_K - 1)
                    tile_load16<16>(sk, stage_k_addr(t) + 1024u * i);
                else
                    tile_load16<64>(sk, stage_k_addr(t) + 1024u * i);
            } else {
                v_src(i - NDMA_K, row, pos);
                const __bf16 *sv = vbase + (int64_t)min(t * kBC + row, Tk - 1) * p.vs[2] + pos * 8;
                tile_load16<64>(sv, stage_v_addr(t) + 1024u * (i - NDMA_K));
            }
        }
    };
    static_assert(kDist == 2, "the wait below leaves exactly tile 1 in flight");
    if constexpr (!PREP) {
        if constexpr (SPARSE) {  // (the clamping form only: it needs no per-lane offsets kept alive)
#pragma unroll
            for (int t = 0; t < kDist; ++t) dma_tile(tile_at(t), t);
        } else if (Tk >= kDist * kBC) {  // workgroup-uniform
#pragma unroll
            for (int t = 0; t < kDist; ++t) dma_full_tile(t, t);
        } else {
#pragma unroll
            for (int t = 0; t < kDist; ++t) dma_tile(t, t);
        }
        zero_state();
    } else {
        // Normalise, rotate and round this wave's Q and R rows where they landed (nobody else
        // reads them). Per row: sum of squares over the CPR lanes of the row, y = x / sqrt(mean
        // + eps) * gamma, then the adjacent pairs (2i, 2i + 1) turned by the row's angle.
        // (Issuing the loads of the first two key tiles between the row passes instead of in
        // front of them was tried: no faster.)
#pragma unroll
        for (int n = 0; n < kDist * kTileLoads; ++n) initial_load(n);
        zero_state();
        // this wave's Q and R rows (and the table entries) are there; the two tiles may still travel
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kDist * kTileLoads) : "memory");
        const int lr = lane % CPR, lrow = lane / CPR;
        u32x4 *zq = lds + QZONE + w * WAVE_TILE_CHUNKS, *zr = lds + RZONE + w * WAVE_TILE_CHUNKS;
        const float inv_d = 1.0f / (float)D;
        // sum of squares of the 8 bf16 values of a chunk (dot products of the packed pairs with
        // themselves), over the CPR lanes of the row; 1 / rms
        auto inv_rms = [&](const u32x4 &c) __attribute__((always_inline)) {
            float ss = 0.f;
#pragma unroll
            for (int e = 0; e < 3; ++e) asm("v_dot2c_f32_bf16_e32 %0, %1, %1" : "+v"(ss) : "v"(c[e]));
            // (the result of a dot product needs three wait states before another kind of
            // instruction reads it; the compiler does not see the instruction, so they are here)
            asm("v_dot2c_f32_bf16_e32 %0, %1, %1\n\ts_nop 2" : "+v"(ss) : "v"(c[3]));
            ss = lane_group_sum<CPR>(ss);  // the CPR lanes of a row are an aligned group
            return __builtin_amdgcn_rsqf(fmaf(ss, inv_d, p.prep.eps));
        };
        // gamma, then (unless ROT is off) the rotation of the four pairs; NOT the 1 / rms factor
        auto scale_rotate = [&](auto rot_tag, const u32x4 &c, const f32x4(&gam)[2], const f32x4(&tab)[2])
                                __attribute__((always_inline)) {
            u32x4 out;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float y0 = bf16_lo_f32(c[j]) * gam[j >> 1][2 * (j & 1)];
                float y1 = bf16_hi_f32(c[j]) * gam[j >> 1][2 * (j & 1) + 1];
                if constexpr (decltype(rot_tag)::value) {
                    const float cs = tab[j >> 1][2 * (j & 1)], sn = tab[j >> 1][2 * (j & 1) + 1];
                    const float r0 = y0 * cs - y1 * sn, r1 = y0 * sn + y1 * cs;
                    y0 = r0, y1 = r1;
                }
                out[j] = pack_bf16(y0, y1);
            }
            return out;
        };
        // The 1 / rms of a row goes to the padding chunk of the row (no fragment reads it), from
        // where the lane that owns the row in the MFMA layout picks it up below.
        auto prep_rows = [&](auto rot_q_tag, auto rot_r_tag) __attribute__((always_inline)) {
#pragma unroll
            for (int it = 0; it < PREP_NIT; ++it) {
                const int row = it * PREP_RPI + lrow, slot = row * KROW + lr;
                const u32x4 cq = zq[slot], cr = zr[slot];
                const float iq = inv_rms(cq), ir = inv_rms(cr);
                zq[slot] = scale_rotate(rot_q_tag, cq, prep_gq, prep_tab[it]);
                zr[slot] = scale_rotate(rot_r_tag, cr, prep_gr, prep_tab[it]);
                if (lr == 0) {
                    *(float *)&zq[row * KROW + CPR] = iq;
                    *(float *)&zr[row * KROW + CPR] = ir;
                }
            }
        };
        // (rotation switches are uniform over the launch: one specialised copy of the pass each)
        if (p.prep.rope_q != 0 && p.prep.rope_r != 0)
            prep_rows(std::true_type{}, std::true_type{});
        else if (p.prep.rope_q != 0)
            prep_rows(std::true_type{}, std::false_type{});
        else
            prep_rows(std::false_type{}, std::false_type{});
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        row_scale = scale_log2 * *(const float *)&zq[col * KROW + CPR];
        r_gain = *(const float *)&zr[col * KROW + CPR];
    }
    tile_barrier<kTileLoads>();  // Q, R and tile 0 have landed
    {
        // B operands: column = query row, k-elements = the 8 dims of chunk 2*ks + h
        const u32x4 *zq = lds + QZONE + w * WAVE_TILE_CHUNKS + col * KROW + h;
        const u32x4 *zr = lds + RZONE + w * WAVE_TILE_CHUNKS + col * KROW + h;
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) {
            qf[ks] = zq[2 * ks];
            if constexpr (USE_R) rf[ks] = zr[2 * ks];
        }
    }
    int stage = 0;
    f32x16 sa1, sa2, sb1, sb2;
    {
        // Pipeline prologue: scores of block (0, 0); reference = its row maximum (key 0 is
        // visible to every row); lower key group -> P. (Everything the loops read from registers
        // loaded out of global memory -- the Q, R fragments -- is consumed here first, so the
        // loops contain no wait on the vector-memory counter, which the tile loads in flight
        // would turn into a full memory round trip.)
        scores(0, half, sa1, sa2);
        if constexpr (!PAIR)
#pragma unroll
            for (int f = 0; f < kLookAhead; ++f) load_kfrag(k_block_ptr(0, 1), f);
        int kb0 = tile_at(0) * kBC;  // 0 unless block-sparse
        if constexpr (SPARSE) asm volatile("" : "+s"(kb0));  // (opaque, for the same reason as n_tiles)
        float neg_m;
        int lim0, lo0;
        float tmax = kNegInf, tall = kNegInf;
        if constexpr (PAIR) {
            // both waves of a pair take the maximum of block (0, 0): P as a whole row block forms it
            f32x16 s0;
#pragma unroll
            for (int r = 0; r < 16; ++r) s0[r] = 0.f;
#pragma unroll
            for (int ks = 0; ks < KSTEPS; ++ks) s0 = mfma32(k_block_ptr(0, 0)[2 * ks], qf[ks], s0);
#pragma unroll
            for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, key_ok(0, r) ? s0[r] : kNegInf);
            if constexpr (WINDOW) {
#pragma unroll
                for (int r = 0; r < 16; ++r) tall = fmaxf(tall, s0[r]);
            }
        } else if constexpr (SPLIT) {
            // Every range takes the reference of the whole launch, so that it forms and rounds the very
            // same P. (A range of its own block's maximum would be as safe, but rounds P
            // against another scale: outputs apart by the bf16 bound, and by 2^-9 from exact where one key
            // has all the weight.) A range far below the reference adds what it would add there.
            f32x16 s0;
#pragma unroll
            for (int r = 0; r < 16; ++r) s0[r] = 0.f;
#pragma unroll
            for (int ks = 0; ks < KSTEPS; ++ks) s0 = mfma32(k_ref[ks], qf[ks], s0);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int key = 8 * (r >> 2) + 4 * h + (r & 3);
                tmax = fmaxf(tmax, key < p.Tk && (!CAUSAL || key <= my_row + (p.Tk - T)) ? s0[r] : kNegInf);
            }
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, key_ok(kb0, r) ? sa1[r] : kNegInf);
        }
        tmax = halves_max(tmax);
        if constexpr (WINDOW || SPARSE) {
            // a row whose window starts behind this block takes the block's plain maximum: any
            // finite reference will do (the check after the loops catches one that was too far off)
            if constexpr (!PAIR) {
#pragma unroll
                for (int r = 0; r < 16; ++r) tall = fmaxf(tall, sa1[r]);
            }
            tall = halves_max(tall);
            tmax = tmax == kNegInf ? tall : tmax;
        }
        m_ref = tmax * row_scale;
        neg_m = -m_ref;
        lim0 = row_lim - kb0 - half * kKB - 4 * h;
        lo0 = row_lo - kb0 - half * kKB - 4 * h;
#pragma unroll
        for (int sl = 0; sl < 12; ++sl)
            exp_stages(std::true_type{}, std::false_type{}, sa1, sa2, 0, sl, 0, 12, neg_m, lim0, lo0, msum1, msum2);
        pb1[0] = pack_group(sa1, 0);
        if constexpr (USE_R) pb2[0] = pack_group(sa2, 0);
    }
    // kt: key tile in `stage`, kt_next: key tile in `next_stage` (kt + 1 unless block-sparse)
    auto tile_steps = [&](auto masked_tag, auto dma_tag, int kt, int kt_next, int stage, int next_stage, f32x16 &sa1,
                          f32x16 &sa2, f32x16 &sb1, f32x16 &sb2) __attribute__((always_inline)) {
        if constexpr (PAIR) {
            // block (kt, half) -> P, PV; scores of (kt_next, half), whose first fragments are read now
            const u32x4 *tk_next = k_block_ptr(next_stage, half);
#pragma unroll
            for (int f = 0; f < kLookAhead; ++f) load_kfrag(tk_next, f);
            pipeline_step(masked_tag, dma_tag, kt * kBC + half * kKB, kt_next * kBC + half * kKB, tk_next,
                          v_block_ptr(stage, half), nullptr, sa1, sa2, sb1, sb2);
            return;
        }
        // block (kt,0) -> P, PV; scores of (kt,1); K fragments of (kt_next,0); loads of the tile after
        pipeline_step(masked_tag, dma_tag, kt * kBC, kt * kBC + kKB, k_block_ptr(stage, 1),
                      v_block_ptr(stage, 0), k_block_ptr(next_stage, 0), sa1, sa2, sb1, sb2);
        // block (kt,1) -> P, PV; scores of (kt_next,0); K fragments of (kt_next,1)
        pipeline_step(masked_tag, std::false_type{}, kt * kBC + kKB, kt_next * kBC, k_block_ptr(next_stage, 0),
                      v_block_ptr(stage, 1), k_block_ptr(next_stage, 1), sb1, sb2, sa1, sa2);
    };
    // One tile of the pipeline with per-lane key masks. Blocks a wave cannot see at all
    // contribute exact zeros.
    auto masked_tile = [&](int kt, f32x16 &sa1, f32x16 &sa2, f32x16 &sb1, f32x16 &sb2)
                           __attribute__((always_inline)) {
        const int next_stage = stage == STAGES - 1 ? 0 : stage + 1;
        const int free_stage = stage == 0 ? STAGES - 1 : stage - 1;
        tile_barrier();
        if (kt + kDist < n_tiles) {              // workgroup-uniform
            const int k2 = tile_at(kt + kDist);
            if (!SPARSE && (k2 + 1) * kBC <= Tk)  // the tile exists completely
                dma_full_tile(k2, free_stage);
            else
                dma_tile(k2, free_stage);
        }
        tile_steps(std::true_type{}, std::false_type{}, tile_at(kt), tile_at(kt + 1), stage, next_stage, sa1, sa2, sb1, sb2);
        stage = next_stage;
    };
    // PAIR: tiles go by twos, as a step hands its score registers over to the next one in the other set; the
    // odd last tile is a step of its own (left by a break, the loop spills)
    auto masked_tiles = [&](int &kt, int end) __attribute__((always_inline)) {
        while (kt < end) {
            masked_tile(kt, sa1, sa2, sb1, sb2);
            ++kt;
            if constexpr (PAIR) {
                masked_tile(kt, sb1, sb2, sa1, sa2);
                ++kt;
            }
        }
    };
    int kt = 0;
    // Sliding window: the leading tiles are cut by the left edge of some row's window.
    if constexpr (WINDOW) masked_tiles(kt, PAIR ? min((n_left + 1) & ~1, n_tiles & ~1) : n_left);
    // Tiles whose keys -- and those of the tile after -- are visible to every row: no masks, a
    // branch-free body. (A step also prepares the lower half of the NEXT block, hence the -1.)
    dma_tk = (const char *)kbase + (kt + kDist) * k_tile_bytes;
    dma_tv = (const char *)vbase + (kt + kDist) * v_tile_bytes;
    auto full_tile = [&](int kt, f32x16 &sa1, f32x16 &sa2, f32x16 &sb1, f32x16 &sb2)
                         __attribute__((always_inline)) {
        const int next_stage = stage == STAGES - 1 ? 0 : stage + 1;
        const int free_stage = stage == 0 ? STAGES - 1 : stage - 1;  // held tile kt - 1
        // tile kt + 1 has landed; the kDist - 2 tiles after it may still be in flight
        tile_barrier<(kDist - 2) * kTileLoads>();
        dma_dk = stage_k_addr(free_stage);  // tile kt + kDist <= T/64 - 1 in this loop: complete
        dma_dv = stage_v_addr(free_stage);
        if constexpr (SPARSE) {
            // (a list that does not ascend gives wrong results, but never a read past the last key)
            const int k2 = min(tile_at(kt + kDist), Tk / kBC - 1);
            dma_tk = (const char *)kbase + k2 * k_tile_bytes;
            dma_tv = (const char *)vbase + k2 * v_tile_bytes;
        }
        tile_steps(std::false_type{}, std::true_type{}, tile_at(kt), tile_at(kt + 1), stage, next_stage, sa1, sa2, sb1, sb2);
        if constexpr (!SPARSE) {
            dma_tk += k_tile_bytes;
            dma_tv += v_tile_bytes;
        }
        stage = next_stage;
    };
    const int full_end = PAIR ? kt + (max(n_full - 1 - kt, 0) & ~1) : n_full - 1;
    for (; kt < full_end; ++kt) {
        full_tile(kt, sa1, sa2, sb1, sb2);
        if constexpr (PAIR) full_tile(++kt, sb1, sb2, sa1, sa2);
    }
    // Remaining tiles (diagonal / tail): the same pipeline with per-lane key masks.
    masked_tiles(kt, PAIR ? n_tiles & ~1 : n_tiles);
    if (PAIR && kt < n_tiles) {
        masked_tile(kt, sa1, sa2, sb1, sb2);
        keep_blocks(sb1, sb2);  // (unused, but nothing else may move in before they are written)
    }
    // ---- closing formula into the wave's staging tile, and the check of the fast pass -------
    // O^T register r of block n <-> dim 32n + 8*(r/4) + 4h + r%4 of row my_row. A lane owns one
    // output ROW, so direct stores would scatter 8 bytes over 32 rows per instruction; the wave
    // instead transposes its 32 x D tile through LDS (its Q landing zone, which nobody else
    // touches) and later writes whole 256-byte rows, 16 bytes a lane.
    // The same pass over the accumulators decides whether the fixed reference held: an inf / NaN
    // anywhere in the sums or accumulators (the reference was too small) shows as a non-finite
    // row sum or output. Only then the workgroup redoes its rows with the online update below
    // and comes back here once more.
    constexpr int OROW = CPR + 1;  // padded row of the staging tile, in 16-byte chunks
    static_assert(OROW == KROW, "the staging tile is the wave's Q tile");
    u32x4 *otile = lds + QZONE + (PAIR ? w & 1 : w) * WAVE_TILE_CHUNKS;  // (PAIR: of both waves, each its dimensions)
    unsigned short *otile16 = (unsigned short *)otile;
    float inv, dsum1, dsum2s;
    // PAIR: the sums of the two waves of a pair, each exact on its keys under its own reference (the same one
    // unless they took the online update). Through the ring, which nobody reads any more: a wave hands over
    // the other's half of the dimensions and the row scalars, and ends up with everything of its own half.
    constexpr int NOWN = PAIR ? NDB / 2 : NDB;
    auto owned = [&](int n) __attribute__((always_inline)) { return !PAIR || n / NOWN == half; };  // (wave-uniform)
    float psum1 = 0.f, psum2 = 0.f, pfsum1 = 0.f, pfsum2 = 0.f;  // PAIR: row sums of both waves
    auto merge_halves = [&]() __attribute__((always_inline)) {
        constexpr int ACC = 2 * NOWN * 4 * 64, ROWSC = 5 * 64 / 4;  // chunks per wave: accumulators, row scalars
        static_assert(!PAIR || 4 * (ACC + ROWSC) <= QZONE, "the ring");
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // tile loads past the end have landed
        __syncthreads();
        f32x4 *mine = (f32x4 *)lds + w * (ACC + ROWSC), *theirs = (f32x4 *)lds + (w ^ 2) * (ACC + ROWSC);
        float *sc = (float *)(mine + ACC) + lane, *osc = (float *)(theirs + ACC) + lane;
        float d1, d2;  // (as in stage_outputs)
        if constexpr (MFMA_SUMS) {
            d1 = dacc[0] + halves_sum(vsum1[0] + vsum1[1]);
            d2 = dacc[8] + halves_sum(vsum2[0] + vsum2[1]);
        } else {
            d1 = halves_sum(rsum1 + vsum1[0] + vsum1[1]);
            d2 = halves_sum(rsum2 + vsum2[0] + vsum2[1]);
        }
        const float f1 = halves_sum(vsum1[0] + vsum1[1] + msum1[0] + msum1[1]);
        const float f2 = halves_sum(vsum2[0] + vsum2[1] + msum2[0] + msum2[1]);
        sc[0] = m_ref, sc[64] = d1, sc[128] = d2;
        if constexpr (STATS) sc[192] = f1, sc[256] = f2;
        auto give = [&](auto first) __attribute__((always_inline)) {
#pragma unroll
            for (int n = 0; n < NOWN; ++n)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    const f32x16 &x = o1[decltype(first)::value + n], &y = o2[decltype(first)::value + n];
                    mine[lane + 64 * (4 * n + q4)] = f32x4{x[4 * q4], x[4 * q4 + 1], x[4 * q4 + 2], x[4 * q4 + 3]};
                    if constexpr (USE_R)
                        mine[lane + 64 * (4 * (NOWN + n) + q4)] = f32x4{y[4 * q4], y[4 * q4 + 1], y[4 * q4 + 2], y[4 * q4 + 3]};
                }
        };
        const std::integral_constant<int, 0> lower{};
        const std::integral_constant<int, PAIR ? NOWN : 0> upper{};
        // (the empty statements keep the two branches apart: merged, they would pick their accumulators
        // through a pointer, and those would live in scratch memory)
        if (half == 0) {  // (wave-uniform)
            give(upper);
            asm volatile("; upper dimensions handed over");
        } else {
            give(lower);
        }
        __syncthreads();
        const float m = fmaxf(m_ref, osc[0]), m_use = m == kNegInf ? 0.f : m;
        const float fm = fast_exp2(m_ref - m_use), ft = fast_exp2(osc[0] - m_use);  // (1 under one reference)
        psum1 = d1 * fm + osc[64] * ft, psum2 = d2 * fm + osc[128] * ft;
        if constexpr (STATS) pfsum1 = f1 * fm + osc[192] * ft, pfsum2 = f2 * fm + osc[256] * ft;
        m_ref = m;
        auto take = [&](auto first) __attribute__((always_inline)) {
#pragma unroll
            for (int n = 0; n < NOWN; ++n)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    f32x16 &x = o1[decltype(first)::value + n], &y = o2[decltype(first)::value + n];
                    const f32x4 u = theirs[lane + 64 * (4 * n + q4)];
#pragma unroll
                    for (int i = 0; i < 4; ++i) x[4 * q4 + i] = x[4 * q4 + i] * fm + u[i] * ft;
                    if constexpr (USE_R) {
                        const f32x4 v = theirs[lane + 64 * (4 * (NOWN + n) + q4)];
#pragma unroll
                        for (int i = 0; i < 4; ++i) y[4 * q4 + i] = y[4 * q4 + i] * fm + v[i] * ft;
                    }
                }
        };
        if (half == 0) {
            take(lower);
            asm volatile("; lower dimensions complete");
        } else {
            take(upper);
        }
    };
    if constexpr (PAIR) merge_halves();
    auto stage_outputs = [&]() __attribute__((always_inline)) {
        float chk = 0.f;
        // Every row of the MFMA row-sum accumulators holds the sum over this lane's query row;
        // the per-lane partial sums cover this lane's keys only: add the other half-wave's.
        float dsum2;
        if constexpr (PAIR) {
            dsum1 = psum1, dsum2 = psum2;
        } else if constexpr (MFMA_SUMS) {
            dsum1 = dacc[0] + halves_sum(vsum1[0] + vsum1[1]);
            dsum2 = dacc[8] + halves_sum(vsum2[0] + vsum2[1]);
        } else {
            dsum1 = halves_sum(rsum1 + vsum1[0] + vsum1[1]);
            dsum2 = halves_sum(rsum2 + vsum2[0] + vsum2[1]);
        }
        if constexpr (PREP) dsum2 *= r_gain;
        if constexpr (SPLIT) dsum2s = dsum2;
        inv = dsum1 > 0.f ? 1.f / dsum1 : 0.f;  // empty key set: zeros
        const float gain = inv * (1.f + dsum2 * inv);
        const float inv2 = PREP ? inv * r_gain : inv;
        chk = fmaf(dsum1 + dsum2, 0.f, chk);  // inf or NaN -> NaN
#pragma unroll
        for (int n = 0; n < NDB; ++n)
            if (owned(n))
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    float y[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int r = 4 * q4 + i;
                        y[i] = o1[n][r] * gain - (USE_R ? o2[n][r] * inv2 : 0.f);
                        chk = fmaf(y[i], 0.f, chk);
                    }
                    const u32x2 packed = {pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3])};
                    *(u32x2 *)(otile16 + col * (OROW * 8) + 32 * n + 8 * q4 + 4 * h) = packed;
                }
        return chk;
    };
    if constexpr (TWO && !PAIR) {  // (the staging tiles reach into ring stage 2)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    }
    float chk = stage_outputs();
    if constexpr (WINDOW || SPARSE) {
        // the reference of a row may come from keys outside its window; if it was so far above
        // the row's own scores that the sum underflowed, take the exact path as well
        // (block-sparse: only for rows that do see a listed key -- the list is ascending, so that
        // is decided by its first tile)
        if (my_row < T && (!SPARSE || tile_at(0) * kBC <= row_lim) && !(dsum1 > 1e-30f)) chk = 1.f;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // tile loads past the end have landed
    const bool overflow = __syncthreads_or(chk != 0.f);  // NaN != 0 is true; all waves agree

    // =========================== fallback: online max / rescale ============================
    if (overflow) {
        zero_state();
        vsum1[0] = vsum1[1] = vsum2[0] = vsum2[1] = 0.f;
        msum1[0] = msum1[1] = msum2[0] = msum2[1] = 0.f;
        m_ref = kNegInf;
        dma_tile(tile_at(0), 0);
        stage = 0;
        for (int t = 0; t < n_tiles; ++t) {
            const int next_stage = stage == STAGES - 1 ? 0 : stage + 1;
            tile_barrier();  // tile t has landed; tile t-2's stage is free for tile t+1
            dma_tile(tile_at(t + 1), next_stage);
#pragma unroll 1
            for (int kb = 0; kb < kBC / kKB; ++kb) {
                if (PAIR && kb != half) continue;
                const int key_base = tile_at(t) * kBC + kb * kKB;
                if (!block_visible(key_base)) continue;
                scores(stage, kb, sa1, sa2);
                float tmax = kNegInf;
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    tmax = fmaxf(tmax, key_ok(key_base, r) ? sa1[r] * row_scale : kNegInf);
                tmax = halves_max(tmax);
                const float m_new = fmaxf(m_ref, tmax);
                const float m_use = m_new == kNegInf ? 0.f : m_new;
                const float alpha = fast_exp2(m_ref - m_use);  // 0 while m_ref = -inf
                m_ref = m_new;
                if constexpr (STATS) {
                    msum1[0] *= alpha, msum1[1] *= alpha;
                    msum2[0] *= alpha, msum2[1] *= alpha;
                }
                if constexpr (!MFMA_SUMS) rsum1 *= alpha, rsum2 *= alpha;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    if constexpr (MFMA_SUMS) dacc[r] *= alpha;
#pragma unroll
                    for (int n = 0; n < NDB; ++n) {
                        o1[n][r] *= alpha;
                        if constexpr (USE_R) o2[n][r] *= alpha;
                    }
                }
                probs(std::true_type{}, key_base, sa1, sa2, pb1, pb2);
                accumulate(stage, kb, pb1, pb2);
            }
            stage = next_stage;
        }
        tile_barrier();  // outstanding tile loads land before the workgroup may exit
        if constexpr (PAIR) merge_halves();
        (void)stage_outputs();
        if constexpr (PAIR) __syncthreads();
    }

    // ---- SPLIT, more than one key range: the record of every row ----------------------------
    // Laid out by accumulator: [float4 block (O1, O2; dimension block n, q4)][half-wave][row], so that
    // every store of a wave is one contiguous KB, then the row scalars.
    // A range keeps its reference (the maximum of the first 32 keys of all) as long as its sums are finite,
    // so it may weigh up to 2^128 times that, beside ranges that took the online update and have
    // another. Its record is therefore scaled by 2^-exponent of d1 (exact) with
    // the exponent added to the reference: every d1 is in [0.5, 1), the references compare what the
    // ranges weigh, and the merge neither overflows nor flushes the weight of a range that counts.
    if constexpr (SPLIT)
        if (n_ranges > 1) {
            const int64_t slot = ((int64_t)b * p.Hq + hq) * p.items_per_head + item;
            if (row0 >= T) return;  // (wave-uniform) no such rows
            float *rec = p.ws + (slot * 4 + w) * prefill_record_floats(D);
            f32x4 *ob = (f32x4 *)rec + 32 * h + col;
            const int e = __builtin_amdgcn_frexp_expf(dsum1);  // (0 for 0, inf and NaN)
            auto scaled = [&](float x) __attribute__((always_inline)) { return __builtin_amdgcn_ldexpf(x, -e); };
            auto scaled4 = [&](const f32x16 &x, int q4) __attribute__((always_inline)) {
                return f32x4{scaled(x[4 * q4]), scaled(x[4 * q4 + 1]), scaled(x[4 * q4 + 2]), scaled(x[4 * q4 + 3])};
            };
#pragma unroll
            for (int n = 0; n < NDB; ++n)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    ob[64 * (4 * n + q4)] = scaled4(o1[n], q4);
                    if constexpr (USE_R) ob[64 * (4 * (NDB + n) + q4)] = scaled4(o2[n], q4);
                }
            float fsum1 = 0.f, fsum2 = 0.f;  // row cache: sums of the unrounded P1, P2 (see msum1)
            if constexpr (STATS) {
                fsum1 = halves_sum(vsum1[0] + vsum1[1] + msum1[0] + msum1[1]);
                fsum2 = halves_sum(vsum2[0] + vsum2[1] + msum2[0] + msum2[1]);
            }
            if (h == 0) {
                float *row = rec + 64 * D + col;  // [m | d1 | d2 | sums of the unrounded P1 | P2][32 rows]
                row[0] = dsum1 > 0.f ? m_ref + (float)e : kNegInf;
                row[32] = scaled(dsum1);
                row[64] = scaled(dsum2s);
                if constexpr (STATS) row[96] = scaled(fsum1), row[128] = scaled(fsum2);
            }
            return;
        }

    // ---- epilogue: the staged rows go out as whole rows ------------------------------------
    {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        __bf16 *obase = (__bf16 *)p.o + b * p.os[0] + hq * p.os[1];
        constexpr int RPI = 64 / CPR;  // rows covered by one wave-wide 16-byte store
        constexpr int NIT = (PAIR ? WROWS / 2 : WROWS) / RPI;  // PAIR: each wave stores half of the rows
        const int rr0 = PAIR ? half * (WROWS / 2) : 0;
#pragma unroll
        for (int i = 0; i < NIT; ++i) {
            const int rr = rr0 + i * RPI + lane / CPR, chunk = lane % CPR;
            const int row = row0 + rr;
            if (row < T) *(u32x4 *)(obase + (int64_t)row * p.os[2] + chunk * 8) = otile[rr * OROW + chunk];
        }
        if constexpr (STATS) {
            // Row cache for the backward pass (App. D): vbar_i = O1 / d1 through the same
            // staging tile, and per row the log-sum-exp of the scaled scores in the exp2 domain
            // (P1 = exp2(S1 * scale * log2 e - lse) needs no further division) and ubar = d2 / d1.
            // (from the fp32 sums of the unrounded P1, P2 -- see msum1 above)
            const float fsum1 = PAIR ? pfsum1 : halves_sum(vsum1[0] + vsum1[1] + msum1[0] + msum1[1]);
            const float fsum2 = PAIR ? pfsum2 : halves_sum(vsum2[0] + vsum2[1] + msum2[0] + msum2[1]);
            if (h == 0 && half == 0 && my_row < T) {
                float *st = p.row_stats + (((int64_t)b * p.Hq + hq) * T + my_row) * 2;
                // (a row with no visible key stores +inf: the backward's exp2(S1 - lse) is then
                // zero for every pair of the row, whatever the mask arithmetic does)
                st[0] = fsum1 > 0.f ? m_ref + log2f(fsum1) : -kNegInf;
                st[1] = fsum1 > 0.f ? fsum2 / fsum1 : 0.f;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if constexpr (PAIR) __syncthreads();  // (the other wave has read its rows)
#pragma unroll
            for (int n = 0; n < NDB; ++n)
                if (owned(n))
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4) {
                        const u32x2 packed = {pack_bf16(o1[n][4 * q4] * inv, o1[n][4 * q4 + 1] * inv),
                                              pack_bf16(o1[n][4 * q4 + 2] * inv, o1[n][4 * q4 + 3] * inv)};
                        *(u32x2 *)(otile16 + col * (OROW * 8) + 32 * n + 8 * q4 + 4 * h) = packed;
                    }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            if constexpr (PAIR) __syncthreads();
            __bf16 *vbase_out = (__bf16 *)p.vbar + b * p.os[0] + hq * p.os[1];
#pragma unroll
            for (int i = 0; i < NIT; ++i) {
                const int rr = rr0 + i * RPI + lane / CPR, chunk = lane % CPR;
                const int row = row0 + rr;
                if (row < T)
                    *(u32x4 *)(vbase_out + (int64_t)row * p.os[2] + chunk * 8) = otile[rr * OROW + chunk];
            }
        }
    }
}


// Merge of the key ranges of a SPLIT launch (App. C) and the closing formula. A wave finishes one
// block of 32 output dimensions of 32 rows: lane (row, h) holds dimensions 8 q4 + 4 h .. + 3, as the
// records do, so every load is one contiguous KB. Row blocks with one range were written by the
// prefill kernel itself. Memory bound: the records travel twice, 2 x 1 KB per row and range at d = 128
// (512 rows over 16384 keys, 16 heads: 8192 rows x 4 ranges, 34 MB each way).
template <int D, bool USE_R, bool STATS>
__global__ __launch_bounds__(256) void prefill_combine_kernel(PrefillParams p) {
    constexpr int NDB = D / 32, ROWS = 128;
    const int lane = threadIdx.x & 63, col = lane & 31, h = lane >> 5;
    const int nrb = (p.T + ROWS - 1) / ROWS;
    int64_t id = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);  // (batch, head, row block, 32 rows, n)
    const int n = (int)(id % NDB);
    id /= NDB;
    const int sub = (int)(id % 4);
    id /= 4;
    const int rbi = (int)(id % nrb);
    const int64_t bh = id / nrb;
    if (bh >= (int64_t)p.B * p.Hq) return;  // (whole waves)
    const int rb = p.causal ? nrb - 1 - rbi : rbi;
    const int row = rb * ROWS + 32 * sub + col;
    if (rb * ROWS + 32 * sub >= p.T) return;
    int item0 = 0, n_ranges = 1;
    for (int i = 0; i <= rbi; ++i) {
        item0 += i > 0 ? n_ranges : 0;
        const PrefillRanges r(p.causal ? min(p.Tk, (nrb - i) * ROWS + (p.Tk - p.T)) : p.Tk, p.split_tiles);
        n_ranges = r.count;
    }
    if (n_ranges == 1) return;
    auto record = [&](int i) {
        return p.ws + ((bh * p.items_per_head + item0 + i) * 4 + sub) * prefill_record_floats(D);
    };
    float m = kNegInf;
#pragma unroll 8
    for (int i = 0; i < n_ranges; ++i) m = fmaxf(m, record(i)[64 * D + col]);
    const float m_use = m == kNegInf ? 0.f : m;
    float d1 = 0.f, d2 = 0.f, f1 = 0.f, f2 = 0.f;
    f32x4 o1[4], o2[4];
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) o1[q4] = o2[q4] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int i = 0; i < n_ranges; ++i) {
        const float *rec = record(i), *sc = rec + 64 * D + col;
        const f32x4 *ob = (const f32x4 *)rec + 32 * h + col;
        const float wt = fast_exp2(sc[0] - m_use);  // 0 where the range shows the row nothing
        d1 += wt * sc[32], d2 += wt * sc[64];
        if constexpr (STATS) f1 += wt * sc[96], f2 += wt * sc[128];
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            o1[q4] += wt * ob[64 * (4 * n + q4)];
            if constexpr (USE_R) o2[q4] += wt * ob[64 * (4 * (NDB + n) + q4)];
        }
    }
    if (row >= p.T) return;
    const float inv = d1 > 0.f ? 1.f / d1 : 0.f, gain = inv * (1.f + d2 * inv);
    const int64_t b = bh / p.Hq, hq = bh % p.Hq, at = b * p.os[0] + hq * p.os[1] + (int64_t)row * p.os[2] + 32 * n + 4 * h;
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
        f32x4 y = o1[q4] * gain;
        if constexpr (USE_R) y -= o2[q4] * inv;
        *(u32x2 *)((__bf16 *)p.o + at + 8 * q4) = u32x2{pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3])};
        if constexpr (STATS) {
            const f32x4 v = o1[q4] * inv;
            *(u32x2 *)((__bf16 *)p.vbar + at + 8 * q4) = u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
        }
    }
    if constexpr (STATS)
        if (n == 0 && h == 0) {
            float *st = p.row_stats + (bh * p.T + row) * 2;
            st[0] = f1 > 0.f ? m_use + log2f(f1) : -kNegInf;
            st[1] = f1 > 0.f ? f2 / f1 : 0.f;
        }
}

// ---- which form a launch takes -------------------------------------------------------------------
// The estimates below are in us, from three quantities of a launch: its longest workgroup, the load dealt over
// the chip, and what the last round of workgroups finds left to do. Fitted to (and the choice checked on) 3000 launches of
// every form: 1 - 64 heads, 17 - 16384 rows behind 0 - 16384 keys, causal and full, windows, K and V not in the
// L2. The form taken is 0.4 % (d = 64) and 0.2 % (d = 128) behind the fastest one on average, and more than a tenth in 6
// of 2095 and 1 of 901 launches.
struct LaunchCosts {
    double start, tile;            // a workgroup alone on its compute unit: to start and finish, per 64-key tile
    double shared;                 // per tile of a second workgroup on the unit (d = 64)
    double load_start, load_tile;  // per workgroup and tile of a chip that is full
    double tail;                   // of the longest workgroup (in tiles at d = 64), where there are more than fit at once
    double bandwidth;              // bytes per us at which all workgroups get their tiles
};
struct PrefillCosts {
    LaunchCosts whole, pair;                       // 128 rows per workgroup; 64 (PAIR)
    double merge, merge_byte, merge_range;         // key ranges: the second launch, per byte of records written or read, per range of a row
    int resident;                                  // workgroups per compute unit
};
static constexpr PrefillCosts kPrefillCosts64 = {{5.9, 0.765, 0.715, 0.0, 0.82, 0.31, 7.7e6},
                                                 {5.3, 0.61, 0.125, 1.1, 0.50, 0.1, 9.1e6}, 4.7, 0.15e-6, 0.89, 2};
static constexpr PrefillCosts kPrefillCosts128 = {{7.2, 1.145, 0.0, 6.0, 1.43, 0.25, 13.0e6},
                                                  {8.3, 0.755, 0.0, 7.2, 0.70, 0.18, 8.5e6}, 5.0, 0.134e-6, 0.95, 1};

// n workgroups, the longest and the mean of them in tiles; at(rank): tiles of the workgroup of that rank, long ones first
template <class At>
static double launch_us(const LaunchCosts &c, int resident, int num_cus, double n, double longest, double mean,
                        double tile_bytes, At at) {
    const double alone = std::max(c.start + c.tile * longest, n * mean * tile_bytes / c.bandwidth);
    if (n <= num_cus) return alone;
    if (resident == 1) {
        // (workgroup k * num_cus starts behind k others, none of them shorter)
        const double rounds = std::floor((n - 1) / num_cus);
        return std::max({alone, n * (c.load_start + mean * c.load_tile) / num_cus + c.tail * alone,
                         (rounds + 1) * (c.start + c.tile * at(rounds * num_cus))});
    }
    const double both = c.tile + c.shared;  // a unit's two workgroups, per tile of each
    double us = std::max(alone + c.shared * at(num_cus), c.start + n * (c.load_start + mean * c.load_tile) / num_cus +
                                                              (n > 2.0 * num_cus ? c.tail * longest : 0.0));
    const double rounds = std::floor((n - 1) / (2.0 * num_cus)), left = n - 2.0 * rounds * num_cus;
    if (rounds > 0) {
        const double last = at(2.0 * rounds * num_cus);
        us = std::max(us, c.start + rounds * both * last + c.tile * last +
                              (left > num_cus ? c.shared * at((2.0 * rounds + 1) * num_cus) : 0.0));
    }
    return us;
}

// A launch without key ranges, `rows` query rows per workgroup
static double unsplit_us(const PrefillParams &p, int num_cus, int rows, const LaunchCosts &c, int resident) {
    const double heads = (double)p.B * p.Hq, blocks = (p.T + rows - 1) / rows, all = (p.Tk + kBC - 1) / kBC;
    const double span = p.window > 0 ? (p.window + rows - 1.0) / kBC + 1 : 1e30;
    // row block j (from 1) sees `before` + j * `step` tiles under a causal mask
    const double before = (p.Tk - p.T + kBC - 1) / kBC, step = rows / kBC, longest = std::min(all, span);
    double sum = blocks * longest;
    if (p.causal) {
        const double inside = std::min(std::max(std::floor((longest - before) / step), 0.0), blocks);  // blocks below `longest`
        sum = inside * before + step * inside * (inside + 1) / 2 + (blocks - inside) * longest;
    }
    auto at = [&](double rank) {
        return p.causal ? std::min(longest, before + step * (blocks - std::floor(rank / heads))) : longest;
    };
    return launch_us(c, resident, num_cus, heads * blocks, longest, sum / blocks, 4.0 * kBC * p.d, at);
}

// 64 rows per workgroup (PAIR) or 128. Measured us, 128 rows / 64, K and V not in the L2: 16 query heads, d = 128, 200
// rows 11.6 / 10.9, 777 21.2 / 18.2, 1000 24.3 / 20.6, 1500 33.1 / 28.8, 2048 43.7 / 42.1, but 128 8.7 / 9.0, 2500 58.7 / 64.8; 32
// heads, 500 16.5 / 14.8, 777 22.2 / 23.4, 300 over 3300 keys 59.5 / 46.4; 8 heads, 4096 79 / 71, 6000 136 / 144; 64 heads, 267
// over 7471 keys (320 workgroups of 64 rows: two rounds) 152 / 197; d = 64, 32 heads, 300 9.6 / 8.6, 777 15.9 / 13.7, 1500 28.3 /
// 28.5, 64 heads, 777 20.3 / 21.6; 8 heads, 2000 28.6 / 23.9, 4096 52.7 / 45.9, 4 x 250 over 6188 75 / 65.
// The forms differ in the last bits: they add the keys' fp32 terms in different orders, and a tile that only some row of a
// workgroup sees in part (so: other tiles, as workgroups have other rows) is summed after the rounding of P, the others
// before it. 1 x 16 heads x 777 rows, d = 128: 4e-4 apart (relative L2), each 1.7e-3 from 64 bits.
static bool pair_possible(const PrefillParams &p) {
    return p.causal && p.use_r && p.sparse_row_ptr == nullptr && !(p.d == 128 && p.Tk <= 2 * kBC);
}

// Key ranges: the tiles per range with the smallest estimate, where that is below `limit`; 0 = none is.
// A range's workgroup costs what one of 128 rows costs; merging costs a launch, the records' bytes there and
// back, and a step per range of a row. Measured us against the number of ranges of the longest row block, 16 heads, d =
// 128: 512 rows over 16384 keys whole 267, 2 160, 3 128, 4 (the rule) 114, 5 160, 8 135; 1024 over 16384 whole
// 302, 2 (the rule) 207, 3 250, 4 226; 17 over 5000 whole 86, 8 30, 16 34; d = 64 (whole, PAIR, ranges): 8 heads, 28
// rows over 3678 keys 47, 42, 4 24, 6 (the rule) 22, 29 42; 694 over 4540 64, 55, 3 37, 5 (the rule) 36, 9 40; 32 heads, 272 over 13224
// 157, 135, 3 92, 5 (the rule) 86, 8 95; 4 x 8 heads, 250 over 5938 75, 65, 3 40, 4 (the rule) 39, 8 44. A split has to be 3 % ahead.
// The plan is made on every call, on the host (0.6 - 2 us, 7 for 16000 rows), so it estimates no more than it has to: once for row
// blocks that see the same keys (full attention) and for range counts that come to the same tiles, and
// only those counts whose lower bound (the longest and the load alone, as if tiles divided evenly) can still win.
static int choose_split_tiles(const PrefillParams &p, int num_cus, const PrefillCosts &c, double limit, int *items_per_head) {
    constexpr int rows = 128;
    const int nrb = (p.T + rows - 1) / rows;
    const double heads = (double)p.B * p.Hq;
    // A launch that keeps more than half of the units busy leaves most of them two ranges: at d = 128 none of 130 such
    // gained 3 %; at d = 64 a few do where the estimate is well ahead, and more of those with more row blocks than units
    // (3 x 32 heads, 383 rows over 13721 keys 315 whole, 259) unless the row blocks see keys of all lengths: the ranges of the
    // long ones come first, whole long ones behind them (4 heads, 14891 rows square 226, 294).
    const double n_whole = heads * nrb;
    if (nrb > 128 || n_whole >= 2.0 * num_cus || (c.resident == 1 && 2 * n_whole > num_cus)) return 0;
    if (n_whole > num_cus && p.causal && p.T > p.Tk / 4) return 0;
    if (2 * n_whole > num_cus) limit *= n_whole <= num_cus ? 0.88 : 0.97;
    const int kinds = p.causal ? nrb : 1, alike = p.causal ? 1 : nrb;  // row blocks by the keys they see
    auto keys = [&](int i) { return p.causal ? std::min(p.Tk, (nrb - i) * rows + (p.Tk - p.T)) : p.Tk; };
    auto tiles_of = [&](int i) { return (keys(i) + kBC - 1) / kBC; };
    // records of 32 rows of a range, all row blocks of the kind together
    auto subs_of = [&](int i) { return p.causal ? (std::min(rows, p.T - (nrb - 1 - i) * rows) + 31) / 32 : (p.T + 31) / 32; };
    const double record_us = 2 * c.merge_byte * (double)prefill_record_floats(p.d) * sizeof(float), tile_bytes = 4.0 * kBC * p.d;
    double all = 0;
    for (int i = 0; i < kinds; ++i) all += alike * tiles_of(i);
    auto estimate = [&](int tiles, int *items) {
        int64_t n = 0, records = 0;
        for (int i = 0; i < kinds; ++i) {
            const PrefillRanges r(keys(i), tiles);
            n += alike * r.count, records += r.count > 1 ? r.count * subs_of(i) : 0;
        }
        auto at = [&](double rank) {
            double before = 0;
            for (int i = 0;; ++i) {
                const PrefillRanges r(keys(i), tiles);
                before += heads * alike * r.count;
                if (rank < before || i == kinds - 1) return (double)r.tiles;
            }
        };
        *items = (int)n;
        const PrefillRanges longest(keys(0), tiles);
        return launch_us(c.whole, c.resident, num_cus, heads * n, longest.tiles, all / n, tile_bytes, at) + c.merge +
               record_us * heads * records + c.merge_range * longest.count;
    };
    int best = 0, last = tiles_of(0), cut = 0;
    double cut_tiles = 0, cut_records = 0;  // of the row blocks with more than one range: tiles, tiles x records
    for (int ranges = 2; ranges <= 32; ++ranges) {
        const int tiles = (tiles_of(0) + ranges - 1) / ranges;
        if (tiles < 2) break;
        if (tiles == last) continue;
        last = tiles;
        for (; cut < kinds && tiles_of(cut) > tiles; ++cut)  // (ever fewer tiles from row block to row block)
            cut_tiles += alike * tiles_of(cut), cut_records += (double)tiles_of(cut) * subs_of(cut);
        const PrefillRanges longest(keys(0), tiles);
        const double n = heads * (cut_tiles / tiles + alike * (kinds - cut));
        double least = c.whole.start + c.whole.tile * longest.tiles;
        if (n > num_cus)
            least = std::max(least, (n * c.whole.load_start + heads * all * c.whole.load_tile) / num_cus);
        least += c.merge + record_us * heads * cut_records / tiles + c.merge_range * longest.count;
        if (least * (1.0 - 1e-9) >= limit) continue;
        int items;
        const double us = estimate(tiles, &items);
        if (us < limit) limit = us, best = tiles, *items_per_head = items;
    }
    return best;
}

size_t plan_prefill_bf16(PrefillParams &p, int num_cus, bool with_ranges) {
    p.rows = 128;
    p.split_tiles = 0;
    if (p.sparse_row_ptr != nullptr) return 0;
    const PrefillCosts &c = p.d == 128 ? kPrefillCosts128 : kPrefillCosts64;
    const bool ranges = with_ranges && p.window <= 0 && p.prep.gamma_q == nullptr;
    if (!ranges && !pair_possible(p)) return 0;
    double us = unsplit_us(p, num_cus, 128, c.whole, c.resident);
    if (pair_possible(p)) {
        const double pair = unsplit_us(p, num_cus, 64, c.pair, c.resident);
        if (pair < us) us = pair, p.rows = 64;
    }
    if (!ranges) return 0;
    p.split_tiles = choose_split_tiles(p, num_cus, c, 0.97 * us, &p.items_per_head);
    if (p.split_tiles == 0) return 0;
    return (size_t)p.B * p.Hq * p.items_per_head * 4 * prefill_record_floats(p.d) * sizeof(float);
}

template <int D>
static hipError_t launch_prefill_split(const PrefillParams &p, hipStream_t stream) {
    const long long total = (long long)p.items_per_head * p.Hq * p.B;
    const int rows = 128;
    const long long waves = (long long)((p.T + rows - 1) / rows) * p.Hq * p.B * 4 * (D / 32);
    const dim3 grid((unsigned)total), merge((unsigned)((waves + 3) / 4)), block(256);
    auto run = [&](auto use_r, auto causal, auto stats) {
        constexpr bool R = decltype(use_r)::value, C = decltype(causal)::value, ST = decltype(stats)::value;
        hipLaunchKernelGGL((prefill_bf16_kernel<D, R, C, false, ST, false, false, true>), grid, block, 0, stream, p);
        if (hipError_t err = hipGetLastError()) return err;
        hipLaunchKernelGGL((prefill_combine_kernel<D, R, ST>), merge, block, 0, stream, p);
        return hipGetLastError();
    };
    const std::true_type yes;
    const std::false_type no;
    if (p.row_stats != nullptr) return p.causal ? run(yes, yes, yes) : run(yes, no, yes);
    if (p.use_r) return p.causal ? run(yes, yes, no) : run(yes, no, no);
    return p.causal ? run(no, yes, no) : run(no, no, no);
}

// Block-sparse tile iterator (use_r, no window): lists per 128 query rows.
template <int D>
static hipError_t launch_prefill_sparse(const PrefillParams &p, hipStream_t stream) {
    const long long total = (long long)((p.T + 127) / 128) * p.Hq * p.B;
    if (total > 0x7fffffffLL) return hipErrorInvalidValue;
    const dim3 grid((unsigned)total), block(256);
    if (p.row_stats != nullptr) {  // with the row cache of the backward pass
        if (p.causal)
            hipLaunchKernelGGL((prefill_bf16_kernel<D, true, true, false, true, true>), grid, block, 0, stream, p);
        else
            hipLaunchKernelGGL((prefill_bf16_kernel<D, true, false, false, true, true>), grid, block, 0, stream, p);
        return hipGetLastError();
    }
    if (p.causal)
        hipLaunchKernelGGL((prefill_bf16_kernel<D, true, true, false, false, true>), grid, block, 0, stream, p);
    else
        hipLaunchKernelGGL((prefill_bf16_kernel<D, true, false, false, false, true>), grid, block, 0, stream, p);
    return hipGetLastError();
}

// Dense causal forward, 64 rows per workgroup
template <int D>
static hipError_t launch_prefill_pair(const PrefillParams &p, hipStream_t stream) {
    const long long total = (long long)((p.T + 63) / 64) * p.Hq * p.B;
    if (total > 0x7fffffffLL) return hipErrorInvalidValue;
    const dim3 grid((unsigned)total), block(256);
    if (p.prep.gamma_q != nullptr)
        hipLaunchKernelGGL((prefill_bf16_kernel<D, true, true, false, false, false, true, false, true>), grid, block, 0, stream, p);
    else if (p.row_stats != nullptr && p.window > 0)
        hipLaunchKernelGGL((prefill_bf16_kernel<D, true, true, true, true, false, false, false, true>), grid, block, 0, stream, p);
    else if (p.row_stats != nullptr)
        hipLaunchKernelGGL((prefill_bf16_kernel<D, true, true, false, true, false, false, false, true>), grid, block, 0, stream, p);
    else if (p.window > 0)
        hipLaunchKernelGGL((prefill_bf16_kernel<D, true, true, true, false, false, false, false, true>), grid, block, 0, stream, p);
    else
        hipLaunchKernelGGL((prefill_bf16_kernel<D, true, true, false, false, false, false, false, true>), grid, block, 0, stream, p);
    return hipGetLastError();
}

// Dense kernels, 128 rows per workgroup
template <int D>
static hipError_t launch_prefill_dense(const PrefillParams &p, hipStream_t stream) {
    const int rows = 128;
    const long long total = (long long)((p.T + rows - 1) / rows) * p.Hq * p.B;
    if (total > 0x7fffffffLL) return hipErrorInvalidValue;
    const dim3 grid((unsigned)total), block(256);
    if (p.prep.gamma_q != nullptr) {  // RMSNorm + RoPE on q, rho in the prologue (use_r, no window, no row cache)
        if (p.causal)
            hipLaunchKernelGGL((prefill_bf16_kernel<D, true, true, false, false, false, true>), grid, block, 0, stream, p);
        else
            hipLaunchKernelGGL((prefill_bf16_kernel<D, true, false, false, false, false, true>), grid, block, 0, stream, p);
        return hipGetLastError();
    }
    if (p.row_stats != nullptr && p.window > 0) {  // row cache + sliding window (causal, use_r)
        hipLaunchKernelGGL((prefill_bf16_kernel<D, true, true, true, true, false>), grid, block, 0, stream, p);
    } else if (p.row_stats != nullptr) {  // with the row cache of the backward pass (use_r)
        if (p.causal)
            hipLaunchKernelGGL((prefill_bf16_kernel<D, true, true, false, true, false>), grid, block, 0, stream, p);
        else
            hipLaunchKernelGGL((prefill_bf16_kernel<D, true, false, false, true, false>), grid, block, 0, stream, p);
    } else if (p.window > 0) {  // causal only (checked by the caller)
        if (p.use_r)
            hipLaunchKernelGGL((prefill_bf16_kernel<D, true, true, true, false, false>), grid, block, 0, stream, p);
        else
            hipLaunchKernelGGL((prefill_bf16_kernel<D, false, true, true, false, false>), grid, block, 0, stream, p);
    } else if (p.use_r) {
        if (p.causal)
            hipLaunchKernelGGL((prefill_bf16_kernel<D, true, true, false, false, false>), grid, block, 0, stream, p);
        else
            hipLaunchKernelGGL((prefill_bf16_kernel<D, true, false, false, false, false>), grid, block, 0, stream, p);
    } else {
        if (p.causal)
            hipLaunchKernelGGL((prefill_bf16_kernel<D, false, true, false, false, false>), grid, block, 0, stream, p);
        else
            hipLaunchKernelGGL((prefill_bf16_kernel<D, false, false, false, false, false>), grid, block, 0, stream, p);
    }
    return hipGetLastError();
}

hipError_t launch_prefill_bf16(const PrefillParams &p, hipStream_t stream) {  // (planned by plan_prefill_bf16)
    if (p.ws != nullptr)
        return p.d == 128 ? launch_prefill_split<128>(p, stream) : launch_prefill_split<64>(p, stream);
    if (p.sparse_row_ptr != nullptr)
        return p.d == 128 ? launch_prefill_sparse<128>(p, stream) : launch_prefill_sparse<64>(p, stream);
    if (p.rows == 64) return p.d == 128 ? launch_prefill_pair<128>(p, stream) : launch_prefill_pair<64>(p, stream);
    return p.d == 128 ? launch_prefill_dense<128>(p, stream) : launch_prefill_dense<64>(p, stream);
}

}  // namespace plx
