// fp32 Parallax: forward (decode and prefill) and backward for every head dimension up to 256 (large prefill launches at
// d = 64 go to prefill_f32.hip), on
// the fp32 matrix instructions of gfx950 (v_mfma_f32_16x16x4_f32: fp32 operands, fp32
// accumulation, one rounding per step, as a chain of fused multiply-adds has). Algorithm 1 of the
// paper (Sec. 3.3) with the running state (m, d1, d2, O1, O2), closed with
// O1/d1 * (1 + d2/d1) - O2/d1; gradients by the closed forms of App. D.
//
// Layout, the same in all three kernels. A workgroup owns 16 COLUMNS of the matrix tiles (query
// rows in the forward and in the dQ / dR pass, keys in the dK / dV pass) and its four waves
// deal the other side out among themselves in blocks of 16 (wave w: blocks w, w + 4, ...), each
// with a state of its own; the states meet in LDS at the end. No barrier in the loops, work
// for four waves even where there are 16 rows only, and one kernel serves prefill (16 rows of a
// head) and decode (the heads of a GQA group x query rows, keys split over workgroups as well).
//   scores   S^T = K Q^T: A = 16 keys, read straight from global memory (lane (c, g): chunk 4 j + g
//            of row c, the four values of a chunk are four k-steps), B = the 16 columns, kept in LDS.
//   outputs  the accumulator of a score block (lane (c, g): column c, keys 4 g .. 4 g + 3) IS the
//            B operand of O^T += V^T P^T, k-step r taking key 4 g + r from lane group g, so P never
//            leaves its lane. A = V^T: lane (c, g) holds dimensions 64 m + 4 c .. + 3 of key 4 g + r,
//            again whole 16-byte loads from global memory, fully coalesced.
//   Where a tensor is needed in both orders (K in the dQ / dR pass; Q, R, dO in the dK / dV pass)
//   the wave turns it round in a 16-row LDS tile of its own.
// What bounds it: the matrix pipe, at 64 flop per clock and SIMD (157 TFLOP/s nominal on the chip):
// a 16-key block costs DP matrix instructions of 32 clocks (two score products of DP / 4, two output
// products of DP / 4) against 2 * 16 * DP * 4 bytes of loads, 16 bytes per clock and compute unit. One row, one
// key at a time on the vector ALU (one workgroup per row, the kernels these replaced), the step of 8
// sequences x 8 heads x 512 rows, d = 64, forward and backward, took 7800 us, 6286 of them in
// dK / dV; these take 187 us = 86 TFLOP/s (206 with the row pointers formed per lane, padding tests
// where d = 64 needs none, and the two sums merged one after the other; 191 with the rare path of
// f32_take_out_not_finite as a loop). At 4 x 8 heads x 2048 rows the forward reaches 95 TFLOP/s.
// 2 x 8 heads x 500 rows, forward / backward: d = 128 38 / 95 us (273 / 3440 before), d = 256 68 / 194
// (394 / 7100), d = 132 62 / 159 (304 / 3690). Tiles padded beyond d skip the matrix instructions of the
// padding. The one call that one workgroup per row served better: d > 128 over 65 to about 130 keys in a
// single split, two rounds of a wave where a column holds two heads (d = 256, 100 keys: 17.4 -> 19.3 us).
// Tried and slower: a wave alone with its columns (no merge; 8 x 8 x 512: 64 -> 82 us forward), four
// waves per SIMD for d = 64 (spills; 62 -> 67, dK / dV 82 -> 109); no gain: all four waves adding up and
// finishing a quarter of the dimensions each at d = 256.
// A decode step over 4 sequences x 2048 keys, 8 key heads, d = 64: 320 -> 16 us (half of that by
// splitting the keys over workgroups).
#include "plx_f32.h"

namespace plx {

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

// 16 rows (columns of the matrix tiles) in LDS: [16][DP + 4] floats, the padding makes 16 rows at one
// chunk fall into 16 different bank groups. Chunks past d and dead rows hold zeros.
template <int DP>
struct F32Rows {
    float x[16][DP + 4];
};

// One 16 x 16 score block: acc += A (lane (c, g): chunks 4 j + g of row c) x rows, up to dimension d. (The
// offset of the lane is made opaque: seeing that the operand never changes, the compiler would otherwise
// keep all of it in registers around the loop, and the registers decide how many waves a SIMD holds.)
template <int DP>
__device__ __forceinline__ f32x4 f32_scores(const f32x4 (&a)[DP / 16], const F32Rows<DP> &rows, int d, int c, int g) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    int at = c * (DP + 4) + 4 * g;
    asm volatile("" : "+v"(at));
#pragma unroll
    for (int j = 0; j < DP / 16; ++j) {
        if (16 * j >= d) break;
        const f32x4 b = *(const f32x4 *)(&rows.x[0][0] + at + 16 * j);
#pragma unroll
        for (int i = 0; i < 4; ++i) acc = mfma_f32(a[j][i], b[i], acc);
    }
    return acc;
}

// acc[4 m + i] += A^T p over 16 keys: a[r][m] = dimensions 64 m + 4 c .. + 3 of key 4 g + r, p[r] =
// weight of key 4 g + r for column c. In accumulator register rr of acc[4 m + i] lane (c, g) then
// holds dimension 64 m + 4 (4 g + rr) + i of column c.
template <int DP>
__device__ __forceinline__ void f32_outputs(const f32x4 (&a)[4][DP / 64], const f32x4 &p, int d, f32x4 (&acc)[DP / 16]) {
#pragma unroll
    for (int m = 0; m < DP / 64; ++m) {
        if (64 * m >= d) break;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[4 * m + i] = mfma_f32(a[r][m][i], p[r], acc[4 * m + i]);
    }
}

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

// The chunks 4 j + g of a row in global memory (zeros past d)
template <int DP>
__device__ __forceinline__ void f32_load_row(f32x4 (&a)[DP / 16], const float *row, int d, int g) {
#pragma unroll
    for (int j = 0; j < DP / 16; ++j) {
        const int dim = 4 * (4 * j + g);
        a[j] = dim < d ? *(const f32x4 *)(row + dim) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
}
// The wave's private 16-row tile: rows in (chunk order of f32_load_row), transposed operands out
template <int DP>
__device__ __forceinline__ void f32_turn(const f32x4 (&in)[DP / 16], F32Rows<DP> &tile, f32x4 (&out)[4][DP / 64], int c,
                                         int g) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < DP / 16; ++j) *(f32x4 *)&tile.x[c][4 * (4 * j + g)] = in[j];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int m = 0; m < DP / 64; ++m) out[r][m] = *(const f32x4 *)&tile.x[4 * g + r][64 * m + 4 * c];
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

// ---- forward -------------------------------------------------------------------------------
template <int DP>
union F32ForwardLds {
    F32Rows<DP> rows[2];                  // q, rho of the 16 columns
    f32x4 merge[2 * 2 * (DP / 16) * 64];  // the accumulators of two waves
};

// FULL: d == DP, nothing to pad
template <int DP, bool PAGED, bool USE_R, bool FULL>
__global__ __launch_bounds__(kF32Threads, DP <= 128 ? 2 : 1) void f32_forward_kernel(F32Forward p) {
    __shared__ F32ForwardLds<DP> lds;
    __shared__ float sm[3][kF32Waves][16];
    constexpr int NA = DP / 16;

    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int c = lane & 15, g = lane >> 4, d = FULL ? DP : p.d;
    int64_t id = f32_block_id();
    if (id >= (int64_t)p.n_blocks * p.B * p.heads * p.S) return;
    const int split = (int)(id % p.S);
    id /= p.S;
    const int hgrp = (int)(id % p.heads);
    id /= p.heads;
    const int b = (int)(id % p.B);
    const int blk = p.n_blocks - 1 - (int)(id / p.B);  // causal: the longest rows first
    const int hk = hgrp * p.gcols / p.G;

    // columns of this workgroup: key range [lo, end) of each, their union and intersection
    const int len = p.seq_lens ? min(max(p.seq_lens[b], 0), p.Lk) : p.Lk;
    auto row_end = [&](int t) { return max(p.tail ? len - (p.Tq - 1 - t) : len, 0); };
    auto row_lo = [&](int t) { return p.window > 0 ? max(row_end(t) - p.window, 0) : 0; };
    const int x_last = min(16 * blk + 15, p.n_cols - 1);
    const int t0 = 16 * blk / p.gcols, t1 = x_last / p.gcols;
    const int x = min(16 * blk + c, x_last);
    const int t = x / p.gcols, head = hgrp * p.gcols + x % p.gcols;
    const int my_end = row_end(t), my_lo = row_lo(t);
    const int all_lo = row_lo(t1), all_end = row_end(t0);  // every column sees [all_lo, all_end)
    int lo = row_lo(t0) / 16, hi = (row_end(t1) + 15) / 16;  // 16-key blocks of the union
    const int last_key = row_end(t1) - 1;
    if (p.S > 1) {
        const int per = (hi - lo + p.S - 1) / p.S;
        lo += split * per;
        hi = min(lo + per, hi);
    }

    for (int e = tid; e < 16 * (DP / 4); e += kF32Threads) {
        const int row = e / (DP / 4), dim = 4 * (e % (DP / 4));
        const int xr = 16 * blk + row;
        f32x4 qv = {0.f, 0.f, 0.f, 0.f}, rv = {0.f, 0.f, 0.f, 0.f};
        if (xr < p.n_cols && dim < d) {
            const int64_t tr = xr / p.gcols, hr = hgrp * p.gcols + xr % p.gcols;
            qv = *(const f32x4 *)(p.q + b * p.qs[0] + hr * p.qs[1] + tr * p.qs[2] + dim);
            if constexpr (USE_R) rv = *(const f32x4 *)(p.r + b * p.rs[0] + hr * p.rs[1] + tr * p.rs[2] + dim);
        }
        *(f32x4 *)&lds.rows[0].x[row][dim] = qv;
        *(f32x4 *)&lds.rows[1].x[row][dim] = rv;
    }

    const float *kb = p.k + (PAGED ? 0 : b * p.ks[0]) + hk * p.ks[1];
    const float *vb = p.v + (PAGED ? 0 : b * p.vs[0]) + hk * p.vs[1];
    // row of a key; keys behind the last one any column sees re-read that one (masked below)
    auto row_of = [&](const float *base, const int64_t (&st)[3], int key) -> const float * {
        key = min(key, last_key);
        if constexpr (PAGED) {
            const int pg = min(max(p.block_table[(int64_t)b * p.table_stride + key / p.page_size], 0), p.num_pages - 1);
            return base + (int64_t)pg * st[0] + (int64_t)(key % p.page_size) * st[2];
        } else {
            return base + (int64_t)key * st[2];
        }
    };
    // (the rows of a whole block of a contiguous cache: a uniform base plus this lane's own offset)
    const int64_t k_lane = (int64_t)c * p.ks[2], v_lane = (int64_t)(4 * g) * p.vs[2];
    f32x4 kf[NA], vf[4][DP / 64];
    auto load_k = [&](int kblk) {
        const bool plain = !PAGED && 16 * kblk + 15 <= last_key;  // uniform
        const float *row = plain ? kb + (int64_t)(16 * kblk) * p.ks[2] + k_lane : row_of(kb, p.ks, 16 * kblk + c);
        f32_load_row<DP>(kf, row, d, g);
    };
    auto load_v = [&](int kblk) {
        const bool plain = !PAGED && 16 * kblk + 15 <= last_key;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float *row = plain ? vb + (int64_t)(16 * kblk + r) * p.vs[2] + v_lane : row_of(vb, p.vs, 16 * kblk + 4 * g + r);
#pragma unroll
            for (int m = 0; m < DP / 64; ++m) {
                const int dim = 64 * m + 4 * c;
                vf[r][m] = dim < d ? *(const f32x4 *)(row + dim) : f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }
    };

    const float scale_log2 = p.scale * kLog2e;
    float m_run = kNegInf, d1 = 0.f, d2 = 0.f;  // column c; the sums over this lane's keys only
    f32x4 o1[NA], o2[NA];
#pragma unroll
    for (int n = 0; n < NA; ++n) o1[n] = o2[n] = f32x4{0.f, 0.f, 0.f, 0.f};

    int kblk = lo + w;
    if (kblk < hi) load_k(kblk), load_v(kblk);
    __syncthreads();
    for (; kblk < hi; kblk += kF32Waves) {
        const int key0 = 16 * kblk, next = kblk + kF32Waves;
        f32x4 s1 = f32_scores<DP>(kf, lds.rows[0], d, c, g);
        f32x4 s2 = {0.f, 0.f, 0.f, 0.f};
        if constexpr (USE_R) s2 = f32_scores<DP>(kf, lds.rows[1], d, c, g);
        // the next block's K rows travel under the exponentials and the V product, its V rows (below)
        // under its scores: each register set is refilled as soon as it has been used
        if (next < hi) load_k(next);

        const bool whole = key0 >= all_lo && key0 + 16 <= all_end;  // uniform
        unsigned seen = 15u;
        float tmax = kNegInf;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            s1[r] *= scale_log2;
            if (!whole) {
                const int key = key0 + 4 * g + r;
                const bool ok = key >= my_lo && key < my_end;
                if (!ok) s1[r] = kNegInf, s2[r] = 0.f, seen &= ~(1u << r);
            }
            tmax = fmaxf(tmax, s1[r]);
        }
        tmax = rows_max(tmax);
        const float m_new = fmaxf(m_run, tmax);
        const float m_use = m_new == kNegInf ? 0.f : m_new;
        const float alpha = fast_exp2(m_run - m_use);  // 0 on the first block that is seen
        m_run = m_new;
        f32x4 p1, p2;
        float a1 = 0.f, a2 = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            p1[r] = fast_exp2(s1[r] - m_use);  // 0 if masked
            p2[r] = p1[r] * s2[r];
            a1 += p1[r], a2 += p2[r];
        }
        d1 = d1 * alpha + a1;
        d2 = d2 * alpha + a2;
        if (!__all(alpha == 1.f)) {
#pragma unroll
            for (int n = 0; n < NA; ++n) o1[n] *= alpha, o2[n] *= alpha;
        }
        if (__builtin_expect(!whole && f32_not_finite<DP>(vf), 0)) {
            if constexpr (USE_R)
                f32_take_out_not_finite<DP, 2>(vf, {&p1, &p2}, seen, {&o1, &o2});
            else
                f32_take_out_not_finite<DP, 1>(vf, {&p1}, seen, {&o1});
        }
        f32_outputs<DP>(vf, p1, d, o1);
        if constexpr (USE_R) f32_outputs<DP>(vf, p2, d, o2);
        if (next < hi) load_v(next);
    }

    // ---- the four waves' states on one reference, summed into wave 0 ------------------------
    d1 = rows_sum(d1), d2 = rows_sum(d2);
    if (g == 0) sm[0][w][c] = m_run, sm[1][w][c] = d1, sm[2][w][c] = d2;
    __syncthreads();
    float m_all = kNegInf;
#pragma unroll
    for (int i = 0; i < kF32Waves; ++i) m_all = fmaxf(m_all, sm[0][i][c]);
    d1 = d2 = 0.f;
#pragma unroll
    for (int i = 0; i < kF32Waves; ++i) {
        const float wt = sm[0][i][c] == kNegInf ? 0.f : fast_exp2(sm[0][i][c] - m_all);
        d1 += wt * sm[1][i][c], d2 += wt * sm[2][i][c];
    }
    const float wt = m_run == kNegInf ? 0.f : fast_exp2(m_run - m_all);
#pragma unroll
    for (int n = 0; n < NA; ++n) o1[n] *= wt, o2[n] *= wt;
    f32_sum_waves<NA>(o1, o2, lds.merge, w, lane, hi - lo);
    if (w != 0 || 16 * blk + c >= p.n_cols) return;

    // lane (c, g): dimensions 64 m + 16 g + 4 rr .. + 3 of column c, float4 by float4
    const float inv = d1 > 0.f ? 1.f / d1 : 0.f;
    if (p.S > 1) {
        float *rec = p.ws + ((((int64_t)b * p.Hq + head) * p.Tq + t) * p.S + split) * (2 * d + 4);
        if (g == 0) *(f32x4 *)rec = f32x4{m_all, d1, d2, 0.f};
#pragma unroll
        for (int m = 0; m < DP / 64; ++m)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                const int dim = 64 * m + 16 * g + 4 * rr;
                if (dim >= d) continue;
                *(f32x4 *)(rec + 4 + dim) = f32x4{o1[4 * m][rr], o1[4 * m + 1][rr], o1[4 * m + 2][rr], o1[4 * m + 3][rr]};
                *(f32x4 *)(rec + 4 + d + dim) = f32x4{o2[4 * m][rr], o2[4 * m + 1][rr], o2[4 * m + 2][rr], o2[4 * m + 3][rr]};
            }
        return;
    }
    const int64_t orow = b * p.os[0] + head * p.os[1] + t * p.os[2];
#pragma unroll
    for (int m = 0; m < DP / 64; ++m)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            const int dim = 64 * m + 16 * g + 4 * rr;
            if (dim >= d) continue;
            f32x4 out = {0.f, 0.f, 0.f, 0.f}, mean = out;  // empty key set: zeros
            if (d1 > 0.f)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    mean[i] = o1[4 * m + i][rr] * inv;
                    out[i] = mean[i] * (1.f + d2 * inv) - o2[4 * m + i][rr] * inv;
                }
            *(f32x4 *)(p.o + orow + dim) = out;
            if (p.vbar) *(f32x4 *)(p.vbar + orow + dim) = mean;
        }
    if (p.row_stats && g == 0) {
        float *st = p.row_stats + (((int64_t)b * p.Hq + head) * p.Tq + t) * 2;
        st[0] = d1 > 0.f ? m_all + log2f(d1) : kNegInf;
        st[1] = d1 > 0.f ? d2 * inv : 0.f;
    }
}

// Merge of the split records (App. C), one workgroup per output row: 64 dimension lanes (float4
// each) x 4 split lanes, eight records per thread in flight.
__global__ __launch_bounds__(256) void f32_combine_kernel(F32Forward p) {
    __shared__ float hdr[4][3];
    __shared__ f32x4 acc[4][2][64];
    const int dl = threadIdx.x & 63, sl = threadIdx.x >> 6, d = p.d, dim = 4 * dl;
    const int64_t row = f32_block_id();  // (b, head, t)
    if (row >= (int64_t)p.B * p.Hq * p.Tq) return;
    const float *rec0 = p.ws + row * p.S * (2 * d + 4);
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    float m = kNegInf, d1 = 0.f, d2 = 0.f;
    f32x4 a1 = zero, a2 = zero;
    for (int s0 = sl; s0 < p.S; s0 += 32) {
        f32x4 h[8], x1[8], x2[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int s = s0 + 4 * u;
            const float *rec = rec0 + (int64_t)min(s, p.S - 1) * (2 * d + 4);
            h[u] = s < p.S ? *(const f32x4 *)rec : f32x4{kNegInf, 0.f, 0.f, 0.f};
            x1[u] = dim < d ? *(const f32x4 *)(rec + 4 + dim) : zero;
            x2[u] = dim < d ? *(const f32x4 *)(rec + 4 + d + dim) : zero;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            // (uniform per split lane) nothing there, or no key seen; a reference of -inf with a sum that is
            // not zero is a record of NaN scores only, which must reach the result
            if (h[u][0] == kNegInf && h[u][1] == 0.f) continue;
            const float m_new = fmaxf(m, h[u][0]), m_use = m_new == kNegInf ? 0.f : m_new;
            const float w_old = fast_exp2(m - m_use), w_new = fast_exp2(h[u][0] - m_use);
            m = m_new;
            d1 = w_old * d1 + w_new * h[u][1], d2 = w_old * d2 + w_new * h[u][2];
            a1 = w_old * a1 + w_new * x1[u], a2 = w_old * a2 + w_new * x2[u];
        }
    }
    if (dl == 0) hdr[sl][0] = m, hdr[sl][1] = d1, hdr[sl][2] = d2;
    acc[sl][0][dl] = a1, acc[sl][1][dl] = a2;
    __syncthreads();
    if (sl != 0 || dim >= d) return;
    float m_all = kNegInf;
#pragma unroll
    for (int i = 0; i < 4; ++i) m_all = fmaxf(m_all, hdr[i][0]);
    d1 = d2 = 0.f, a1 = a2 = zero;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float wt = hdr[i][0] == kNegInf ? 0.f : fast_exp2(hdr[i][0] - m_all);  // (0 * NaN stays NaN)
        d1 += wt * hdr[i][1], d2 += wt * hdr[i][2];
        a1 += wt * acc[i][0][dl], a2 += wt * acc[i][1][dl];
    }
    f32x4 out = zero;
    if (d1 > 0.f) {
        const float inv = 1.f / d1;
        out = (a1 * inv) * (1.f + d2 * inv) - a2 * inv;
    }
    const int t = (int)(row % p.Tq);
    const int64_t bh = row / p.Tq;
    *(f32x4 *)(p.o + (bh / p.Hq) * p.os[0] + (bh % p.Hq) * p.os[1] + t * p.os[2] + dim) = out;
}

static hipError_t launch_forward(F32Forward &g, hipStream_t stream) {
    g.n_blocks = (g.n_cols + 15) / 16;
    const dim3 grid = f32_grid((int64_t)g.n_blocks * g.B * g.heads * g.S), block(kF32Threads);
    auto pick = [&](auto paged, auto use_r) {
        constexpr bool P = decltype(paged)::value, R = decltype(use_r)::value;
        if (g.d == 64)
            hipLaunchKernelGGL((f32_forward_kernel<64, P, R, true>), grid, block, 0, stream, g);
        else if (g.d < 64)
            hipLaunchKernelGGL((f32_forward_kernel<64, P, R, false>), grid, block, 0, stream, g);
        else if (g.d == 128)
            hipLaunchKernelGGL((f32_forward_kernel<128, P, R, true>), grid, block, 0, stream, g);
        else if (g.d < 128)
            hipLaunchKernelGGL((f32_forward_kernel<128, P, R, false>), grid, block, 0, stream, g);
        else if (g.d == 256)
            hipLaunchKernelGGL((f32_forward_kernel<256, P, R, true>), grid, block, 0, stream, g);
        else
            hipLaunchKernelGGL((f32_forward_kernel<256, P, R, false>), grid, block, 0, stream, g);
    };
    const std::true_type yes;
    const std::false_type no;
    if (g.block_table)
        g.use_r ? pick(yes, yes) : pick(yes, no);
    else
        g.use_r ? pick(no, yes) : pick(no, no);
    if (hipError_t err = hipGetLastError()) return err;
    if (g.S > 1) {
        hipLaunchKernelGGL(f32_combine_kernel, f32_grid((int64_t)g.B * g.Hq * g.Tq), dim3(256), 0, stream, g);
        return hipGetLastError();
    }
    return hipSuccess;
}

hipError_t launch_decode_f32(const DecodeParams &p, hipStream_t stream) {
    F32Forward g{};
    g.q = (const float *)p.q, g.r = (const float *)p.r, g.k = (const float *)p.k, g.v = (const float *)p.v;
    g.o = (float *)p.o;
    g.seq_lens = p.seq_lens;
    g.B = p.B, g.Hq = p.Hq, g.G = p.G, g.Tq = p.Tq, g.Lk = p.Lmax, g.d = p.d;
    g.heads = p.Hkv, g.gcols = p.G, g.n_cols = p.G * p.Tq;
    g.qs[0] = g.rs[0] = g.os[0] = (int64_t)p.Hq * p.Tq * p.d;
    g.qs[1] = g.rs[1] = g.os[1] = (int64_t)p.Tq * p.d;
    g.qs[2] = g.rs[2] = g.os[2] = p.d;
    g.ks[0] = p.ksb, g.ks[1] = p.ksh, g.ks[2] = p.ksl;
    g.vs[0] = p.vsb, g.vs[1] = p.vsh, g.vs[2] = p.vsl;
    g.scale = p.scale, g.use_r = p.use_r, g.tail = 1, g.window = p.window;
    g.block_table = p.block_table;
    g.page_size = p.page_size, g.table_stride = p.table_stride, g.num_pages = p.num_pages;
    g.S = p.S, g.ws = p.ws;
    return launch_forward(g, stream);
}

int32_t prefill_form_f32(const PrefillParams &p) {
    return f32_thirds_pay(p.d, p.T, p.Tk, p.causal, p.window, f32_thirds_blocks(p.T, p.B, p.Hq)) ? kF32ThirdsColumns : 0;
}

hipError_t launch_prefill_f32(const PrefillParams &p, hipStream_t stream) {
    if (prefill_form_f32(p)) return launch_forward_thirds(p, stream);
    F32Forward g{};
    g.q = (const float *)p.q, g.r = (const float *)p.r, g.k = (const float *)p.k, g.v = (const float *)p.v;
    g.o = (float *)p.o;
    g.B = p.B, g.Hq = p.Hq, g.G = p.G, g.Tq = p.T, g.Lk = p.Tk, g.d = p.d;
    g.heads = p.Hq, g.gcols = 1, g.n_cols = p.T;
    for (int a = 0; a < 3; ++a)
        g.qs[a] = p.qs[a], g.rs[a] = p.rs[a], g.ks[a] = p.ks[a], g.vs[a] = p.vs[a], g.os[a] = p.os[a];
    g.scale = p.scale, g.use_r = p.use_r, g.tail = p.causal, g.window = p.window;
    g.vbar = (float *)p.vbar, g.row_stats = p.row_stats;
    g.S = 1;
    return launch_forward(g, stream);
}

// ---- backward (closed forms of the paper's App. D) -------------------------------------------
// dQ, dR: 16 query rows per workgroup, the waves deal out the keys. It first forms tau = dO.o and
// beta = dO.vbar of its rows and leaves (lse, ubar, tau, beta) in the workspace for the dK / dV pass.
template <int DP>
struct F32RowsLds {
    F32Rows<DP> rows[3];             // q, rho, dO
    union {
        F32Rows<DP> tile[kF32Waves];     // K blocks on their way into the other operand order
        f32x4 merge[2 * 2 * (DP / 16) * 64];
    };
};

template <int DP, bool FULL>
__global__ __launch_bounds__(kF32Threads, DP <= 128 ? 2 : 1) void f32_bwd_rows_kernel(PrefillBwdParams p) {
    __shared__ F32RowsLds<DP> lds;
    __shared__ f32x4 scalars[16];
    constexpr int NA = DP / 16;
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int c = lane & 15, g = lane >> 4, d = FULL ? DP : p.d, off = p.Tk - p.T;
    const int n_blocks = (p.T + 15) / 16;
    int64_t id = f32_block_id();
    if (id >= (int64_t)n_blocks * p.B * p.Hq) return;
    const int h = (int)(id % p.Hq);
    id /= p.Hq;
    const int b = (int)(id % p.B);
    const int i0 = 16 * (n_blocks - 1 - (int)(id / p.B));  // first row
    const int64_t head = ((int64_t)b * p.Hq + h) * p.T;
    const int64_t khead = ((int64_t)b * p.Hkv + h / p.G) * p.Tk;

    {  // 16 lanes per row: rows into LDS, tau and beta on the way
        const int row = tid >> 4, l = tid & 15;
        const int64_t e0 = (head + min(i0 + row, p.T - 1)) * d;
        float tau = 0.f, beta = 0.f;
        for (int dim = 4 * l; dim < DP; dim += 64) {
            f32x4 x[3] = {};
            if (dim < d) {
                x[0] = *(const f32x4 *)((const float *)p.q + e0 + dim);
                x[1] = *(const f32x4 *)((const float *)p.r + e0 + dim);
                x[2] = *(const f32x4 *)((const float *)p.d_o + e0 + dim);
                const f32x4 o = *(const f32x4 *)((const float *)p.o + e0 + dim);
                const f32x4 vb = *(const f32x4 *)((const float *)p.vbar + e0 + dim);
#pragma unroll
                for (int i = 0; i < 4; ++i) tau = fmaf(x[2][i], o[i], tau), beta = fmaf(x[2][i], vb[i], beta);
            }
#pragma unroll
            for (int n = 0; n < 3; ++n) *(f32x4 *)&lds.rows[n].x[row][dim] = x[n];
        }
        tau = lane_group_sum<16>(tau), beta = lane_group_sum<16>(beta);
        if (l == 0) {
            const int64_t r = head + min(i0 + row, p.T - 1);
            const f32x4 s = {p.row_stats[2 * r], p.row_stats[2 * r + 1], tau, beta};
            scalars[row] = s;
            if (i0 + row < p.T) ((f32x4 *)p.row_cache)[r] = s;
        }
    }
    const int my_end = p.causal ? min(min(i0 + c, p.T - 1) + 1 + off, p.Tk) : p.Tk;
    const int my_lo = p.window > 0 ? max(my_end - p.window, 0) : 0;
    const int last = min(i0 + 15, p.T - 1);
    const int end = p.causal ? min(last + 1 + off, p.Tk) : p.Tk, first_end = p.causal ? min(i0 + 1 + off, p.Tk) : p.Tk;
    const int lo = p.window > 0 ? max(first_end - p.window, 0) / 16 : 0;
    const int all_lo = p.window > 0 ? max(end - p.window, 0) : 0;
    const float *k = (const float *)p.k + khead * d, *v = (const float *)p.v + khead * d;
    f32x4 kf[NA], vf[NA];
    auto load = [&](f32x4(&x)[NA], const float *base, int kblk) {
        f32_load_row<DP>(x, base + (int64_t)min(16 * kblk + c, end - 1) * d, d, g);
    };
    f32x4 dq[NA], dr[NA];
#pragma unroll
    for (int n = 0; n < NA; ++n) dq[n] = dr[n] = f32x4{0.f, 0.f, 0.f, 0.f};
    const float scale_log2 = p.scale * kLog2e;
    const int hi = (end + 15) / 16;
    int kblk = lo + w;
    if (kblk < hi) load(kf, k, kblk), load(vf, v, kblk);
    __syncthreads();
    const f32x4 sc = scalars[c];
    for (; kblk < hi; kblk += kF32Waves) {
        const int key0 = 16 * kblk, next = kblk + kF32Waves;
        const f32x4 a = f32_scores<DP>(vf, lds.rows[2], d, c, g);
        if (next < hi) load(vf, v, next);
        const f32x4 s1 = f32_scores<DP>(kf, lds.rows[0], d, c, g);
        const f32x4 s2 = f32_scores<DP>(kf, lds.rows[1], d, c, g);
        f32x4 kt[4][DP / 64];
        f32_turn<DP>(kf, lds.tile[w], kt, c, g);
        if (next < hi) load(kf, k, next);
        const bool whole = key0 >= all_lo && key0 + 16 <= first_end;
        unsigned seen = 15u;
        f32x4 g1, g2;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float pr = fast_exp2(s1[r] * scale_log2 - sc[0]);
            const float dlt = a[r] - sc[3];
            g1[r] = pr * (a[r] - sc[2] + (sc[1] - s2[r]) * dlt);
            g2[r] = -pr * dlt;
            if (!whole) {
                const int key = key0 + 4 * g + r;
                if (!(key >= my_lo && key < my_end)) g1[r] = g2[r] = 0.f, seen &= ~(1u << r);
            }
        }
        if (__builtin_expect(!whole && f32_not_finite<DP>(kt), 0)) f32_take_out_not_finite<DP, 2>(kt, {&g1, &g2}, seen, {&dq, &dr});
        f32_outputs<DP>(kt, g1, d, dq);
        f32_outputs<DP>(kt, g2, d, dr);
    }
    f32_sum_waves<NA>(dq, dr, lds.merge, w, lane, hi - lo);
    if (w != 0 || i0 + c >= p.T) return;
    const int64_t e0 = (head + i0 + c) * d;
#pragma unroll
    for (int m = 0; m < DP / 64; ++m)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            const int dim = 64 * m + 16 * g + 4 * rr;
            if (dim >= d) continue;
            f32x4 x, y;
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = dq[4 * m + i][rr] * p.scale, y[i] = dr[4 * m + i][rr];
            *(f32x4 *)((float *)p.dq + e0 + dim) = x;
            *(f32x4 *)((float *)p.dr + e0 + dim) = y;
        }
}

// dK, dV: 16 keys per workgroup, the waves deal out the 16-row blocks of all query heads of the group.
template <int DP>
struct F32ColsLds {
    F32Rows<DP> rows[2];  // k, v
    union {
        F32Rows<DP> tile[kF32Waves];
        f32x4 merge[2 * 2 * (DP / 16) * 64];
    };
};

template <int DP, bool FULL>
__global__ __launch_bounds__(kF32Threads, DP <= 128 ? 2 : 1) void f32_bwd_cols_kernel(PrefillBwdParams p) {
    __shared__ F32ColsLds<DP> lds;
    constexpr int NA = DP / 16;
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int c = lane & 15, g = lane >> 4, d = FULL ? DP : p.d, off = p.Tk - p.T;
    const int n_blocks = (p.Tk + 15) / 16;
    int64_t id = f32_block_id();
    if (id >= (int64_t)n_blocks * p.B * p.Hkv) return;
    const int hk = (int)(id % p.Hkv);
    id /= p.Hkv;
    const int b = (int)(id % p.B);
    const int j0 = 16 * (int)(id / p.B);  // first key; causal: the first keys are seen by most rows
    const int64_t khead = ((int64_t)b * p.Hkv + hk) * p.Tk;
    for (int e = tid; e < 16 * (DP / 4); e += kF32Threads) {
        const int row = e / (DP / 4), dim = 4 * (e % (DP / 4));
        f32x4 x = {0.f, 0.f, 0.f, 0.f}, y = x;
        if (j0 + row < p.Tk && dim < d) {
            x = *(const f32x4 *)((const float *)p.k + (khead + j0 + row) * d + dim);
            y = *(const f32x4 *)((const float *)p.v + (khead + j0 + row) * d + dim);
        }
        *(f32x4 *)&lds.rows[0].x[row][dim] = x;
        *(f32x4 *)&lds.rows[1].x[row][dim] = y;
    }
    // rows [lo, end) see key j
    auto key_lo = [&](int j) { return p.causal ? max(j - off, 0) : 0; };
    auto key_end = [&](int j) { return p.window > 0 ? min(p.T, max(j - off + p.window, 0)) : p.T; };
    const int j_last = min(j0 + 15, p.Tk - 1), j = min(j0 + c, j_last);
    const int my_lo = key_lo(j), my_end = key_end(j);
    const int lo = key_lo(j0) / 16, end = key_end(j_last);  // union (both bounds grow with the key)
    const int all_lo = key_lo(j_last), all_end = key_end(j0);
    const int per_head = max((end + 15) / 16 - lo, 0), n_items = per_head * p.G;

    f32x4 xq[NA], xr[NA], xg[NA];
    auto load = [&](f32x4(&x)[NA], const void *base, int item) {
        const int64_t head = ((int64_t)b * p.Hq + hk * p.G + item / per_head) * p.T;
        const int i = min(16 * (lo + item % per_head) + c, end - 1);
        f32_load_row<DP>(x, (const float *)base + (head + i) * d, d, g);
    };
    f32x4 dk[NA], dv[NA];
#pragma unroll
    for (int n = 0; n < NA; ++n) dk[n] = dv[n] = f32x4{0.f, 0.f, 0.f, 0.f};
    const float scale_log2 = p.scale * kLog2e;
    int item = w;
    if (item < n_items) load(xq, p.q, item), load(xr, p.r, item), load(xg, p.d_o, item);
    __syncthreads();
    for (; item < n_items; item += kF32Waves) {
        const int next = item + kF32Waves;
        const int i0 = 16 * (lo + item % per_head);
        const int64_t head = ((int64_t)b * p.Hq + hk * p.G + item / per_head) * p.T;
        f32x4 sc[4];  // (lse, ubar, tau, beta) of rows i0 + 4 g + r
#pragma unroll
        for (int r = 0; r < 4; ++r) sc[r] = ((const f32x4 *)p.row_cache)[head + min(i0 + 4 * g + r, end - 1)];
        const f32x4 s1 = f32_scores<DP>(xq, lds.rows[0], d, c, g);
        const f32x4 s2 = f32_scores<DP>(xr, lds.rows[0], d, c, g);
        const f32x4 a = f32_scores<DP>(xg, lds.rows[1], d, c, g);
        const bool whole = i0 >= all_lo && i0 + 16 <= all_end;
        unsigned seen = 15u;
        f32x4 wt, g1, g2;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float pr = fast_exp2(s1[r] * scale_log2 - sc[r][0]);
            const float um = sc[r][1] - s2[r], dlt = a[r] - sc[r][3];
            wt[r] = pr * (1.f + um);
            g1[r] = pr * (a[r] - sc[r][2] + um * dlt) * p.scale;
            g2[r] = -pr * dlt;
            if (!whole) {
                const int i = i0 + 4 * g + r;
                if (!(i >= my_lo && i < my_end)) wt[r] = g1[r] = g2[r] = 0.f, seen &= ~(1u << r);
            }
        }
        auto add = [&](f32x4(&x)[NA], const void *base, const f32x4 &weights, f32x4(&acc)[NA]) {
            f32x4 xt[4][DP / 64];
            f32_turn<DP>(x, lds.tile[w], xt, c, g);
            if (next < n_items) load(x, base, next);
            if (__builtin_expect(!whole && f32_not_finite<DP>(xt), 0)) f32_take_out_not_finite<DP, 1>(xt, {&weights}, seen, {&acc});
            f32_outputs<DP>(xt, weights, d, acc);
        };
        add(xq, p.q, g1, dk);
        add(xr, p.r, g2, dk);
        add(xg, p.d_o, wt, dv);
    }
    f32_sum_waves<NA>(dk, dv, lds.merge, w, lane, n_items);
    if (w != 0 || j0 + c >= p.Tk) return;
    const int64_t e0 = (khead + j0 + c) * d;
#pragma unroll
    for (int m = 0; m < DP / 64; ++m)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            const int dim = 64 * m + 16 * g + 4 * rr;
            if (dim >= d) continue;
            *(f32x4 *)((float *)p.dk + e0 + dim) = f32x4{dk[4 * m][rr], dk[4 * m + 1][rr], dk[4 * m + 2][rr], dk[4 * m + 3][rr]};
            *(f32x4 *)((float *)p.dv + e0 + dim) = f32x4{dv[4 * m][rr], dv[4 * m + 1][rr], dv[4 * m + 2][rr], dv[4 * m + 3][rr]};
        }
}

int32_t backward_form_f32(const PrefillBwdParams &p) {
    // (each pass by itself: with several query heads to a key head there are fewer key blocks)
    auto pay = [&](int n, int heads) { return f32_thirds_pay(p.d, p.T, p.Tk, p.causal, p.window, f32_thirds_blocks(n, p.B, heads)); };
    return (pay(p.Tk, p.Hkv) ? kF32ThirdsColumns : 0) + 256 * (pay(p.T, p.Hq) ? kF32ThirdsColumns : 0);
}

template <int DP, bool FULL>
static hipError_t launch_backward(const PrefillBwdParams &p, hipStream_t stream) {
    const int32_t form = backward_form_f32(p);
    const int64_t row_blocks = (p.T + 15) / 16, key_blocks = (p.Tk + 15) / 16;
    if (form / 256) {
        if (hipError_t err = launch_bwd_rows_thirds(p, stream)) return err;
    } else {
        hipLaunchKernelGGL((f32_bwd_rows_kernel<DP, FULL>), f32_grid(row_blocks * p.B * p.Hq), dim3(kF32Threads), 0, stream, p);
        if (hipError_t err = hipGetLastError()) return err;
    }
    if (form % 256) return launch_bwd_cols_thirds(p, stream);
    hipLaunchKernelGGL((f32_bwd_cols_kernel<DP, FULL>), f32_grid(key_blocks * p.B * p.Hkv), dim3(kF32Threads), 0, stream, p);
    return hipGetLastError();
}

hipError_t launch_prefill_bwd_f32(const PrefillBwdParams &p, hipStream_t stream) {
    return p.d == 64    ? launch_backward<64, true>(p, stream)
           : p.d < 64   ? launch_backward<64, false>(p, stream)
           : p.d == 128 ? launch_backward<128, true>(p, stream)
           : p.d < 128  ? launch_backward<128, false>(p, stream)
           : p.d == 256 ? launch_backward<256, true>(p, stream)
                        : launch_backward<256, false>(p, stream);
}

}  // namespace plx
