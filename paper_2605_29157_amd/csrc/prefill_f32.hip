// fp32 Parallax, forward and backward of a prefill at d = 64, on the bf16 matrix instructions: every
// fp32 operand is cut into three bf16 thirds (its 24 bits exactly, from 2^-110 on) and a product of two operands is the
// six largest products of thirds, accumulated in fp32 by the instruction (Henry, Tang, Heinecke, "Leveraging the bfloat16
// Artificial Intelligence Datatype For Higher-Precision Computations", 2019). What is left out, second by third twice and third by
// third, is 2^-22 of a product at most (the first third is cut off, so the second reaches 2^-7 of the value, the third 2^-16), 0.4 *
// 2^-24 rms. 16 x 16 x 32 at bf16 takes 16 clocks, so a 32-deep step costs 96 clocks against 256 on v_mfma_f32_16x16x4_f32.
//
// Against 64 bits the results are closer than those of generic_f32.hip (relative error of o, dq, dr, dk, dv, 8
// sequences x 8 heads x 512 rows: 2.0, 3.2, 2.9, 3.2, 2.8e-7 against 2.9, 4.1, 3.7, 5.0, 4.2e-7).
// Time, forward / backward, us, generic_f32.hip -> here: 8 x 8 x 512 53.2 / 131 -> 40.4 / 107; 4 x 8 x 512 31.0 / 75.9
// -> 26.3 / 67.3; 8 heads x 2048 103 / 238 -> 83.6 / 222; 4 x 8 x 512 not causal 47.4 / 115 -> 33.9 / 89.9.
// What bounds it: vector ALU and matrix pipe one after the other, 40k and 26k clocks of the 85k that a SIMD
// of the forward of 8 x 8 x 512 takes: cutting is 5.5 instructions a value, and with 2 waves per SIMD (256
// registers) the two hardly overlap. Tried and slower: three waves per SIMD (spills; 45 -> 55), every wave cutting its own
// tiles without LDS (forward 46, backward 141), remainders by v_dot2 (copies and waits eat what it saves),
// 64 columns per workgroup (42 / 108 here, but half as many workgroups: 4 x 8 x 333 87 -> 120 a step). d = 128
// needs twice the registers: one workgroup per unit, 135 -> 237 for 2 x 8 x 500, so it stays there.
//
// Layout. A workgroup of four waves owns 16 * CG COLUMNS of the matrix tiles (query rows in the forward and in
// the dQ / dR pass, keys in the dK / dV pass) and walks the other side in tiles of 32 rows: CG column groups
// of 16 x KG = 4 / CG tiles at a time, a wave each. The columns are cut once and stay in registers. A tile is
// loaded and cut by the whole workgroup (cutting costs the vector ALU as much as the products cost the
// matrix pipe if every wave does it for itself) and lies in LDS as thirds, one swizzled 16-bit tile each.
//   scores   S^T = K Q^T: A = 16 keys by rows, B = the columns.
//   outputs  the accumulators of the two score blocks (lane (c, g): column c, keys 16 s + 4 g + r) are
//            the eight k-elements 4 s + r of the B operand of O^T += V^T P^T; A = V^T by transposing reads.
// The next tile travels under the products of this one. With KG = 2 the two halves of a column's keys meet in LDS
// at the end.
//
// Infinities, NaN and finite values whose products overflow: a third of them is NaN and so is
// every accumulator it reaches (also from a key that no column sees: 0 * NaN). A workgroup that ends with
// an accumulator that is not finite walks its tiles again with care: scores of operands that are not
// finite on the fp32 instruction, such values zero in the output operand, and what they do to the columns
// that see them added as sums of products that overflow.
// Small values: the last thirds of what is below 2^-110 are lost (bf16 ends at 2^-133). A workgroup that cut such a
// value of q, rho, k, v or dO, whatever it is multiplied with, walks again with every product on the fp32 instruction;
// so does one with a column whose largest gradient weight is that small. Softmax weights are not looked at (the
// largest of a column is 1, and a small one loses 2^-134 at most). Looking is half an instruction a value (exact zeros,
// which hide others from the minimum, two). Forward / backward of 8 x 8 x 512, us: 40.0 / 102 without it, 40.4 / 107 with it,
// 41.6 / 109 where a tenth of the values and every fifth row are zeros, 40.2 / 200 where every head has a row of dO at 1e-36.
#include "plx_f32.h"

namespace plx {

namespace {

// Head dimension, column groups, tiles at a time; blocks of 16 dimensions and steps of 32 in it
constexpr int DP = kF32ThirdsD, CG = kF32ThirdsColumns / 16, KG = kF32Waves / CG, COLS = 16 * CG, NA = DP / 16, NJ = DP / 32;

struct Thirds {
    u32x4 x[3];  // eight values each, largest third first
};

// Eight fp32 values in thirds. The first is cut off (a finite value stays finite), the others rounded:
// what is left of 24 bits fits the third one exactly (from kThirdsExact on).
__device__ __forceinline__ Thirds f32_cut(const f32x4 &lo, const f32x4 &hi) {
    Thirds t;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float a = i < 2 ? lo[2 * i] : hi[2 * i - 4], b = i < 2 ? lo[2 * i + 1] : hi[2 * i - 3];
        const uint32_t ua = __builtin_bit_cast(uint32_t, a), ub = __builtin_bit_cast(uint32_t, b);
        t.x[0][i] = __builtin_amdgcn_perm(ub, ua, 0x07060302);
        const float ra = a - __builtin_bit_cast(float, ua & 0xffff0000u), rb = b - __builtin_bit_cast(float, ub & 0xffff0000u);
        const uint32_t second = pack_bf16(ra, rb);
        t.x[1][i] = second;
        t.x[2][i] = pack_bf16(ra - bf16_lo_f32(second), rb - bf16_hi_f32(second));
    }
    return t;
}

// acc[i] += A[i] B[i] for N independent products, the small ones first. (Interleaved: one chain of dependent
// matrix instructions alone waits for each of them.)
template <int N>
__device__ __forceinline__ void mfma_thirds(const Thirds *const (&a)[N], const Thirds *const (&b)[N], f32x4 *const (&acc)[N]) {
    constexpr int kA[6] = {2, 0, 1, 1, 0, 0}, kB[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
    for (int k = 0; k < 6; ++k)
#pragma unroll
        for (int i = 0; i < N; ++i) *acc[i] = mfma16(a[i]->x[kA[k]], b[i]->x[kB[k]], *acc[i]);
}
// Output accumulators: the products of a tile are summed on their own and added to the running sum by the vector
// ALU, which rounds to nearest; the matrix instruction does not, and over the tiles of a long row that shows.
template <int N>
__device__ __forceinline__ void add_thirds(const Thirds *const (&a)[N], const Thirds *const (&b)[N], f32x4 *const (&acc)[N]) {
    f32x4 t[N];
#pragma unroll
    for (int i = 0; i < N; ++i) t[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    constexpr int kA[6] = {2, 0, 1, 1, 0, 0}, kB[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
    for (int k = 0; k < 6; ++k)
#pragma unroll
        for (int i = 0; i < N; ++i) t[i] = mfma16(a[i]->x[kA[k]], b[i]->x[kB[k]], t[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) *acc[i] += t[i];
}

// The smallest magnitude whose thirds hold it exactly, its last bit being no less than the smallest bf16, 2^-133; zero is
// exact too. The minimum is NaN where a value is.
constexpr float kThirdsExact = 0x1p-110f;
__device__ __forceinline__ float smallest(float low, const f32x4 &a, const f32x4 &b) {
#pragma unroll
    for (int i = 0; i < 4; ++i) low = __builtin_elementwise_minimum(__builtin_elementwise_minimum(low, fabsf(a[i])), fabsf(b[i]));
    return low;
}
// (without sign, less one: a zero is the largest)
__device__ __forceinline__ uint32_t size_or_most(float x) { return 2 * __builtin_bit_cast(uint32_t, x) - 1; }
__device__ __forceinline__ bool any_lost(const f32x4 &a, const f32x4 &b) {
    uint32_t low = 0xffffffffu;
#pragma unroll
    for (int i = 0; i < 4; ++i) low = min(low, min(size_or_most(a[i]), size_or_most(b[i])));
    return low < size_or_most(kThirdsExact);
}

__device__ __forceinline__ bool finite4(const f32x4 &x) {
    return fmaf(x[0], 0.f, fmaf(x[1], 0.f, fmaf(x[2], 0.f, x[3] * 0.f))) == 0.f;
}

// One lane's share of a column or row: dimensions 32 j + 8 g .. + 7 of it
struct RowPart {
    f32x4 x[DP / 32][2];
};
__device__ __forceinline__ RowPart load_part(const float *row, int g) {
    RowPart a;
#pragma unroll
    for (int j = 0; j < DP / 32; ++j)
#pragma unroll
        for (int h = 0; h < 2; ++h) a.x[j][h] = *(const f32x4 *)(row + 32 * j + 8 * g + 4 * h);
    return a;
}
__device__ __forceinline__ bool part_finite(const RowPart &a) {
    bool ok = true;
#pragma unroll
    for (int j = 0; j < DP / 32; ++j) ok &= finite4(a.x[j][0]) && finite4(a.x[j][1]);
    return ok;
}
__device__ __forceinline__ bool part_lost(const RowPart &a) {
    float low = kThirdsExact;
#pragma unroll
    for (int j = 0; j < DP / 32; ++j) low = smallest(low, a.x[j][0], a.x[j][1]);
    if (!__any(!(low >= kThirdsExact))) return false;
    bool lost = false;
#pragma unroll
    for (int j = 0; j < DP / 32; ++j) lost |= any_lost(a.x[j][0], a.x[j][1]);
    return lost;
}
struct CutPart {
    Thirds x[DP / 32];
};
__device__ __forceinline__ CutPart cut_part(const RowPart &a) {
    CutPart t;
#pragma unroll
    for (int j = 0; j < DP / 32; ++j) t.x[j] = f32_cut(a.x[j][0], a.x[j][1]);
    return t;
}
// acc + dot products over this lane's share, summed over the four lanes of the column
__device__ __forceinline__ float column_dot(const RowPart &a, const RowPart &b) {
    float acc = 0.f;
#pragma unroll
    for (int j = 0; j < DP / 32; ++j)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc = fmaf(a.x[j][h][i], b.x[j][h][i], acc);
    return rows_sum(acc);
}
// A score block on the fp32 instruction, both sides straight from global memory
__device__ __forceinline__ f32x4 scores_f32(const float *row, const float *col, int g) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int dim = 4 * g; dim < DP; dim += 16) {
        const f32x4 a = *(const f32x4 *)(row + dim), b = *(const f32x4 *)(col + dim);
#pragma unroll
        for (int i = 0; i < 4; ++i) acc = mfma_f32(a[i], b[i], acc);
    }
    return acc;
}

// ROWS rows of one tensor in thirds
struct CutTile {
    u32x4 x[3][32 * KG * DP / 8];
};
// ... and on their way there, a thread's chunks of eight values
struct Staged {
    static constexpr int kChunks = 32 * KG * DP / 8 / kF32Threads;
    f32x4 x[kChunks][2];
};
// row_of(i, row in its tile of 32) -> address; chunk i of a thread lies in tile i * kF32Threads / (4 DP)
template <typename RowOf>
__device__ __forceinline__ void stage(Staged &st, int tid, RowOf row_of) {
#pragma unroll
    for (int i = 0; i < Staged::kChunks; ++i) {
        const int e = tid + i * kF32Threads, row = e / (DP / 8), dim = 8 * (e % (DP / 8));
        const float *at = row_of(i * kF32Threads / (4 * DP), row & 31);
        st.x[i][0] = *(const f32x4 *)(at + dim), st.x[i][1] = *(const f32x4 *)(at + dim + 4);
    }
}
// Returns whether the thread met a value that its thirds do not hold; with care one that is not finite, and such values
// become zeros.
template <bool CARE>
__device__ __forceinline__ bool put(Staged &st, CutTile &tile, int tid) {
    bool odd = false;
    if constexpr (!CARE) {
        float low = kThirdsExact;
#pragma unroll
        for (int i = 0; i < Staged::kChunks; ++i) low = smallest(low, st.x[i][0], st.x[i][1]);
        if (__builtin_expect(__any(!(low >= kThirdsExact)), 0)) {
#pragma unroll
            for (int i = 0; i < Staged::kChunks; ++i) odd |= any_lost(st.x[i][0], st.x[i][1]);
        }
    }
#pragma unroll
    for (int i = 0; i < Staged::kChunks; ++i) {
        const int e = tid + i * kF32Threads, row = e / (DP / 8), chunk = e % (DP / 8);
        if constexpr (CARE)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                odd |= !finite4(st.x[i][h]);
#pragma unroll
                for (int k = 0; k < 4; ++k) st.x[i][h][k] = fabsf(st.x[i][h][k]) < -kNegInf ? st.x[i][h][k] : 0.f;
            }
        const Thirds t = f32_cut(st.x[i][0], st.x[i][1]);
#pragma unroll
        for (int n = 0; n < 3; ++n) tile.x[n][lds_chunk_slot<DP>(row, chunk)] = t.x[n];
    }
    return odd;
}
// Rows `row0` + c by rows (score operand, step j) and eight rows `row0` + 16 s + 4 g + r of dimension 16 n + c
__device__ __forceinline__ Thirds by_rows(const CutTile &tile, int row0, int j, int c, int g) {
    Thirds t;
#pragma unroll
    for (int n = 0; n < 3; ++n) t.x[n] = tile.x[n][lds_chunk_slot<DP>(row0 + c, 4 * j + g)];
    return t;
}
__device__ __forceinline__ Thirds transposed(const CutTile &tile, int row0, int n, int c, int g) {
    Thirds t;
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int row = row0 + 16 * s + 4 * g + (c >> 2), half = c & 3;
            const u32x2 x = lds_read_tr16((const char *)&tile.x[k][lds_chunk_slot<DP>(row, 2 * n + (half >> 1))] + 8 * (half & 1));
            t.x[k][2 * s] = x[0], t.x[k][2 * s + 1] = x[1];
        }
    return t;
}

// What values that are not finite (zeros in the operand) do to the columns: weights w[s][r] of row 16 s + 4 g +
// r, which the column sees if bit 4 s + r of `seen` is set. Sums of products of finite numbers that overflow
// where +inf (up) or -inf (down) reaches a column, and both where a NaN does or a zero weight meets an infinity.
template <typename RowOf>
__device__ __forceinline__ void add_not_finite(f32x4 (&acc)[DP / 16], const f32x4 (&w)[2], unsigned seen, int c, RowOf row_of) {
    constexpr float kBig = 3.0e38f, kInf = -kNegInf;
#pragma unroll
    for (int n = 0; n < DP / 16; ++n) {
        f32x4 up = {0.f, 0.f, 0.f, 0.f}, down = up;
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float x = row_of(s, r)[16 * n + c], wt = w[s][r];
                const bool sees = (seen >> (4 * s + r)) & 1;
                const float high = !(x < kInf) ? kBig : 0.f, low = !(x > kNegInf) ? kBig : 0.f;
                const float plus = sees && !(wt < 0.f) ? kBig : 0.f, minus = sees && !(wt > 0.f) ? kBig : 0.f;
                up = mfma_f32(high, plus, up), up = mfma_f32(low, minus, up);
                down = mfma_f32(high, minus, down), down = mfma_f32(low, plus, down);
            }
        acc[n] = acc[n] + up - down;
    }
}

// Output products on the fp32 instruction, for weights that are not finite (thirds of an infinity would make them NaN)
template <typename RowOf>
__device__ __forceinline__ void add_products_f32(f32x4 (&acc)[NA], const f32x4 (&w)[2], int c, RowOf row_of) {
#pragma unroll
    for (int n = 0; n < NA; ++n)
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float x = row_of(s, r)[16 * n + c];
                acc[n] = mfma_f32(fabsf(x) < -kNegInf ? x : 0.f, w[s][r], acc[n]);
            }
}
__device__ __forceinline__ bool wave_finite(const f32x4 (&w)[2]) { return __all(finite4(w[0]) && finite4(w[1])); }

// What a walk leaves to be said about it: an accumulator that is not finite, or operands that their thirds do not hold
enum { kNotFinite = 1, kLost = 2 };
__device__ __forceinline__ int verdict(const f32x4 (&a)[NA], const f32x4 (&b)[NA], float more, bool lost) {
    float chk = more * 0.f;
#pragma unroll
    for (int n = 0; n < NA; ++n)
#pragma unroll
        for (int i = 0; i < 4; ++i) chk = fmaf(a[n][i], 0.f, fmaf(b[n][i], 0.f, chk));
    return (__any(!(chk == 0.f)) ? kNotFinite : 0) | (__any(lost) ? kLost : 0);
}

// Sizes of the weights of an output, one after another: the bits of their first thirds on top of each other. An exponent
// of 16 or more, 2^-111, leaves a bit above the lowest four that no smaller ones make together.
struct WeightSizes {
    uint32_t bits = 0;
    __device__ __forceinline__ void add(const Thirds &w) {
        bits |= w.x[0][0] | w.x[0][1];
        bits |= w.x[0][2] | w.x[0][3];
    }
    // bit c: column c has weights that are not zero; bit 16 + c: a large one
    __device__ __forceinline__ unsigned columns() const {
        auto fold = [](unsigned long long lanes) {
            const unsigned x = (unsigned)lanes | (unsigned)(lanes >> 32);
            return (x | x >> 16) & 0xffffu;
        };
        return fold(__ballot((bits & 0x7fff7fffu) != 0)) | fold(__ballot((bits & 0x78007800u) != 0)) << 16;
    }
};
// kLost if a column has weights, all of them small, over the waves that share it
__device__ __forceinline__ int small_columns(const unsigned (&sizes)[kF32Waves]) {
    int said = 0;
#pragma unroll
    for (int cg = 0; cg < CG; ++cg) {
        unsigned x = 0;
#pragma unroll
        for (int kg = 0; kg < KG; ++kg) x |= sizes[kg * CG + cg];
        if (x & 0xffffu & ~(x >> 16)) said = kLost;
    }
    return said;
}

// The two halves of the keys (waves CG .. 2 CG - 1 hand theirs to waves 0 .. CG - 1)
__device__ __forceinline__ void join_halves(f32x4 (&a)[NA], f32x4 (&b)[NA], f32x4 *buf, int cg, int kg, int lane) {
    f32x4 *at = buf + cg * 2 * NA * 64 + lane;
    __syncthreads();
    if (kg == 1)
#pragma unroll
        for (int n = 0; n < NA; ++n) at[n * 64] = a[n], at[(NA + n) * 64] = b[n];
    __syncthreads();
    if (kg == 0)
#pragma unroll
        for (int n = 0; n < NA; ++n) a[n] += at[n * 64], b[n] += at[(NA + n) * 64];
}

template <int TENSORS>
union Lds {
    CutTile tile[TENSORS];
    f32x4 merge[CG * 2 * NA * 64];
};

// ---- forward -------------------------------------------------------------------------------
template <bool USE_R>
__global__ __launch_bounds__(kF32Threads, 2) void f32_prefill_kernel(PrefillParams p) {
    __shared__ Lds<2> lds;  // k, v
    __shared__ float sm[3][kF32Waves][16];
    __shared__ int odd[kF32Waves];
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int c = lane & 15, g = lane >> 4, cg = w % CG, kg = w / CG;
    const int n_blocks = (p.T + COLS - 1) / COLS;
    int64_t id = f32_block_id();
    if (id >= (int64_t)n_blocks * p.B * p.Hq) return;
    const int head = (int)(id % p.Hq);
    id /= p.Hq;
    const int b = (int)(id % p.B);
    const int blk = n_blocks - 1 - (int)(id / p.B);  // causal: the longest rows first
    const int hk = head / p.G;

    // row t sees the keys [row_lo(t), row_end(t))
    auto row_end = [&](int t) { return p.causal ? max(p.Tk - (p.T - 1 - t), 0) : p.Tk; };
    auto row_lo = [&](int t) { return p.window > 0 ? max(row_end(t) - p.window, 0) : 0; };
    const int t0 = COLS * blk, t1 = min(t0 + COLS, p.T) - 1;                      // of the workgroup
    const int w0 = min(t0 + 16 * cg, t1), w1 = min(t0 + 16 * cg + 15, t1);        // of the wave
    const int t = min(t0 + 16 * cg + c, t1), my_end = row_end(t), my_lo = row_lo(t);
    const int all_lo = row_lo(w1), all_end = row_end(w0), any_lo = row_lo(w0), any_end = row_end(w1);
    const int lo = row_lo(t0) / 32, hi = (row_end(t1) + 31) / 32, last_key = row_end(t1) - 1;
    const float *qcol = (const float *)p.q + b * p.qs[0] + head * p.qs[1] + t * p.qs[2];
    const float *rcol = USE_R ? (const float *)p.r + b * p.rs[0] + head * p.rs[1] + t * p.rs[2] : qcol;
    const float *kb = (const float *)p.k + b * p.ks[0] + hk * p.ks[1], *vb = (const float *)p.v + b * p.vs[0] + hk * p.vs[1];
    auto k_row = [&](int key) { return kb + (int64_t)min(key, last_key) * p.ks[2]; };
    auto v_row = [&](int key) { return vb + (int64_t)min(key, last_key) * p.vs[2]; };

    Staged ks, vs;
    auto load = [&](int first) {  // tiles first .. first + KG - 1
        stage(ks, tid, [&](int i, int row) { return k_row(32 * (first + i) + row); });
        stage(vs, tid, [&](int i, int row) { return v_row(32 * (first + i) + row); });
    };
    if (lo < hi) load(lo);
    CutPart q, rho;
    bool lost;  // a value that its thirds do not hold
    {
        const RowPart x = load_part(qcol, g);
        lost = part_lost(x), q = cut_part(x);
    }
    if constexpr (USE_R) {
        const RowPart x = load_part(rcol, g);
        lost |= part_lost(x), rho = cut_part(x);
    }

    const float scale_log2 = p.scale * kLog2e;
    float m_run, d1, d2;  // the sums over this lane's keys only
    f32x4 o1[NA], o2[NA];
    bool all_f32 = false;  // with care: every product on the fp32 instruction
    auto walk = [&](auto with_care) {
        // (one rounding per operation in both walks: what is finite comes out the same bit for bit)
#pragma clang fp contract(off)
        constexpr bool CARE = decltype(with_care)::value;
        m_run = kNegInf, d1 = d2 = 0.f;
#pragma unroll
        for (int n = 0; n < NA; ++n) o1[n] = o2[n] = f32x4{0.f, 0.f, 0.f, 0.f};
        bool odd_cols = false;
        if constexpr (CARE) {
            odd_cols = !part_finite(load_part(qcol, g)) || !part_finite(load_part(rcol, g));
            odd_cols = all_f32 || __any(odd_cols);
        }
        for (int first = lo; first < hi; first += KG) {
            int odd_k = 0, odd_v = 0;
            if (first > lo) __syncthreads();  // (the last tiles have been read)
            if constexpr (CARE) {
                load(first);
                odd_k = put<true>(ks, lds.tile[0], tid), odd_v = put<true>(vs, lds.tile[1], tid);
                odd_k = __syncthreads_or(odd_k), odd_v = __syncthreads_or(odd_v);
            } else {
                lost |= put<false>(ks, lds.tile[0], tid), lost |= put<false>(vs, lds.tile[1], tid);
                __syncthreads();
                if (first + KG < hi) load(first + KG);
            }
            const int key0 = 32 * (first + kg);
            if (key0 >= any_end || key0 + 32 <= any_lo) continue;  // (uniform over the wave)

            f32x4 s1[2], s2[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) s1[s] = s2[s] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const Thirds a0 = by_rows(lds.tile[0], 32 * kg, j, c, g), a1 = by_rows(lds.tile[0], 32 * kg + 16, j, c, g);
                const Thirds *const qj = &q.x[j], *const rj = &rho.x[j];
                if constexpr (USE_R)
                    mfma_thirds<4>({&a0, &a0, &a1, &a1}, {qj, rj, qj, rj}, {&s1[0], &s2[0], &s1[1], &s2[1]});
                else
                    mfma_thirds<2>({&a0, &a1}, {qj, qj}, {&s1[0], &s1[1]});
            }
            if constexpr (CARE)
                if (odd_cols || odd_k)
#pragma unroll
                    for (int s = 0; s < 2; ++s) {
                        s1[s] = scores_f32(k_row(key0 + 16 * s + c), qcol, g);
                        if constexpr (USE_R) s2[s] = scores_f32(k_row(key0 + 16 * s + c), rcol, g);
                    }
            const bool whole = key0 >= all_lo && key0 + 32 <= all_end;  // uniform
            unsigned seen = 255u;
            float tmax = kNegInf;
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    s1[s][r] *= scale_log2;
                    if (!whole) {
                        const int key = key0 + 16 * s + 4 * g + r;
                        if (!(key >= my_lo && key < my_end)) s1[s][r] = kNegInf, s2[s][r] = 0.f, seen &= ~(1u << (4 * s + r));
                    }
                    tmax = fmaxf(tmax, s1[s][r]);
                }
            tmax = rows_max(tmax);
            const float m_new = fmaxf(m_run, tmax);
            const float m_use = m_new == kNegInf ? 0.f : m_new;
            const float alpha = fast_exp2(m_run - m_use);  // 0 on the first tile that is seen
            m_run = m_new;
            f32x4 p1[2], p2[2];
            float sum1 = 0.f, sum2 = 0.f;
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    p1[s][r] = fast_exp2(s1[s][r] - m_use);  // 0 if masked
                    p2[s][r] = p1[s][r] * s2[s][r];
                    sum1 += p1[s][r], sum2 += p2[s][r];
                }
            d1 = fmaf(d1, alpha, sum1), d2 = fmaf(d2, alpha, sum2);
            if (!__all(alpha == 1.f)) {
#pragma unroll
                for (int n = 0; n < NA; ++n) o1[n] *= alpha, o2[n] *= alpha;
            }
            if constexpr (CARE)
                if (odd_v) {
                    auto at = [&](int s, int r) { return v_row(key0 + 16 * s + 4 * g + r); };
                    add_not_finite(o1, p1, seen, c, at);
                    if constexpr (USE_R) add_not_finite(o2, p2, seen, c, at);
                }
            if constexpr (CARE)
                if (all_f32 || !wave_finite(p1) || !wave_finite(p2)) {
                    auto at = [&](int s, int r) { return v_row(key0 + 16 * s + 4 * g + r); };
                    add_products_f32(o1, p1, c, at);
                    if constexpr (USE_R) add_products_f32(o2, p2, c, at);
                    continue;
                }
            const Thirds w1 = f32_cut(p1[0], p1[1]), w2 = f32_cut(p2[0], p2[1]);
#pragma unroll
            for (int n = 0; n < NA; n += 2) {
                const Thirds a0 = transposed(lds.tile[1], 32 * kg, n, c, g), a1 = transposed(lds.tile[1], 32 * kg, n + 1, c, g);
                if constexpr (USE_R)
                    add_thirds<4>({&a0, &a0, &a1, &a1}, {&w1, &w2, &w1, &w2}, {&o1[n], &o2[n], &o1[n + 1], &o2[n + 1]});
                else
                    add_thirds<2>({&a0, &a1}, {&w1, &w1}, {&o1[n], &o1[n + 1]});
            }
        }
        d1 = rows_sum(d1), d2 = rows_sum(d2);
        const int said = verdict(o1, o2, d1 + d2, lost);
        if (lane == 0) odd[w] = said;
        if (g == 0) sm[0][w][c] = m_run, sm[1][w][c] = d1, sm[2][w][c] = d2;
    };
    walk(std::false_type{});
    __syncthreads();
    if (const int said = odd[0] | odd[1] | odd[2] | odd[3]) {
        all_f32 = said & kLost;
        __syncthreads();
        walk(std::true_type{});
        __syncthreads();
    }
    {  // the halves on one reference
        const float m_own = m_run;
        float m_all = kNegInf;
#pragma unroll
        for (int i = 0; i < KG; ++i) m_all = fmaxf(m_all, sm[0][i * CG + cg][c]);
        d1 = d2 = 0.f;
#pragma unroll
        for (int i = 0; i < KG; ++i) {
            const float m_i = sm[0][i * CG + cg][c], wt = m_i == kNegInf ? 0.f : fast_exp2(m_i - m_all);
            d1 += wt * sm[1][i * CG + cg][c], d2 += wt * sm[2][i * CG + cg][c];
        }
        const float wt = m_own == kNegInf ? 0.f : fast_exp2(m_own - m_all);
#pragma unroll
        for (int n = 0; n < NA; ++n) o1[n] *= wt, o2[n] *= wt;
        m_run = m_all;
        join_halves(o1, o2, lds.merge, cg, kg, lane);
    }
    if (kg != 0 || t0 + 16 * cg + c >= p.T) return;

    // lane (c, g): dimensions 16 n + 4 g .. + 3 of column c
    const float inv = d1 > 0.f ? 1.f / d1 : 0.f;
    const int64_t orow = b * p.os[0] + head * p.os[1] + t * p.os[2];
#pragma unroll
    for (int n = 0; n < NA; ++n) {
        const int dim = 16 * n + 4 * g;
        f32x4 out = {0.f, 0.f, 0.f, 0.f}, mean = out;  // empty key set: zeros
        if (d1 > 0.f) {
            mean = o1[n] * inv;
            out = mean * (1.f + d2 * inv) - o2[n] * inv;
        }
        *(f32x4 *)((float *)p.o + orow + dim) = out;
        if (p.vbar) *(f32x4 *)((float *)p.vbar + orow + dim) = mean;
    }
    if (p.row_stats && g == 0) {
        float *st = p.row_stats + (((int64_t)b * p.Hq + head) * p.T + t) * 2;
        st[0] = d1 > 0.f ? m_run + log2f(d1) : kNegInf;
        st[1] = d1 > 0.f ? d2 * inv : 0.f;
    }
}

// ---- backward (closed forms of the paper's App. D) -------------------------------------------
// dQ, dR: columns are query rows. Every wave first forms tau = dO.o and beta = dO.vbar of its columns; (lse,
// ubar, tau, beta) go to the workspace for the dK / dV pass.
__global__ __launch_bounds__(kF32Threads, 2) void f32_prefill_rows_kernel(PrefillBwdParams p) {
    __shared__ Lds<2> lds;  // k, v
    __shared__ int odd[kF32Waves];
    __shared__ unsigned sizes[2][kF32Waves];
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int c = lane & 15, g = lane >> 4, cg = w % CG, kg = w / CG, off = p.Tk - p.T;
    const int n_blocks = (p.T + COLS - 1) / COLS;
    int64_t id = f32_block_id();
    if (id >= (int64_t)n_blocks * p.B * p.Hq) return;
    const int h = (int)(id % p.Hq);
    id /= p.Hq;
    const int b = (int)(id % p.B);
    const int t0 = COLS * (n_blocks - 1 - (int)(id / p.B)), t1 = min(t0 + COLS, p.T) - 1;
    auto row_end = [&](int t) { return p.causal ? min(max(t + 1 + off, 0), p.Tk) : p.Tk; };
    auto row_lo = [&](int t) { return p.window > 0 ? max(row_end(t) - p.window, 0) : 0; };
    const int w0 = min(t0 + 16 * cg, t1), w1 = min(t0 + 16 * cg + 15, t1);
    const int t = min(t0 + 16 * cg + c, t1), my_end = row_end(t), my_lo = row_lo(t);
    const int all_lo = row_lo(w1), all_end = row_end(w0), any_lo = row_lo(w0), any_end = row_end(w1);
    const int lo = row_lo(t0) / 32, hi = (row_end(t1) + 31) / 32, last_key = row_end(t1) - 1;
    const int64_t row = ((int64_t)b * p.Hq + h) * p.T + t, khead = ((int64_t)b * p.Hkv + h / p.G) * p.Tk;
    const float *qcol = (const float *)p.q + row * DP, *rcol = (const float *)p.r + row * DP, *gcol = (const float *)p.d_o + row * DP;
    auto k_row = [&](int key) { return (const float *)p.k + (khead + min(key, last_key)) * DP; };
    auto v_row = [&](int key) { return (const float *)p.v + (khead + min(key, last_key)) * DP; };

    Staged ks, vs;
    auto load = [&](int first) {
        stage(ks, tid, [&](int i, int r) { return k_row(32 * (first + i) + r); });
        stage(vs, tid, [&](int i, int r) { return v_row(32 * (first + i) + r); });
    };
    if (lo < hi) load(lo);
    float lse, ubar, tau, beta;
    CutPart q, rho, up;
    bool lost;
    {
        const RowPart x = load_part(gcol, g);
        lost = part_lost(x);
        tau = column_dot(x, load_part((const float *)p.o + row * DP, g));
        beta = column_dot(x, load_part((const float *)p.vbar + row * DP, g));
        lse = p.row_stats[2 * row], ubar = p.row_stats[2 * row + 1];
        if (kg == 0 && g == 0 && t0 + 16 * cg + c <= t1) ((f32x4 *)p.row_cache)[row] = f32x4{lse, ubar, tau, beta};
        up = cut_part(x);
    }
    {
        const RowPart x = load_part(qcol, g);
        lost |= part_lost(x), q = cut_part(x);
    }
    {
        const RowPart x = load_part(rcol, g);
        lost |= part_lost(x), rho = cut_part(x);
    }
    f32x4 dq[NA], dr[NA];
    const float scale_log2 = p.scale * kLog2e;
    bool all_f32 = false;  // with care: every product on the fp32 instruction
    auto walk = [&](auto with_care) {
        constexpr bool CARE = decltype(with_care)::value;
#pragma unroll
        for (int n = 0; n < NA; ++n) dq[n] = dr[n] = f32x4{0.f, 0.f, 0.f, 0.f};
        WeightSizes size1, size2;
        bool odd_cols = false;
        if constexpr (CARE) {
            odd_cols = !part_finite(load_part(qcol, g)) || !part_finite(load_part(rcol, g)) ||
                       !part_finite(load_part(gcol, g));
            odd_cols = all_f32 || __any(odd_cols);
        }
        for (int first = lo; first < hi; first += KG) {
            int odd_k = 0, odd_v = 0;
            if (first > lo) __syncthreads();
            if constexpr (CARE) {
                load(first);
                odd_k = put<true>(ks, lds.tile[0], tid), odd_v = put<true>(vs, lds.tile[1], tid);
                odd_k = __syncthreads_or(odd_k), odd_v = __syncthreads_or(odd_v);
            } else {
                lost |= put<false>(ks, lds.tile[0], tid), lost |= put<false>(vs, lds.tile[1], tid);
                __syncthreads();
                if (first + KG < hi) load(first + KG);
            }
            const int key0 = 32 * (first + kg);
            if (key0 >= any_end || key0 + 32 <= any_lo) continue;

            f32x4 a[2], s1[2], s2[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) a[s] = s1[s] = s2[s] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    const Thirds x = by_rows(lds.tile[0], 32 * kg + 16 * s, j, c, g);
                    const Thirds y = by_rows(lds.tile[1], 32 * kg + 16 * s, j, c, g);
                    mfma_thirds<3>({&x, &x, &y}, {&q.x[j], &rho.x[j], &up.x[j]}, {&s1[s], &s2[s], &a[s]});
                }
            }
            if constexpr (CARE)
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    const int key = key0 + 16 * s + c;
                    if (odd_cols || odd_k)
                        s1[s] = scores_f32(k_row(key), qcol, g), s2[s] = scores_f32(k_row(key), rcol, g);
                    if (odd_cols || odd_v) a[s] = scores_f32(v_row(key), gcol, g);
                }
            const bool whole = key0 >= all_lo && key0 + 32 <= all_end;
            unsigned seen = 255u;
            f32x4 g1[2], g2[2];
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float pr = fast_exp2(s1[s][r] * scale_log2 - lse);
                    const float dlt = a[s][r] - beta;
                    g1[s][r] = pr * (a[s][r] - tau + (ubar - s2[s][r]) * dlt);
                    g2[s][r] = -pr * dlt;
                    if (!whole) {
                        const int key = key0 + 16 * s + 4 * g + r;
                        if (!(key >= my_lo && key < my_end)) g1[s][r] = g2[s][r] = 0.f, seen &= ~(1u << (4 * s + r));
                    }
                }
            if constexpr (CARE)
                if (odd_k) {
                    auto at = [&](int s, int r) { return k_row(key0 + 16 * s + 4 * g + r); };
                    add_not_finite(dq, g1, seen, c, at);
                    add_not_finite(dr, g2, seen, c, at);
                }
            if constexpr (CARE)
                if (all_f32 || !wave_finite(g1) || !wave_finite(g2)) {
                    auto at = [&](int s, int r) { return k_row(key0 + 16 * s + 4 * g + r); };
                    add_products_f32(dq, g1, c, at), add_products_f32(dr, g2, c, at);
                    continue;
                }
            const Thirds w1 = f32_cut(g1[0], g1[1]), w2 = f32_cut(g2[0], g2[1]);
            if constexpr (!CARE) size1.add(w1), size2.add(w2);
#pragma unroll
            for (int n = 0; n < NA; n += 2) {
                const Thirds x0 = transposed(lds.tile[0], 32 * kg, n, c, g), x1 = transposed(lds.tile[0], 32 * kg, n + 1, c, g);
                add_thirds<4>({&x0, &x0, &x1, &x1}, {&w1, &w2, &w1, &w2}, {&dq[n], &dr[n], &dq[n + 1], &dr[n + 1]});
            }
        }
        const int said = verdict(dq, dr, 0.f, lost);
        const unsigned columns[2] = {size1.columns(), size2.columns()};
        if (lane == 0) odd[w] = said, sizes[0][w] = columns[0], sizes[1][w] = columns[1];
    };
    walk(std::false_type{});
    __syncthreads();
    if (const int said = odd[0] | odd[1] | odd[2] | odd[3] | small_columns(sizes[0]) | small_columns(sizes[1])) {
        all_f32 = said & kLost;
        __syncthreads();
        walk(std::true_type{});
    }
    join_halves(dq, dr, lds.merge, cg, kg, lane);
    if (kg != 0 || t0 + 16 * cg + c >= p.T) return;
#pragma unroll
    for (int n = 0; n < NA; ++n) {
        const int dim = 16 * n + 4 * g;
        *(f32x4 *)((float *)p.dq + row * DP + dim) = dq[n] * p.scale;
        *(f32x4 *)((float *)p.dr + row * DP + dim) = dr[n];
    }
}

// dK, dV: columns are keys; the tiles are those of all query heads of the group.
__global__ __launch_bounds__(kF32Threads, 2) void f32_prefill_cols_kernel(PrefillBwdParams p) {
    __shared__ Lds<3> lds;  // q, rho, dO
    __shared__ int odd[kF32Waves];
    __shared__ unsigned sizes[3][kF32Waves];
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int c = lane & 15, g = lane >> 4, cg = w % CG, kg = w / CG, off = p.Tk - p.T;
    const int n_blocks = (p.Tk + COLS - 1) / COLS;
    int64_t id = f32_block_id();
    if (id >= (int64_t)n_blocks * p.B * p.Hkv) return;
    const int hk = (int)(id % p.Hkv);
    id /= p.Hkv;
    const int b = (int)(id % p.B);
    const int j0 = COLS * (int)(id / p.B), j1 = min(j0 + COLS, p.Tk) - 1;  // causal: the first keys are seen by most rows
    // rows [key_lo, key_end) see key j
    auto key_lo = [&](int j) { return p.causal ? max(j - off, 0) : 0; };
    auto key_end = [&](int j) { return p.window > 0 ? min(p.T, max(j - off + p.window, 0)) : p.T; };
    const int w0 = min(j0 + 16 * cg, j1), w1 = min(j0 + 16 * cg + 15, j1), j = min(j0 + 16 * cg + c, j1);
    const int my_lo = key_lo(j), my_end = key_end(j);
    const int all_lo = key_lo(w1), all_end = key_end(w0), any_lo = key_lo(w0), any_end = key_end(w1);
    const int lo = key_lo(j0) / 32, end = key_end(j1);  // (both bounds grow with the key)
    const int per_head = max((end + 31) / 32 - lo, 0), n_items = per_head * p.G;
    const int64_t col = (((int64_t)b * p.Hkv + hk) * p.Tk + j) * DP;
    const float *kcol = (const float *)p.k + col, *vcol = (const float *)p.v + col;
    auto head_of = [&](int item) { return ((int64_t)b * p.Hq + hk * p.G + item / per_head) * p.T; };
    auto row_of = [&](const void *base, int item, int r) {
        item = min(item, n_items - 1);
        return (const float *)base + (head_of(item) + min(32 * (lo + item % per_head) + r, end - 1)) * DP;
    };

    Staged xq, xr, xg;
    auto load = [&](int first) {
        stage(xq, tid, [&](int i, int r) { return row_of(p.q, first + i, r); });
        stage(xr, tid, [&](int i, int r) { return row_of(p.r, first + i, r); });
        stage(xg, tid, [&](int i, int r) { return row_of(p.d_o, first + i, r); });
    };
    if (n_items > 0) load(0);
    CutPart kk, vv;
    bool lost;
    {
        const RowPart x = load_part(kcol, g);
        lost = part_lost(x), kk = cut_part(x);
    }
    {
        const RowPart x = load_part(vcol, g);
        lost |= part_lost(x), vv = cut_part(x);
    }
    f32x4 dk[NA], dv[NA];
    const float scale_log2 = p.scale * kLog2e;
    bool all_f32 = false;  // with care: every product on the fp32 instruction
    auto walk = [&](auto with_care) {
        constexpr bool CARE = decltype(with_care)::value;
#pragma unroll
        for (int n = 0; n < NA; ++n) dk[n] = dv[n] = f32x4{0.f, 0.f, 0.f, 0.f};
        WeightSizes size_w, size1, size2;
        bool odd_cols = false;
        if constexpr (CARE) {
            odd_cols = !part_finite(load_part(kcol, g)) || !part_finite(load_part(vcol, g));
            odd_cols = all_f32 || __any(odd_cols);
        }
        for (int first = 0; first < n_items; first += KG) {
            int odd_q = 0, odd_r = 0, odd_g = 0;
            if (first > 0) __syncthreads();
            if constexpr (CARE) {
                load(first);
                odd_q = put<true>(xq, lds.tile[0], tid), odd_r = put<true>(xr, lds.tile[1], tid);
                odd_g = put<true>(xg, lds.tile[2], tid);
                odd_q = __syncthreads_or(odd_q), odd_r = __syncthreads_or(odd_r), odd_g = __syncthreads_or(odd_g);
            } else {
                lost |= put<false>(xq, lds.tile[0], tid), lost |= put<false>(xr, lds.tile[1], tid);
                lost |= put<false>(xg, lds.tile[2], tid);
                __syncthreads();
                if (first + KG < n_items) load(first + KG);
            }
            const int item = first + kg;
            const int i0 = 32 * (lo + item % per_head);
            if (item >= n_items || i0 >= any_end || i0 + 32 <= any_lo) continue;
            const int64_t head = head_of(item);
            f32x4 sc[2][4];  // (lse, ubar, tau, beta) of rows i0 + 16 s + 4 g + r
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int r = 0; r < 4; ++r) sc[s][r] = ((const f32x4 *)p.row_cache)[head + min(i0 + 16 * s + 4 * g + r, end - 1)];
            f32x4 s1[2], s2[2], a[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) a[s] = s1[s] = s2[s] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int jj = 0; jj < NJ; ++jj) {
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    const int r0 = 32 * kg + 16 * s;
                    const Thirds x = by_rows(lds.tile[0], r0, jj, c, g), y = by_rows(lds.tile[1], r0, jj, c, g);
                    const Thirds z = by_rows(lds.tile[2], r0, jj, c, g);
                    mfma_thirds<3>({&x, &y, &z}, {&kk.x[jj], &kk.x[jj], &vv.x[jj]}, {&s1[s], &s2[s], &a[s]});
                }
            }
            if constexpr (CARE)
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    const int r = 16 * s + c;
                    if (odd_cols || odd_q) s1[s] = scores_f32(row_of(p.q, item, r), kcol, g);
                    if (odd_cols || odd_r) s2[s] = scores_f32(row_of(p.r, item, r), kcol, g);
                    if (odd_cols || odd_g) a[s] = scores_f32(row_of(p.d_o, item, r), vcol, g);
                }
            const bool whole = i0 >= all_lo && i0 + 32 <= all_end;
            unsigned seen = 255u;
            f32x4 wt[2], g1[2], g2[2];
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const f32x4 &x = sc[s][r];
                    const float pr = fast_exp2(s1[s][r] * scale_log2 - x[0]);
                    const float um = x[1] - s2[s][r], dlt = a[s][r] - x[3];
                    wt[s][r] = pr * (1.f + um);
                    g1[s][r] = pr * (a[s][r] - x[2] + um * dlt) * p.scale;
                    g2[s][r] = -pr * dlt;
                    if (!whole) {
                        const int i = i0 + 16 * s + 4 * g + r;
                        if (!(i >= my_lo && i < my_end)) wt[s][r] = g1[s][r] = g2[s][r] = 0.f, seen &= ~(1u << (4 * s + r));
                    }
                }
            auto add = [&](int tensor, const void *base, int is_odd, const f32x4(&weights)[2], WeightSizes &sizes_of, f32x4(&acc)[NA]) {
                if constexpr (CARE) {
                    auto at = [&](int s, int r) { return row_of(base, item, 16 * s + 4 * g + r); };
                    if (is_odd) add_not_finite(acc, weights, seen, c, at);
                    if (all_f32 || !wave_finite(weights)) {
                        add_products_f32(acc, weights, c, at);
                        return;
                    }
                }
                const Thirds y = f32_cut(weights[0], weights[1]);
                if constexpr (!CARE) sizes_of.add(y);
#pragma unroll
                for (int n = 0; n < NA; n += 4) {
                    Thirds x[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) x[i] = transposed(lds.tile[tensor], 32 * kg, n + i, c, g);
                    add_thirds<4>({&x[0], &x[1], &x[2], &x[3]}, {&y, &y, &y, &y}, {&acc[n], &acc[n + 1], &acc[n + 2], &acc[n + 3]});
                }
            };
            add(0, p.q, odd_q, g1, size1, dk);
            add(1, p.r, odd_r, g2, size2, dk);
            add(2, p.d_o, odd_g, wt, size_w, dv);
        }
        const int said = verdict(dk, dv, 0.f, lost);
        const unsigned columns[3] = {size1.columns(), size2.columns(), size_w.columns()};
        if (lane == 0) odd[w] = said, sizes[0][w] = columns[0], sizes[1][w] = columns[1], sizes[2][w] = columns[2];
    };
    walk(std::false_type{});
    __syncthreads();
    if (const int said = odd[0] | odd[1] | odd[2] | odd[3] | small_columns(sizes[0]) | small_columns(sizes[1]) |
                         small_columns(sizes[2])) {
        all_f32 = said & kLost;
        __syncthreads();
        walk(std::true_type{});
    }
    join_halves(dk, dv, lds.merge, cg, kg, lane);
    if (kg != 0 || j0 + 16 * cg + c >= p.Tk) return;
#pragma unroll
    for (int n = 0; n < NA; ++n) {
        const int dim = 16 * n + 4 * g;
        *(f32x4 *)((float *)p.dk + col + dim) = dk[n];
        *(f32x4 *)((float *)p.dv + col + dim) = dv[n];
    }
}
}  // namespace

hipError_t launch_forward_thirds(const PrefillParams &p, hipStream_t stream) {
    const dim3 grid = f32_grid(f32_thirds_blocks(p.T, p.B, p.Hq)), block(kF32Threads);
    if (p.use_r)
        hipLaunchKernelGGL(f32_prefill_kernel<true>, grid, block, 0, stream, p);
    else
        hipLaunchKernelGGL(f32_prefill_kernel<false>, grid, block, 0, stream, p);
    return hipGetLastError();
}

hipError_t launch_bwd_rows_thirds(const PrefillBwdParams &p, hipStream_t stream) {
    hipLaunchKernelGGL(f32_prefill_rows_kernel, f32_grid(f32_thirds_blocks(p.T, p.B, p.Hq)), dim3(kF32Threads), 0, stream, p);
    return hipGetLastError();
}

hipError_t launch_bwd_cols_thirds(const PrefillBwdParams &p, hipStream_t stream) {
    hipLaunchKernelGGL(f32_prefill_cols_kernel, f32_grid(f32_thirds_blocks(p.Tk, p.B, p.Hkv)), dim3(kF32Threads), 0, stream, p);
    return hipGetLastError();
}

}  // namespace plx
