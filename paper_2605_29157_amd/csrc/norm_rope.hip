// RMSNorm over the head dimension followed by rotary position embedding, for up to three
// tensors (q, rho, k of one layer) in ONE launch -- the operations the paper's language-model
// runs apply to q, k and rho in front of the attention call (experiment setup of Sec. 5 and the
// backbone appendix: RMSNorm on q, k, rho; RoPE with base 1e6). Standard formulas:
//     y = x / sqrt(mean_c(x_c^2) + eps) * gamma
//     (y_2i, y_2i+1) rotated by pos * theta^(-2i/d)   (adjacent pairs)
// HBM bound: every element is read once and written once, 16 bytes per lane; the lanes of one row
// (d * element size / 16 of them) share the sum of squares, rows of 8 and 16 lanes without a trip through the LDS. The angle is
// formed and reduced modulo 2 pi in double precision (pos * frequency reaches 1e5 and more, where
// fp32 would lose the fraction), sine and cosine are taken in single precision -- once per
// (position, pair), for all heads of all tensors.
#include <algorithm>
#include <cmath>

#include "plx_device.h"
#include "plx_kernels.h"

namespace plx {

constexpr int kNormRopeTripHeads = 4;

template <typename T>
struct Chunk;  // 16 bytes of a row
template <>
struct Chunk<__bf16> {
    static constexpr int E = 8;
    u32x4 raw;
    __device__ float get(int e) const { return (e & 1) ? bf16_hi_f32(raw[e >> 1]) : bf16_lo_f32(raw[e >> 1]); }
    __device__ void set_pair(int j, float a, float b) { raw[j] = pack_bf16(a, b); }
};
template <>
struct Chunk<float> {
    static constexpr int E = 4;
    f32x4 raw;
    __device__ float get(int e) const { return raw[e]; }
    __device__ void set_pair(int j, float a, float b) { raw[2 * j] = a, raw[2 * j + 1] = b; }
};

// A wave owns 64 / (lanes per row) consecutive positions of one sequence and walks over some of the
// trips there, a trip being four heads of one tensor, all four in flight (the first trip's loads are
// issued before the trigonometry).
// A wave that walked all 40 heads of a layer alone would compute sine and cosine of a (position, pair)
// once, but is a chain of 10 dependent memory round trips: two trips a wave are faster at every size
// (many positions are bound by memory, 4.9 - 5.4 TB/s), one where there are few positions.
// q, rho [1,16,777,128] and k [1,8,777,128]: 6.2 us, 6.9 with the powers taken here and sums by lane shuffles; one row
// each 4.5 (5.2), [4,..,4096,128] 67 - 69 either way.
template <typename T>
__global__ __launch_bounds__(256) void norm_rope_kernel(NormRopeParams p) {
    constexpr int E = Chunk<T>::E;
    constexpr int UNROLL = kNormRopeTripHeads;     // heads in flight per lane
    using raw_t = decltype(Chunk<T>::raw);
    const int lpr = p.d / E;                       // lanes per row (a power of two <= 64)
    const int rows_per_wave = 64 / lpr;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lr = lane % lpr;                     // this lane's chunk of its row
    const int t_per_seq = (p.T + rows_per_wave - 1) / rows_per_wave;  // position groups per sequence
    const int64_t wid_all = (int64_t)blockIdx.x * 4 + wave;
    if (wid_all >= (int64_t)p.B * t_per_seq * p.trip_chunks) return;   // whole waves only: no barrier below
    const int first_trip = (int)(wid_all % p.trip_chunks) * p.trips_per_wave;
    const int64_t wid = wid_all / p.trip_chunks;
    const int b = (int)(wid / t_per_seq);
    const int t = (int)(wid % t_per_seq) * rows_per_wave + lane / lpr;
    const bool live = t < p.T;
    const int ld_t = live ? t : p.T - 1;

    // trip -> tensor and first head; loads of its heads (heads past the last re-read that one)
    int ten_i = 0, h0 = first_trip * UNROLL;
    for (; ten_i < p.n_tensors && h0 >= p.t[ten_i].H; ++ten_i) h0 -= (p.t[ten_i].H + UNROLL - 1) / UNROLL * UNROLL;
    if (ten_i >= p.n_tensors) return;
    Chunk<T> c[UNROLL];
    float gam[E];
    NormRopeTensor ten;
    auto load_trip = [&]() {
        const raw_t *src = (const raw_t *)ten.x;
#pragma unroll
        for (int u = 0; u < UNROLL; ++u)
            c[u].raw = src[(((int64_t)b * ten.H + min(h0 + u, ten.H - 1)) * p.T + ld_t) * lpr + lr];
    };
    auto take_tensor = [&]() {
        ten = p.t[ten_i];
#pragma unroll
        for (int e = 0; e < E; ++e) gam[e] = ten.gamma[lr * E + e];
    };
    take_tensor();
    load_trip();

    float cs[E / 2], sn[E / 2];
    if (p.table != nullptr) {  // (uniform) from the caller's table: E floats = this lane's E / 2 pairs
        const int64_t pos = min(max((p.pos0 ? p.pos0[b] : 0) + ld_t, 0), p.n_pos - 1);
        const float *e = p.table + (pos * (p.d / 2) + lr * (E / 2)) * 2;
#pragma unroll
        for (int j = 0; j < E / 2; j += 2) {
            const f32x4 v = *(const f32x4 *)(e + 2 * j);
            cs[j] = v[0], sn[j] = v[1], cs[j + 1] = v[2], sn[j + 1] = v[3];
        }
    } else {
        // theta^(-dim/d) for this lane's first pair (from the host: a power in double precision per lane took 0.5 us of
        // a small launch), then pair by pair times theta^(-2/d) (at most four roundings more than a power per pair,
        // 5e-16 of the angle)
        const double pos = (double)((p.pos0 ? p.pos0[b] : 0) + ld_t);
        double freq = p.freq[lr];
#pragma unroll
        for (int j = 0; j < E / 2; ++j) {
            double ang = pos * freq;
            ang -= floor(ang * 0.15915494309189535) * 6.283185307179586;  // modulo 2 pi
            sincosf((float)ang, &sn[j], &cs[j]);
            freq *= p.pair_ratio;
        }
    }
    const float inv_d = 1.0f / (float)p.d;
    for (int n = 0; n < p.trips_per_wave; ++n) {
        raw_t *dst = (raw_t *)ten.y;
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            float ss = 0.f;
#pragma unroll
            for (int e = 0; e < E; ++e) ss = fmaf(c[u].get(e), c[u].get(e), ss);
            if (lpr == 16)  // (uniform; the same sums in the same order, without a trip through the LDS)
                ss = lane_group_sum<16>(ss);
            else if (lpr == 8)
                ss = lane_group_sum<8>(ss);
            else
                for (int off = 1; off < lpr; off <<= 1) ss += __shfl_xor(ss, off, 64);
            const float rinv = 1.0f / sqrtf(ss * inv_d + p.eps);
#pragma unroll
            for (int j = 0; j < E / 2; ++j) {
                float y0 = c[u].get(2 * j) * rinv * gam[2 * j];
                float y1 = c[u].get(2 * j + 1) * rinv * gam[2 * j + 1];
                if (ten.rope) {
                    const float r0 = y0 * cs[j] - y1 * sn[j], r1 = y0 * sn[j] + y1 * cs[j];
                    y0 = r0, y1 = r1;
                }
                c[u].set_pair(j, y0, y1);
            }
            if (live && h0 + u < ten.H)
                dst[(((int64_t)b * ten.H + h0 + u) * p.T + t) * lpr + lr] = c[u].raw;
        }
        if (n + 1 == p.trips_per_wave) break;  // (all uniform)
        h0 += UNROLL;
        if (h0 >= ten.H) {
            if (++ten_i >= p.n_tensors) break;
            h0 = 0;
            take_tensor();
        }
        load_trip();
    }
}

// (cos, sin) of pos * theta^(-2i/d), one thread per (position, pair): the same double-precision
// angle reduction as above for the attention kernels that apply the rotation themselves. (The power is
// taken for every pair here, where the kernel above multiplies on from a lane's first: the angles agree to
// four roundings of double precision, before they are taken to single.)
__global__ __launch_bounds__(256) void rope_table_kernel(float *table, int n_pos, int d, float theta) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int half = d / 2;
    if (idx >= (int64_t)n_pos * half) return;
    const int pos = (int)(idx / half), i = (int)(idx % half);
    double ang = (double)pos * exp2(-(double)(2 * i) / (double)d * log2((double)theta));
    ang -= floor(ang * 0.15915494309189535) * 6.283185307179586;  // modulo 2 pi
    float sn, cs;
    sincosf((float)ang, &sn, &cs);
    table[2 * idx] = cs;
    table[2 * idx + 1] = sn;
}

hipError_t launch_rope_table(float *table, int n_pos, int d, float theta, hipStream_t stream) {
    const int64_t blocks = ((int64_t)n_pos * (d / 2) + 255) / 256;
    if (blocks <= 0 || blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(rope_table_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, table, n_pos, d, theta);
    return hipGetLastError();
}

hipError_t launch_norm_rope(const NormRopeParams &p_in, bool f32, hipStream_t stream) {
    NormRopeParams p = p_in;
    const int elems = f32 ? 4 : 8;
    const int rows_per_wave = 64 / (p.d / elems);
    const int64_t groups = (int64_t)p.B * ((p.T + rows_per_wave - 1) / rows_per_wave);
    // trips per wave: one, or two from where that leaves eight waves per SIMD. Measured us, 16 / 16 / 8 heads
    // (10 trips), for all trips in a wave, two, one: d = 128, 16384 positions 65, 64 - 69, 69; 32768 positions
    // 141, 125 - 128, 131 - 143; d = 64, 65536 positions 154, 126, 129; d = 128, 4096 positions 29, 16.6,
    // 18.4; d = 64, 4096 positions 26, 13.4, 13.3. 40 / 40 / 5 heads (22 trips), 32768 positions 300, 269, 278.
    int trips = 0;
    for (int i = 0; i < p.n_tensors; ++i) trips += (p.t[i].H + kNormRopeTripHeads - 1) / kNormRopeTripHeads;
    int64_t chunks = std::max<int64_t>((8192 + groups - 1) / groups, (trips + 1) / 2);
    if (chunks > trips) chunks = trips;
    p.trips_per_wave = (trips + (int)chunks - 1) / (int)chunks;
    p.trip_chunks = (trips + p.trips_per_wave - 1) / p.trips_per_wave;
    const double log2_theta = std::log2((double)p.theta);
    p.pair_ratio = std::exp2(-2.0 / (double)p.d * log2_theta);
    double step[4] = {1.0};  // (every fourth lane by a power, one rounding more in between: six powers for 16 lanes, not fifteen)
    for (int i = 1; i < 4; ++i) step[i] = std::exp2(-(double)(i * elems) / (double)p.d * log2_theta);
    for (int i = 0; i < p.d / elems; i += 4) {
        const double first = i == 0 ? 1.0 : std::exp2(-(double)(i * elems) / (double)p.d * log2_theta);
        for (int k = 0; k < 4; ++k) p.freq[i + k] = first * step[k];
    }
    const int64_t waves = groups * p.trip_chunks;
    const int64_t blocks = (waves + 3) / 4;
    if (blocks <= 0 || blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    if (f32)
        hipLaunchKernelGGL(norm_rope_kernel<float>, dim3((unsigned)blocks), dim3(256), 0, stream, p);
    else
        hipLaunchKernelGGL(norm_rope_kernel<__bf16>, dim3((unsigned)blocks), dim3(256), 0, stream, p);
    return hipGetLastError();
}

}  // namespace plx
