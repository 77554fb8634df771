// First-layer contraction of the fp32 heads on the fp64 matrix cores: shared by the forward heads and their training.
//
// v_mfma_f64_16x16x4: a lane gives row / column (lane & 15) and one of four k = lane >> 4; its four results are rows
// 4 v + (lane >> 4), column lane & 15.  The order of k inside a chunk of 16 is free, so a lane reads four consecutive
// floats.  A wavefront takes 16 output units x 64 samples (the weights, the larger operand, are read once) over a
// range of k, the four wavefronts of a workgroup neighbouring ranges.
// The inputs are cut by d alone into up to 32 ranges, four neighbouring ranges are a group, and ranges and groups are added
// in order.  Either every group has a workgroup (and the next kernel adds the groups), so that few tiles fill the chip, or
// a workgroup takes all groups of its tile one after the other: the same order both ways, so a result does not depend on
// what shares the call, be it samples or other heads.
// 64 x 2560 -> 2 x 256: 32 us with vector FMAs (four units x four samples per workgroup), 43 us with a wavefront per
// result, 8.4 us here (bound by the latency of gathering the rows and of the 80 dependent MFMAs of a wavefront).
#pragma once

#include "common.hpp"

namespace brl {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f_u __attribute__((ext_vector_type(4), aligned(4)));      // rows of the flat buffers start anywhere

constexpr int L1_GROUPS = 8, L1_RANGES = 4 * L1_GROUPS;

// chunks of 16 inputs in a range, and groups of four ranges
__host__ __device__ inline int first_layer_range_chunks(int d) { return ((d + 15) / 16 + L1_RANGES - 1) / L1_RANGES; }
__host__ __device__ inline int first_layer_groups(int d) {
    const int group = 4 * 16 * first_layer_range_chunks(d);
    return (d + group - 1) / group;
}

// workgroups that share a tile: one per group up to L1_SHARED_TILES tiles, then one
constexpr int L1_SHARED_TILES = 1024;
inline int first_layer_splits(int tiles, int btiles, int d) {
    return (long)tiles * btiles <= L1_SHARED_TILES ? first_layer_groups(d) : 1;
}

// rows of partial sums (splits x samples) that hold every launch of up to B samples: the splits drop where a batch passes
// a block of 64 samples, so a smaller batch can need more rows than B itself
inline size_t first_layer_rows(int tiles, int B, int d) {
    size_t rows = 0;
    for (int bt = 1; bt <= (B + 63) / 64; ++bt) {
        const int splits = first_layer_splits(tiles, bt, d), b = bt * 64L < B ? bt * 64 : B;
        if ((size_t)splits * b > rows) rows = (size_t)splits * b;
        if (splits == 1) return rows > (size_t)B ? rows : (size_t)B;
    }
    return rows;
}

// four inputs k .. k + 3 of a row of n values, zeros past the end
__device__ inline v4f_u four_inputs(const float* row, int k, int n) {
    if (k + 4 <= n) return *reinterpret_cast<const v4f_u*>(row + k);
    v4f_u r;
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = k + e < n ? row[k + e] : 0.f;
    return r;
}

// the wavefronts' sums, [wavefront][4 * sample tile + v][lane], and running totals over the groups
template <bool ALL, int QT>
struct FirstLayerSums {
    double part[4][4 * QT][64];
    double total[ALL ? 4 * QT : 1][64];
};
// WHOLE: rows are whole chunks of 16 inputs, so every load is unconditional; a bounds test per load costs a branch each
// (2560 -> 512 units from 64 samples: 9.4 us with them, 8.4 us without).
template <bool WHOLE, int QT>
__device__ __forceinline__ void first_layer_range(const float* wrow, const float* const (&hrow)[QT], int d, int c0, int c1, v4d (&acc)[QT]) {
    const int kk = (threadIdx.x & 63) >> 4;
    auto inputs = [&](const float* row, int k) { return WHOLE ? *reinterpret_cast<const v4f_u*>(row + k) : four_inputs(row, k, d); };
    constexpr int NC = 5;                            // chunks requested together (2560 inputs over 32 wavefronts: all of them)
    for (int cb = c0; cb < c1; cb += NC) {
        v4f_u w[NC], x[NC][QT];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int k = min(cb + c, c1 - 1) * 16 + 4 * kk;
            w[c] = inputs(wrow, k);
#pragma unroll
            for (int q = 0; q < QT; ++q) x[c][q] = inputs(hrow[q], k);
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if (cb + c >= c1) break;
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int q = 0; q < QT; ++q)
                    acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)x[c][q][e], (double)w[c][e], acc[q], 0, 0, 0);
        }
    }
}

// wrow: the lane's weight row; hrow: its rows of the QT sample tiles; ALL: every group of the tile, else group `split`.
// sum[u] = the workgroup's part for sample 16 u + 4 wave + (lane >> 4), output unit lane & 15.  The running totals live in LDS: in registers they would cost a wavefront per SIMD (8192 samples of 2560 ->
// 512 units: 475 us, 550 us that way).
template <bool ALL, int QT>
__device__ __forceinline__ void first_layer_sums(const float* wrow, const float* const (&hrow)[QT], int d, int split,
                                                 FirstLayerSums<ALL, QT>& s, double (&sum)[QT]) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int chunks = (d + 15) / 16, per = first_layer_range_chunks(d);
    auto group = [&](int g) {
        const int c0 = (g * 4 + wave) * per, c1 = min(chunks, c0 + per);
        v4d acc[QT] = {};
        if (d % 16 == 0) first_layer_range<true, QT>(wrow, hrow, d, c0, c1, acc);
        else first_layer_range<false, QT>(wrow, hrow, d, c0, c1, acc);
        if (ALL && g) __syncthreads();               // the group before has been read
#pragma unroll
        for (int q = 0; q < QT; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) s.part[wave][q * 4 + v][lane] = acc[q][v];
        __syncthreads();
    };
    auto group_sum = [&](int qv) { return ((s.part[0][qv][lane] + s.part[1][qv][lane]) + s.part[2][qv][lane]) + s.part[3][qv][lane]; };
    if constexpr (ALL) {
        const int groups = first_layer_groups(d);
        for (int g = 0; g < groups; ++g) {
            group(g);
#pragma unroll
            for (int u = 0; u < QT; ++u) {
                double v = group_sum(u * 4 + wave);
                if (g) v = s.total[u * 4 + wave][lane] + v;
                s.total[u * 4 + wave][lane] = v;     // (read by the same thread)
                sum[u] = v;
            }
        }
    } else {
        group(split);
#pragma unroll
        for (int u = 0; u < QT; ++u) sum[u] = group_sum(u * 4 + wave);
    }
}

// the groups of one first-layer result, in order
__device__ inline double first_layer_total(const double* __restrict__ z, int splits, size_t stride) {
    double p[L1_GROUPS];
#pragma unroll
    for (int sp = 0; sp < L1_GROUPS; ++sp) p[sp] = z[(size_t)min(sp, splits - 1) * stride];
    double v = p[0];
#pragma unroll
    for (int sp = 1; sp < L1_GROUPS; ++sp) v += sp < splits ? p[sp] : 0.0;
    return v;
}

__device__ inline double wave_sum(double v) { return wave_total(v); }
__device__ inline double activate(double z, int act) { return act == BRL_ACT_RELU ? fmax(z, 0.0) : tanh(z); }

// sum_i w[i] x[i] over a group of LG adjacent lanes (every lane of the group gets it), 32 weights of a lane in flight
template <int LG>
__device__ inline double group_dot(const float* __restrict__ w, const double* x, int n) {
    double v = 0.0;
    int i = threadIdx.x % LG;
    for (; i + 31 * LG < n; i += 32 * LG) {
        float wv[32];
#pragma unroll
        for (int t = 0; t < 32; ++t) wv[t] = w[i + t * LG];
#pragma unroll
        for (int t = 0; t < 32; ++t) v += (double)wv[t] * x[i + t * LG];
    }
#pragma unroll 4
    for (; i < n; i += LG) v += (double)w[i] * x[i];
    static_assert(LG == 1 || LG == 2 || LG == 4 || LG == 8 || LG == 16, "groups inside a row of 16 lanes");
    if constexpr (LG > 1) v += lane_exchange<DPP_XOR1>(v);
    if constexpr (LG > 2) v += lane_exchange<DPP_XOR2>(v);
    if constexpr (LG > 4) v += lane_exchange<DPP_HALF_MIRROR>(v);
    if constexpr (LG > 8) v += lane_exchange<DPP_MIRROR>(v);
    return v;
}

}  // namespace brl
