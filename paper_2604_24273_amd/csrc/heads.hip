// Forward pass of the fp32 MLP heads (policy and value, or an ensemble of value heads): all heads of a call together.
//
// The first layers of every head are one fp64 matrix-core contraction (mlp_f64.hpp).  What is above them is small (256 ->
// 18, 256 -> 1): one workgroup per sample for all of it and, for an ensemble, the mean; or a launch per layer level where a
// workgroup would be long at it or its LDS too small.  Every sum runs in an order of its own layer's width alone, so
// the bits of a head do not depend on the launch form, the batch or the heads beside it: an ensemble's member gives what
// it gives as a value head.
// One launch per layer and head with a wavefront per result took 86 us for 64 samples of 2560 -> 256 -> 18 and 1 (four
// launches; 81 us even for one sample: 40 dependent rounds of loads per wavefront); the two launches take 13.5 us for 64
// samples, 9.0 us for one, 71 us for 1024 (the launches per layer and head 1147 us).
#include <climits>
#include <cstring>

#include "mlp_f64.hpp"

namespace brl {

namespace {

constexpr int HEAD_MAX_UNITS = 4096;           // layer outputs of all heads together: 32 KB of LDS
// threads of a sample's workgroup: 512 up to two workgroups per compute unit, where every loop over units costs its
// latency (2560 -> 256 -> 256 -> 18 and 1, 128 samples: 34.8 us, 45.3 us with 256; 512 samples: 69.1 us, 77.8 us), 256
// beyond (2560 -> 256 -> 18 and 1, 1024 samples: 70.8 us, 73.9 us with 512; 4096 samples: 246 us, 260 us)
constexpr int HEAD_TAIL_FEW = 512;

// What is the same for every form.  Units of a layer level lie head after head; a head that has no such layer has none.
struct SetArgs {
    MlpSet s;
    int splits, btiles, depth;
    int tile_end[MAX_HEADS];                         // first-layer tiles of 16 units, cumulative
    int unit_end[MAX_MLP_LAYERS][MAX_HEADS];         // outputs of a level, cumulative
    double* z;                                       // [splits][B][units of level 0]
};

// the head that entry u of a cumulative table belongs to
__device__ inline int head_of(const int (&end)[MAX_HEADS], int n, int u) {
    int hd = 0;
#pragma unroll
    for (int e = 0; e + 1 < MAX_HEADS; ++e) hd += (e + 1 < n && u >= end[e]) ? 1 : 0;
    return hd;
}

// ALL: a workgroup takes all of its tile's inputs (a.splits is 1).  QT: tiles of 16 samples of a workgroup, one where the
// call has no more than 16 (five members of 2560 -> 256 -> 1, one sample: 21.4 us with four, 14.9 us with one).
template <bool ALL, int QT>
__global__ __launch_bounds__(256, 3) void heads_first_kernel(SetArgs a) {
    __shared__ FirstLayerSums<ALL, QT> part;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int tiles = a.tile_end[a.s.n - 1];
    const int split = blockIdx.x % a.splits, tile = (blockIdx.x / a.splits) % tiles, bt = blockIdx.x / (a.splits * tiles);
    const int hd = head_of(a.tile_end, a.s.n, tile);
    const int d = a.s.dims[hd][0], od = a.s.dims[hd][1];
    const int o0 = (tile - (hd ? a.tile_end[hd - 1] : 0)) * 16;
    const float* hrow[QT];
#pragma unroll
    for (int q = 0; q < QT; ++q) hrow[q] = a.s.h + (size_t)min(bt * 64 + q * 16 + (lane & 15), a.s.B - 1) * d;
    double sum[QT];
    first_layer_sums<ALL, QT>(a.s.W[hd][0] + (size_t)min(o0 + (lane & 15), od - 1) * d, hrow, d, split, part, sum);
    const int ncol = a.unit_end[0][a.s.n - 1], col0 = hd ? a.unit_end[0][hd - 1] : 0;
#pragma unroll
    for (int u = 0; u < QT; ++u) {
        const int b = bt * 64 + u * 16 + 4 * wave + (lane >> 4), o = o0 + (lane & 15);
        if (b < a.s.B && o < od) a.z[((size_t)split * a.s.B + b) * ncol + col0 + o] = sum[u];
    }
}

// mean over the heads in head order, in fp64, rounded once
__device__ inline float head_mean(const float* vals, int n, size_t stride) {
    double t = 0.0;
    for (int e = 0; e < n; ++e) t += (double)vals[e * stride];
    return (float)(t / (double)n);
}

constexpr int LG = 8;                                // lanes per output unit above the first layer

template <int THREADS>
__global__ __launch_bounds__(THREADS) void heads_tail_kernel(SetArgs a) {
    __shared__ double out[HEAD_MAX_UNITS];           // layer outputs, level by level
    __shared__ float last[MAX_HEADS];                // results of width 1 (for the mean)
    const int tid = threadIdx.x, b = blockIdx.x;
    const int ncol = a.unit_end[0][a.s.n - 1];
    for (int c = tid; c < ncol; c += THREADS) {
        const int hd = head_of(a.unit_end[0], a.s.n, c), o = c - (hd ? a.unit_end[0][hd - 1] : 0);
        const double v = first_layer_total(a.z + (size_t)b * ncol + c, a.splits, (size_t)a.s.B * ncol) + (double)a.s.bias[hd][0][o];
        if (a.s.layers[hd] > 1) {
            out[c] = activate(v, a.s.act);
        } else {
            a.s.out[hd][(size_t)b * a.s.dims[hd][1] + o] = (float)v;
            if (o == 0) last[hd] = (float)v;
        }
    }
    __syncthreads();
    constexpr int GROUPS = THREADS / LG;
    int in_base = 0, out_base = ncol;
    for (int l = 1; l < a.depth; ++l) {
        const int total = a.unit_end[l][a.s.n - 1];
        for (int u = tid / LG; u < (total + GROUPS - 1) / GROUPS * GROUPS; u += GROUPS) {
            const int uc = min(u, total - 1), hd = head_of(a.unit_end[l], a.s.n, uc), o = uc - (hd ? a.unit_end[l][hd - 1] : 0);
            const int id = a.s.dims[hd][l], od = a.s.dims[hd][l + 1];
            double v = group_dot<LG>(a.s.W[hd][l] + (size_t)o * id, out + in_base + (hd ? a.unit_end[l - 1][hd - 1] : 0), id);
            if (tid % LG == 0 && u < total) {
                v += (double)a.s.bias[hd][l][o];
                if (l + 1 < a.s.layers[hd]) {
                    v = activate(v, a.s.act);
                } else {
                    a.s.out[hd][(size_t)b * od + o] = (float)v;
                    if (o == 0) last[hd] = (float)v;
                }
                out[out_base + u] = v;
            }
        }
        in_base = out_base;
        out_base += total;
        __syncthreads();
    }
    if (a.s.mean && tid == 0) a.s.mean[b] = head_mean(last, a.s.n, 1);
}

// One layer level of every head and sample: a thread per result of the first layer, LG lanes per result above
struct LevelArgs {
    SetArgs a;
    int level;
    const double* in;                                // [B][units of the level below]
    double* out;                                     // [B][units of the level]
};
template <bool FIRST>
__global__ __launch_bounds__(256) void heads_level_kernel(LevelArgs g) {
    const SetArgs& a = g.a;
    const int l = FIRST ? 0 : g.level, total = a.unit_end[l][a.s.n - 1];
    const size_t n = (size_t)a.s.B * total, r = ((size_t)blockIdx.x * 256 + threadIdx.x) / (FIRST ? 1 : LG);
    const size_t rc = r < n ? r : n - 1;             // (every lane of a group has to be there)
    const int b = (int)(rc / total), u = (int)(rc % total);
    const int hd = head_of(a.unit_end[l], a.s.n, u), o = u - (hd ? a.unit_end[l][hd - 1] : 0);
    const int id = a.s.dims[hd][l], od = a.s.dims[hd][l + 1];
    double v;
    if constexpr (FIRST) {
        v = first_layer_total(a.z + (size_t)b * total + u, a.splits, n);
    } else {
        const int in0 = hd ? a.unit_end[l - 1][hd - 1] : 0;
        v = group_dot<LG>(a.s.W[hd][l] + (size_t)o * id, g.in + (size_t)b * a.unit_end[l - 1][a.s.n - 1] + in0, id);
    }
    if (r >= n || (!FIRST && threadIdx.x % LG != 0)) return;
    v += (double)a.s.bias[hd][l][o];
    if (l + 1 == a.s.layers[hd]) a.s.out[hd][(size_t)b * od + o] = (float)v;
    else g.out[(size_t)b * total + u] = activate(v, a.s.act);
}

__global__ __launch_bounds__(256) void heads_mean_kernel(MlpSet s) {
    const int b = blockIdx.x * 256 + threadIdx.x;
    if (b < s.B) s.mean[b] = head_mean(s.out[0] + b, s.n, (size_t)s.B);      // the members' results lie one after another
}

SetArgs set_layout(const MlpSet& s) {
    SetArgs a;
    memset(&a, 0, sizeof(a));
    a.s = s;
    int tiles = 0;
    a.depth = 1;
    for (int e = 0; e < s.n; ++e) {
        a.tile_end[e] = tiles += (s.dims[e][1] + 15) / 16;
        if (s.layers[e] > a.depth) a.depth = s.layers[e];
        for (int l = 0; l < MAX_MLP_LAYERS; ++l)
            a.unit_end[l][e] = (e ? a.unit_end[l][e - 1] : 0) + (l < s.layers[e] ? s.dims[e][l + 1] : 0);
    }
    a.btiles = (s.B + 63) / 64;
    a.splits = first_layer_splits(tiles, a.btiles, s.dims[0][0]);
    return a;
}

// the first layers' partial sums (never less than a smaller batch needs)
size_t sums_bytes(const SetArgs& a) {
    const MlpSet& s = a.s;
    return round_up_sz(first_layer_rows(a.tile_end[s.n - 1], s.B, s.dims[0][0]) * a.unit_end[0][s.n - 1] * sizeof(double), 256);
}

// Weights above the first layers that a lone workgroup goes through before a launch per level would be done, and the batch
// from which there are workgroups enough to fill the chip.  2560 inputs, one workgroup per sample / a launch per level, us:
// five members of 64, 64 (21 k weights) on 1 sample 18.9 / 15.5, on 64 23.1 / 21.9, on 200 28.3 / 33.2; policy and value
// head of 256 (5 k) 9.5 / 10.6, 14.1 / 16.2, 26.3 / 28.3; of 256, 256 (136 k) 27.3 / 15.7, 32.0 / 26.1, 43.9 / 53.7.
constexpr size_t HEAD_TAIL_WEIGHTS = 1 << 14;
constexpr int HEAD_TAIL_BATCH = 128;

// samples below which a call takes a launch per level instead
int level_batch(const SetArgs& a) {
    size_t units = 0, weights = 0;
    for (int l = 0; l < a.depth; ++l) units += (size_t)a.unit_end[l][a.s.n - 1];
    for (int e = 0; e < a.s.n; ++e)
        for (int l = 1; l < a.s.layers[e]; ++l) weights += (size_t)a.s.dims[e][l] * a.s.dims[e][l + 1];
    if (units > (size_t)HEAD_MAX_UNITS) return INT_MAX;
    return weights > HEAD_TAIL_WEIGHTS ? HEAD_TAIL_BATCH : 0;
}

// the hidden layers of the launch-per-level form, for every batch up to this one that takes it
size_t hidden_bytes(const SetArgs& a) {
    size_t units = 0;
    for (int l = 0; l + 1 < a.depth; ++l) units += (size_t)a.unit_end[l][a.s.n - 1];
    const int below = level_batch(a);
    const size_t rows = below == 0 ? 0 : a.s.B < below ? a.s.B : below - 1;
    return round_up_sz(rows * units * sizeof(double), 256);
}

}  // namespace

size_t heads_workspace_bytes(const MlpSet& s) {
    const SetArgs a = set_layout(s);
    return sums_bytes(a) + hidden_bytes(a);
}

int launch_heads(const MlpSet& s, void* workspace, hipStream_t stream) {
    LaunchTimer tm(BRL_KC_OTHER, stream);
    LevelArgs g;
    memset(&g, 0, sizeof(g));
    SetArgs& a = g.a;
    a = set_layout(s);
    a.z = static_cast<double*>(workspace);
    const dim3 grid((unsigned)a.tile_end[s.n - 1] * (unsigned)a.splits * (unsigned)a.btiles);
    const bool few = s.B <= 16;
    if (a.splits == 1 && few) hipLaunchKernelGGL((heads_first_kernel<true, 1>), grid, dim3(256), 0, stream, a);
    else if (a.splits == 1) hipLaunchKernelGGL((heads_first_kernel<true, 4>), grid, dim3(256), 0, stream, a);
    else if (few) hipLaunchKernelGGL((heads_first_kernel<false, 1>), grid, dim3(256), 0, stream, a);
    else hipLaunchKernelGGL((heads_first_kernel<false, 4>), grid, dim3(256), 0, stream, a);
    if (s.B >= level_batch(a)) {
        if (s.B <= HEAD_TAIL_FEW) hipLaunchKernelGGL(heads_tail_kernel<512>, dim3((unsigned)s.B), dim3(512), 0, stream, a);
        else hipLaunchKernelGGL(heads_tail_kernel<256>, dim3((unsigned)s.B), dim3(256), 0, stream, a);
    } else {
        g.out = reinterpret_cast<double*>(static_cast<char*>(workspace) + sums_bytes(a));
        for (g.level = 0; g.level < a.depth; ++g.level) {
            const size_t results = (size_t)s.B * a.unit_end[g.level][s.n - 1];
            if (g.level == 0) hipLaunchKernelGGL(heads_level_kernel<true>, dim3((unsigned)((results + 255) / 256)), dim3(256), 0, stream, g);
            else hipLaunchKernelGGL(heads_level_kernel<false>, dim3((unsigned)((results * LG + 255) / 256)), dim3(256), 0, stream, g);
            g.in = g.out;
            g.out += results;
        }
        if (s.mean) hipLaunchKernelGGL(heads_mean_kernel, dim3((s.B + 255) / 256), dim3(256), 0, stream, s);
    }
    BRL_LAUNCH_CHECK("heads");
    return BRL_OK;
}

}  // namespace brl
