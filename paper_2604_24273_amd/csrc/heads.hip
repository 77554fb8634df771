// Forward pass of the fp32 MLP heads (policy and value, or an ensemble of value heads): all heads of a call together.
//
// Two launches: the first layers of every head as one fp64 matrix-core contraction (mlp_f64.hpp), then one workgroup
// per sample for everything above (the layers there are small: 256 -> 18, 256 -> 1) and, for an ensemble, the mean.
// One launch per layer and head with a wavefront per result took 86 us for 64 samples of 2560 -> 256 -> 18 and 1 (four
// launches; 81 us even for one sample: 40 dependent rounds of loads per wavefront), this takes 18 us from one to 64
// samples; 1024 samples 1167 -> 90 us (78 us of it the contraction).  Heads whose upper layers are too wide for a workgroup per sample keep a launch per layer level.
#include <cstring>

#include "mlp_f64.hpp"

namespace brl {

namespace {

constexpr int HEAD_MAX_UNITS = 4096;           // layer outputs of all heads together: 32 KB of LDS
constexpr size_t HEAD_MAX_WEIGHTS = 1 << 18;   // weights above the first layers: every sample's workgroup reads them all

struct SetArgs {
    MlpSet s;
    int splits, btiles;
    int tile_end[MAX_HEADS], col_end[MAX_HEADS];     // first-layer tiles of 16 units / columns, cumulative
    double* z;                                       // [splits][B][col_end[n - 1]]
};

__global__ __launch_bounds__(256) void heads_first_kernel(SetArgs a) {
    __shared__ FirstLayerSums part;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int tiles = a.tile_end[a.s.n - 1];
    const int split = blockIdx.x % a.splits, tile = (blockIdx.x / a.splits) % tiles, bt = blockIdx.x / (a.splits * tiles);
    int hd = 0;
    while (tile >= a.tile_end[hd]) ++hd;
    const int d = a.s.dims[hd][0], od = a.s.dims[hd][1];
    const int o0 = (tile - (hd ? a.tile_end[hd - 1] : 0)) * 16;
    const float* hrow[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) hrow[q] = a.s.h + (size_t)min(bt * 64 + q * 16 + (lane & 15), a.s.B - 1) * d;
    first_layer_sums(a.s.W[hd][0] + (size_t)min(o0 + (lane & 15), od - 1) * d, hrow, d, split * 4 + wave, a.splits * 4, part);
    const int ncol = a.col_end[a.s.n - 1], col0 = hd ? a.col_end[hd - 1] : 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int qv = u * 4 + wave;
        const int b = bt * 64 + (qv >> 2) * 16 + 4 * (qv & 3) + (lane >> 4), o = o0 + (lane & 15);
        if (b < a.s.B && o < od) a.z[((size_t)split * a.s.B + b) * ncol + col0 + o] = first_layer_sum(part, qv, lane);
    }
}

// mean over the heads in head order, in fp64, rounded once
__device__ inline float head_mean(const float* vals, int n, size_t stride) {
    double t = 0.0;
    for (int e = 0; e < n; ++e) t += (double)vals[e * stride];
    return (float)(t / (double)n);
}

__global__ __launch_bounds__(256) void heads_tail_kernel(SetArgs a) {
    __shared__ double out[HEAD_MAX_UNITS];           // layer outputs, level by level, head by head inside a level
    __shared__ float last[MAX_HEADS];                // results of width 1 (for the mean)
    const int tid = threadIdx.x, b = blockIdx.x;
    const int ncol = a.col_end[a.s.n - 1];
    int depth = 1;
    for (int e = 0; e < a.s.n; ++e) depth = max(depth, a.s.layers[e]);
    for (int c = tid; c < ncol; c += 256) {
        int hd = 0;
        while (c >= a.col_end[hd]) ++hd;
        const int o = c - (hd ? a.col_end[hd - 1] : 0);
        const double v = first_layer_total(a.z + (size_t)b * ncol + c, a.splits, (size_t)a.s.B * ncol) + (double)a.s.bias[hd][0][o];
        if (a.s.layers[hd] > 1) {
            out[c] = activate(v, a.s.act);
        } else {
            a.s.out[hd][(size_t)b * a.s.dims[hd][1] + o] = (float)v;
            if (o == 0) last[hd] = (float)v;
        }
    }
    __syncthreads();
    constexpr int LG = 8;                            // lanes per output unit
    int in_base = 0, out_base = ncol;
    for (int l = 1; l < depth; ++l) {
        int total = 0;
        for (int e = 0; e < a.s.n; ++e) total += l < a.s.layers[e] ? a.s.dims[e][l + 1] : 0;
        for (int u = tid / LG; u < (total + 31) / 32 * 32; u += 256 / LG) {
            // head of this unit, its place in the level, and where its inputs start in the level below
            int hd = 0, o = min(u, total - 1), in0 = in_base;
            for (;;) {
                const int od = l < a.s.layers[hd] ? a.s.dims[hd][l + 1] : 0;
                if (o < od) break;
                o -= od;
                in0 += l <= a.s.layers[hd] ? a.s.dims[hd][l] : 0;
                ++hd;
            }
            const int id = a.s.dims[hd][l], od = a.s.dims[hd][l + 1];
            double v = group_dot<LG>(a.s.W[hd][l] + (size_t)o * id, out + in0, id);
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

// One layer level of every head, a wavefront per result
struct LevelArgs {
    MlpSet s;
    int level;
    size_t first[MAX_HEADS + 1];                     // first result of each head
    const double* in64[MAX_HEADS];                   // null on the first level: every head reads h
    double* out64[MAX_HEADS];
};
__global__ __launch_bounds__(256) void heads_level_kernel(LevelArgs a) {
    const size_t wid = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (wid >= a.first[a.s.n]) return;
    int hd = 0;
    while (wid >= a.first[hd + 1]) ++hd;
    const int id = a.s.dims[hd][a.level], od = a.s.dims[hd][a.level + 1];
    const int b = (int)((wid - a.first[hd]) / od), o = (int)((wid - a.first[hd]) % od);
    const float* w = a.s.W[hd][a.level] + (size_t)o * id;
    const double* x64 = a.in64[hd] ? a.in64[hd] + (size_t)b * id : nullptr;
    const float* x32 = a.s.h + (size_t)b * id;
    double acc = 0.0;
#pragma unroll 4
    for (int i = lane; i < id; i += 64) acc += (double)w[i] * (x64 ? x64[i] : (double)x32[i]);
    acc = wave_sum(acc);
    if (lane == 0) {
        const double z = acc + (double)a.s.bias[hd][a.level][o];
        if (a.level + 1 == a.s.layers[hd]) a.s.out[hd][(size_t)b * od + o] = (float)z;
        else a.out64[hd][(size_t)b * od + o] = activate(z, a.s.act);
    }
}

__global__ __launch_bounds__(256) void heads_mean_kernel(MlpSet s) {
    const int b = blockIdx.x * 256 + threadIdx.x;
    if (b < s.B) s.mean[b] = head_mean(s.out[0] + b, s.n, (size_t)s.B);      // the members' results lie one after another
}

size_t hidden_units(const MlpSet& s) {
    size_t t = 0;
    for (int e = 0; e < s.n; ++e)
        for (int l = 1; l < s.layers[e]; ++l) t += (size_t)s.dims[e][l];
    return t;
}

bool tail_fits(const MlpSet& s) {
    size_t units = 0, weights = 0;
    for (int e = 0; e < s.n; ++e)
        for (int l = 0; l < s.layers[e]; ++l) {
            units += (size_t)s.dims[e][l + 1];
            if (l > 0) weights += (size_t)s.dims[e][l] * s.dims[e][l + 1];
        }
    return units <= (size_t)HEAD_MAX_UNITS && weights <= HEAD_MAX_WEIGHTS;
}

void first_layer_layout(const MlpSet& s, SetArgs& a) {
    int tiles = 0, cols = 0;
    for (int e = 0; e < s.n; ++e) {
        a.tile_end[e] = tiles += (s.dims[e][1] + 15) / 16;
        a.col_end[e] = cols += s.dims[e][1];
    }
    a.btiles = (s.B + 63) / 64;
    a.splits = first_layer_splits(tiles, a.btiles, s.dims[0][0]);
}

}  // namespace

// scratch: the first layers' partial sums, or (wide heads) every hidden layer's outputs; never less than a smaller batch needs
size_t heads_workspace_bytes(const MlpSet& s) {
    if (!tail_fits(s)) return round_up_sz((size_t)s.B * hidden_units(s) * sizeof(double), 256) + 256;
    SetArgs a;
    first_layer_layout(s, a);
    return first_layer_rows(a.tile_end[s.n - 1], s.B, s.dims[0][0]) * a.col_end[s.n - 1] * sizeof(double);
}

int launch_heads(const MlpSet& s, void* workspace, hipStream_t stream) {
    LaunchTimer tm(BRL_KC_OTHER, stream);
    if (tail_fits(s)) {
        SetArgs a;
        memset(&a, 0, sizeof(a));
        a.s = s;
        first_layer_layout(s, a);
        a.z = static_cast<double*>(workspace);
        hipLaunchKernelGGL(heads_first_kernel, dim3((unsigned)(a.tile_end[s.n - 1] * a.splits * a.btiles)), dim3(256), 0, stream, a);
        hipLaunchKernelGGL(heads_tail_kernel, dim3((unsigned)s.B), dim3(256), 0, stream, a);
        BRL_LAUNCH_CHECK("heads");
        return BRL_OK;
    }
    int depth = 1;
    for (int e = 0; e < s.n; ++e) depth = s.layers[e] > depth ? s.layers[e] : depth;
    double* next = static_cast<double*>(workspace);
    const double* in[MAX_HEADS] = {};
    for (int l = 0; l < depth; ++l) {
        LevelArgs a;
        memset(&a, 0, sizeof(a));
        a.s = s;
        a.level = l;
        for (int e = 0; e < s.n; ++e) {
            const bool runs = l < s.layers[e];
            a.first[e + 1] = a.first[e] + (runs ? (size_t)s.B * s.dims[e][l + 1] : 0);
            a.in64[e] = in[e];
            if (runs && l + 1 < s.layers[e]) {
                a.out64[e] = next;
                in[e] = next;
                next += (size_t)s.B * s.dims[e][l + 1];
            }
        }
        hipLaunchKernelGGL(heads_level_kernel, dim3((unsigned)((a.first[s.n] + 3) / 4)), dim3(256), 0, stream, a);
    }
    if (s.mean) hipLaunchKernelGGL(heads_mean_kernel, dim3((s.B + 255) / 256), dim3(256), 0, stream, s);
    BRL_LAUNCH_CHECK("heads");
    return BRL_OK;
}

}  // namespace brl
