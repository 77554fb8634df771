// Small kernels around the BitLinear core: embedding gather, final RMSNorm +
// mean-pool (paper Sec. 3.1, Eq. 3: h_t).
#include "common.hpp"

namespace brl {

namespace {

// x[m, :] = widen(E[clamp(ids[m]), :]); eight bf16 per thread
__global__ void embed_kernel(const uint16_t* __restrict__ table, const int32_t* __restrict__ ids, int M, int d,
                             int vocab, float* __restrict__ x) {
    const int per_row = d / 8;
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (size_t)M * per_row) return;
    const int m = (int)(idx / per_row), c = (int)(idx % per_row) * 8;
    int id = ids[m];
    id = id < 0 ? 0 : (id >= vocab ? vocab - 1 : id);
    const uint4 raw = *reinterpret_cast<const uint4*>(table + (size_t)id * d + c);
    float4 lo, hi;
    lo.x = __uint_as_float(raw.x << 16); lo.y = __uint_as_float(raw.x & 0xffff0000u);
    lo.z = __uint_as_float(raw.y << 16); lo.w = __uint_as_float(raw.y & 0xffff0000u);
    hi.x = __uint_as_float(raw.z << 16); hi.y = __uint_as_float(raw.z & 0xffff0000u);
    hi.z = __uint_as_float(raw.w << 16); hi.w = __uint_as_float(raw.w & 0xffff0000u);
    float* o = x + (size_t)m * d + c;
    *reinterpret_cast<float4*>(o) = lo;
    *reinterpret_cast<float4*>(o + 4) = hi;
}

// rinv[m] = fp32(1 / sqrt(mean_k x[m,k]^2 + eps)), statistic in fp64; one wavefront per row
__global__ __launch_bounds__(256) void row_rinv_kernel(const float* __restrict__ x, int M, int d, float eps,
                                                        float* __restrict__ rinv) {
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= M) return;
    const float* p = x + (size_t)row * d;
    double ss = 0.0;
    for (int k = 4 * lane; k < d; k += 256) {
        const float4 v = *reinterpret_cast<const float4*>(p + k);
        ss += (double)v.x * (double)v.x;
        ss += (double)v.y * (double)v.y;
        ss += (double)v.z * (double)v.z;
        ss += (double)v.w * (double)v.w;
    }
    ss = wave_total(ss);
    if (lane == 0) rinv[row] = (float)(1.0 / sqrt(ss / (double)d + (double)eps));
}

// h[b, c] = fp32( sum_{s < len_b} fp64((x[b,s,c] * rinv[b,s]) * g[c]) / len_b ), positions in order
__global__ void pool_kernel(const float* __restrict__ x, const float* __restrict__ rinv, const float* __restrict__ gain,
                            int B, int S, int d, const int32_t* __restrict__ lengths, SeqMap sm, float* __restrict__ h) {
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (size_t)B * d) return;
    const int b = (int)(idx / d), c = (int)(idx % d);
    int len = sm.cu ? seq_len(sm, b, S) : (lengths ? lengths[b] : S);
    len = len < 1 ? 1 : (len > S ? S : len);
    const size_t m0 = (size_t)seq_row0(sm, b, S);
    const float g = gain[c];
    double acc = 0.0;
#pragma unroll 8                 // eight rows in flight (64 x 128 positions of 2560: 45 -> 14 us)
    for (int s = 0; s < len; ++s) {
        const size_t m = m0 + s;
        const float v = (x[m * d + c] * rinv[m]) * g;
        acc += (double)v;
    }
    h[idx] = (float)(acc / (double)len);
}

}  // namespace

int launch_embed(const uint16_t* table, const int32_t* ids, int M, int d, int vocab, float* x, hipStream_t s) {
    const size_t n = (size_t)M * (d / 8);
    LaunchTimer tm(BRL_KC_OTHER, s);
    hipLaunchKernelGGL(embed_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, table, ids, M, d, vocab, x);
    BRL_LAUNCH_CHECK("embed_kernel");
    return BRL_OK;
}

int launch_final_pool(const float* x, const float* gain, int B, int S, int M, int d, const int32_t* lengths,
                      const SeqMap& sm, float eps_norm, float* rinv, float* h, hipStream_t s) {
    LaunchTimer tm(BRL_KC_OTHER, s);
    hipLaunchKernelGGL(row_rinv_kernel, dim3((M + 3) / 4), dim3(256), 0, s, x, M, d, eps_norm, rinv);
    BRL_LAUNCH_CHECK("row_rinv_kernel");
    const size_t n = (size_t)B * d;
    hipLaunchKernelGGL(pool_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, x, rinv, gain, B, S, d, lengths, sm, h);
    BRL_LAUNCH_CHECK("pool_kernel");
    return BRL_OK;
}

}  // namespace brl
