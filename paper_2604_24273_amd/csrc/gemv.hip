// BitLinear for a handful of tokens in one launch: y = dequant(codes . quant(x)).
//
// gemv_kernel (1 .. 4 tokens):
// One workgroup of 16 wavefronts owns one block of 32 output rows over the whole
// k range, so no partial sums ever cross workgroups (no atomics, no fences).
// The packed weights are streamed once with 16-byte-per-lane loads (a wavefront
// reads contiguous 1 KB blocks of 32 rows x 128 columns), all of them issued
// before anything is waited for: the whole matrix is in flight while the activation
// rows are quantised (every workgroup redoes that cheap step on its own).  Loads return
// in order, so the activations, which are needed first, are requested first, then the
// weights, then what the finishing threads need; all of them unconditionally (clamped
// addresses), so that none waits for another.
// The 2-bit fields are expanded in registers to offset codes c = code + 1 and
// contracted with v_dot4_i32_i8 against the int8 activations held in LDS;
// sum_k q is subtracted at the end.
#include <type_traits>

#include "common.hpp"

namespace brl {

namespace {

constexpr int GV_THREADS = 1024;
constexpr int GV_WAVES = GV_THREADS / 64;
constexpr int GV_MAX_SB = MAX_K / SBK;                                   // 72 super-blocks
constexpr int GV_X4 = (MAX_K / 4 + GV_THREADS - 1) / GV_THREADS;         // float4 of one row per thread in the batched kernel: 3
struct GemvArgs {
    const void* x;
    int x_dtype;
    int M, K, N, nsb;
    const uint4* packed;
    const float* beta;
    float eps_act;
    float* y;
    const float* residual;
    int8_t* xq_dbg;
    float* absmax_dbg;
    int32_t* acc_dbg;
};

__device__ inline float4 load_x4(const void* x, int dtype, size_t idx) {
    if (dtype == BRL_BF16) {
        const uint2 raw = *reinterpret_cast<const uint2*>(reinterpret_cast<const uint16_t*>(x) + idx);
        return make_float4(__uint_as_float(raw.x << 16), __uint_as_float(raw.x & 0xffff0000u),
                           __uint_as_float(raw.y << 16), __uint_as_float(raw.y & 0xffff0000u));
    }
    return *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(x) + idx);
}

// NX float4 of a row per thread (K <= 4096 NX), NS super-blocks per wavefront
template <int MT, int NX, int NS>
__global__ __launch_bounds__(GV_THREADS) void gemv_kernel(GemvArgs g) {
    __shared__ __attribute__((aligned(16))) int xq[MT][NX * GV_THREADS];     // int8 activations as dwords (zero padded)
    __shared__ float wmax[MT][GV_WAVES];
    __shared__ int wsum[MT][GV_WAVES];
    __shared__ int red[GV_WAVES][MT][32];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int nb = blockIdx.x;
    const int K = g.K, Kp = g.nsb * SBK;
    const bool bf16 = g.x_dtype == BRL_BF16;

    // 1. everything this workgroup reads
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    typedef const __attribute__((address_space(1))) char* gptr;
    u32x4 raw[MT][NX];
    if (bf16) {
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int u = 0; u < NX; ++u) {
                const int k = min(4 * ((int)threadIdx.x + GV_THREADS * u), K - 4);
                const u32x2 r = *(const __attribute__((address_space(1))) u32x2*)((gptr)g.x + (size_t)min(t, g.M - 1) * K * 2 + (unsigned)k * 2u);
                raw[t][u].xy = r;
            }
    } else {
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int u = 0; u < NX; ++u) {
                const int k = min(4 * ((int)threadIdx.x + GV_THREADS * u), K - 4);
                raw[t][u] = *(const __attribute__((address_space(1))) u32x4*)((gptr)g.x + (size_t)min(t, g.M - 1) * K * 4 + (unsigned)k * 4u);
            }
    }
    u32x4 wreg[NS];                                   // (super-blocks past the end of k are never contracted)
    const __attribute__((address_space(1))) u32x4* wp = (const __attribute__((address_space(1))) u32x4*)g.packed + (size_t)nb * g.nsb * 64;
#pragma unroll
    for (int u = 0; u < NS; ++u) wreg[u] = wp[(unsigned)(min(wave + GV_WAVES * u, g.nsb - 1) * 64 + lane)];
    const float beta = *g.beta;
    const int t_of = threadIdx.x >> 5, r_of = threadIdx.x & 31;          // the finishing threads' (token, row)
    const bool finishes = t_of < MT && t_of < g.M && nb * 32 + r_of < g.N;
    const size_t o = (size_t)t_of * g.N + nb * 32 + r_of;
    const float res = g.residual && finishes ? g.residual[o] : 0.f;

    // 2. per-token absmax
    float4 xv[MT][NX];
    float tmax[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        tmax[t] = 0.f;
#pragma unroll
        for (int u = 0; u < NX; ++u) {
            const bool in = t < g.M && 4 * ((int)threadIdx.x + GV_THREADS * u) < K;
            const u32x4 r = raw[t][u];
            float4 v;
            v.x = in ? __uint_as_float(bf16 ? r.x << 16 : r.x) : 0.f;
            v.y = in ? __uint_as_float(bf16 ? r.x & 0xffff0000u : r.y) : 0.f;
            v.z = in ? __uint_as_float(bf16 ? r.y << 16 : r.z) : 0.f;
            v.w = in ? __uint_as_float(bf16 ? r.y & 0xffff0000u : r.w) : 0.f;
            xv[t][u] = v;
            tmax[t] = fmaxf(tmax[t], fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
        }
        tmax[t] = wave_max(tmax[t]);
        if (lane == 0) wmax[t][wave] = tmax[t];
    }
    __syncthreads();

    // 3. quantise into LDS
    float ac[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        float m = wmax[t][0];
#pragma unroll
        for (int w = 1; w < GV_WAVES; ++w) m = fmaxf(m, wmax[t][w]);
        ac[t] = fmaxf(m, g.eps_act);
        const float sc = 127.0f / ac[t];
        int qsum = 0;
#pragma unroll
        for (int u = 0; u < NX; ++u) {
            const int k = 4 * ((int)threadIdx.x + GV_THREADS * u);
            if (k < Kp) {
                const int word = (int)quantise_four(xv[t][u], sc);
                qsum = __builtin_amdgcn_sdot4(word, 0x01010101, qsum, false);
                xq[t][k >> 2] = word;
                if (g.xq_dbg && nb == 0 && t < g.M && k < K) *reinterpret_cast<int*>(g.xq_dbg + (size_t)t * K + k) = word;
            }
        }
        qsum = wave_total(qsum);
        if (lane == 0) wsum[t][wave] = qsum;
    }
    if (g.absmax_dbg && nb == 0 && threadIdx.x == 0) {
#pragma unroll
        for (int t = 0; t < MT; ++t)
            if (t < g.M) g.absmax_dbg[t] = ac[t];
    }
    __syncthreads();

    // 4. contract: lane (r, hh) holds row 32 nb + r, k-half hh of each 32-column step
    int acc[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[t] = 0;
    const int hh = lane >> 5;
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        const int sb = wave + GV_WAVES * u;
        if (sb >= g.nsb) continue;
        const uint32_t wd[4] = {wreg[u].x, wreg[u].y, wreg[u].z, wreg[u].w};
#pragma unroll
        for (int dd = 0; dd < 4; ++dd) {
            const uint32_t p = wd[dd];
            const int c0 = (int)(p & 0x03030303u), c1 = (int)((p >> 2) & 0x03030303u);
            const int c2 = (int)((p >> 4) & 0x03030303u), c3 = (int)((p >> 6) & 0x03030303u);
            const int xoff = (sb * 128 + dd * 32 + hh * 16) / 4;
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                const int4 xw = *reinterpret_cast<const int4*>(&xq[t][xoff]);
                acc[t] = __builtin_amdgcn_sdot4(c0, xw.x, acc[t], false);
                acc[t] = __builtin_amdgcn_sdot4(c1, xw.y, acc[t], false);
                acc[t] = __builtin_amdgcn_sdot4(c2, xw.z, acc[t], false);
                acc[t] = __builtin_amdgcn_sdot4(c3, xw.w, acc[t], false);
            }
        }
    }
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        acc[t] += __shfl_xor(acc[t], 32, 64);
        if (lane < 32) red[wave][t][lane] = acc[t];
    }
    __syncthreads();

    // 5. finish: threads 0 .. 32 MT - 1 each own one (token, row)
    if (finishes) {
        int part = 0, sq = 0;
        float m = wmax[t_of][0];
#pragma unroll
        for (int w = 0; w < GV_WAVES; ++w) {
            part += red[w][t_of][r_of];
            sq += wsum[t_of][w];
            m = fmaxf(m, wmax[t_of][w]);
        }
        part -= sq;
        const float d = fmaxf(m, g.eps_act) / 127.0f;
        float val = ((float)part * d) * beta;
        if (g.residual) val = val + res;
        g.y[o] = val;
        if (g.acc_dbg) g.acc_dbg[o] = part;
    }
}

// ---------------------------------------------------------------------------
// 3 .. 32 tokens in one launch, on the matrix cores.  A workgroup of 16 wavefronts owns 32 output rows over all of k, as in
// gemv_kernel; every wavefront quantises whole tokens (RW of them, in its registers: no exchange between wavefronts), the
// codes meet in LDS in MFMA operand order, a wavefront contracts every 16th super-block and the parts are added in LDS.
// Every workgroup quantises all tokens again (what a compute unit spends its time on: some 20 vector instructions per four
// values), a price that grows with tokens x k, against a launch, a pass through memory and the gap between two kernels.
// Calls back to back, us, quantisation and product as two launches / here: 16 x 2048 x 2048 8.6 / 5.4 (what the host takes
// for a call; by GPU time 6.5 / 4.8), 16 x 2560 x 5120 8.7 / 7.0.  Where the line lies: rows_product_eligible below.
// In LDS the 16-byte piece p (16 columns) of token r stands at slot (r + p) % (16 RW) of the piece's row: the dwords a
// wavefront writes (one token, 16 pieces) and the pieces it reads (one super-block step, all tokens) fall on different banks.
// Ternary weights only: a form for int8 blobs, whose few-token products run gemm_direct_kernel, has not been built.
// ---------------------------------------------------------------------------
typedef int rp_v4i __attribute__((ext_vector_type(4)));
typedef int rp_v16i __attribute__((ext_vector_type(16)));
typedef unsigned int rp_u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int rp_u32x2 __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(1))) char* rp_gptr;

template <int RW, int NX, bool BF16>
__global__ __launch_bounds__(GV_THREADS) void rows_product_kernel(GemvArgs g) {
    constexpr int TOK = 16 * RW;                     // tokens the operand rows in LDS hold
    constexpr int NS = (NX * 2 + 15) / 16;           // super-blocks of a wavefront
    __shared__ __attribute__((aligned(16))) char aq[NX * 16 * TOK * 16];
    __shared__ int red[GV_WAVES][16][64];
    __shared__ float tok_d[TOK];
    __shared__ int tok_sq[TOK];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int nb = blockIdx.x, K = g.K;

    // everything the workgroup reads: activations first (needed first, and loads return in order), weights, the finishing
    // threads' operands; all with clamped addresses, so that none waits for another
    rp_u32x4 raw[RW][NX];
#pragma unroll
    for (int t = 0; t < RW; ++t) {
        const rp_gptr row = (rp_gptr)g.x + (size_t)min(wave + 16 * t, g.M - 1) * K * (BF16 ? 2 : 4);
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const unsigned k = (unsigned)min(4 * (lane + 64 * i), K - 4);
            if constexpr (BF16) raw[t][i].xy = *(const __attribute__((address_space(1))) rp_u32x2*)(row + k * 2u);
            else raw[t][i] = *(const __attribute__((address_space(1))) rp_u32x4*)(row + k * 4u);
        }
    }
    rp_u32x4 w[NS];
    const __attribute__((address_space(1))) rp_u32x4* wp = (const __attribute__((address_space(1))) rp_u32x4*)g.packed + (size_t)nb * g.nsb * 64;
#pragma unroll
    for (int u = 0; u < NS; ++u) w[u] = wp[(unsigned)(min(wave + 16 * u, g.nsb - 1) * 64 + lane)];
    const float beta = *g.beta;
    const int m = threadIdx.x >> 5, c = threadIdx.x & 31;            // the element this thread finishes
    const bool finishes = m < g.M && nb * 32 + c < g.N;
    const size_t o = (size_t)m * g.N + nb * 32 + c;
    const float res = g.residual && finishes ? g.residual[o] : 0.f;

#pragma unroll
    for (int t = 0; t < RW; ++t) {
        const int r = wave + 16 * t;
        // (past the end of k a lane holds the row's last four values again: the maximum is the same, the code is zero)
        float v[NX][4], amax = 0.f;
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const rp_u32x4 q = raw[t][i];
            v[i][0] = __uint_as_float(BF16 ? q.x << 16 : q.x);
            v[i][1] = __uint_as_float(BF16 ? q.x & 0xffff0000u : q.y);
            v[i][2] = __uint_as_float(BF16 ? q.y << 16 : q.z);
            v[i][3] = __uint_as_float(BF16 ? q.y & 0xffff0000u : q.w);
            amax = fmaxf(fmaxf(fmaxf(fmaxf(amax, fabsf(v[i][0])), fabsf(v[i][1])), fabsf(v[i][2])), fabsf(v[i][3]));
        }
        const float ac = fmaxf(wave_max(amax), g.eps_act);
        const float s = 127.0f / ac;
        char* const at = aq + (lane >> 2) * (TOK * 16) + 4 * (lane & 3);
        const int slot = (r + (lane >> 2)) % TOK;
        int sum = 0;
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const uint32_t word = quantise_four(v[i], s) & (4 * (lane + 64 * i) < K ? ~0u : 0u);
            sum = __builtin_amdgcn_sdot4((int)word, 0x01010101, sum, false);
            *reinterpret_cast<uint32_t*>(at + i * (TOK * 256) + ((slot + 16 * i) % TOK) * 16) = word;
        }
        sum = wave_total(sum);
        if (lane == 0) {
            tok_d[r] = ac / 127.0f;
            tok_sq[r] = sum;
            if (g.absmax_dbg && nb == 0 && r < g.M) g.absmax_dbg[r] = ac;
        }
    }
    __syncthreads();

    if (g.xq_dbg && nb == 0) {
        for (int i = threadIdx.x; i < g.M * (K / 4); i += GV_THREADS) {
            const int t = i / (K / 4), k = 4 * (i % (K / 4)), p = k >> 4;
            *reinterpret_cast<uint32_t*>(g.xq_dbg + (size_t)t * K + k) =
                *reinterpret_cast<const uint32_t*>(aq + p * (TOK * 16) + ((t + p) % TOK) * 16 + (k & 15));
        }
    }

    rp_v16i acc = {};
    const int r = lane & (TOK - 1), hh = lane >> 5;                  // (RW = 1: rows 16 .. 31 repeat the first ones)
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        const int sb = wave + 16 * u;
        if (sb >= g.nsb) break;
#pragma unroll
        for (int dd = 0; dd < 4; ++dd) {
            const int p = sb * 8 + dd * 2 + hh;
            const rp_v4i a = *reinterpret_cast<const rp_v4i*>(aq + p * (TOK * 16) + ((r + p) % TOK) * 16);
            const uint32_t pw = w[u][dd];
            const rp_v4i b = {(int)(pw & 0x03030303u), (int)((pw >> 2) & 0x03030303u), (int)((pw >> 4) & 0x03030303u),
                              (int)((pw >> 6) & 0x03030303u)};
            acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, acc, 0, 0, 0);
        }
    }
    const int parts = min(GV_WAVES, g.nsb);
    if (wave < parts) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
            if (RW == 2 || v < 8) red[wave][v][lane] = acc[v];
    }
    __syncthreads();

    if (finishes) {
        // register 4 (m / 8) + m % 4 of lane c + 32 (m / 4 % 2)
        const int v = 4 * (m >> 3) + (m & 3), l = c + 32 * ((m >> 2) & 1);
        int part = -tok_sq[m];
        for (int q = 0; q < parts; ++q) part += red[q][v][l];
        float val = ((float)part * tok_d[m]) * beta;
        if (g.residual) val = val + res;
        g.y[o] = val;
        if (g.acc_dbg) g.acc_dbg[o] = part;
    }
}

// ---------------------------------------------------------------------------
// Many independent problems of one shape in a single launch.  Work item i is row block
// i % nwg of problem i / nwg.  A persistent workgroup takes a contiguous run of items and
// quantises the activations of a problem once (into LDS) for all of that problem's row
// blocks it owns.  Inside a problem every wavefront owns whole row blocks: it streams the
// block's packed weights in chunks of CH super-blocks (CH chosen to divide k evenly where it can), the next chunk (also across
// row blocks) requested before the current one is contracted, and finishes the 32 rows by
// itself - no partial sums cross wavefronts and no barrier is met until the problem changes.
// ---------------------------------------------------------------------------
struct GemvBatchArgs {
    const uint4* const* packed;   // device arrays of device pointers, one entry per problem
    const float* const* beta;
    const void* const* x;
    float* const* y;
    int x_dtype;
    int M, K, N, nsb, nwg, count;
    float eps_act;
};

// CH = super-blocks (1 KB wavefront loads) per chunk: 4, 5 or 6

// Loads are unconditional (super-blocks past the end of k are clamped to the last one and never
// contracted): with straight-line requests the compiler can count the loads still in flight and
// waits only for the chunk it is about to contract, not for the one just requested.  The weight
// pointers come out of a device array, so they are marked as global memory by hand: generic
// (flat) loads would tie the vector-memory and LDS counters together and force full waits.
typedef unsigned int gb_u32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) gb_u32x4* gb_wptr;
template <int CH>
__device__ inline void gb_request(gb_wptr blk, int c, int nsb, uint4 (&w)[CH]) {
#pragma unroll
    for (int u = 0; u < CH; ++u) {
        const int sb = min(c * CH + u, nsb - 1);
        const gb_u32x4 v = blk[(size_t)sb * 64];
        w[u] = make_uint4(v.x, v.y, v.z, v.w);
    }
}

// No conditions here either: the activations in LDS are zero from the end of k up to a whole number of
// chunks, so the clamped super-blocks of the last chunk contribute nothing.
template <int MT, int CH>
__device__ inline void gb_contract(const uint4 (&w)[CH], int c, int hh, const int (*xq)[MAX_K / 4], int (&acc)[MT]) {
#pragma unroll
    for (int u = 0; u < CH; ++u) {
        const int sb = c * CH + u;
        const uint32_t wd[4] = {w[u].x, w[u].y, w[u].z, w[u].w};
#pragma unroll
        for (int dd = 0; dd < 4; ++dd) {
            const uint32_t pw = wd[dd];
            const int c0 = (int)(pw & 0x03030303u), c1 = (int)((pw >> 2) & 0x03030303u);
            const int c2 = (int)((pw >> 4) & 0x03030303u), c3 = (int)((pw >> 6) & 0x03030303u);
            const int xoff = (sb * 128 + dd * 32 + hh * 16) / 4;
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                const int4 xw = *reinterpret_cast<const int4*>(&xq[t][xoff]);
                acc[t] = __builtin_amdgcn_sdot4(c0, xw.x, acc[t], false);
                acc[t] = __builtin_amdgcn_sdot4(c1, xw.y, acc[t], false);
                acc[t] = __builtin_amdgcn_sdot4(c2, xw.z, acc[t], false);
                acc[t] = __builtin_amdgcn_sdot4(c3, xw.w, acc[t], false);
            }
        }
    }
}

// ANY_EPS: codes past the row are zero also where the scale may be infinite (then a zero's is -127, and in a last chunk that
// is no whole one it would meet real weights).  A variant of its own: the mask takes scalar registers from the loads' cursors,
// four tokens x 2304 x 1792, 9 problems each way 43 -> 54 us.
template <int MT, int CH, bool ANY_EPS = false>
__global__ __launch_bounds__(GV_THREADS) void gemv_batch_kernel(GemvBatchArgs g) {
    __shared__ __attribute__((aligned(16))) int xq[MT][MAX_K / 4];   // CH = 5 is only launched where it divides k
    __shared__ float wmax[MT][GV_WAVES];
    __shared__ int wsum[MT][GV_WAVES];
    constexpr int GB_SLOTS = MT == 4 ? 3 : 16 / MT;          // row blocks a wavefront parks before it stores them
    __shared__ float ypark[GV_WAVES][GB_SLOTS][MT][32];

    // the wavefront index as a scalar: everything derived from it (row blocks, cursors, loop bounds) then lives in
    // scalar registers and branches on it are uniform
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int K = g.K;
    const long items = (long)g.count * g.nwg;
    const long i0 = items * blockIdx.x / gridDim.x, i1 = items * (blockIdx.x + 1) / gridDim.x;
    const int hh = lane >> 5;
    const int nchunks = (g.nsb + CH - 1) / CH;
    const int Kc = nchunks * CH * SBK;                       // the xq rows hold a whole number of chunks

    long it = i0;
    while (it < i1) {
        const int p = (int)(it / g.nwg);
        const long p_end = min(i1, (long)(p + 1) * g.nwg);     // this workgroup's items of problem p: [it, p_end)

        // ---- this wavefront's row blocks: it + wave, + 16, ...; a flat walk over (row block, chunk).  The first
        // chunk does not depend on the activations: it is requested ahead of their quantisation.
        const gb_wptr wp = (gb_wptr)g.packed[p];
        const long first = it + wave;
        const int mine = first < p_end ? (int)((p_end - first + GV_WAVES - 1) / GV_WAVES) : 0;
        const int total = mine * nchunks;
        const int nb_first = (int)(first % g.nwg);              // row blocks of one problem are consecutive
        const size_t blk_stride = (size_t)GV_WAVES * g.nsb * 64;
        uint4 wa[CH], wb[CH];
        // request cursor (runs ahead of the contraction cursor over the same sequence)
        gb_wptr rq_blk = wp + (size_t)nb_first * g.nsb * 64 + lane;
        int rq_c = 0, rq_left = total;
        auto request = [&](uint4 (&w)[CH]) {
            gb_request<CH>(rq_blk, rq_c, g.nsb, w);
            if (rq_left > 1) {                 // past the end the last chunk is requested again and dropped
                --rq_left;
                if (++rq_c == nchunks) { rq_c = 0; rq_blk += blk_stride; }
            }
        };
        if (total > 0) request(wa);

        // ---- quantise the activations of problem p into LDS
        __syncthreads();                   // every wavefront is done with the previous problem's xq
        float dsc[MT];                     // a / 127 per token
        int sq[MT];                        // sum_k q per token
        {
            const void* x = (const void*)(const __attribute__((address_space(1))) char*)g.x[p];
            float4 xv[MT][GV_X4];
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                float tm = 0.f;
#pragma unroll
                for (int u = 0; u < GV_X4; ++u) {
                    const int k = 4 * ((int)threadIdx.x + GV_THREADS * u);
                    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (t < g.M && k < K) v = load_x4(x, g.x_dtype, (size_t)t * K + k);
                    xv[t][u] = v;
                    tm = fmaxf(tm, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
                }
                tm = wave_max(tm);
                if (lane == 0) wmax[t][wave] = tm;
            }
            __syncthreads();
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                float m = wmax[t][0];
#pragma unroll
                for (int w = 1; w < GV_WAVES; ++w) m = fmaxf(m, wmax[t][w]);
                const float ac = fmaxf(m, g.eps_act);
                dsc[t] = ac / 127.0f;
                const float sc = 127.0f / ac;
                int qsum = 0;
#pragma unroll
                for (int u = 0; u < GV_X4; ++u) {
                    const int k = 4 * ((int)threadIdx.x + GV_THREADS * u);
                    if (k < Kc) {          // zeros from K to a whole number of chunks
                        const int word = (int)(quantise_four(xv[t][u], sc) & (ANY_EPS && k >= K ? 0u : ~0u));
                        qsum = __builtin_amdgcn_sdot4(word, 0x01010101, qsum, false);
                        xq[t][k >> 2] = word;
                    }
                }
                qsum = wave_total(qsum);
                if (lane == 0) wsum[t][wave] = qsum;
            }
            __syncthreads();
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                int sum = 0;
#pragma unroll
                for (int w = 0; w < GV_WAVES; ++w) sum += wsum[t][w];
                sq[t] = sum;
            }
        }
        const float beta = *(const __attribute__((address_space(1))) float*)g.beta[p];
        __attribute__((address_space(1))) float* yp = (__attribute__((address_space(1))) float*)g.y[p];
        int acc[MT];
#pragma unroll
        for (int t = 0; t < MT; ++t) acc[t] = 0;

        if (total > 0) {
            int cc = 0, nb = nb_first;         // chunk and row block being contracted
            int slot = 0, nb_slot0 = nb_first; // results parked in LDS: row blocks nb_slot0, + 16, ... (slot of them)
            // Results go to LDS first and to memory in groups: a store in flight between the weight loads would
            // make every later wait a wait for everything (loads and stores share one counter).
            auto flush = [&]() {
                for (int sl = 0; sl < slot; ++sl) {
                    const int n = (nb_slot0 + sl * GV_WAVES) * 32 + (lane & 31);
#pragma unroll
                    for (int t = 0; t < MT; ++t)
                        if (lane < 32 && t < g.M && n < g.N) yp[(size_t)t * g.N + n] = ypark[wave][sl][t][lane];
                }
                slot = 0;
            };
            auto contract = [&](const uint4 (&w)[CH]) {
                gb_contract<MT, CH>(w, cc, hh, xq, acc);
                if (++cc == nchunks) {
                    // last chunk of a row block: fold the two k-halves, rescale, park 32 rows per token
                    if (slot == 0) nb_slot0 = nb;
#pragma unroll
                    for (int t = 0; t < MT; ++t) {
                        const int full = acc[t] + __shfl_xor(acc[t], 32, 64);
                        if (lane < 32) ypark[wave][slot][t][lane] = ((float)(full - sq[t]) * dsc[t]) * beta;
                        acc[t] = 0;
                    }
                    cc = 0;
                    nb += GV_WAVES;
                    if (++slot == GB_SLOTS) flush();
                }
            };

            for (int q = 0; q < total; q += 2) {
                request(wb);
                contract(wa);
                request(wa);
                if (q + 1 < total) contract(wb);
            }
            flush();
        }
        it = p_end;
    }
}

template <int MT, int CH, bool ANY_EPS = false>
int launch_batch_ch(const GemvBatchArgs& g, hipStream_t s) {
    static const int slots = [] {        // workgroups the device holds at once
        int dev = 0, cus = 0, per_cu = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, gemv_batch_kernel<MT, CH, ANY_EPS>, GV_THREADS, 0) != hipSuccess ||
            cus <= 0 || per_cu <= 0) {
            (void)hipGetLastError();
            cus = 256;
            per_cu = 1;
        }
        return cus * per_cu;
    }();
    const long items = (long)g.count * g.nwg;
    const int grid = (int)(items < slots ? items : slots);
    hipLaunchKernelGGL((gemv_batch_kernel<MT, CH, ANY_EPS>), dim3(grid), dim3(GV_THREADS), 0, s, g);
    return BRL_OK;
}

// chunk length: one that divides the number of super-blocks (no clamped tail loads), else 4
template <int MT>
int launch_batch_one(const GemvBatchArgs& g, hipStream_t s) {
    if (g.nsb % 4 == 0) return launch_batch_ch<MT, 4>(g, s);
    if (g.nsb % 6 == 0) return launch_batch_ch<MT, 6>(g, s);
    if (g.nsb % 5 == 0) return launch_batch_ch<MT, 5>(g, s);
    if (127.0f / g.eps_act > 3.4028235e38f) return launch_batch_ch<4, 4, true>(g, s);
    return launch_batch_ch<MT, 4>(g, s);
}

}  // namespace

int launch_gemv(const void* x, int x_dtype, int M, int K, int N, const uint32_t* packed, const float* beta,
                float eps_act, float* y, const float* residual, int8_t* xq_dbg, float* absmax_dbg,
                int32_t* acc_dbg, hipStream_t s) {
    GemvArgs g;
    g.x = x; g.x_dtype = x_dtype; g.M = M; g.K = K; g.N = N;
    g.nsb = round_up(K, SBK) / SBK;
    if (g.nsb > GV_MAX_SB) {
        set_error("gemv: K = %d exceeds the supported %d", K, MAX_K);
        return BRL_EINVAL;
    }
    g.packed = reinterpret_cast<const uint4*>(packed);
    g.beta = beta; g.eps_act = eps_act; g.y = y; g.residual = residual;
    g.xq_dbg = xq_dbg; g.absmax_dbg = absmax_dbg; g.acc_dbg = acc_dbg;
    const int grid = round_up(N, NB) / NB;
    LaunchTimer tm(BRL_KC_GEMV, s);
    auto launch = [&](auto mt) {
        constexpr int MT = decltype(mt)::value;
        if (K <= 4096) hipLaunchKernelGGL((gemv_kernel<MT, 1, 2>), dim3(grid), dim3(GV_THREADS), 0, s, g);
        else if (K <= 8192) hipLaunchKernelGGL((gemv_kernel<MT, 2, 4>), dim3(grid), dim3(GV_THREADS), 0, s, g);
        else hipLaunchKernelGGL((gemv_kernel<MT, 3, 5>), dim3(grid), dim3(GV_THREADS), 0, s, g);
    };
    switch (M) {
        case 1: launch(std::integral_constant<int, 1>()); break;
        case 2: launch(std::integral_constant<int, 2>()); break;
        case 3:
        case 4: launch(std::integral_constant<int, 4>()); break;
        default: set_error("gemv: M = %d out of range 1..4", M); return BRL_EINVAL;
    }
    BRL_LAUNCH_CHECK("gemv_kernel");
    return BRL_OK;
}

// Does launch_rows_product take this product?  From three tokens on (gemv_kernel / here, us a call: 2 x 4096 x 4096 5.4 /
// 6.4, 2 x 6912 x 2560 5.4 / 5.4, 3 x 6912 x 2560 6.2 / 5.4, 4 x 4096 x 4096 7.0 / 6.1, 4 x 2560 x 5120 8.0 / 6.9); one
// workgroup per compute unit and round, so not past 256 of them.  Up to 16 tokens as far as a wavefront's registers and the
// operand rows beside the parts' 64 KB of LDS reach, 5120 columns: ahead there also by GPU time alone, in a captured graph whose
// weights no other call reads (two launches / here: 16 x 8192 x 4096 8.5 / 7.2, x 5120 9.0 / 8.3; bf16, where this instance
// spills four registers, 9.5 / 8.6, 16 x 2560 x 5120 9.3 / 8.3; on weights that every call reads again the bf16 one is level
// from 4097 columns on, 0.93 to 1.05).  17 to 32 tokens only up to 2048: ahead by GPU time up to 1024 columns (1.23 to 1.32 over
// 3700 shapes), within 3 % from there on (fp32 1.01 up to 1536 and 0.99 up to 2048, bf16 0.99 and 0.97; from 2048 rows on 2 %
// less), a launch less for the host (32 x 8192 x 2048 8.2 / 7.3); at 2560 behind (24 x 4096 7.8 / 8.1, 32 x 128 7.3 / 7.8, 32 x
// 8192 on resident weights 7.2 / 7.9) for 0 to 17 % of a call's time from the host.
bool rows_product_eligible(int M, int N, int K) {
    return M >= 3 && M <= 32 && round_up(N, NB) / NB <= 256 && K <= (M <= 16 ? 5120 : 2048);
}

int launch_rows_product(const void* x, int x_dtype, int M, int K, int N, const uint32_t* packed, const float* beta,
                        float eps_act, float* y, const float* residual, int8_t* xq_dbg, float* absmax_dbg,
                        int32_t* acc_dbg, hipStream_t s) {
    GemvArgs g;
    g.x = x; g.x_dtype = x_dtype; g.M = M; g.K = K; g.N = N;
    g.nsb = round_up(K, SBK) / SBK;
    g.packed = reinterpret_cast<const uint4*>(packed);
    g.beta = beta; g.eps_act = eps_act; g.y = y; g.residual = residual;
    g.xq_dbg = xq_dbg; g.absmax_dbg = absmax_dbg; g.acc_dbg = acc_dbg;
    LaunchTimer tm(BRL_KC_GEMM_NARROW, s, 2.0 * (double)M * (double)N * (double)K);
    const dim3 grid(round_up(N, NB) / NB);
    auto launch = [&](auto rw, auto nx) {
        constexpr int RW = decltype(rw)::value, NX = decltype(nx)::value;
        if (x_dtype == BRL_BF16) hipLaunchKernelGGL((rows_product_kernel<RW, NX, true>), grid, dim3(GV_THREADS), 0, s, g);
        else hipLaunchKernelGGL((rows_product_kernel<RW, NX, false>), grid, dim3(GV_THREADS), 0, s, g);
    };
    typedef std::integral_constant<int, 1> one;
    typedef std::integral_constant<int, 2> two;
    if (!rows_product_eligible(M, N, K)) {
        set_error("rows product: %d tokens, %d x %d", M, N, K);
        return BRL_EINVAL;
    }
    if (M <= 16) {
        if (K <= 1024) launch(one(), std::integral_constant<int, 4>());
        else if (K <= 2048) launch(one(), std::integral_constant<int, 8>());
        else if (K <= 2560) launch(one(), std::integral_constant<int, 10>());
        else if (K <= 4096) launch(one(), std::integral_constant<int, 16>());
        else launch(one(), std::integral_constant<int, 20>());
    } else {
        if (K <= 1024) launch(two(), std::integral_constant<int, 4>());
        else launch(two(), std::integral_constant<int, 8>());
    }
    BRL_LAUNCH_CHECK("rows_product_kernel");
    return BRL_OK;
}

int launch_gemv_batch(const void* const* packed, const float* const* beta, int N, int K, const void* const* x,
                      int x_dtype, int M, float eps_act, float* const* y, int count, hipStream_t s) {
    GemvBatchArgs g;
    g.packed = reinterpret_cast<const uint4* const*>(packed);
    g.beta = beta; g.x = x; g.y = y; g.x_dtype = x_dtype;
    g.M = M; g.K = K; g.N = N;
    g.nsb = round_up(K, SBK) / SBK;
    g.nwg = round_up(N, NB) / NB;
    g.count = count;
    g.eps_act = eps_act;
    if (g.nsb > GV_MAX_SB) {
        set_error("gemv batch: K = %d exceeds the supported %d", K, MAX_K);
        return BRL_EINVAL;
    }
    if (count == 0) return BRL_OK;
    LaunchTimer tm(BRL_KC_GEMV, s);
    switch (M) {
        case 1: launch_batch_one<1>(g, s); break;
        case 2: launch_batch_one<2>(g, s); break;
        case 3:
        case 4: launch_batch_one<4>(g, s); break;
        default: set_error("gemv batch: M = %d out of range 1..4", M); return BRL_EINVAL;
    }
    BRL_LAUNCH_CHECK("gemv_batch_kernel");
    return BRL_OK;
}

}  // namespace brl
