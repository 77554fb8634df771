// Rotary causal grouped-query attention on the matrix cores: fp16 hi + lo split
// operands, fp32 accumulation and softmax.
//
// Every fp32 operand x is carried as hi = fp16(x), lo = fp16(x - hi); a product is
// taken as hi*hi + hi*lo + lo*hi (three v_mfma_f32_32x32x16_f16 per step), which
// keeps about 21 mantissa bits - the accuracy of fp32 attention at matrix-core speed.
//
// Two kernels:
//  attn_pack_kernel   reads the fp32 k | v rows once, applies the rotary
//                     embedding to k and writes hi / lo fp16 MFMA operand
//                     fragments: 1 KB pieces in lane order, so that every later
//                     load of them is a linear, fully coalesced copy.  (q rows
//                     are used by exactly one wavefront and are rotated and
//                     split by that wavefront itself.)
//  attention_frag_kernel  a wavefront owns 32 queries of one head (lane & 31 =
//                     query, lane >> 5 = k-group).  Per block of 32 keys it
//                     computes the transposed scores S^T = K Q^T, so a lane ends
//                     up with 16 scores of ITS query: the softmax is lane-local
//                     apart from one exchange with lane ^ 32.  The probabilities
//                     stay in registers and become the B operand of
//                     O^T = V^T P^T, which again keeps one query per lane.  The
//                     four wavefronts of a workgroup (the heads of one key/value
//                     group on one query block, so all four need the same
//                     causal range of keys) share each K / V block through LDS,
//                     filled by direct global->LDS loads, double buffered.
// V fragments are stored transposed with the keys of a block permuted so that
// the 8 keys a lane's probabilities stand for are 16 contiguous bytes.
// Where the q | k | v product has written the v fragments (uniform batches, other head sizes), attn_keys_kernel
// takes the pack kernel's place.
// Where the q | k | v product has already written the fragments (its epilogue does for
// uniform batches at head_dim 128, q included), only attention_frag_kernel runs, in the
// form that reads its q fragments straight into registers (launch_attention_mfma_prepacked).
#include "common.hpp"


namespace brl {

namespace {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

struct PackArgs {
    const float* qkv;     // [B*S, ld]: q heads | k heads | v heads
    int ld, B, S, NRB, Hq, Hkv, dh;   // S: rows per state, or the bound on the state lengths with a SeqMap
    SeqMap sm;
    const float* cos_t;   // [S, dh/2]
    const float* sin_t;
    uint4* KVF;           // [B][Hkv][NRB][ K: [KS][hi,lo] | V: [DB][2][hi,lo] ][64 lanes]
    int by_xcd;           // neighbouring heads on one XCD (pack_by_xcd), else the order of the workgroups
};

__device__ inline uint4 pack8h(const float (&x)[8], bool lo_part) {
    v8h r;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const _Float16 hi = (_Float16)x[e];
        r[e] = lo_part ? (_Float16)(x[e] - (float)hi) : hi;
    }
    return __builtin_bit_cast(uint4, r);
}

// a value the compiler must round to fp32: it would fold the last multiply into a conversion that follows (one rounding
// instead of two), for one use of the value and not for another
__device__ __forceinline__ float rounded(float x) {
    asm("" : "+v"(x));
    return x;
}

// fp16 hi and lo of two values.  x - hi is exact in fp32, so the mixed-precision multiply-add (x * 1 - hi, fp16 operand and
// result) rounds once, as subtraction and conversion would: two instructions for a pair of low parts instead of five.
__device__ __forceinline__ void split_pair(float x0, float x1, uint32_t& hi, uint32_t& lo) {
    typedef _Float16 v2h __attribute__((ext_vector_type(2)));
    v2h h = {(_Float16)x0, (_Float16)x1};
    hi = __builtin_bit_cast(uint32_t, h);
    float one = 1.0f;                                // (opaque: a literal would turn the multiply-add back into a subtraction;
    asm("" : "+s"(one));                             // likewise the pair, into two more conversions)
    asm("" : "+v"(hi));
    h = __builtin_bit_cast(v2h, hi);
    const v2h l = {(_Float16)__builtin_fmaf(x0, one, -(float)h[0]), (_Float16)__builtin_fmaf(x1, one, -(float)h[1])};
    lo = __builtin_bit_cast(uint32_t, l);
}

// k-steps of 16 components of a score.  Heads of 100 end in the seventh, the eighth would multiply zeros; so may all of up to 112
// whose rotary halves are not whole quads, and wider ones of that kind are refused (attn_head_dim_ok).
template <int DHP, int VW> constexpr int k_steps = DHP == 128 && VW == 2 ? 7 : DHP / 16;

template <int VW> struct VecOf;
template <> struct VecOf<4> { typedef float4 type; };
template <> struct VecOf<2> { typedef float2 type; };

// --- staging of one 32-row block of a q or k head -------------------------------------------
// A wavefront reads the rows with fully coalesced loads (VW floats per lane, one or two rows per
// instruction), rotates pairs (i, i + dh/2), scales, splits into fp16 hi / lo and parks both in a
// wave-private LDS region of 128 * DHP bytes: plane hi [32 rows][DHP halfs], then plane lo.  The
// 16-byte chunks of a row are XOR-swizzled so that the later fragment reads (lane = row) spread
// over all banks.  Components beyond dh and rows beyond n_valid are zero.
template <int DHP>
__device__ inline int plane_offset(int r, int chunk) {
    constexpr int RS = DHP * 2, CH = DHP / 8, RPB = 256 / RS;
    return r * RS + ((chunk ^ ((r / RPB) & (CH - 1))) << 4);
}

// NIT of the block's load instructions, from it_begin on: a share of the rows for each of several wavefronts.  The count
// is a template argument so that a wavefront's loads can be in flight together (at most 32 / VW of them); the compiler decides
// how many are, by the registers it wants.  AT_ONCE: all of them, whatever it wants.  For attention_short_kernel on heads of
// up to 32, where it had come to take four trips to memory (heads of 32, 1 state of 32 tokens 8.3 us, 6.7 at once; 1024 states 31.0 /
// 28.7); wider heads need the wavefronts more (100, 64 states of 32 tokens 31.3 / 32.6; 64 level).
template <int DHP, int VW, int NIT = 32 / (64 / (DHP / VW)), bool AT_ONCE = false>
__device__ __forceinline__ void stage_rope_rows(const float* rows, int ld, int n_valid, const float* cp, const float* sp,
                                                int dh, float scale, char* region, int lane, int it_begin = 0) {
    typedef typename VecOf<VW>::type V;
    constexpr int LPR = DHP / VW, RPI = 64 / LPR;     // lanes per row, rows per instruction
    const int half = dh / 2;
    const int c = lane % LPR, d = c * VW;
    // loads are unconditional (addresses clamped into the block, results masked) so that the
    // loads of many iterations can be in flight together
    const bool in_head = d < dh;
    const bool first = d < half;
    const int ds = in_head ? d : 0;
    const int i = in_head ? (first ? d : d - half) : 0;
    const int dp = in_head ? (first ? d + half : d - half) : 0;
    static_assert(!AT_ONCE || NIT * VW <= 16, "64 registers of a lane");
    V xs[NIT], xp[NIT], cs[NIT], sn[NIT];
    auto request = [&](int u) {
        const int rc = min((it_begin + u) * RPI + lane / LPR, n_valid - 1);
        const float* row = rows + (size_t)rc * ld;
        xs[u] = *reinterpret_cast<const V*>(row + ds);
        xp[u] = *reinterpret_cast<const V*>(row + dp);
        cs[u] = *reinterpret_cast<const V*>(cp + (size_t)rc * half + i);
        sn[u] = *reinterpret_cast<const V*>(sp + (size_t)rc * half + i);
    };
    if constexpr (AT_ONCE) {
#pragma unroll
        for (int u = 0; u < NIT; ++u) request(u);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll(NIT < 32 / VW ? NIT : 32 / VW)
    for (int u = 0; u < NIT; ++u) {
        if constexpr (!AT_ONCE) request(u);
        const int r = (it_begin + u) * RPI + lane / LPR;
        const float* fs = reinterpret_cast<const float*>(&xs[u]);
        const float* fp = reinterpret_cast<const float*>(&xp[u]);
        const float* fc = reinterpret_cast<const float*>(&cs[u]);
        const float* fn = reinterpret_cast<const float*>(&sn[u]);
        const bool keep = in_head && r < n_valid;
        float v[VW];
#pragma unroll
        for (int e = 0; e < VW; ++e) {
            const float t = (first ? (fs[e] * fc[e] - fp[e] * fn[e]) : (fs[e] * fc[e] + fp[e] * fn[e])) * scale;
            v[e] = keep ? t : 0.f;
        }
        typedef _Float16 hv __attribute__((ext_vector_type(VW)));
        hv hi, lo;
#pragma unroll
        for (int e = 0; e < VW; ++e) {
            hi[e] = (_Float16)v[e];
            lo[e] = (_Float16)(v[e] - (float)hi[e]);
        }
        const int off = plane_offset<DHP>(r, d >> 3) + (d & 7) * 2;
        *reinterpret_cast<hv*>(region + off) = hi;
        *reinterpret_cast<hv*>(region + 64 * DHP + off) = lo;
    }
}

// fragment of k-step ks for lane (row = lane & 31, kg = lane >> 5): components 16 ks + 8 kg + 0..7
template <int DHP>
__device__ inline uint4 staged_fragment(const char* region, int ks, int lane, int lo_plane) {
    return *reinterpret_cast<const uint4*>(region + lo_plane * 64 * DHP +
                                           plane_offset<DHP>(lane & 31, 2 * ks + (lane >> 5)));
}

// --- the 32 query rows of a wavefront ----------------------------------------------------------------------------
// Four lanes read 64 neighbouring bytes of a row's first half and the rotary partners of these components (every element
// once, every load in flight together), rotate, scale and split them into the same planes.  dh / 2 need not be a multiple of
// four: the last lanes then repeat components of their neighbours.  Rows past the last repeat it (no one stores them).
// Against stage_rope_rows (every element twice, a quarter of the loads in flight): heads of 100, 1 state of 128 tokens 22.6 ->
// 21.1 us, 64 states 234 -> 203, pack kernel included; 16 / 16 heads of 64, 16 states of 96 tokens 20.4 -> 16.4.  Not ahead
// everywhere: 256 states of 128 tokens with 16 / 16 heads of 64, which memory bounds, 218 -> 227, one state of 64 with heads of 16 10.2
// -> 10.6 (with the read-ahead of compute).
template <int DHP, int VW>
struct QueryRows {
    static constexpr int NQ = DHP / 32;               // groups of 16 components of a first half
    typedef float v4 __attribute__((ext_vector_type(4), aligned(8)));      // (dh / 2 is even)
    v4 x[2][NQ], y[2][NQ], c[2][NQ], s[2][NQ];
    static __device__ __forceinline__ int comp(int ks, int half) { return min(16 * ks + 4 * (int)(threadIdx.x & 3), half - 4); }
    __device__ __forceinline__ void request(const float* rows, int ld, int n_valid, const float* cp, const float* sp, int half) {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = min((lane >> 2) + 16 * i, n_valid - 1);
            const float* row = rows + (size_t)r * ld;
#pragma unroll
            for (int ks = 0; ks < NQ; ++ks) {
                const int d = comp(ks, half);
                x[i][ks] = *reinterpret_cast<const v4*>(row + d);
                y[i][ks] = *reinterpret_cast<const v4*>(row + half + d);
                c[i][ks] = *reinterpret_cast<const v4*>(cp + (size_t)r * half + d);
                s[i][ks] = *reinterpret_cast<const v4*>(sp + (size_t)r * half + d);
            }
        }
    }
    __device__ __forceinline__ void park(char* region, int half, float scale) const {
        typedef _Float16 hv __attribute__((ext_vector_type(VW)));
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = (lane >> 2) + 16 * i;
#pragma unroll
            for (int ks = 0; ks < NQ; ++ks) {
                const int d = comp(ks, half);
#pragma unroll
                for (int e = 0; e < 4; e += VW) {
                    hv h1, l1, h2, l2;
#pragma unroll
                    for (int q = 0; q < VW; ++q) {
                        const float xv = x[i][ks][e + q], yv = y[i][ks][e + q], cv = c[i][ks][e + q], sv = s[i][ks][e + q];
                        const float t1 = rounded((xv * cv - yv * sv) * scale), t2 = rounded((yv * cv + xv * sv) * scale);
                        h1[q] = (_Float16)t1; l1[q] = (_Float16)(t1 - (float)h1[q]);
                        h2[q] = (_Float16)t2; l2[q] = (_Float16)(t2 - (float)h2[q]);
                    }
                    const int d1 = d + e, d2 = half + d + e;          // VW components never cross a chunk of eight
                    const int o1 = plane_offset<DHP>(r, d1 >> 3) + (d1 & 7) * 2, o2 = plane_offset<DHP>(r, d2 >> 3) + (d2 & 7) * 2;
                    *reinterpret_cast<hv*>(region + o1) = h1;
                    *reinterpret_cast<hv*>(region + 64 * DHP + o1) = l1;
                    *reinterpret_cast<hv*>(region + o2) = h2;
                    *reinterpret_cast<hv*>(region + 64 * DHP + o2) = l2;
                }
            }
        }
        // components past the head
        const int r = lane & 31, plane = (lane >> 5) * 64 * DHP;
        for (int d = 2 * half; d < DHP; d += 2) *reinterpret_cast<uint32_t*>(region + plane + plane_offset<DHP>(r, d >> 3) + (d & 7) * 2) = 0u;
    }
};

template <int DHP, int VW>
__global__ __launch_bounds__(256) void attn_pack_kernel(PackArgs a) {
    constexpr int KS = k_steps<DHP, VW>, DB = DHP / 32;
    constexpr int KVFR = KS * 2 + DB * 4;             // 1 KB fragments per key block
    __shared__ __attribute__((aligned(16))) char park[128 * DHP];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n_work = a.B * a.NRB * a.Hkv, per_xcd = (n_work + 7) >> 3;
    const int w = a.by_xcd ? (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
    if (w >= n_work) return;
    const int hd = w % a.Hkv;
    const int rb = (w / a.Hkv) % a.NRB;
    const int b = w / (a.Hkv * a.NRB);
    const int half = a.dh / 2;
    const int dq = a.Hq * a.dh, dkv = a.Hkv * a.dh;
    const int n_valid = min(32, seq_len(a.sm, b, a.S) - rb * 32);
    if (n_valid <= 0) return;             // this state has no such key block (never read either)
    const float* rows = a.qkv + ((size_t)seq_row0(a.sm, b, a.S) + rb * 32) * a.ld;
    uint4* dst = a.KVF + ((size_t)(b * a.Hkv + hd) * a.NRB + rb) * KVFR * 64;

    // k head: each wavefront stages a quarter of the rows, then writes a quarter of the fragments
    constexpr int ITS = 32 / (64 / (DHP / VW));
    stage_rope_rows<DHP, VW, ITS / 4>(rows + dq + hd * a.dh, a.ld, n_valid, a.cos_t + (size_t)rb * 32 * half,
                                      a.sin_t + (size_t)rb * 32 * half, a.dh, 1.0f, park, lane, wave * (ITS / 4));
    __syncthreads();
#pragma unroll
    for (int q = 0; q < (KS + 1) / 2; ++q) {
        const int fr = q * 4 + wave;                  // fragment = (k-step, plane)
        if (KS % 2 && fr >= 2 * KS) break;
        dst[fr * 64 + lane] = staged_fragment<DHP>(park, fr >> 1, lane, fr & 1);
    }
    // v head, transposed: lane (d, h) of (block r, step t) holds the keys 16 t + 8 (e >> 2) + 4 h + (e & 3)
    const int col0 = dq + dkv + hd * a.dh;
    for (int t = threadIdx.x; t < 128 * DB; t += 256) {
        const int dl = t & 31, h = (t >> 5) & 1, tt = (t >> 6) & 1, r = t >> 7;
        const int d = 32 * r + dl;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int row = 16 * tt + 8 * (e >> 2) + 4 * h + (e & 3);
            v[e] = (row < n_valid && d < a.dh) ? rows[(size_t)row * a.ld + col0 + d] : 0.f;
        }
        const int ln = h * 32 + dl;
        dst[(KS * 2 + (r * 2 + tt) * 2 + 0) * 64 + ln] = pack8h(v, false);
        dst[(KS * 2 + (r * 2 + tt) * 2 + 1) * 64 + ln] = pack8h(v, true);
    }
}

// The k fragments alone, where the product has written the v fragments (whole key blocks, no ragged states).  Bound by
// memory: a wavefront takes a key block of one head, every element read once, 16 bytes per lane and all of them in flight.
// (64 states of 512 tokens, 32 heads of 100: 220 us, 0.89 GB; the pack kernel without its v part 294, with it 411.  Half a block
// per wavefront, twice the wavefronts: 231.)
template <int DHP, int VW>
__global__ __launch_bounds__(256) void attn_keys_kernel(PackArgs a) {
    constexpr int KS = k_steps<DHP, VW>, DB = DHP / 32, KVFR = KS * 2 + DB * 4;
    __shared__ __attribute__((aligned(16))) char park[4][128 * DHP];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n_work = a.B * a.NRB * a.Hkv, per_xcd = (n_work + 7) >> 3;          // neighbouring heads on one XCD, as above
    const int at = (int)(blockIdx.x >> 3) * 4 + wave, w = (int)(blockIdx.x & 7) * per_xcd + at;
    if (at >= per_xcd || w >= n_work) return;
    const int hd = w % a.Hkv, rb = (w / a.Hkv) % a.NRB, b = w / (a.Hkv * a.NRB), half = a.dh / 2;
    QueryRows<DHP, VW> k;
    k.request(a.qkv + ((size_t)b * a.S + rb * 32) * a.ld + (a.Hq + hd) * a.dh, a.ld, 32, a.cos_t + (size_t)rb * 32 * half,
              a.sin_t + (size_t)rb * 32 * half, half);
    k.park(park[wave], half, 1.0f);
    __builtin_amdgcn_wave_barrier();
    uint4* dst = a.KVF + ((size_t)(b * a.Hkv + hd) * a.NRB + rb) * KVFR * 64;
#pragma unroll
    for (int fr = 0; fr < 2 * KS; ++fr) dst[fr * 64 + lane] = staged_fragment<DHP>(park[wave], fr >> 1, lane, fr & 1);
}

struct FragArgs {
    const float* qkv;     // [B*S, ld]: the q heads are read from here
    int ld;
    const float* cos_t;
    const float* sin_t;
    float qscale;         // softmax scale in log2 units, folded into q
    const uint4* KVF;
    const uint4* QF;      // q fragments [B][Hq][NRB][KS][hi,lo][64 lanes] (only where the producer wrote them)
    int B, S, NRB, Hq, Hkv, dh;
    SeqMap sm;
    int n_work;           // B * Hkv * chunks
    int turn;             // 1: the chunks of queries start one further on from head to head (chunk_turn)
    float* out;           // [B*S, Hq*dh]
};

template <int DHP, int VW>
struct AttnTile {
    static constexpr int KS = k_steps<DHP, VW>, DB = DHP / 32;
    static constexpr int KVFR = KS * 2 + DB * 4;      // 1 KB fragments per key block (K hi/lo, then V hi/lo)
    static constexpr int STAGE = (KVFR > DHP / 4 ? KVFR : DHP / 4) * 64;      // a block, or two wavefronts' parked queries
    // the WPG wavefronts of a workgroup copy KVFR / WPG fragments each
    template <int WPG>
    static __device__ inline void issue(const uint4* src, uint4* st, int wave, int lane) {
#pragma unroll
        for (int c = 0; c < (KVFR + WPG - 1) / WPG; ++c) {
            const int f = c * WPG + wave;
            if (KVFR % WPG == 0 || f < KVFR) __builtin_amdgcn_global_load_lds(src + f * 64 + lane, st + f * 64, 16, 0, 0);
        }
    }

    // scores of one block of 32 keys against the wavefront's 32 queries, kf(ks, plane) = key fragment
    template <class KF>
    static __device__ __forceinline__ v16f scores(KF&& kf, const v8h (&qh)[KS], const v8h (&ql)[KS]) {
        v16f s;
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const v8h kfh = kf(ks, 0), kfl = kf(ks, 1);
            s = __builtin_amdgcn_mfma_f32_32x32x16_f16(kfl, qh[ks], s, 0, 0, 0);
            s = __builtin_amdgcn_mfma_f32_32x32x16_f16(kfh, ql[ks], s, 0, 0, 0);
            s = __builtin_amdgcn_mfma_f32_32x32x16_f16(kfh, qh[ks], s, 0, 0, 0);
        }
        return s;
    }

    // running softmax: probabilities of the block as fp16 hi / lo, returns the factor of what was accumulated before
    template <bool DIAG>
    static __device__ __forceinline__ float softmax(v16f& s, float& m_run, float& l_run, int lane, v8h (&ph)[2], v8h (&pl)[2]) {
        const int qi = lane & 31, h = lane >> 5;
        float bmax = -INFINITY;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int key = 8 * (v >> 2) + 4 * h + (v & 3);     // position inside the block
            if (DIAG && key > qi) s[v] = -INFINITY;             // causal: keys of later blocks are never visited
            bmax = fmaxf(bmax, s[v]);
        }
        bmax = fmaxf(bmax, __shfl_xor(bmax, 32, 64));
        const float m_new = fmaxf(m_run, bmax);                 // finite: key 0 of the block is visible
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
        float psum = 0.f;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            uint32_t hi[4], lo[4];
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
                const float p0 = __builtin_amdgcn_exp2f(s[8 * t + e] - m_new), p1 = __builtin_amdgcn_exp2f(s[8 * t + e + 1] - m_new);
                psum += p0;
                psum += p1;
                split_pair(p0, p1, hi[e / 2], lo[e / 2]);
            }
            ph[t] = __builtin_bit_cast(v8h, make_uint4(hi[0], hi[1], hi[2], hi[3]));
            pl[t] = __builtin_bit_cast(v8h, make_uint4(lo[0], lo[1], lo[2], lo[3]));
        }
        l_run = l_run * alpha + psum;
        m_run = m_new;
        return alpha;
    }

    // o += V^T P^T for 32 components, vf(t, plane) = transposed value fragment
    template <class VF>
    static __device__ __forceinline__ void values(VF&& vf, const v8h (&ph)[2], const v8h (&pl)[2], v16f& o) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const v8h vfh = vf(t, 0), vfl = vf(t, 1);
            o = __builtin_amdgcn_mfma_f32_32x32x16_f16(vfl, ph[t], o, 0, 0, 0);
            o = __builtin_amdgcn_mfma_f32_32x32x16_f16(vfh, pl[t], o, 0, 0, 0);
            o = __builtin_amdgcn_mfma_f32_32x32x16_f16(vfh, ph[t], o, 0, 0, 0);
        }
    }

    // one staged block of 32 keys against the wavefront's 32 queries
    template <bool DIAG>
    static __device__ __forceinline__ void compute(const uint4* st, const v8h (&qh)[KS], const v8h (&ql)[KS], v16f (&o)[DB],
                                          float& m_run, float& l_run, int lane) {
        v16f s = scores([&](int ks, int plane) { return __builtin_bit_cast(v8h, st[(ks * 2 + plane) * 64 + lane]); }, qh, ql);
        // the key fragments two steps ahead of their products: left to itself the compiler reads each one right before its
        // use, a trip to LDS per product
        __builtin_amdgcn_sched_group_barrier(SCHED_LDS_READ, 4, 0);
#pragma unroll
        for (int ks = 2; ks < KS; ++ks) {
            __builtin_amdgcn_sched_group_barrier(SCHED_MFMA, 3, 0);
            __builtin_amdgcn_sched_group_barrier(SCHED_LDS_READ, 2, 0);
        }
        __builtin_amdgcn_sched_group_barrier(SCHED_MFMA, 6, 0);
        v8h ph[2], pl[2];
        const float alpha = softmax<DIAG>(s, m_run, l_run, lane, ph, pl);
#pragma unroll
        for (int r = 0; r < DB; ++r) {
#pragma unroll
            for (int v = 0; v < 16; ++v) o[r][v] *= alpha;
            values([&](int t, int plane) { return __builtin_bit_cast(v8h, st[(KS * 2 + (r * 2 + t) * 2 + plane) * 64 + lane]); }, ph, pl, o[r]);
        }
    }
    static constexpr int SCHED_MFMA = 0x8, SCHED_LDS_READ = 0x100;
};

// WPG wavefronts (a multiple of 4) = WPG units of one key/value head share every K / V block.
// Four is what is launched: eight halved the K / V traffic but ran 12-19 % slower on both
// measured shapes (fewer resident workgroups, longer tails).
constexpr int ATTN_WPG = 4;
// QPRE: the q rows arrive as fragments (rotated, scaled, split by the kernel that produced them) and are read
// straight into the operand registers; otherwise they are staged from the fp32 rows here.
template <int DHP, int VW, int WPG, bool QPRE = false>
__global__ __launch_bounds__(WPG * 64, 2) void attention_frag_kernel(FragArgs a) {
    using T = AttnTile<DHP, VW>;
    constexpr int KS = T::KS, DB = T::DB;
    __shared__ __attribute__((aligned(1024))) uint4 stage0[T::STAGE];
    __shared__ __attribute__((aligned(1024))) uint4 stage1[T::STAGE];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int group = a.Hq / a.Hkv;
    const int U = group * a.NRB;                      // (query block, head in group) units of one key/value head
    const int chunks = (U + WPG - 1) / WPG;
    // Consecutive work items (the chunks of one key/value head) run on one XCD and share its L2; the longest chunks of a head
    // come first, unless that would put them all on one shader engine (chunk_turn).
    const int per_xcd = (a.n_work + 7) >> 3;
    const int w = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (w >= a.n_work) return;
    const int c = chunks - 1 - (w + a.turn * (w / chunks)) % chunks;
    const int j = (w / chunks) % a.Hkv;
    const int b = w / (chunks * a.Hkv);
    const int len = seq_len(a.sm, b, a.S);
    const int nrb = (len + 31) >> 5;                  // query / key blocks this state really has
    const size_t row0 = (size_t)seq_row0(a.sm, b, a.S);
    // unit u = (query block u / group, head u % group of the group): the wavefronts of a workgroup sit on
    // the same query block (or neighbouring ones), so they need the same key blocks and finish together
    const int u0 = WPG * c, u1 = min(U, u0 + WPG) - 1;
    if (u0 / group >= nrb) return;                    // none of the units exists in this state
    const int kb_max = min(u1 / group, nrb - 1);
    const int u = u0 + wave;
    const bool live = u < U && u / group < nrb;
    const int head = j * group + (live ? u % group : 0);
    const int qb = live ? u / group : -1;

    v8h qh[KS], ql[KS];
    const int qpos = qb * 32 + (lane & 31);
    if constexpr (QPRE) {
        const uint4* qf = a.QF + ((size_t)(b * a.Hq + head) * a.NRB + max(qb, 0)) * (KS * 2 * 64) + lane;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            qh[ks] = __builtin_bit_cast(v8h, qf[(ks * 2 + 0) * 64]);
            ql[ks] = __builtin_bit_cast(v8h, qf[(ks * 2 + 1) * 64]);
        }
    } else {
        // the stage buffers are free before the first key block arrives: the q rows are parked there,
        // four wavefronts at a time
        char* region = reinterpret_cast<char*>((wave & 2) ? stage1 : stage0) + (wave & 1) * (128 * DHP);
#pragma unroll
        for (int rnd = 0; rnd < WPG / 4; ++rnd) {
            const bool mine = (wave >> 2) == rnd;
            if (mine && live) {
                const int half = a.dh / 2;
                QueryRows<DHP, VW> q;
                q.request(a.qkv + (row0 + qb * 32) * a.ld + head * a.dh, a.ld, min(32, len - qb * 32),
                          a.cos_t + (size_t)qb * 32 * half, a.sin_t + (size_t)qb * 32 * half, half);
                q.park(region, half, a.qscale);
            }
            __syncthreads();
            if (mine) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    qh[ks] = __builtin_bit_cast(v8h, staged_fragment<DHP>(region, ks, lane, 0));
                    ql[ks] = __builtin_bit_cast(v8h, staged_fragment<DHP>(region, ks, lane, 1));
                }
            }
            __syncthreads();
        }
    }
    v16f o[DB];
#pragma unroll
    for (int r = 0; r < DB; ++r)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[r][v] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;

    const uint4* kv = a.KVF + (size_t)(b * a.Hkv + j) * a.NRB * T::KVFR * 64;
    T::template issue<WPG>(kv, stage0, wave, lane);
    // (two forms of compute: at heads of 64 they cost a fourth wavefront per SIMD, 164 registers where one that always tests the
    // mask takes 122; it was ahead for states of up to 128 tokens (1.00 to 1.05), behind for most longer ones (0.95 to 1.03): 0.984 over 2500 shapes)
    auto block = [&](const uint4* st, int kb) {
        if (kb < qb) T::template compute<false>(st, qh, ql, o, m_run, l_run, lane);
        else if (kb == qb) T::template compute<true>(st, qh, ql, o, m_run, l_run, lane);
    };
    int kb = 0;
    for (; kb + 1 <= kb_max; kb += 2) {
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        T::template issue<WPG>(kv + (size_t)(kb + 1) * T::KVFR * 64, stage1, wave, lane);
        block(stage0, kb);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (kb + 2 <= kb_max) T::template issue<WPG>(kv + (size_t)(kb + 2) * T::KVFR * 64, stage0, wave, lane);
        block(stage1, kb + 1);
    }
    if (kb <= kb_max) {
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        block(stage0, kb);
    }

    const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
    const int pos = qpos;
    if (live && pos < len) {
        const float inv = 1.0f / l_tot;
        const int h = lane >> 5;
        float* op = a.out + (row0 + pos) * ((size_t)a.Hq * a.dh) + (size_t)head * a.dh;
#pragma unroll
        for (int r = 0; r < DB; ++r)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                const int d = 32 * r + 8 * g4 + 4 * h;
                if (d < a.dh) {
                    float4 v;
                    v.x = o[r][4 * g4 + 0] * inv; v.y = o[r][4 * g4 + 1] * inv;
                    v.z = o[r][4 * g4 + 2] * inv; v.w = o[r][4 * g4 + 3] * inv;
                    *reinterpret_cast<float4*>(op + d) = v;
                }
            }
    }
}

// States of at most 32 tokens (one key block): one kernel, no fragment round trip through memory.  A workgroup = one
// query head of one state; such a launch is latency bound, so everything is requested at once by as many wavefronts as
// the work splits into: DB wavefronts stage a share of the q rows each and request the v components they will multiply
// (32 of them, straight into the operand layout), DB more stage a share of the k rows.  After one barrier each of the
// first DB wavefronts takes the whole 32 x 32 scores (redundant, but side by side) and finishes its 32 components.
// Same MFMAs in the same order as the general kernel: same bits.
// Heads of up to 32 ask for five wavefronts per SIMD: left to itself the compiler keeps the rows in flight in 107 registers, four
// wavefronts, and beyond 2048 query heads that is a round sooner (heads of 16, 10 / 2, 291 states of 6 tokens 10.7 -> 9.7 us, 8 / 4, 358
// of 28 12.1 -> 11.4; over 1900 shapes of heads of 16 and 32 1.01, 0.97 to 1.11).
template <int DHP, int VW>
__global__ __launch_bounds__(DHP * 4, DHP == 32 && VW == 4 ? 5 : 1) void attention_short_kernel(FragArgs a) {
    using T = AttnTile<DHP, VW>;
    constexpr int KS = T::KS, DB = T::DB;                 // 2 DB wavefronts
    constexpr int REG = 128 * DHP;                        // bytes of one staged 32-row block (hi and lo planes)
    __shared__ __attribute__((aligned(1024))) char qpark[REG];
    __shared__ __attribute__((aligned(1024))) char kpark[REG];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int head = blockIdx.x % a.Hq, b = blockIdx.x / a.Hq;
    const int j = head / (a.Hq / a.Hkv);
    const int len = seq_len(a.sm, b, a.S);                // 1 .. 32
    if (len <= 0) return;
    const size_t row0 = (size_t)seq_row0(a.sm, b, a.S);
    const int dq = a.Hq * a.dh, dkv = a.Hkv * a.dh;
    const float* rows = a.qkv + row0 * a.ld;
    const int dl = lane & 31, h = lane >> 5;
    constexpr int ITS = 32 / (64 / (DHP / VW));           // load instructions per 32-row block
    static_assert(ITS % DB == 0, "the rows split evenly over DB wavefronts");
    const bool first = wave < DB;
    const int share = first ? wave : wave - DB;
    float vv[2][8];
    // lane (dl, h) of step tt: keys 16 tt + 8 (e >> 2) + 4 h + (e & 3) of component 32 wave + dl.  Keys past the state's
    // end repeat its last row (their probabilities are exactly zero), components past the head are never stored: no
    // condition on a load, which would keep the next one waiting
    if (first) {
        const int d = 32 * wave + dl;
        const float* col = rows + dq + dkv + j * a.dh + min(d, a.dh - 1);
#pragma unroll
        for (int tt = 0; tt < 2; ++tt)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int row = 16 * tt + 8 * (e >> 2) + 4 * h + (e & 3);
                vv[tt][e] = col[(unsigned)(min(row, len - 1) * a.ld)];
            }
    }
    stage_rope_rows<DHP, VW, ITS / DB, DHP == 32>(rows + (first ? head * a.dh : dq + j * a.dh), a.ld, len, a.cos_t, a.sin_t, a.dh,
                                       first ? a.qscale : 1.0f, first ? qpark : kpark, lane, share * (ITS / DB));
    __syncthreads();
    if (!first) return;

    v8h qh[KS], ql[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        qh[ks] = __builtin_bit_cast(v8h, staged_fragment<DHP>(qpark, ks, lane, 0));
        ql[ks] = __builtin_bit_cast(v8h, staged_fragment<DHP>(qpark, ks, lane, 1));
    }
    v16f s = T::scores([&](int ks, int plane) { return __builtin_bit_cast(v8h, staged_fragment<DHP>(kpark, ks, lane, plane)); }, qh, ql);
    float m_run = -INFINITY, l_run = 0.f;
    v8h ph[2], pl[2];
    T::template softmax<true>(s, m_run, l_run, lane, ph, pl);
    v16f o;
#pragma unroll
    for (int v = 0; v < 16; ++v) o[v] = 0.f;
    T::values([&](int t, int plane) { return __builtin_bit_cast(v8h, pack8h(vv[t], plane == 1)); }, ph, pl, o);

    const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
    if (dl < len) {
        const float inv = 1.0f / l_tot;
        float* op = a.out + (row0 + dl) * ((size_t)a.Hq * a.dh) + (size_t)head * a.dh;
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
            const int d = 32 * wave + 8 * g4 + 4 * h;
            if (d < a.dh) {
                float4 v;
                v.x = o[4 * g4 + 0] * inv; v.y = o[4 * g4 + 1] * inv;
                v.z = o[4 * g4 + 2] * inv; v.w = o[4 * g4 + 3] * inv;
                *reinterpret_cast<float4*>(op + d) = v;
            }
        }
    }
}

// The same states with a workgroup = (state, key/value head, up to four query heads of its group): k and v are staged once
// for four heads.  All global reads are requested in one phase by two sets of wavefronts side by side: four stage one q head
// each, four stage a quarter of the k rows each and hold v in registers; after one barrier the k and v fragments are laid
// out in LDS exactly as attn_pack_kernel lays them out in memory, and the block is computed by the same code as in the
// general kernel: same bits.  Where each form runs and what it measured: short_form below.
template <int DHP, int VW>
__global__ __launch_bounds__(512) void attention_group_kernel(FragArgs a) {
    using T = AttnTile<DHP, VW>;
    constexpr int KS = T::KS, DB = T::DB;
    constexpr int REG = 128 * DHP;                        // bytes of one staged 32-row block (hi and lo planes)
    __shared__ __attribute__((aligned(1024))) char qpark[4 * REG];
    __shared__ __attribute__((aligned(1024))) char kpark[REG];
    __shared__ __attribute__((aligned(1024))) uint4 kvst[T::KVFR * 64];

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int group = a.Hq / a.Hkv;
    const int chunks = (group + 3) / 4;
    const int w = blockIdx.x;
    const int c = w % chunks;
    const int j = (w / chunks) % a.Hkv;
    const int b = w / (chunks * a.Hkv);
    const int len = seq_len(a.sm, b, a.S);                // 1 .. 32
    if (len <= 0) return;
    const size_t row0 = (size_t)seq_row0(a.sm, b, a.S);
    const bool qside = wave < 4;                          // wavefronts 0-3: one q head each; 4-7: k and v
    const int u = 4 * c + (wave & 3);
    const bool live = qside && u < group;
    const int head = j * group + (live ? u : 0);
    const int dq = a.Hq * a.dh, dkv = a.Hkv * a.dh;
    const float* rows = a.qkv + row0 * a.ld;

    // ---- one phase of global reads, the two sides in parallel
    char* region = qpark + (wave & 3) * REG;
    constexpr int ITS = 32 / (64 / (DHP / VW));
    constexpr int VR = (128 * DB + 255) / 256;            // v: thread t of 128 * DB owns lane slot (d, h) of (block r, step tt)
    float vv[VR][8];
    const int tk = threadIdx.x - 256;
    if (qside) {
        if (live) stage_rope_rows<DHP, VW>(rows + head * a.dh, a.ld, len, a.cos_t, a.sin_t, a.dh, a.qscale, region, lane);
    } else {
        const int col0 = dq + dkv + j * a.dh;
#pragma unroll
        for (int q = 0; q < VR; ++q) {
            const int t = tk + 256 * q;
            const int dl = t & 31, h = (t >> 5) & 1, tt = (t >> 6) & 1, r = t >> 7;
            const int d = 32 * r + dl;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int row = 16 * tt + 8 * (e >> 2) + 4 * h + (e & 3);
                vv[q][e] = (t < 128 * DB && row < len && d < a.dh) ? rows[(size_t)row * a.ld + col0 + d] : 0.f;
            }
        }
        stage_rope_rows<DHP, VW, ITS / 4>(rows + dq + j * a.dh, a.ld, len, a.cos_t, a.sin_t, a.dh, 1.0f, kpark, lane,
                                          (wave - 4) * (ITS / 4));
    }
    __syncthreads();

    v8h qh[KS], ql[KS];
    if (qside) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            qh[ks] = __builtin_bit_cast(v8h, staged_fragment<DHP>(region, ks, lane, 0));
            ql[ks] = __builtin_bit_cast(v8h, staged_fragment<DHP>(region, ks, lane, 1));
        }
    } else {
#pragma unroll
        for (int q = 0; q < (KS + 1) / 2; ++q) {
            const int fr = q * 4 + wave - 4;              // fragment = (k-step, plane)
            if (KS % 2 && fr >= 2 * KS) break;
            kvst[fr * 64 + lane] = staged_fragment<DHP>(kpark, fr >> 1, lane, fr & 1);
        }
#pragma unroll
        for (int q = 0; q < VR; ++q) {
            const int t = tk + 256 * q;
            if (t < 128 * DB) {
                const int dl = t & 31, h = (t >> 5) & 1, tt = (t >> 6) & 1, r = t >> 7;
                const int ln = h * 32 + dl;
                kvst[(KS * 2 + (r * 2 + tt) * 2 + 0) * 64 + ln] = pack8h(vv[q], false);
                kvst[(KS * 2 + (r * 2 + tt) * 2 + 1) * 64 + ln] = pack8h(vv[q], true);
            }
        }
    }
    __syncthreads();
    if (!qside) return;

    v16f o[DB];
#pragma unroll
    for (int r = 0; r < DB; ++r)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[r][v] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;
    T::template compute<true>(kvst, qh, ql, o, m_run, l_run, lane);

    const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
    const int pos = lane & 31;
    if (live && pos < len) {
        const float inv = 1.0f / l_tot;
        const int h = lane >> 5;
        float* op = a.out + (row0 + pos) * ((size_t)a.Hq * a.dh) + (size_t)head * a.dh;
#pragma unroll
        for (int r = 0; r < DB; ++r)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                const int d = 32 * r + 8 * g4 + 4 * h;
                if (d < a.dh) {
                    float4 v;
                    v.x = o[r][4 * g4 + 0] * inv; v.y = o[r][4 * g4 + 1] * inv;
                    v.z = o[r][4 * g4 + 2] * inv; v.w = o[r][4 * g4 + 3] * inv;
                    *reinterpret_cast<float4*>(op + d) = v;
                }
            }
    }
}

// States of at most 64 tokens with heads of 128: no fragments through memory.  Bound by memory and by how much of it is in
// flight: the pair of kernels above writes K and V once and reads them twice more than needed, waits for q before it asks
// for them, and gives the queries past row 32, a few rows of each head, a wavefront per head.  Here a workgroup asks for the
// fp32 rows of up to four query heads and of their key/value head at once, and stages the rotated K and the transposed V in
// LDS itself (fragments as attn_pack_kernel lays them out).  The first 32 queries: a wavefront per head, one 32-column block
// of the result at a time (one key block needs no running sums).  The queries beyond: workgroups of their own (ahead in the
// grid, they take longer), all heads' rows one after the other in units of 32, a unit's columns shared out over the
// wavefronts that have no unit.  The arithmetic per element and its order are those of the pair: same bits.
// 1024 states of 15 .. 40 tokens, 20 / 5 heads: pack 80 + fragments 309 us, 213 here (725 MB once; 225 with q read in operand
// order, 236 as two launches); 64 states 36 -> 19, 1 state 17 -> 11.  What other sizes take: short_form below.  (The layout of
// rows and fragments is that of heads of 128; none for other head sizes has been built, they keep the pair past 32 tokens.)
constexpr int ROWS_D = 128, ROWS_KS = AttnTile<ROWS_D, 4>::KS;
constexpr int ROWS_STAGE = AttnTile<ROWS_D, 4>::KVFR * 64;
struct RowsBlock {                                    // what a thread of 256 stages of a key block
    float4 k[4], c[2], s[2];                          // eight components of a k row and their eight partners; rotary factors
    float v[2][8];
    // rows: the state's first row; kb: key block; rows past the state's end repeat the last one (never seen by a query)
    __device__ __forceinline__ void request(const float* rows, int ld, int kcol, int vcol, int kb, int len, const float* cos_t,
                                            const float* sin_t) {
        const int t = threadIdx.x;
        const int r = min(kb * 32 + (t >> 3), len - 1), comp = 16 * ((t >> 1) & 3) + 8 * (t & 1);
        const float* kr = rows + (unsigned)(r * ld) + kcol + comp;
        k[0] = *reinterpret_cast<const float4*>(kr);
        k[1] = *reinterpret_cast<const float4*>(kr + 4);
        k[2] = *reinterpret_cast<const float4*>(kr + 64);
        k[3] = *reinterpret_cast<const float4*>(kr + 68);
        c[0] = *reinterpret_cast<const float4*>(cos_t + r * 64 + comp);
        c[1] = *reinterpret_cast<const float4*>(cos_t + r * 64 + comp + 4);
        s[0] = *reinterpret_cast<const float4*>(sin_t + r * 64 + comp);
        s[1] = *reinterpret_cast<const float4*>(sin_t + r * 64 + comp + 4);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int i = t + 256 * q, h = (i >> 5) & 1, tt = (i >> 6) & 1, d = 32 * (i >> 7) + (i & 31);
#pragma unroll
            for (int e = 0; e < 8; ++e)
                v[q][e] = rows[(unsigned)(min(kb * 32 + 16 * tt + 8 * (e >> 2) + 4 * h + (e & 3), len - 1) * ld) + vcol + d];
        }
    }
    __device__ __forceinline__ void commit(uint4* st) const;
};

// N components x and their partners y (64 components on), rotated and scaled, as fp16 hi and lo
template <int N>
__device__ __forceinline__ void rotate_split(const float (&x)[N], const float (&y)[N], const float (&c)[N], const float (&s)[N],
                                             float scale, _Float16 __attribute__((ext_vector_type(N))) (&first)[2],
                                             _Float16 __attribute__((ext_vector_type(N))) (&second)[2]) {
#pragma unroll
    for (int e = 0; e < N; ++e) {
        const float t1 = rounded((x[e] * c[e] - y[e] * s[e]) * scale), t2 = rounded((y[e] * c[e] + x[e] * s[e]) * scale);
        first[0][e] = (_Float16)t1;
        first[1][e] = (_Float16)(t1 - (float)first[0][e]);
        second[0][e] = (_Float16)t2;
        second[1][e] = (_Float16)(t2 - (float)second[0][e]);
    }
}
__device__ __forceinline__ void unpack8(const float4& a, const float4& b, float (&v)[8]) {
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}

// fragments as attn_pack_kernel lays them out in memory
__device__ __forceinline__ void RowsBlock::commit(uint4* st) const {
    const int t = threadIdx.x, r = t >> 3, ks = (t >> 1) & 3, kg = t & 1;
    float x[8], y[8], cf[8], sf[8];
    unpack8(k[0], k[1], x);
    unpack8(k[2], k[3], y);
    unpack8(c[0], c[1], cf);
    unpack8(s[0], s[1], sf);
    v8h a[2], b[2];
    rotate_split<8>(x, y, cf, sf, 1.0f, a, b);
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        st[(ks * 2 + p) * 64 + kg * 32 + r] = __builtin_bit_cast(uint4, a[p]);
        st[((ks + 4) * 2 + p) * 64 + kg * 32 + r] = __builtin_bit_cast(uint4, b[p]);
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int i = t + 256 * q, tt = (i >> 6) & 1, rb = i >> 7;
        st[(ROWS_KS * 2 + (rb * 2 + tt) * 2 + 0) * 64 + (i & 63)] = pack8h(v[q], false);
        st[(ROWS_KS * 2 + (rb * 2 + tt) * 2 + 1) * 64 + (i & 63)] = pack8h(v[q], true);
    }
}

// The q fragments of a wavefront's 32 queries: four lanes read 64 neighbouring bytes of a row (and the 64 bytes of their
// rotary partners), rotate and split them, and the wavefront's 16 KB of LDS turn them into operand order.  Read straight in
// operand order a lane's 16 bytes have no neighbour in the same 64: 15 .. 40 tokens, 64 states 21.8 us, 19.2 this way.
struct RowsQuery {
    float4 x[2][4], y[2][4];
    const float *cp[2], *sp[2];
    // row(r), pos(r): the row of the head and the position of query r
    template <class Row, class Pos>
    __device__ __forceinline__ void request(Row&& row, Pos&& pos, const float* cos_t, const float* sin_t) {
        const int lane = threadIdx.x & 63, part = 4 * (lane & 3);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = (lane >> 2) + 16 * i;
            const float* p = row(r) + part;
            cp[i] = cos_t + pos(r) * 64 + part;
            sp[i] = sin_t + pos(r) * 64 + part;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                x[i][ks] = *reinterpret_cast<const float4*>(p + 16 * ks);
                y[i][ks] = *reinterpret_cast<const float4*>(p + 64 + 16 * ks);
            }
        }
    }
    __device__ __forceinline__ void fragments(uint4* mine, float scale, v8h (&qh)[ROWS_KS], v8h (&ql)[ROWS_KS]) const {
        typedef _Float16 v4h __attribute__((ext_vector_type(4)));
        const int lane = threadIdx.x & 63, part = lane & 3;
        char* at = reinterpret_cast<char*>(mine) + (part >> 1) * 512 + (lane >> 2) * 16 + (part & 1) * 8;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const float4 cv = *reinterpret_cast<const float4*>(cp[i] + 16 * ks), sv = *reinterpret_cast<const float4*>(sp[i] + 16 * ks);
                const float xf[4] = {x[i][ks].x, x[i][ks].y, x[i][ks].z, x[i][ks].w}, yf[4] = {y[i][ks].x, y[i][ks].y, y[i][ks].z, y[i][ks].w};
                const float cf[4] = {cv.x, cv.y, cv.z, cv.w}, sf[4] = {sv.x, sv.y, sv.z, sv.w};
                v4h a[2], b[2];
                rotate_split<4>(xf, yf, cf, sf, scale, a, b);
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    *reinterpret_cast<v4h*>(at + (ks * 2 + p) * 1024 + i * 256) = a[p];
                    *reinterpret_cast<v4h*>(at + ((ks + 4) * 2 + p) * 1024 + i * 256) = b[p];
                }
            }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int ks = 0; ks < ROWS_KS; ++ks) {
            qh[ks] = __builtin_bit_cast(v8h, mine[(ks * 2 + 0) * 64 + lane]);
            ql[ks] = __builtin_bit_cast(v8h, mine[(ks * 2 + 1) * 64 + lane]);
        }
    }
};

// 32 columns of the result, normalised
__device__ __forceinline__ void store_columns(const v16f& o, float inv, float* op, int h) {
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
        float4 v;
        v.x = o[4 * g4 + 0] * inv; v.y = o[4 * g4 + 1] * inv;
        v.z = o[4 * g4 + 2] * inv; v.w = o[4 * g4 + 3] * inv;
        *reinterpret_cast<float4*>(op + 8 * g4 + 4 * h) = v;
    }
}

// workgroup w: up to four heads of one key/value head of one state
struct RowsWork {
    int b, j, c, group, len, kcol, vcol;
    size_t row0;
    const float* rows;
    __device__ __forceinline__ RowsWork(const FragArgs& a, int w) {
        group = a.Hq / a.Hkv;
        const int chunks = (group + 3) / 4;
        c = w % chunks;
        j = (w / chunks) % a.Hkv;
        b = w / (chunks * a.Hkv);
        len = seq_len(a.sm, b, a.S);
        row0 = (size_t)seq_row0(a.sm, b, a.S);
        rows = a.qkv + row0 * a.ld;
        kcol = (a.Hq + j) * ROWS_D;
        vcol = (a.Hq + a.Hkv + j) * ROWS_D;
    }
};

__device__ __forceinline__ void rows_first(const FragArgs& a, int w, uint4* st) {
    using T = AttnTile<ROWS_D, 4>;
    const RowsWork k(a, w);
    if (k.len <= 0) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int u = 4 * k.c + wave, head = k.j * k.group + min(u, k.group - 1);
    const int qi = lane & 31, h = lane >> 5, pos = min(qi, k.len - 1);

    RowsQuery q;
    const float* qrows = k.rows + head * ROWS_D;
    q.request([&](int r) { return qrows + (unsigned)(min(r, k.len - 1) * a.ld); }, [&](int r) { return min(r, k.len - 1); }, a.cos_t, a.sin_t);
    RowsBlock kv;
    kv.request(k.rows, a.ld, k.kcol, k.vcol, 0, k.len, a.cos_t, a.sin_t);
    __builtin_amdgcn_sched_barrier(0);
    v8h qh[ROWS_KS], ql[ROWS_KS];
    q.fragments(st + wave * (ROWS_STAGE / 2), a.qscale, qh, ql);
    __syncthreads();
    kv.commit(st);
    __syncthreads();
    if (u >= k.group) return;

    v16f s = T::scores([&](int ks, int plane) { return __builtin_bit_cast(v8h, st[(ks * 2 + plane) * 64 + lane]); }, qh, ql);
    float m_run = -INFINITY, l_run = 0.f;
    v8h ph[2], pl[2];
    T::template softmax<true>(s, m_run, l_run, lane, ph, pl);
    const float inv = 1.0f / (l_run + __shfl_xor(l_run, 32, 64));
    float* op = a.out + (k.row0 + pos) * ((size_t)a.Hq * ROWS_D) + (size_t)head * ROWS_D;
#pragma unroll
    for (int r = 0; r < T::DB; ++r) {
        v16f o;
#pragma unroll
        for (int v = 0; v < 16; ++v) o[v] = 0.f;
        T::values([&](int t, int plane) { return __builtin_bit_cast(v8h, st[(ROWS_KS * 2 + (r * 2 + t) * 2 + plane) * 64 + lane]); }, ph, pl, o);
        if (qi < k.len) store_columns(o, inv, op + 32 * r, h);
    }
}

// both key blocks against the wavefront's unit, NB 32-column blocks of its result from r0 on
template <int NB>
__device__ __forceinline__ void rows_tail_unit(const uint4* stage, const v8h (&qh)[ROWS_KS], const v8h (&ql)[ROWS_KS], int at,
                                               int r0, bool live, float* op) {
    using T = AttnTile<ROWS_D, 4>;
    const int lane = threadIdx.x & 63, h = lane >> 5;
    v16f o[NB];
#pragma unroll
    for (int r = 0; r < NB; ++r)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[r][v] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
        const uint4* st = stage + kb * ROWS_STAGE;
        v16f s = T::scores([&](int ks, int plane) { return __builtin_bit_cast(v8h, st[(ks * 2 + plane) * 64 + lane]); }, qh, ql);
        v8h ph[2], pl[2];
        const float alpha = kb ? T::template softmax<true>(s, m_run, l_run, h * 32 + at, ph, pl)
                               : T::template softmax<false>(s, m_run, l_run, h * 32 + at, ph, pl);
#pragma unroll
        for (int r = 0; r < NB; ++r) {
#pragma unroll
            for (int v = 0; v < 16; ++v) o[r][v] *= alpha;
            T::values([&](int t, int plane) { return __builtin_bit_cast(v8h, st[(ROWS_KS * 2 + ((r0 + r) * 2 + t) * 2 + plane) * 64 + lane]); }, ph, pl, o[r]);
        }
    }
    const float inv = 1.0f / (l_run + __shfl_xor(l_run, 32, 64));
    if (live) {
#pragma unroll
        for (int r = 0; r < NB; ++r) store_columns(o[r], inv, op + 32 * (r0 + r), h);
    }
}

__device__ __forceinline__ void rows_tail(const FragArgs& a, int w, uint4* st) {
    const RowsWork k(a, w);
    const int n_tail = k.len - 32;
    if (n_tail <= 0) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // queries: all rows of the first head, then the next head's; 1, 2 or (3 or) 4 units of 32, a wavefront's share of one
    const int n_q = min(4, k.group - 4 * k.c) * n_tail;
    const int shift = n_q <= 32 ? 2 : n_q <= 64 ? 1 : 0;                  // log2 of the wavefronts of a unit
    const int q0 = (wave >> shift) * 32;
    auto query = [&](int r) { return min(q0 + r, n_q - 1); };
    auto head_of = [&](int qc) { return k.j * k.group + 4 * k.c + qc / n_tail; };
    auto pos_of = [&](int qc) { return 32 + qc % n_tail; };

    RowsQuery q;
    q.request([&](int r) { return k.rows + (unsigned)(pos_of(query(r)) * a.ld) + head_of(query(r)) * ROWS_D; },
              [&](int r) { return pos_of(query(r)); }, a.cos_t, a.sin_t);
    RowsBlock kv0, kv1;
    kv0.request(k.rows, a.ld, k.kcol, k.vcol, 0, k.len, a.cos_t, a.sin_t);
    kv1.request(k.rows, a.ld, k.kcol, k.vcol, 1, k.len, a.cos_t, a.sin_t);
    __builtin_amdgcn_sched_barrier(0);
    v8h qh[ROWS_KS], ql[ROWS_KS];
    q.fragments(st + wave * (ROWS_STAGE / 2), a.qscale, qh, ql);
    __syncthreads();
    kv0.commit(st);
    kv1.commit(st + ROWS_STAGE);
    __syncthreads();
    if ((wave >> shift) * 32 >= n_q) return;
    const int qc = query(lane & 31), pos = pos_of(qc);
    const bool live = q0 + (lane & 31) < n_q;
    float* op = a.out + (k.row0 + pos) * ((size_t)a.Hq * ROWS_D) + (size_t)head_of(qc) * ROWS_D;
    if (shift == 2) rows_tail_unit<1>(st, qh, ql, pos - 32, wave, live, op);
    else if (shift == 1) rows_tail_unit<2>(st, qh, ql, pos - 32, 2 * (wave & 1), live, op);
    else rows_tail_unit<4>(st, qh, ql, pos - 32, 0, live, op);
}

template <bool TAIL>
__global__ __launch_bounds__(256, 2) void attention_rows_kernel(FragArgs a) {
    __shared__ __attribute__((aligned(1024))) uint4 st[2 * ROWS_STAGE];
    if constexpr (TAIL) {
        const int half = gridDim.x >> 1, w = (int)blockIdx.x;
        if (w < half) rows_tail(a, w, st);
        else rows_first(a, w - half, st);
    } else {
        rows_first(a, (int)blockIdx.x, st);
    }
}

constexpr int padded_head_dim(int dh) { return dh <= 32 ? 32 : (dh <= 64 ? 64 : 128); }
constexpr int head_k_steps(int dh) {
    const int dhp = padded_head_dim(dh);
    return dhp == 128 ? ((dh / 2) % 4 ? k_steps<128, 2> : k_steps<128, 4>) : dhp / 16;
}
// what the kernels can do: rows of whole quads, rotary halves that hold one (QueryRows), no component past the last k-step
constexpr bool attn_head_dim_ok(int dh) { return dh % 4 == 0 && dh >= 8 && dh <= 128 && dh <= 16 * head_k_steps(dh); }
static_assert(attn_head_dim_ok(16) && attn_head_dim_ok(32) && attn_head_dim_ok(64) && attn_head_dim_ok(100) && attn_head_dim_ok(128),
              "the head sizes the entry points accept");
static_assert(!attn_head_dim_ok(4) && !attn_head_dim_ok(102) && attn_head_dim_ok(108) && !attn_head_dim_ok(116) &&
              attn_head_dim_ok(120) && !attn_head_dim_ok(124) && !attn_head_dim_ok(132), "and what no kernel can do");

}  // namespace

size_t attention_mfma_ws_bytes(int B, int S, int n_heads, int n_kv_heads, int head_dim) {
    (void)n_heads;
    const int dhp = padded_head_dim(head_dim);
    const size_t nrb = (size_t)(S + 31) / 32, ks = dhp / 16, db = dhp / 32;
    return (size_t)B * n_kv_heads * nrb * (ks * 2 + db * 4) * 1024;
}

namespace {

// Which form states of one key block take, and at heads of 128 states of two.  N (HEAD): a workgroup per (state, query head),
// O (GROUP): per (state, four query heads of one key/value head), R (ROWS): likewise, q, k and v from the rows, P (PAIR): the
// pack and fragment kernels.  All give the same bits.  Times of 1 .. 2048 states in us:
// - heads of 128, one block: N up to 512 query heads and for groups of one, else R (20 / 5, 20 tokens, 16 states 10.1 / 10.9,
//   32 states 13.3 / 11.5, 64 states 19.7 / 15.7, 1024 states 212 (P) / 151; 12 / 4, 32 tokens, 32 states 11.0 / 11.6, 48 states
//   14.7 / 12.2; 16 / 8, 20 tokens, 64 states 17.2 / 15.1; 16 / 16, 20 tokens, 512 states 106 / 131).  Groups of two and five leave
//   wavefronts of R idle: N while some compute units have a second workgroup of R but none more than three of N, or a third
//   of R but none more than six (groups of two: five) of N.  R / N, over 1300 shapes: groups of two, 257 to 384 and 513 to 640
//   workgroups of R 1.05 and 1.06 (0.95 to 1.12), 385 to 512 0.83 to 0.95, 641 to 768 0.95 to 1.02; of five, 257 to 304 1.10, 308
//   to 352 0.97, 513 to 608 1.07, 610 and 612 1.04 to 1.07.
//   Two blocks: R (20 / 5, 15 .. 40 tokens, P / R: 1 state 16.9 / 11.2, 64 states 36 / 19, 1024 states 374 / 213; 64 tokens: 16
//   states 23.1 / 15.5, 1024 states 499 / 446; 16 / 16, 64 tokens, 64 states 54 / 51; never behind in 120 of them) but P for
//   workgroups half empty of which there are many (30 / 6, 64 tokens, 32 states 37.9 / 33.7, 64 states 52.7 / 58.2).
// - up to 32: N; beyond 1024 query heads, where at least three of O's four wavefronts have a head, O (16 / 4 heads
//   of 32, 32 tokens, 64 states 8.2 / 8.9, 256 states 17.4 / 15.0, 2048 states 121 / 84; 16 / 8: 17.2 / 18.6).
// - up to 64: O where three of its four wavefronts have a head (16 / 4, 32 tokens, 1 state 8.7 / 8.6, 256 states 31 / 23 and
//   P 28), P beyond 2048 workgroups where a group has more than one (32 / 4, 32 tokens, 384 states 55 / 51).  Groups of one,
//   two and five: O up to one, four and four workgroups per compute unit, then N (16 / 16, 32 tokens, 4 states 8.8 / 8.2, 64
//   states 11.9 / 14.7; 16 / 8, 32 tokens, 128 states 19.7 / 17.5, 8 tokens, 512 states 39 / 42; 30 / 6, 8 tokens, 64 states
//   14.5 / 13.3, 256 states 37 / 42), of five P beyond 8192 query heads (8 tokens, 1024 states 127 / 110).
// - between 64 and 128 (100; N / O / P): N; O where N has more than three workgroups per compute unit but O, with three of four
//   wavefronts busy, at most one; P for full groups of many states (20 / 5, 20 tokens, 32 states 14.1 / 13.8 / 16.4, 38 states 14.1 /
//   13.9 / 16.6, 48 states 16.5 / 14.5 / 17.4, 56 states 18.9 / 23.6 / 21.1, 1024 states 257 / 249 / 190; 32 tokens, 512 states 158 / 168 /
//   123; 32 / 32, 32 tokens, 64 states 30 / 82 / 52, 1024 states 565 / 1574 / 874).  P's line was drawn for heads of 128: at 100 P is
//   ahead of it already in full groups of 256 states (20 tokens 54 / 55 / 44, 32 tokens 62 / 66 / 55; 409 of 32 95 / 103 / 102) and
//   in groups of five (30 / 6, 20 tokens, 1024 states 378 / 549 / 334).
enum class ShortForm { HEAD, GROUP, ROWS, PAIR };
ShortForm short_form(int dh, int nrb, int B, int Hq, int Hkv) {
    constexpr long CUS = 256;
    const int dhp = padded_head_dim(dh);
    const long group = Hq / Hkv, chunks = (group + 3) / 4, heads = (long)B * Hq, work = (long)B * Hkv * chunks;
    const bool three_of_four = group >= 3 * chunks, full = 2 * group >= 7 * chunks;
    if (dh == ROWS_D && nrb == 2) return group > 4 && !three_of_four && work > 2 * CUS ? ShortForm::PAIR : ShortForm::ROWS;
    if (nrb > 1) return ShortForm::PAIR;
    if (dh == ROWS_D) {
        const bool few = (work > CUS && heads <= 3 * CUS) || (work > 2 * CUS && heads <= (group == 2 ? 5 : 6) * CUS);
        return group > 1 && heads > 2 * CUS && (three_of_four || !few) ? ShortForm::ROWS : ShortForm::HEAD;
    }
    if (dhp == 32) return three_of_four && heads > 4 * CUS ? ShortForm::GROUP : ShortForm::HEAD;
    if (dhp == 64) {
        if (!three_of_four) {
            if (work <= (group == 1 ? 1 : 4) * CUS) return ShortForm::GROUP;
            return group > 4 && heads > 32 * CUS ? ShortForm::PAIR : ShortForm::HEAD;
        }
        return chunks > 1 && work > 8 * CUS ? ShortForm::PAIR : ShortForm::GROUP;
    }
    if (three_of_four && heads > 3 * CUS && work <= CUS) return ShortForm::GROUP;
    const bool many = chunks > 1 ? heads >= 16 * CUS : heads > 32 * CUS;
    return full && many ? ShortForm::PAIR : ShortForm::HEAD;
}

// The pack kernel's work by XCD: neighbouring heads then share lines where a head is no whole number of them (heads of 100: 1.09
// GB fetched for 0.84 in the order of the workgroups; 398 -> 383 us for 64 states of 512 tokens), and the fragment kernel finds
// what its XCD wrote in that L2 (gain up to 32 MB of fragments: 1.0 to 1.28, any head size).  Heads of 128 are whole lines; from 100 MB
// of their fragments on the plain order is level or ahead (16 / 16, by XCD / plain: 64 states of 72 tokens, 96 MB 60.3 / 61.3, of 128,
// 128 MB 106 / 104, of 256, 256 MB 238 / 228, 128 of 96, 192 MB 172 / 162; 20 / 5, 120 to 160 MB 0.994 to 1.004).  Heads of 64: 0.97 to 1.06
// there, of 32 and 16 1.0 to 1.16.
bool pack_by_xcd(int head_dim, size_t fragment_bytes) { return head_dim != 128 || fragment_bytes <= (size_t)100 << 20; }

// Workgroups go to the four shader engines of an XCD in turn, whether or not one of them has room, and a later chunk of queries
// has more keys: where a head has a multiple of four chunks, one engine would get all the long ones (four chunks, heads of 100, 64
// states of 512 tokens: 1.2 wavefronts per SIMD instead of 2, 715 -> 597 us).  Then the chunks start one further on from head
// to head.  That gives up the order by length, so it takes enough heads to make up for it, more for many chunks.  Gain at 1 / 4 / 8
// / 16 / 48 heads per XCD, heads of 64, 100 and 128 alike: 4 chunks 1 / 1 / 1 / 1 / 1.05, 8 chunks 1 / 1 / 1.09 / 1.08 / 1.10, 12 chunks
// 1 / 0.95 / 0.89 to 1 / 1.03 / 1.08 (1.04 at 12), 16 chunks 1 / 1.05 / 1.01 / 1.04 / 1.07 (0.92 at 6), 20 chunks 1 / 0.85 to 1 / 1 /
// 1.02 / 1.04, 32 chunks 1 / 0.91 / 0.98 / 1.01 / 1.02; any other number at most 1.04, mostly a loss (3: 0.93 to 1, 5: 0.92 to 1.01, 7: 0.85
// to 1, 40 chunks of one head per XCD 0.80).
int chunk_turn(int chunks, int heads) {
    const int per_xcd = heads / 8;
    return chunks % 4 == 0 && (chunks <= 8 || (per_xcd >= 12 && 2 * per_xcd >= chunks)) ? 1 : 0;
}

template <int DHP, int VW>
void launch_pair(const PackArgs& p, const FragArgs& f, dim3 pgrid, int n_work, bool values_ready, hipStream_t s) {
    const ShortForm form = values_ready ? ShortForm::PAIR : short_form(f.dh, p.NRB, f.B, f.Hq, f.Hkv);
    if (form == ShortForm::HEAD) {
        hipLaunchKernelGGL((attention_short_kernel<DHP, VW>), dim3((unsigned)(f.B * f.Hq)), dim3(DHP * 4), 0, s, f);
        return;
    }
    if constexpr (DHP == ROWS_D && VW == 4) {             // heads of 128: never a workgroup per group
        if (form == ShortForm::ROWS) {
            const unsigned work = (unsigned)(f.B * f.Hkv * ((f.Hq / f.Hkv + 3) / 4));
            if (p.NRB == 2) hipLaunchKernelGGL(attention_rows_kernel<true>, dim3(2 * work), dim3(256), 0, s, f);
            else hipLaunchKernelGGL(attention_rows_kernel<false>, dim3(work), dim3(256), 0, s, f);
            return;
        }
    } else if (form == ShortForm::GROUP) {                // (NRB is 1: n_work counts the same workgroups)
        hipLaunchKernelGGL((attention_group_kernel<DHP, VW>), dim3((unsigned)n_work), dim3(512), 0, s, f);
        return;
    }
    if (values_ready) {
        const unsigned per_xcd = (unsigned)(((size_t)p.B * p.NRB * p.Hkv + 7) / 8);
        hipLaunchKernelGGL((attn_keys_kernel<DHP, VW>), dim3(8 * ((per_xcd + 3) / 4)), dim3(256), 0, s, p);
    } else {
        hipLaunchKernelGGL((attn_pack_kernel<DHP, VW>), pgrid, dim3(256), 0, s, p);
    }
    const dim3 agrid((unsigned)(8 * ((n_work + 7) / 8)));
    hipLaunchKernelGGL((attention_frag_kernel<DHP, VW, ATTN_WPG>), agrid, dim3(ATTN_WPG * 64), 0, s, f);
}

}  // namespace

int launch_attention_mfma(const float* qkv, int ld, int B, int S, const SeqMap& sm, int n_heads, int n_kv_heads,
                          int head_dim, const float* cos_t, const float* sin_t, void* frag_ws, float* out, hipStream_t s,
                         bool values_ready) {
    if (!attn_head_dim_ok(head_dim) || ld % 4 != 0) {
        set_error("attention: head_dim %d must be a multiple of 4 from 8 to 112, or of 8 up to 128 (row stride %d a multiple of 4)",
                  head_dim, ld);
        return BRL_EINVAL;
    }
    const int dhp = padded_head_dim(head_dim);
    const int nrb = (S + 31) / 32;
    const int group = n_heads / n_kv_heads;
    const int chunks = (group * nrb + ATTN_WPG - 1) / ATTN_WPG;
    PackArgs p;
    p.qkv = qkv; p.ld = ld; p.B = B; p.S = S; p.NRB = nrb; p.Hq = n_heads; p.Hkv = n_kv_heads; p.dh = head_dim;
    p.sm = sm;
    p.cos_t = cos_t; p.sin_t = sin_t;
    p.KVF = static_cast<uint4*>(frag_ws);
    p.by_xcd = pack_by_xcd(head_dim, attention_mfma_ws_bytes(B, S, n_heads, n_kv_heads, head_dim)) ? 1 : 0;
    FragArgs f;
    f.qkv = qkv; f.ld = ld; f.cos_t = cos_t; f.sin_t = sin_t;
    f.qscale = (float)(1.0 / sqrt((double)head_dim)) * 1.4426950408889634f;
    f.KVF = p.KVF; f.QF = nullptr; f.B = B; f.S = S; f.NRB = nrb; f.Hq = n_heads; f.Hkv = n_kv_heads; f.dh = head_dim;
    f.sm = sm;
    f.n_work = B * n_kv_heads * chunks;
    f.turn = chunk_turn(chunks, B * n_kv_heads);
    f.out = out;
    const dim3 pgrid((unsigned)(8 * (((size_t)B * nrb * n_kv_heads + 7) / 8)));
    const bool v4 = (head_dim / 2) % 4 == 0;          // rotary halves and head rows 16-byte aligned
    LaunchTimer tm(BRL_KC_ATTENTION, s);
    if (dhp == 32) {
        if (v4) launch_pair<32, 4>(p, f, pgrid, f.n_work, values_ready, s); else launch_pair<32, 2>(p, f, pgrid, f.n_work, values_ready, s);
    } else if (dhp == 64) {
        if (v4) launch_pair<64, 4>(p, f, pgrid, f.n_work, values_ready, s); else launch_pair<64, 2>(p, f, pgrid, f.n_work, values_ready, s);
    } else {
        if (v4) launch_pair<128, 4>(p, f, pgrid, f.n_work, values_ready, s); else launch_pair<128, 2>(p, f, pgrid, f.n_work, values_ready, s);
    }
    BRL_LAUNCH_CHECK("attention_mfma");
    return BRL_OK;
}

void attention_key_block(int head_dim, int& k_fragments, int& fragments) {
    const int dhp = padded_head_dim(head_dim);
    k_fragments = 2 * head_k_steps(head_dim);
    fragments = k_fragments + dhp / 8;                // two steps of 16 keys, hi and lo, for each 32 components
}

// The fragments (K / V and q) were written by the epilogue of the q | k | v product.
int launch_attention_mfma_prepacked(int B, int S, int n_heads, int n_kv_heads, const void* kvf, const void* qf, float* out,
                                    hipStream_t s) {
    constexpr int dh = 128;
    if (S % 32 != 0 || n_heads % n_kv_heads != 0) {
        set_error("attention: prepacked operands need 32 | S (S = %d) and whole head groups", S);
        return BRL_EINVAL;
    }
    const int nrb = S / 32;
    const int group = n_heads / n_kv_heads;
    const int chunks = (group * nrb + ATTN_WPG - 1) / ATTN_WPG;
    FragArgs f;
    f.qkv = nullptr; f.ld = 0; f.cos_t = nullptr; f.sin_t = nullptr;
    f.qscale = 0.f;
    f.KVF = static_cast<const uint4*>(kvf);
    f.QF = static_cast<const uint4*>(qf);
    f.B = B; f.S = S; f.NRB = nrb; f.Hq = n_heads; f.Hkv = n_kv_heads; f.dh = dh;
    f.sm.cu = nullptr; f.sm.b0 = 0;
    f.n_work = B * n_kv_heads * chunks;
    f.turn = chunk_turn(chunks, B * n_kv_heads);
    f.out = out;
    LaunchTimer tm(BRL_KC_ATTENTION, s);
    const dim3 agrid((unsigned)(8 * ((f.n_work + 7) / 8)));
    hipLaunchKernelGGL((attention_frag_kernel<128, 4, ATTN_WPG, true>), agrid, dim3(ATTN_WPG * 64), 0, s, f);
    BRL_LAUNCH_CHECK("attention_mfma (prepacked)");
    return BRL_OK;
}

}  // namespace brl
