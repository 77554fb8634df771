// Ternary x int8 GEMM on the gfx950 int8 matrix cores, fused dequant epilogue.
//
//   acc[m, n] = sum_k q[m, k] * code[n, k]                       (int32, exact)
//   y[m, n]   = (float(acc) * (a_m / 127)) * beta (+ residual)    (fp32, in that order)
//
// Both operands arrive in v_mfma_i32_32x32x32_i8 fragment order, so every load
// is a fully coalesced 1 KB wavefront read and no shuffles are needed:
//   * activations: tiled int8 buffer written by the quantisation kernel,
//   * weights: 2-bit packed blob; a lane's 32-bit word holds its 16 k-values for
//     one MFMA, as offset codes c = code + 1.  Four shift/and pairs expand it to
//     the 16-byte operand.  The MFMA therefore accumulates sum_k q * c, and the
//     epilogue subtracts sum_k q (from the quantisation kernel) to get acc.
// Integer sums are order independent, so the k-order inside a fragment only
// has to agree between the two operands - it does, by construction of the layouts.
// Int8 weights (the higher-precision critic variant) come in the activations' own
// fragment layout and feed the MFMA as they are: no expansion, no offset correction.
//
// Kernels:
//   gemm_lds_kernel    many tokens: both operand tiles of a workgroup (128 tokens
//                      x 128 k, and 256 or 128 weight rows x 128 k still packed)
//                      are staged in LDS with direct global->LDS loads, double
//                      buffered; in GLU mode the epilogue writes
//                      h = max(G,0)^2 U from interleaved gate / up blocks.
//                      Launches of up to 450 tiles of 128 x 128 put eight wavefronts
//                      of 64 x 32 on the tile.
//                      gemm_lds_attn_kernel is the wide tile on the q | k | v product of a
//                      uniform batch at head_dim 128: its epilogue rotates q and k and
//                      writes them and v as the fp16 hi / lo fragments the attention
//                      kernel reads (no fp32 rows, no pack kernel).
//                      gemm_lds_values_kernel writes v alone, other head sizes.
//                      gemm_lds_w8_kernel is the same loop on int8 weight blobs.
//   gemm_direct_kernel launches that would leave most compute units with one tile or
//                      none: no LDS staging, the 4 to 16 wavefronts of a workgroup
//                      split k and finish the tile together through LDS.
// launch_gemm picks among them by how many workgroups each would make.
#include <cstring>

#include "common.hpp"

namespace brl {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

struct GemmArgs {
    const uint4* A;          // tiled activations, 16 bytes per lane per fragment
    const float* dscale;
    const int32_t* sumq;
    const uint4* wp[3];      // packed weights per segment
    int wfrag;               // uint4 per (32-row block, 128-k super-block) of a weight blob: 64 (2-bit) or 256 (int8)
    const float* beta[3];
    int nb_end[3];
    int n_end[3];
    int nseg;
    int M, nmb, nnb, nsb;
    int tiles_m, tiles_n, group_m;
    float* y;
    int ldy;
    const float* residual;   // [M, ldy] fp32, or bf16 bit patterns when res_bf16 (widened exactly on load)
    int res_bf16;
    int32_t* acc_dbg;
    int fast_epilogue;       // every segment a multiple of 32 rows, ldy % 4 == 0, no debug tap
    double ops;              // int8 operations of the product (for the timing hooks)
    int glu;                 // 1: segments are (gate, up) of equal size, interleaved block by block;
                             //    the epilogue emits h = (max(G,0) * max(G,0)) * U, one column per pair
    // attention-operand epilogue (the q | k | v product of a uniform batch, head_dim 128): instead of fp32 rows the
    // kernel writes what the attention kernel reads - q and k rotated (q also scaled) as fp16 hi / lo MFMA fragments,
    // v transposed fragments - see epilogue_attn
    const float* att_cos;    // [S][64]
    const float* att_sin;
    float att_qscale;
    uint4* att_kvf;          // [B][Hkv][NRB][ K: [8][hi,lo] | V: [4][2][hi,lo] ][64 lanes]
    uint4* att_qf;           // [B][Hq][NRB][8][hi,lo][64 lanes]
    int att_S, att_nrb, att_Hq, att_Hkv;
    // value-operand epilogue (the same product at other head sizes): the column blocks from att_v0 on leave as v fragments
    // only, the others as fp32 rows - see epilogue_values
    int att_v0, att_dh, att_kfr, att_kvfr;   // head size, 1 KB fragments of k and of k and v in a key block
};

// residual element(s) at flat index o (o % 4 == 0 for the four-wide form)
__device__ inline float res_at(const GemmArgs& g, size_t o) {
    if (g.res_bf16) return __uint_as_float((uint32_t)reinterpret_cast<const uint16_t*>(g.residual)[o] << 16);
    return g.residual[o];
}
__device__ inline float4 res4_at(const GemmArgs& g, size_t o) {
    if (g.res_bf16) {
        const uint2 raw = *reinterpret_cast<const uint2*>(reinterpret_cast<const uint16_t*>(g.residual) + o);
        return make_float4(__uint_as_float(raw.x << 16), __uint_as_float(raw.x & 0xffff0000u),
                           __uint_as_float(raw.y << 16), __uint_as_float(raw.y & 0xffff0000u));
    }
    return *reinterpret_cast<const float4*>(g.residual + o);
}

__device__ inline v4i expand_codes(uint32_t p) {
    v4i r;
    r.x = (int)(p & 0x03030303u);
    r.y = (int)((p >> 2) & 0x03030303u);
    r.z = (int)((p >> 4) & 0x03030303u);
    r.w = (int)((p >> 6) & 0x03030303u);
    return r;
}

__device__ inline uint32_t pick(const uint4& v, int dd) {
    return dd == 0 ? v.x : dd == 1 ? v.y : dd == 2 ? v.z : v.w;
}

__device__ inline v4i as_v4i(const uint4& u) {
    v4i r;
    r.x = (int)u.x; r.y = (int)u.y; r.z = (int)u.z; r.w = (int)u.w;
    return r;
}

// XCD-aware tile order: workgroup w runs on XCD (w & 7); each XCD gets a
// contiguous run of tiles, walked in groups of `group_m` row tiles so that the
// tiles resident on one XCD share activation and weight panels in its L2.
__device__ inline bool tile_of_block(const GemmArgs& g, int& tile_m, int& tile_n) {
    const int total = g.tiles_m * g.tiles_n;
    const int per_xcd = (total + 7) / 8;
    const int T = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per_xcd || T >= total) return false;
    const int gsz = g.group_m * g.tiles_n;
    const int grp = T / gsz;
    const int first_m = grp * g.group_m;
    const int rows_in_grp = min(g.group_m, g.tiles_m - first_m);
    tile_m = first_m + (T - grp * gsz) % rows_in_grp;
    tile_n = (T - grp * gsz) / rows_in_grp;
    return true;
}

// Segment, first output column and number of valid columns of global weight block gnb.
// In GLU mode block 2 n is gate block n and block 2 n + 1 is up block n; both map to
// output columns 32 n ...
__device__ inline void block_columns(const GemmArgs& g, int gnb, int& seg, int& col0, int& ncols) {
    if (g.glu) {
        seg = gnb & 1;
        col0 = (gnb >> 1) * 32;
        ncols = gnb < g.nnb ? min(32, g.n_end[0] - col0) : 0;
        return;
    }
    int s = 0;
    if (g.nseg > 1 && gnb >= g.nb_end[0]) s = 1;
    if (g.nseg > 2 && gnb >= g.nb_end[1]) s = 2;
    const int nb_begin = s == 0 ? 0 : g.nb_end[s - 1];
    const int n_begin = s == 0 ? 0 : g.n_end[s - 1];
    seg = s;
    col0 = n_begin + (gnb - nb_begin) * 32;
    ncols = gnb < g.nnb ? min(32, g.n_end[s] - col0) : 0;
}

// Where the TN weight blocks of a wavefront live: segment, packed pointer, output columns.
template <int TN>
struct BCols {
    const uint4* ptr[TN];
    int seg[TN], col0[TN], ncols[TN];
    __device__ inline void init(const GemmArgs& g, int nb0, int lane) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int gnb = min(nb0 + j, g.nnb - 1);      // clamped blocks are computed but never stored
            int s, c0, nc;
            block_columns(g, gnb, s, c0, nc);
            const int lnb = g.glu ? (gnb >> 1) : gnb - (s == 0 ? 0 : g.nb_end[s - 1]);
            seg[j] = s;
            col0[j] = c0;
            ncols[j] = (nb0 + j < g.nnb) ? nc : 0;
            ptr[j] = g.wp[s] + (size_t)lnb * g.nsb * g.wfrag + lane;
        }
    }
};

// Epilogue.  In a 32x32 accumulator tile a lane holds column (lane & 31) and rows
// 8*(v/4) + 4*(lane/32) + v%4.  Each half token block of the wavefront (16 rows x
// TN*32 columns; accumulator registers v < 8 or v >= 8) is turned through a
// private LDS region into row-major order, so that the rescale reads 4
// consecutive columns of one row per lane and the result leaves as 16-byte
// stores (512-byte runs per row for TN = 4):
//     y = (float(acc - sum_q[m]) * dscale[m]) * beta[n] (+ residual)
// Tiles whose column blocks are all full take the 16-byte path (token rows past M are
// masked); tiles on the N edge (or with debug taps, or unaligned rows) take a compact
// per-element loop.
template <int TM, int TN>
struct Epi {
    static constexpr int W = TN * 32, LD = W + 4;
    static constexpr int ROWS = TM * 32;          // token rows of a wavefront: (dscale, sum_q) pairs parked after the turn area
    static constexpr int REGION = 16 * LD + 2 * ROWS;   // ints of LDS per wavefront
};

// accumulator registers half*8 .. half*8+7 of the TN tiles of token block i -> row-major 16 x TN*32 ints in scr
template <int TM, int TN>
__device__ inline void scatter_half(v16i (&acc)[TM][TN], int i, int half, int lane, int* scr) {
    constexpr int LD = Epi<TM, TN>::LD;
    const int cl = lane & 31, rh = (lane >> 5) * 4;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 8; ++v) scr[(8 * (v >> 2) + rh + (v & 3)) * LD + j * 32 + cl] = acc[i][j][half * 8 + v];
    __builtin_amdgcn_wave_barrier();
}

// The per-token scale and code sum of the wavefront's rows are fetched once (one row per lane)
// and parked in LDS behind the turn area, so that the passes below wait on LDS only.
template <int TM, int TN>
__device__ inline const int2* park_rows(const GemmArgs& g, int mb0, int lane, int* scr) {
    int2* rows = reinterpret_cast<int2*>(scr + 16 * Epi<TM, TN>::LD);
#pragma unroll
    for (int r = lane; r < TM * 32; r += 64) {
        const int m = min(mb0 * 32 + r, g.M - 1);
        rows[r] = make_int2(__float_as_int(g.dscale[m]), g.sumq ? g.sumq[m] : 0);   // no offset codes: nothing to subtract
    }
    return rows;
}

// h = (max(G,0) * max(G,0)) * U from the gate / up column pairs; 4 columns of one row per lane
template <int TM, int TN>
__device__ inline void epilogue_glu(const GemmArgs& g, v16i (&acc)[TM][TN], int mb0, int nb0, const float (&beta)[TN],
                                    int lane, int* scr) {
    constexpr int LD = Epi<TM, TN>::LD;
    constexpr int LPR = (TN / 2) * 8;            // lanes per row
    constexpr int RPP = 64 / LPR;
    constexpr int NP = 16 / RPP;                 // passes per half token block
    static_assert(64 % LPR == 0, "TN / 2 must be a power of two");
    const int cg = lane % LPR, r0 = lane / LPR;
    const int jj = cg >> 3, cc = 4 * (cg & 7);
    int row[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) row[p] = p * RPP + r0;
    float bg = beta[0], bu = beta[1];
#pragma unroll
    for (int q = 1; q < TN / 2; ++q)
        if (jj == q) { bg = beta[2 * q]; bu = beta[2 * q + 1]; }
    const int col = (nb0 / 2 + jj) * 32 + cc;
    const int2* rows = park_rows<TM, TN>(g, mb0, lane, scr);
#pragma unroll
    for (int idx = 0; idx < 2 * TM; ++idx) {
        const int mbase = (mb0 + (idx >> 1)) * 32 + (idx & 1) * 16;
        scatter_half<TM, TN>(acc, idx >> 1, idx & 1, lane, scr);
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int2 rw = rows[idx * 16 + row[p]];
            const float d = __int_as_float(rw.x);
            const int sq = rw.y;
            const int4 ga = *reinterpret_cast<const int4*>(&scr[row[p] * LD + (2 * jj) * 32 + cc]);
            const int4 ua = *reinterpret_cast<const int4*>(&scr[row[p] * LD + (2 * jj + 1) * 32 + cc]);
            const int gi[4] = {ga.x, ga.y, ga.z, ga.w}, ui[4] = {ua.x, ua.y, ua.z, ua.w};
            float hv[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float G = ((float)(gi[q] - sq) * d) * bg;
                const float U = ((float)(ui[q] - sq) * d) * bu;
                const float pz = fmaxf(G, 0.f);
                hv[q] = (pz * pz) * U;
            }
            if (mbase + row[p] < g.M)
                *reinterpret_cast<float4*>(g.y + (size_t)(mbase + row[p]) * g.ldy + col) =
                    make_float4(hv[0], hv[1], hv[2], hv[3]);
        }
        __builtin_amdgcn_sched_barrier(0);       // keeps the requests of later half blocks from piling up here
    }
}

// y = (float(acc - sum_q) * dscale) * beta (+ residual); 4 columns of one row per lane
template <int TM, int TN, bool RES>
__device__ inline void epilogue_plain(const GemmArgs& g, v16i (&acc)[TM][TN], int mb0, int nb0,
                                      const float (&beta)[TN], int lane, int* scr) {
    constexpr int LD = Epi<TM, TN>::LD;
    constexpr int LPR = TN * 8;
    constexpr int RPP = 64 / LPR;                // rows per pass (TN a power of two)
    constexpr int NP = 16 / RPP;
    static_assert(64 % LPR == 0, "TN must be a power of two");
    const int c4 = lane % LPR, r0 = lane / LPR;
    int row[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) row[p] = p * RPP + r0;
    float my_beta = beta[0];
#pragma unroll
    for (int j = 1; j < TN; ++j)
        if ((c4 >> 3) == j) my_beta = beta[j];
    const int col = nb0 * 32 + 4 * c4;
    const int2* rows = park_rows<TM, TN>(g, mb0, lane, scr);
#pragma unroll
    for (int idx = 0; idx < 2 * TM; ++idx) {
        const int mbase = (mb0 + (idx >> 1)) * 32 + (idx & 1) * 16;
        // the residual is requested before the LDS turn of this half block and used after it
        constexpr int NPRE = RES ? NP : 1;
        float4 res[NPRE];
        if constexpr (RES) {     // rows past M are clamped for the load and never stored
#pragma unroll
            for (int p = 0; p < NPRE; ++p)
                res[p] = res4_at(g, (size_t)min(mbase + row[p], g.M - 1) * g.ldy + col);
        }
        scatter_half<TM, TN>(acc, idx >> 1, idx & 1, lane, scr);
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int2 rw = rows[idx * 16 + row[p]];
            const float d = __int_as_float(rw.x);
            const int sq = rw.y;
            const int4 a = *reinterpret_cast<const int4*>(&scr[row[p] * LD + 4 * c4]);
            float4 val;
            val.x = ((float)(a.x - sq) * d) * my_beta;
            val.y = ((float)(a.y - sq) * d) * my_beta;
            val.z = ((float)(a.z - sq) * d) * my_beta;
            val.w = ((float)(a.w - sq) * d) * my_beta;
            if constexpr (RES) {
                const float4 r = res[p];
                val.x = val.x + r.x; val.y = val.y + r.y; val.z = val.z + r.z; val.w = val.w + r.w;
            }
            if (mbase + row[p] < g.M) *reinterpret_cast<float4*>(g.y + (size_t)(mbase + row[p]) * g.ldy + col) = val;
        }
        __builtin_amdgcn_sched_barrier(0);       // keeps the requests of later half blocks from piling up here
    }
}

template <int TM, int TN>
__device__ inline void epilogue(const GemmArgs& g, v16i (&acc)[TM][TN], int mb0, int nb0, const float (&beta)[TN],
                                int lane, int* scr) {
    constexpr int W = Epi<TM, TN>::W, LD = Epi<TM, TN>::LD;
    // full column blocks take the 16-byte paths (token rows past M are masked there)
    const bool interior = g.fast_epilogue && mb0 * 32 < g.M && nb0 + TN <= g.nnb;
    if (interior) {
        if (g.glu) {
            if constexpr (TN % 2 == 0) epilogue_glu<TM, TN>(g, acc, mb0, nb0, beta, lane, scr);
        } else if (g.residual) {
            epilogue_plain<TM, TN, true>(g, acc, mb0, nb0, beta, lane, scr);
        } else {
            epilogue_plain<TM, TN, false>(g, acc, mb0, nb0, beta, lane, scr);
        }
        return;
    }

    // tiles on the M / N edge, debug taps, unaligned rows: compact per-element loops
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        if (mb0 + i >= g.nmb) break;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int mbase = (mb0 + i) * 32 + half * 16;
            scatter_half<TM, TN>(acc, i, half, lane, scr);
            if (g.glu) {
#pragma unroll 1
                for (int e = lane; e < 16 * (W / 2); e += 64) {
                    const int row = e / (W / 2), c = e % (W / 2);
                    const int m = mbase + row;
                    const int jj = c >> 5, cc = c & 31;
                    int seg, col0, ncols;
                    block_columns(g, nb0 + 2 * jj, seg, col0, ncols);
                    if (m < g.M && cc < ncols) {
                        const int sq = g.sumq ? g.sumq[m] : 0;
                        const float d = g.dscale[m];
                        const float G = ((float)(scr[row * LD + (2 * jj) * 32 + cc] - sq) * d) * (*g.beta[0]);
                        const float U = ((float)(scr[row * LD + (2 * jj + 1) * 32 + cc] - sq) * d) * (*g.beta[1]);
                        const float pz = fmaxf(G, 0.f);
                        g.y[(size_t)m * g.ldy + col0 + cc] = (pz * pz) * U;
                    }
                }
            } else {
#pragma unroll 1
                for (int e = lane; e < 16 * W; e += 64) {
                    const int row = e / W, c = e % W;
                    const int m = mbase + row;
                    int seg, col0, ncols;
                    block_columns(g, nb0 + (c >> 5), seg, col0, ncols);
                    if (m < g.M && (c & 31) < ncols) {
                        const int a = scr[row * LD + c] - (g.sumq ? g.sumq[m] : 0);
                        const size_t o = (size_t)m * g.ldy + col0 + (c & 31);
                        float val = ((float)a * g.dscale[m]) * (*g.beta[seg]);
                        if (g.residual) val = val + res_at(g, o);
                        g.y[o] = val;
                        if (g.acc_dbg) g.acc_dbg[o] = a;
                    }
                }
            }
        }
    }
}

// Attention operands straight from the q | k | v product (head_dim 128, 32 | S, uniform layout).  A wavefront
// holds two 32-column blocks of one head: columns c .. c + 31 of its first half and the 32 columns 64 further
// on, the rotary partners of the first (the tile loop hands it the weight pieces in that order).  Both blocks
// of a half block of 16 rows are turned through the wavefront's own LDS region; a lane then has eight
// components of a row and their eight partners, rotates both, scales q, splits into fp16 hi / lo and stores
// four whole 16-byte fragment entries.  No other wavefront is involved.  The arithmetic per element is the one
// the separate pack kernel applies to the fp32 rows ((x c -+ x' s) * scale, then hi = fp16, lo = fp16(t - hi))
// on the same fp32 values the plain epilogue would have written, so the fragments hold the same bits.  v needs
// no turn: its transposed fragment order is the accumulator's own lane order.
typedef _Float16 half8 __attribute__((ext_vector_type(8)));

// fp32 -> fp16 of a value the compiler must first round to fp32: without the barrier it folds the last multiply
// into the conversion (v_fma_mixlo_f16, one rounding instead of two), and the hi part used for the lo part then
// differs, on ties, from the one that is stored - and from what the pack kernel makes of the fp32 rows in memory
__device__ inline _Float16 half_of_rounded(float x) {
    asm("" : "+v"(x));
    return (_Float16)x;
}

template <int TM, int TN>
__device__ inline void epilogue_attn(const GemmArgs& g, v16i (&acc)[TM][TN], int mb0, int nb0, const float (&beta)[TN],
                                     int lane, int* scr) {
    static_assert(TN == 2, "a block of a head's first half and the block of its rotary partners");
    constexpr int LD = Epi<TM, TN>::LD;
    constexpr int KS = 8, DB = 4, KVFR = KS * 2 + DB * 4;       // 1 KB fragments per key block at head_dim 128
    int seg, col0, ncols;
    block_columns(g, min(nb0, g.nnb - 1), seg, col0, ncols);
    const bool cols_live = nb0 < g.nnb;
    const int head_all = col0 >> 7;                             // head over q | k | v
    const int sub = (col0 >> 5) & 1;                            // which 32 columns of the head's first half
    const float bsel = beta[0];                                 // both blocks lie in one head, i.e. one matrix
    const int2* rows = park_rows<TM, TN>(g, mb0, lane, scr);
    __builtin_amdgcn_wave_barrier();

    if (seg == 2) {
        if (!cols_live) return;
        // v: lane (column dl of block j, h) holds the keys 16 tt + 8 (e >> 2) + 4 h + (e & 3) of step tt
        const int kvh = head_all - g.att_Hq - g.att_Hkv;
        const int dl = lane & 31, h = lane >> 5;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int mb = mb0 + i;
            if (mb >= g.nmb) continue;
            const int b = (mb * 32) / g.att_S, rb = ((mb * 32) % g.att_S) >> 5;
            uint4* dst = g.att_kvf + ((size_t)(b * g.att_Hkv + kvh) * g.att_nrb + rb) * (KVFR * 64);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int r = sub + 2 * j;                      // 32-column block of the head
#pragma unroll
                for (int tt = 0; tt < 2; ++tt) {
                    half8 hi, lo;
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int v = 8 * tt + e;
                        const int2 rw = rows[i * 32 + 8 * (v >> 2) + 4 * h + (v & 3)];
                        const float y = ((float)(acc[i][j][v] - rw.y) * __int_as_float(rw.x)) * bsel;
                        const _Float16 yh = half_of_rounded(y);
                        hi[e] = yh;
                        lo[e] = (_Float16)(y - (float)yh);
                    }
                    dst[(KS * 2 + (r * 2 + tt) * 2 + 0) * 64 + h * 32 + dl] = __builtin_bit_cast(uint4, hi);
                    dst[(KS * 2 + (r * 2 + tt) * 2 + 1) * 64 + h * 32 + dl] = __builtin_bit_cast(uint4, lo);
                }
            }
        }
        return;
    }
    if (!cols_live) return;

    // q and k: four lanes per row, eight components and their eight partners per lane; one pass per half block
    const int c8 = lane & 3, row = lane >> 2;                     // row of the half block
    const float scale = seg == 0 ? g.att_qscale : 1.0f;
    const int comp = sub * 32 + 8 * c8;                           // first of the lane's components of the first half
    const int ks = comp >> 4, kg = (comp >> 3) & 1;               // the partners are four k-steps on
#pragma unroll
    for (int idx = 0; idx < 2 * TM; ++idx) {
        const int mb = mb0 + (idx >> 1), hb = idx & 1;
        if (mb >= g.nmb) break;
        const int b = (mb * 32) / g.att_S, rb = ((mb * 32) % g.att_S) >> 5;
        // the rotary factors of the lane's row are requested before the turn
        const int pos = rb * 32 + hb * 16 + row;                  // position inside the state
        const float* cp = g.att_cos + (size_t)pos * 64 + comp;
        const float* sp = g.att_sin + (size_t)pos * 64 + comp;
        const float4 c0 = *reinterpret_cast<const float4*>(cp), c1 = *reinterpret_cast<const float4*>(cp + 4);
        const float4 s0 = *reinterpret_cast<const float4*>(sp), s1 = *reinterpret_cast<const float4*>(sp + 4);
        scatter_half<TM, TN>(acc, idx >> 1, hb, lane, scr);
        const int2 rw = rows[idx * 16 + row];
        const float d = __int_as_float(rw.x);
        const int sq = rw.y;
        const int4 a0 = *reinterpret_cast<const int4*>(&scr[row * LD + 8 * c8]);
        const int4 a1 = *reinterpret_cast<const int4*>(&scr[row * LD + 8 * c8 + 4]);
        const int4 p0 = *reinterpret_cast<const int4*>(&scr[row * LD + 32 + 8 * c8]);
        const int4 p1 = *reinterpret_cast<const int4*>(&scr[row * LD + 32 + 8 * c8 + 4]);
        const int ai[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
        const int pi[8] = {p0.x, p0.y, p0.z, p0.w, p1.x, p1.y, p1.z, p1.w};
        const float cf[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
        const float sf[8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
        half8 hi1, lo1, hi2, lo2;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const float x1 = ((float)(ai[q] - sq) * d) * bsel;    // component of the first half
            const float x2 = ((float)(pi[q] - sq) * d) * bsel;    // its partner, 64 components on
            const float t1 = (x1 * cf[q] - x2 * sf[q]) * scale;
            const float t2 = (x2 * cf[q] + x1 * sf[q]) * scale;
            const _Float16 h1 = half_of_rounded(t1), h2 = half_of_rounded(t2);
            hi1[q] = h1; lo1[q] = (_Float16)(t1 - (float)h1);
            hi2[q] = h2; lo2[q] = (_Float16)(t2 - (float)h2);
        }
        uint4* dst = seg == 0
            ? g.att_qf + ((size_t)(b * g.att_Hq + head_all) * g.att_nrb + rb) * (KS * 2 * 64)
            : g.att_kvf + ((size_t)(b * g.att_Hkv + (head_all - g.att_Hq)) * g.att_nrb + rb) * (KVFR * 64);
        uint4* slot = dst + (ks * 2) * 64 + kg * 32 + hb * 16 + row;
        slot[0] = __builtin_bit_cast(uint4, hi1);
        slot[64] = __builtin_bit_cast(uint4, lo1);               // the lo plane is the next 1 KB fragment
        slot[8 * 64] = __builtin_bit_cast(uint4, hi2);           // four k-steps = eight fragments on
        slot[9 * 64] = __builtin_bit_cast(uint4, lo2);
    }
}

// ---------------------------------------------------------------------------
// Many-token kernel: WM x WN wavefronts, each TM x TN tiles; both operands staged
// through LDS with direct global->LDS loads, double buffered.
// ---------------------------------------------------------------------------
template <int TM, int TN, int WM, int WN, bool W8>
struct LdsTile {
    static constexpr int NW = WM * WN;
    // k-steps (of 32) per stage: a whole super-block for the 2-bit weights; half of one for int8
    // weights, whose stage would otherwise be 32 KB and leave two wavefronts per SIMD
    static constexpr int KD = W8 ? 2 : 4;
    static constexpr int SPB = 4 / KD;                // stages per super-block
    static constexpr int AFR = WM * TM * KD;          // 1 KB activation fragments per stage
    static constexpr int BFR = WN * TN * (W8 ? KD : 1);   // 1 KB pieces of weights per stage: a packed 2-bit block, or
                                                      // the k-step fragments of an int8 block
    static constexpr int STAGE = (AFR + BFR) * 64;    // uint4 elements per stage
    static constexpr int APW = (AFR + NW - 1) / NW, BPW = (BFR + NW - 1) / NW;   // pieces copied per wavefront

    // Request stage t (k-steps t * KD ...) of this wavefront's share: piece c of wavefront w is
    // fragment c*NW + w (lane i's 16 bytes land at offset 16 i).
    static __device__ inline void issue(const uint4* const (&asrc)[APW], const uint4* const (&bsrc)[BPW], int t,
                                        uint4* st, int wave) {
#pragma unroll
        for (int c = 0; c < APW; ++c)
            if (AFR % NW == 0 || c * NW + wave < AFR)
                __builtin_amdgcn_global_load_lds(asrc[c] + (size_t)t * (KD * 64), st + (c * NW + wave) * 64, 16, 0, 0);
#pragma unroll
        for (int c = 0; c < BPW; ++c)
            if (BFR % NW == 0 || c * NW + wave < BFR)
                __builtin_amdgcn_global_load_lds(bsrc[c] + (size_t)t * (W8 ? KD * 64 : 64), st + (AFR + c * NW + wave) * 64,
                                                 16, 0, 0);
    }

    // The MFMAs of one stage.  Activation fragments are requested from LDS two uses before the
    // MFMAs that consume them.
    // p0: the wavefront's first weight piece of the tile; its TN pieces are p0, p0 + PSTR, ...
    template <int PSTR = 1>
    static __device__ inline void compute(v16i (&acc)[TM][TN], const uint4* st, int wm, int p0, int lane) {
        const uint4* sa = st + (wm * TM * KD) * 64 + lane;
        const uint4* sbp = st + (AFR + p0 * (W8 ? KD : 1)) * 64 + lane;
        uint4 bq[W8 ? 1 : TN];
        if constexpr (!W8) {
#pragma unroll
            for (int j = 0; j < TN; ++j) bq[j] = sbp[j * PSTR * 64];
        }
        constexpr int NF = KD * TM;
        uint4 fr[NF];
        fr[0] = sa[0];
        if (NF > 1) fr[1] = sa[(TM > 1 ? KD : 1) * 64];
#pragma unroll
        for (int dd = 0; dd < KD; ++dd) {
            v4i bf[TN];
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if constexpr (W8) bf[j] = as_v4i(sbp[(j * PSTR * KD + dd) * 64]);
                else bf[j] = expand_codes(pick(bq[j], dd));
            }
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int g = dd * TM + i;                       // use index of this fragment
                if (g + 2 < NF) {
                    const int g2 = g + 2, dd2 = g2 / TM, i2 = g2 % TM;
                    fr[g2] = sa[(i2 * KD + dd2) * 64];
                }
                const v4i af = as_v4i(fr[g]);
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af, bf[j], acc[i][j], 0, 0, 0);
            }
        }
        // Issue order.  Left to itself the compiler expands the codes of a k-step in one run between two batches of MFMAs, and
        // reads int8 fragments right before their use.  Here each MFMA is followed by its share of the next k-step's
        // expansion or by one read.  Ternary, wide tile, 8192 x 13824 x 2560 231.5 -> 230.7 us, 32768 x 17280 x 3200 1412 -> 1389
        // (the 128-wide tile spills under it: + 2.7 %); int8, 8192 x 3840 x 2560 106 -> 101, 8192 x 13824 x 2560 317 -> 314.
        if constexpr (W8) {
            __builtin_amdgcn_sched_group_barrier(SCHED_LDS_READ, 4, 0);
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                __builtin_amdgcn_sched_group_barrier(SCHED_MFMA, 1, 0);
                __builtin_amdgcn_sched_group_barrier(SCHED_LDS_READ, 1, 0);
            }
            __builtin_amdgcn_sched_group_barrier(SCHED_MFMA, 4, 0);
        } else if constexpr (NW == 8 && TM == 2 && TN == 2) {
            __builtin_amdgcn_sched_group_barrier(SCHED_LDS_READ, 4, 0);
            __builtin_amdgcn_sched_group_barrier(SCHED_VALU, 14, 0);         // the first k-step's codes: 7 per block
#pragma unroll
            for (int g = 0; g < 6; ++g) {
                __builtin_amdgcn_sched_group_barrier(SCHED_MFMA, 1, 0);
                __builtin_amdgcn_sched_group_barrier(SCHED_VALU, 4, 0);
                __builtin_amdgcn_sched_group_barrier(SCHED_LDS_READ, 1, 0);
                __builtin_amdgcn_sched_group_barrier(SCHED_MFMA, 1, 0);
                __builtin_amdgcn_sched_group_barrier(SCHED_VALU, 3, 0);
            }
            __builtin_amdgcn_sched_group_barrier(SCHED_MFMA, 4, 0);
        }
    }
    static constexpr int SCHED_VALU = 0x2, SCHED_MFMA = 0x8, SCHED_LDS_READ = 0x100;
};

// The value columns of the q | k | v product of a uniform batch (32 | S) as the attention kernel's v fragments, any head
// size: a lane's accumulator registers are eight keys of its column in the order of a fragment entry, twice, so nothing
// has to be turned, and a column's head and component only decide where the entries go.  Entries of components past the
// head are left as they are: they only reach output rows that no one stores.  The arithmetic is the plain epilogue's and
// the pack kernel's, so the fragments hold the same bits.
template <int TM, int TN>
__device__ inline void epilogue_values(const GemmArgs& g, v16i (&acc)[TM][TN], int mb0, int nb0, const float (&beta)[TN],
                                       int lane, int* scr) {
    const int2* rows = park_rows<TM, TN>(g, mb0, lane, scr);
    __builtin_amdgcn_wave_barrier();
    const int dl = lane & 31, h = lane >> 5;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        if (nb0 + j >= g.nnb) break;
        const int col = (nb0 + j - g.att_v0) * 32 + dl, kvh = col / g.att_dh, d = col - kvh * g.att_dh;
        const int at = (g.att_kfr + (d >> 5) * 4) * 64 + h * 32 + (d & 31);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int mb = mb0 + i;
            if (mb >= g.nmb) continue;
            const int b = (mb * 32) / g.att_S, rb = ((mb * 32) % g.att_S) >> 5;
            uint4* dst = g.att_kvf + ((size_t)(b * g.att_Hkv + kvh) * g.att_nrb + rb) * ((size_t)g.att_kvfr * 64) + at;
#pragma unroll
            for (int tt = 0; tt < 2; ++tt) {
                half8 hi, lo;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int v = 8 * tt + e;
                    const int2 rw = rows[i * 32 + 8 * (v >> 2) + 4 * h + (v & 3)];
                    const float y = ((float)(acc[i][j][v] - rw.y) * __int_as_float(rw.x)) * beta[j];
                    const _Float16 yh = half_of_rounded(y);
                    hi[e] = yh;
                    lo[e] = (_Float16)(y - (float)yh);
                }
                dst[tt * 128] = __builtin_bit_cast(uint4, hi);
                dst[tt * 128 + 64] = __builtin_bit_cast(uint4, lo);
            }
        }
    }
}

enum class LdsEpi { ROWS, ATTN, VALUES };

template <int TM, int TN, int WM, int WN, bool W8, LdsEpi EPI = LdsEpi::ROWS>
__device__ __forceinline__ void gemm_lds_body(const GemmArgs& g) {
    using Tile = LdsTile<TM, TN, WM, WN, W8>;
    constexpr int NW = Tile::NW;
    constexpr bool ATTN = EPI == LdsEpi::ATTN;
    __shared__ __attribute__((aligned(1024))) uint4 stage0[Tile::STAGE];
    __shared__ __attribute__((aligned(1024))) uint4 stage1[Tile::STAGE];

    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int wn = wave % WN, wm = wave / WN;
    int tile_m, tile_n;
    if (!tile_of_block(g, tile_m, tile_n)) return;

    const int mb_tile0 = tile_m * WM * TM;
    const int mb0 = mb_tile0 + wm * TM;
    const int nb_tile0 = tile_n * WN * TN;
    // weight blocks of the wavefront: TN neighbours, or (attention-operand epilogue) a 32-column block of a head's
    // first half and the block 64 columns on, which holds the rotary partners of its columns
    constexpr int PSTR = ATTN ? 2 : 1;
    const int p0 = ATTN ? (wn >> 1) * 4 + (wn & 1) : wn * TN;
    const int nb0 = nb_tile0 + p0;

    // sources of the stage pieces this wavefront copies (clamped: padding is never stored)
    const uint4* asrc[Tile::APW];
#pragma unroll
    for (int c = 0; c < Tile::APW; ++c) {
        const int f = c * NW + wave;                              // fragment = (token block, k-step of the stage)
        const int mb = min(mb_tile0 + f / Tile::KD, g.nmb - 1);
        asrc[c] = g.A + ((size_t)mb * g.nsb * 4 + f % Tile::KD) * 64 + lane;
    }
    const uint4* bsrc[Tile::BPW];
#pragma unroll
    for (int c = 0; c < Tile::BPW; ++c) {
        const int piece = c * NW + wave;
        BCols<1> one;
        one.init(g, nb_tile0 + (W8 ? piece / Tile::KD : piece), lane);
        bsrc[c] = one.ptr[0] + (W8 ? (piece % Tile::KD) * 64 : 0);
    }

    float beta[TN];
    {
        BCols<TN> bc;
        bc.init(g, nb0, lane);
#pragma unroll
        for (int j = 0; j < TN; ++j) beta[j] = *g.beta[bc.seg[j]];
    }

    v16i acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0;

    // Double buffering with two distinct LDS objects: while one is read, the
    // other is filled.  A stage requested in one step is waited for (vmcnt 0)
    // at the top of the next, so its latency hides behind 4*TM*TN MFMAs.
    const int sb_first = 0, sb_last = g.nsb * Tile::SPB;       // stages
    Tile::issue(asrc, bsrc, sb_first, stage0, wave);
    int sb = sb_first;
    for (; sb + 1 < sb_last; sb += 2) {
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        Tile::issue(asrc, bsrc, sb + 1, stage1, wave);
        __builtin_amdgcn_sched_barrier(0);       // the copy requests stay ahead of the MFMAs that hide them
        Tile::template compute<PSTR>(acc, stage0, wm, p0, lane);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (sb + 2 < sb_last) Tile::issue(asrc, bsrc, sb + 2, stage0, wave);
        __builtin_amdgcn_sched_barrier(0);
        Tile::template compute<PSTR>(acc, stage1, wm, p0, lane);
    }
    if (sb < sb_last) {
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        Tile::template compute<PSTR>(acc, stage0, wm, p0, lane);
    }

    // the stages are free once every wavefront has left the k loop: reuse them for the epilogue
    __syncthreads();
    static_assert((NW / 2) * Epi<TM, TN>::REGION * 4 <= Tile::STAGE * 16, "half of the epilogue regions per stage");
    int* scr = reinterpret_cast<int*>(wave < NW / 2 ? stage0 : stage1) + (wave % (NW / 2)) * Epi<TM, TN>::REGION;
    if constexpr (ATTN) {
        static_assert(WN == 4 && TN == 2, "a 256-column tile is two heads of 128: four wavefronts of 32 + 32 columns");
        epilogue_attn<TM, TN>(g, acc, mb0, nb0, beta, lane, scr);
    } else {
        if constexpr (EPI == LdsEpi::VALUES) {
            if (nb0 >= g.att_v0) {                    // (TN divides att_v0)
                epilogue_values<TM, TN>(g, acc, mb0, nb0, beta, lane, scr);
                return;
            }
        }
        epilogue<TM, TN>(g, acc, mb0, nb0, beta, lane, scr);
    }
}

template <int TM, int TN, int WM, int WN>
__global__ __launch_bounds__(WM * WN * 64, 4) void gemm_lds_kernel(GemmArgs g) {
    gemm_lds_body<TM, TN, WM, WN, false>(g);
}

// the wide tile with the attention-operand epilogue (q | k | v product).  Ternary, 8192 x 3840 x 2560: 82 us and 54 us of
// attention against 92 us, a pack kernel of 19 and 65 us; int8 weights 104 + 53 against 102 + 19 + 65.
template <bool W8>
__global__ __launch_bounds__(512, 4) void gemm_lds_attn_kernel(GemmArgs g) {
    gemm_lds_body<2, 2, 2, 4, W8, LdsEpi::ATTN>(g);
}

// the wide tile with the value-operand epilogue.  32768 tokens x 9600 x 3200, 32 heads of 100: 818 us and 220 of k fragments
// against 811 and a pack kernel of 411.
__global__ __launch_bounds__(512, 4) void gemm_lds_values_kernel(GemmArgs g) {
    gemm_lds_body<2, 2, 2, 4, false, LdsEpi::VALUES>(g);
}

// the same tile loop on int8 weight blobs
template <int TM, int TN, int WM, int WN>
__global__ __launch_bounds__(WM * WN * 64, 4) void gemm_lds_w8_kernel(GemmArgs g) {
    gemm_lds_body<TM, TN, WM, WN, true>(g);
}

// ---------------------------------------------------------------------------
// Few-token kernel: operands straight from L2 to registers; one TM x TN tile per workgroup, WK wavefronts split k.
// D super-blocks of k are in flight per wavefront: with one, each super-block of its share costs a memory latency.
// ---------------------------------------------------------------------------
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) u32x4* gptr16;

// Output item t of a TM x TN tile: E (four or one) consecutive columns of one token row.  `at` is its place in an
// accumulator block parked as [16 registers][64 lanes] (see the epilogues above).
template <int TM, int TN, int E>
struct DirectOut {
    int c, i, j0, m, at, seg, ncols;
    size_t off;
    bool in_tile;
    __device__ inline DirectOut(const GemmArgs& g, int t, int mb0, int nb0) {
        constexpr int IPB = 32 / E;                              // items per row of a 32-column block
        constexpr int GB = TN > 1 ? TN / 2 : 1;                  // output column blocks of the tile in GLU mode (TN otherwise)
        c = E * (t % IPB);
        const int jb = g.glu ? (t / IPB) % GB : (t / IPB) % TN, r = g.glu ? t / (IPB * GB) : t / (IPB * TN), rr = r & 31;
        i = r >> 5;
        j0 = g.glu ? 2 * jb : jb;
        m = mb0 * 32 + r;
        at = (4 * (rr >> 3) + (rr & 3)) * 64 + c + 32 * ((rr >> 2) & 1);
        in_tile = r < TM * 32 && nb0 + j0 < g.nnb;
        int col0;
        block_columns(g, min(nb0 + j0, g.nnb - 1), seg, col0, ncols);
        off = (size_t)m * g.ldy + col0 + c;
    }
    __device__ inline bool live(const GemmArgs& g) const { return in_tile && m < g.M && c < ncols; }
};

template <int TM, int TN, int WK, int D, int OCC, bool W8>
__global__ __launch_bounds__(WK * 64, OCC) void gemm_direct_kernel(GemmArgs g) {
    constexpr int NT = WK * 64;
    constexpr int BW = W8 ? 4 : 1;     // 16-byte weight pieces per lane, 32-row block and super-block
    constexpr int OUT = TM * TN * 1024;
    constexpr bool QUADS = OUT / NT >= 4;             // four columns per thread and pass, 16-byte stores
    constexpr int NP = QUADS ? OUT / NT / 4 : 1;      // passes of the main finishing form
    // What the finishing pass reads from memory is requested with the first loads where the launch is bound by latency
    // (the one-block tile: 0.5 us); held through the k loop it costs the larger tiles wavefronts (256 x 2560 x 6912: 1 us).
    constexpr bool EARLY = TM * TN == 1;
    typedef DirectOut<TM, TN, QUADS ? 4 : 1> Out;
    typedef DirectOut<TM, TN, 1> OutOne;
    static_assert(QUADS || OUT / NT == 1, "one item per thread");
    // One 32 x 32 block: every wavefront parks its part and the finishing threads add them up (64 KB of LDS, one barrier;
    // 0.3 us ahead of atomic adds there).  Larger tiles add into one copy, so that several workgroups fit a compute unit.
    constexpr bool PARK = TM * TN == 1;
    __shared__ __attribute__((aligned(16))) int red[(PARK ? WK : 1) * OUT];
    const int lane = threadIdx.x & 63;
    const int wk = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    int tile_m, tile_n;
    if (!tile_of_block(g, tile_m, tile_n)) return;
    if constexpr (!PARK) {
        for (int t = threadIdx.x; t < OUT; t += NT) red[t] = 0;
        __syncthreads();
    }

    const int mb0 = tile_m * TM, nb0 = tile_n * TN;
    gptr16 aptr[TM], bptr[TN];
    float beta[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) aptr[i] = (gptr16)g.A + (size_t)min(mb0 + i, g.nmb - 1) * g.nsb * 256;
    {
        BCols<TN> bc;
        bc.init(g, nb0, 0);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            bptr[j] = (gptr16)bc.ptr[j];
            beta[j] = *g.beta[bc.seg[j]];
        }
    }

    float early_d = 0.f, early_res = 0.f;
    int early_sq = 0;
    v16i acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0;

    auto request_outputs = [&] {
        OutOne o(g, (int)threadIdx.x, mb0, nb0);
        const int m = min(o.m, g.M - 1);
        early_d = g.dscale[m];
        early_sq = g.sumq ? g.sumq[m] : 0;
        if (g.residual && o.live(g)) early_res = res_at(g, o.off);
    };
    const int sb_begin = wk * g.nsb / WK, sb_end = (wk + 1) * g.nsb / WK;
    if (sb_begin < sb_end) {
        u32x4 aq[D][4][TM], bq[D][BW][TN];
        auto load = [&](int d, int sb) {
#pragma unroll
            for (int q = 0; q < BW; ++q)
#pragma unroll
                for (int j = 0; j < TN; ++j) bq[d][q][j] = bptr[j][(unsigned)((sb * BW + q) * 64 + lane)];
#pragma unroll
            for (int dd = 0; dd < 4; ++dd)
#pragma unroll
                for (int i = 0; i < TM; ++i) aq[d][dd][i] = aptr[i][(unsigned)((sb * 4 + dd) * 64 + lane)];
        };
        auto contract = [&](int d) {
#pragma unroll
            for (int dd = 0; dd < 4; ++dd) {
                v4i bf[TN];
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    if constexpr (W8) bf[j] = __builtin_bit_cast(v4i, bq[d][dd][j]);
                    else bf[j] = expand_codes(bq[d][0][j][dd]);
                }
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(__builtin_bit_cast(v4i, aq[d][dd][i]), bf[j],
                                                                          acc[i][j], 0, 0, 0);
            }
        };
#pragma unroll
        for (int d = 0; d < D; ++d) load(d, min(sb_begin + d, sb_end - 1));
        __builtin_amdgcn_sched_barrier(0);
        if (EARLY) request_outputs();
        __builtin_amdgcn_sched_barrier(0);
        int sb = sb_begin;
        for (; sb + 2 * D <= sb_end; sb += D)
#pragma unroll
            for (int d = 0; d < D; ++d) {
                contract(d);
                load(d, sb + d + D);
                __builtin_amdgcn_sched_barrier(0);
            }
        if (sb + D < sb_end) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                contract(d);
                load(d, min(sb + d + D, sb_end - 1));
                __builtin_amdgcn_sched_barrier(0);
            }
            sb += D;
        }
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (sb + d < sb_end) contract(d);
    } else if (EARLY) {
        request_outputs();
    }

    // The k-parts meet in LDS (integer sums: any order gives the same bits).
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                if constexpr (PARK) red[(wk * 16 + v) * 64 + lane] = acc[i][j][v];
                else atomicAdd(&red[((i * TN + j) * 16 + v) * 64 + lane], acc[i][j][v]);
            }
    __syncthreads();

    if (QUADS && g.fast_epilogue) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            Out o(g, (int)threadIdx.x + p * NT, mb0, nb0);
            if (!o.live(g)) continue;
            const float d = g.dscale[o.m];
            const int sq = g.sumq ? g.sumq[o.m] : 0;
            const int4 a0 = *reinterpret_cast<const int4*>(&red[(o.i * TN + o.j0) * 1024 + o.at]);
            float4 val;
            if (g.glu) {
                const int4 a1 = *reinterpret_cast<const int4*>(&red[(o.i * TN + (TN > 1 ? o.j0 + 1 : 0)) * 1024 + o.at]);
                const int gi[4] = {a0.x, a0.y, a0.z, a0.w}, ui[4] = {a1.x, a1.y, a1.z, a1.w};
                float hv[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float G = ((float)(gi[q] - sq) * d) * beta[0];
                    const float U = ((float)(ui[q] - sq) * d) * beta[TN > 1 ? 1 : 0];
                    const float pz = fmaxf(G, 0.f);
                    hv[q] = (pz * pz) * U;
                }
                val = make_float4(hv[0], hv[1], hv[2], hv[3]);
            } else {
                float bsel = beta[0];
#pragma unroll
                for (int j = 1; j < TN; ++j) bsel = o.j0 == j ? beta[j] : bsel;
                val.x = ((float)(a0.x - sq) * d) * bsel;
                val.y = ((float)(a0.y - sq) * d) * bsel;
                val.z = ((float)(a0.z - sq) * d) * bsel;
                val.w = ((float)(a0.w - sq) * d) * bsel;
                if (g.residual) {
                    const float4 res = res4_at(g, o.off);
                    val.x = val.x + res.x; val.y = val.y + res.y; val.z = val.z + res.z; val.w = val.w + res.w;
                }
            }
            *reinterpret_cast<float4*>(g.y + o.off) = val;
        }
        return;
    }
    // ragged columns, debug taps: an element per thread and pass; what four passes read from memory is requested together
    // (unconditionally: under the bounds test each would be waited for before the next)
    constexpr int P4 = OUT / NT < 4 ? OUT / NT : 4;
#pragma unroll 1
    for (int p0 = 0; p0 < OUT / NT; p0 += P4) {
        float dv[P4], rv[P4];
        int sv[P4];
#pragma unroll
        for (int p = 0; p < P4; ++p) {
            if constexpr (EARLY) {
                dv[p] = early_d; sv[p] = early_sq; rv[p] = early_res;
            } else {
                const OutOne o(g, (int)threadIdx.x + (p0 + p) * NT, mb0, nb0);
                const int m = min(o.m, g.M - 1);
                dv[p] = g.dscale[m];
                sv[p] = g.sumq ? g.sumq[m] : 0;
                rv[p] = g.residual ? res_at(g, o.live(g) ? o.off : 0) : 0.f;
            }
        }
#pragma unroll
        for (int p = 0; p < P4; ++p) {
            const OutOne o(g, (int)threadIdx.x + (p0 + p) * NT, mb0, nb0);
            if (!o.live(g)) continue;
            int a0 = -sv[p];
#pragma unroll
            for (int w = 0; w < (PARK ? WK : 1); ++w) a0 += red[w * OUT + (o.i * TN + o.j0) * 1024 + o.at];
            if (g.glu) {
                const float G = ((float)a0 * dv[p]) * beta[0];
                const float U = ((float)(red[(o.i * TN + (TN > 1 ? o.j0 + 1 : 0)) * 1024 + o.at] - sv[p]) * dv[p]) * beta[TN > 1 ? 1 : 0];
                const float pz = fmaxf(G, 0.f);
                g.y[o.off] = (pz * pz) * U;
            } else {
                float bsel = beta[0];
#pragma unroll
                for (int j = 1; j < TN; ++j) bsel = o.j0 == j ? beta[j] : bsel;
                float val = ((float)a0 * dv[p]) * bsel;
                if (g.residual) val = val + rv[p];
                g.y[o.off] = val;
                if (g.acc_dbg) g.acc_dbg[o.off] = a0;
            }
        }
    }
}

template <int TM, int TN, int WK, int D, int OCC, bool W8>
int launch_direct(GemmArgs& g, hipStream_t s) {
    g.tiles_m = (g.nmb + TM - 1) / TM;
    g.tiles_n = (g.nnb + TN - 1) / TN;
    g.group_m = 4;
    const int total = g.tiles_m * g.tiles_n;
    const int grid = ((total + 7) / 8) * 8;
    LaunchTimer tm(BRL_KC_GEMM_NARROW, s, g.ops);
    hipLaunchKernelGGL((gemm_direct_kernel<TM, TN, WK, D, OCC, W8>), dim3(grid), dim3(WK * 64), 0, s, g);
    BRL_LAUNCH_CHECK("gemm_direct_kernel");
    return BRL_OK;
}

template <int TM, int TN, int WM, int WN, bool W8>
int launch_lds(GemmArgs& g, hipStream_t s) {
    g.tiles_m = (g.nmb + WM * TM - 1) / (WM * TM);
    g.tiles_n = (g.nnb + WN * TN - 1) / (WN * TN);
    g.group_m = 4;
    const int total = g.tiles_m * g.tiles_n;
    const int grid = ((total + 7) / 8) * 8;
    LaunchTimer tm(WN * TN == 8 ? BRL_KC_GEMM : BRL_KC_GEMM_NARROW, s, g.ops);     // 256-column tiles are the wide class
    if constexpr (W8)
        hipLaunchKernelGGL((gemm_lds_w8_kernel<TM, TN, WM, WN>), dim3(grid), dim3(WM * WN * 64), 0, s, g);
    else
        hipLaunchKernelGGL((gemm_lds_kernel<TM, TN, WM, WN>), dim3(grid), dim3(WM * WN * 64), 0, s, g);
    BRL_LAUNCH_CHECK("gemm_lds_kernel");
    return BRL_OK;
}

}  // namespace

namespace {

int device_cus() {
    static const int cus = [] {        // initialised once, thread-safe
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) {
            (void)hipGetLastError();
            n = 256;
        }
        return n;
    }();
    return cus;
}

// would launch_gemm run this many-token product on the 128 x 256 tile?  (the rule at the end of launch_gemm)
bool wide_tile_chosen(int nmb, int nnb) {
    const int cus = device_cus();
    const long t_wide = (long)((nmb + 3) / 4) * ((nnb + 7) / 8);
    const long t_narrow = (long)((nmb + 3) / 4) * ((nnb + 3) / 4);
    const double fill_wide = (double)t_wide / (double)(((t_wide + cus - 1) / cus) * cus);
    const double fill_narrow = (double)t_narrow / (double)(((t_narrow + cus - 1) / cus) * cus);
    return t_wide >= 2 * cus && fill_wide >= 0.95 * fill_narrow;
}

// the q | k | v product on the wide tile
GemmArgs qkv_args(const ActBuf& a, const WeightSegs& w, int M, int K) {
    GemmArgs g;
    memset(&g, 0, sizeof(g));
    g.A = reinterpret_cast<const uint4*>(a.q);
    g.dscale = a.dscale;
    g.sumq = w.w8 ? nullptr : a.sumq;
    g.wfrag = w.w8 ? 256 : 64;
    g.nseg = 3;
    for (int i = 0; i < 3; ++i) {
        g.wp[i] = reinterpret_cast<const uint4*>(w.packed[i]);
        g.beta[i] = w.beta[i];
        g.nb_end[i] = w.nb_end[i];
        g.n_end[i] = w.n_end[i];
    }
    g.M = M;
    g.nmb = M / NB;
    g.nnb = w.nb_end[2];
    g.nsb = round_up(K, SBK) / SBK;
    g.ops = 2.0 * (double)M * (double)w.n_end[2] * (double)K;
    g.tiles_m = (g.nmb + 3) / 4;
    g.tiles_n = (g.nnb + 7) / 8;
    g.group_m = 4;
    return g;
}

}  // namespace

bool gemm_attn_eligible(int M, int n_heads, int n_kv_heads, int head_dim, int S) {
    const int N = (n_heads + 2 * n_kv_heads) * head_dim;
    return head_dim == 128 && S % 32 == 0 && M % 32 == 0 && M % S == 0 && N % 256 == 0 && wide_tile_chosen(M / 32, N / 32);
}

int launch_gemm_attn(const ActBuf& a, const WeightSegs& w, int M, int K, const AttnOperands& out, hipStream_t s) {
    if (w.count != 3 || !gemm_attn_eligible(M, out.n_heads, out.n_kv_heads, 128, out.S) ||
        w.n_end[0] != out.n_heads * 128 || w.n_end[1] - w.n_end[0] != out.n_kv_heads * 128 ||
        w.n_end[2] - w.n_end[1] != out.n_kv_heads * 128) {
        set_error("gemm: the attention-operand epilogue needs the q | k | v product of a uniform batch at head_dim 128");
        return BRL_EINVAL;
    }
    GemmArgs g = qkv_args(a, w, M, K);
    g.att_cos = out.cos_t; g.att_sin = out.sin_t; g.att_qscale = out.qscale;
    g.att_kvf = static_cast<uint4*>(out.kvf); g.att_qf = static_cast<uint4*>(out.qf);
    g.att_S = out.S; g.att_nrb = out.S / 32; g.att_Hq = out.n_heads; g.att_Hkv = out.n_kv_heads;
    LaunchTimer tm(BRL_KC_GEMM_QKV_ATTN, s, g.ops);
    const dim3 grid((unsigned)(((g.tiles_m * g.tiles_n + 7) / 8) * 8));
    if (w.w8) hipLaunchKernelGGL(gemm_lds_attn_kernel<true>, grid, dim3(512), 0, s, g);
    else hipLaunchKernelGGL(gemm_lds_attn_kernel<false>, grid, dim3(512), 0, s, g);
    BRL_LAUNCH_CHECK("gemm_lds_attn_kernel");
    return BRL_OK;
}

// Whole key blocks of a uniform batch and column blocks that are all k or all v, where the wide tile is the one to take.
// Encoders of four layers, width 1024, with / without (us): heads of 100, 8 states of 1024 tokens 2293 / 2499, 76 of 128 (8
// heads) 847 / 970; of 64, 512 states of 64 tokens 4055 / 4433, 128 of 128 (4 of 16 heads have values) 1069 / 1093; of 32, 64 of
// 128 tokens 720 / 758, 128 of 64 (8 of 32) 633 / 630; of 16, 64 of 128 tokens 864 / 957; 2 of 32 of 64, 128 states of 128
// tokens 1556 / 1547, 256 of 64 level.  Heads of 128: gemm_attn_eligible.  int8 weights: that kernel has not been built, they keep
// the pack kernel.
bool gemm_values_eligible(int M, int n_heads, int n_kv_heads, int head_dim, int S, int w8) {
    const int dq = n_heads * head_dim, dkv = n_kv_heads * head_dim;
    return !w8 && head_dim < 128 && S > 32 && S % 32 == 0 && M % S == 0 && dq % 32 == 0 && dkv % 32 == 0 &&
           (dq + dkv) % 64 == 0 && wide_tile_chosen(M / 32, (dq + 2 * dkv) / 32);
}

int launch_gemm_values(const ActBuf& a, const WeightSegs& w, int M, int K, float* y, int ldy, const ValueOperands& out,
                       hipStream_t s) {
    if (w.count != 3 || !gemm_values_eligible(M, out.n_heads, out.n_kv_heads, out.head_dim, out.S, w.w8) ||
        w.n_end[0] != out.n_heads * out.head_dim || w.n_end[1] - w.n_end[0] != out.n_kv_heads * out.head_dim ||
        w.n_end[2] - w.n_end[1] != out.n_kv_heads * out.head_dim) {
        set_error("gemm: the value-operand epilogue needs the q | k | v product of a uniform batch on the wide tile");
        return BRL_EINVAL;
    }
    GemmArgs g = qkv_args(a, w, M, K);
    g.y = y;
    g.ldy = ldy;
    g.fast_epilogue = ldy % 4 == 0 ? 1 : 0;
    g.att_kvf = static_cast<uint4*>(out.kvf);
    g.att_S = out.S; g.att_nrb = out.S / 32; g.att_Hq = out.n_heads; g.att_Hkv = out.n_kv_heads;
    g.att_v0 = w.nb_end[1];
    g.att_dh = out.head_dim; g.att_kfr = out.k_fragments; g.att_kvfr = out.fragments;
    LaunchTimer tm(BRL_KC_GEMM, s, g.ops);
    hipLaunchKernelGGL(gemm_lds_values_kernel, dim3((unsigned)(((g.tiles_m * g.tiles_n + 7) / 8) * 8)), dim3(512), 0, s, g);
    BRL_LAUNCH_CHECK("gemm_lds_values_kernel");
    return BRL_OK;
}

int launch_gemm(const ActBuf& a, const WeightSegs& w, int M, int N, int K, float* y, int ldy,
                const float* residual, int32_t* acc_dbg, int glu, hipStream_t s, int res_bf16) {
    GemmArgs g;
    memset(&g, 0, sizeof(g));
    g.A = reinterpret_cast<const uint4*>(a.q);
    g.dscale = a.dscale;
    g.sumq = w.w8 ? nullptr : a.sumq;
    g.wfrag = w.w8 ? 256 : 64;
    g.nseg = w.count;
    for (int i = 0; i < 3; ++i) {
        g.wp[i] = reinterpret_cast<const uint4*>(w.packed[i < w.count ? i : 0]);
        g.beta[i] = w.beta[i < w.count ? i : 0];
        g.nb_end[i] = w.nb_end[i < w.count ? i : w.count - 1];
        g.n_end[i] = w.n_end[i < w.count ? i : w.count - 1];
    }
    g.M = M;
    g.nmb = round_up(M, NB) / NB;
    g.nnb = w.nb_end[w.count - 1];
    g.glu = glu;
    if (glu) {
        if (w.count != 2 || w.n_end[1] != 2 * w.n_end[0] || residual || acc_dbg) {
            set_error("gemm: GLU mode needs two equal segments, no residual, no tap");
            return BRL_EINVAL;
        }
        g.nnb = 2 * w.nb_end[0];
    }
    g.nsb = round_up(K, SBK) / SBK;
    g.ops = 2.0 * (double)M * (double)w.n_end[w.count - 1] * (double)K;
    g.y = y;
    g.ldy = ldy;
    g.residual = residual;
    g.res_bf16 = residual ? res_bf16 : 0;
    g.acc_dbg = acc_dbg;
    g.fast_epilogue = (acc_dbg == nullptr && ldy % 4 == 0) ? 1 : 0;
    for (int i = 0; i < w.count; ++i)
        if ((w.n_end[i] - (i ? w.n_end[i - 1] : 0)) % 32 != 0) g.fast_epilogue = 0;
    (void)N;
    // Which kernel.  The LDS-staged tiles are ahead once every compute unit has about two of them; below that the
    // direct kernel's smaller tiles, with k over the wavefronts of a workgroup, spread the product evenly.  The limits
    // are counts of tiles, measured at 16 to 2560 tokens, K = 2560 and 6912, N = 2560 to 13824 (times in us, kernel
    // trace, weights from HBM; the tile named first is the one taken).
    const long n32 = (long)g.nmb * g.nnb;                              // 32 x 32
    const long n64 = (long)((g.nmb + 1) / 2) * ((g.nnb + 1) / 2);      // 64 x 64
    const long t_narrow = (long)((g.nmb + 3) / 4) * ((g.nnb + 3) / 4);
    if (w.w8) {
        // int8 blobs: four times the weight bytes, so square tiles earlier (N = 2560, K = 6912: 900 tokens 36 against 54
        // and 1750 tokens 54 against 74 for 128 x 128 tiles, K = 2560: 900 tokens 20 / 26, 1750 tokens 29.5 / 30.2); up to 1600 of
        // them where k is long: 1700 x 2560 of K = 2560 35.0 (128 x 128) / 35.1, 4096 49.2 / 46.0, 9216 104 / 96.7
        if (n32 <= 256 && !glu) return launch_direct<1, 1, 16, 1, 4, true>(g, s);
        if (g.nmb <= 1 || (glu && n32 <= 1024)) return launch_direct<1, 2, 8, 1, 4, true>(g, s);
        if (!glu && (long)((g.nmb + 1) / 2) * g.nnb <= 700) return launch_direct<2, 1, 8, 1, 4, true>(g, s);
        if (n64 <= (g.nsb >= 32 ? 1600 : 1000)) return launch_direct<2, 2, 4, 1, 3, true>(g, s);
        // 128 x 256 tiles, two to a compute unit, or 128 x 128, four to one, whose last round ends sooner.  Wide / narrow in us,
        // quantisation included, 290 shapes in graphs:
        // - the fullest compute unit must not have more to do: 5000 x 2560 x 2560 (2 wide or 4 narrow tiles) 57.3 / 61.7, 8192 x 2048 x
        //   2560 (2, 4) 68.9 / 71.6, 8192 x 3840 x 2560 (4, 8) 112 / 117; but 4096 x 3072 x 2560 (2, 3) 55.0 / 51.9, 6144 x 2048 x 2560 (2,
        //   3) 58.3 / 55.4, 6144 x 3072 x 2560 (3, 5) 81.5 / 77.7;
        // - the last round three quarters full: 7040 x 6624 x 2560 (2.8) 1.02; 8320 x 9152 x 2560 (4.6) 0.995, 4096 x 6592 x 1024 (1.6)
        //   0.96.  But past the first round not all but full (more than nine tenths of it, whole rounds apart): many of those lose, why
        //   is not known (11684 x 2697 x 2888 (1.98) 215 / 196, 3782 x 12803 x 3960 (2.99) 343 / 316, 7330 x 8761 x 1528 (3.96) 276 /
        //   255; 21199 x 1522 x 3744 (1.95) 271 / 282; 44 of them 0.988, 0.91 to 1.04, the 621 others that take the wide tile 1.025,
        //   0.95 to 1.11).  Not so from 32 super-blocks of k on (28 of them 1.024, 0.95 to 1.08) and for gate|up (1094 layers 1.00 to 1.01, 0.97 to 1.03);
        // - from six rounds on neither matters for gate|up or long k (1.01 to 1.04; 6.06 of them at 12032 x 8320: K = 4096 level, 2560 349 /
        //   334), from seven on down to K = 2560 (9600 x 12864 1.02, 12544 x 11008 1.01, 24576 x 9600 of 3200 1.02; 29312 x 4352 0.99);
        // - k not short past the first round: 4864 x 13568 (3.9) of K = 1024 104 / 105, 1536 139.5 / 144; 20184 x 4032 (4.9) 157 / 152, 197 /
        //   202; 7680 x 12928 (6.0) 163 / 160, 212 / 212 (gate|up 16384 x 8192 of K = 1024 still 1.02);
        // - next to no tiles of padding (one in 55 at 2048 x 7008 x 6912: 1.07, one in 75 at N = 9600: 932 / 954; one in 25 at N = 3200: 4096 tokens
        //   60.6 / 59.7, 9000 132 / 129; the worst let through: 1024 x 12928 x 1024 0.965; N = 128, all of them double: 49152 tokens 173 / 160; N = 640, 16384 tokens 81 / 71).
        const long t_wide = (long)((g.nmb + 3) / 4) * ((g.nnb + 7) / 8), cus = device_cus(), slots = 2 * cus;
        const bool padded = 50 * (2 * t_wide - t_narrow) > t_narrow;
        const bool level = 2 * ((t_wide + cus - 1) / cus) <= (t_narrow + cus - 1) / cus;
        const bool brim = !glu && t_wide > slots && g.nsb < 32 && 10 * (t_wide % slots) > 9 * slots;
        const bool full_round = (4 * (t_wide % slots) >= 3 * slots && !brim) || t_wide % slots == 0;
        const bool many = t_wide >= (glu || g.nsb >= 32 ? 6 : 7) * slots && (glu || g.nsb >= 20);
        if (!padded && (many || (level && full_round && (t_wide <= slots || glu || g.nsb >= 12))))
            return launch_lds<2, 2, 2, 4, true>(g, s);
        return launch_lds<2, 2, 2, 2, true>(g, s);                     // 16 KB per stage
    }
    const long n32x64 = (long)g.nmb * ((g.nnb + 1) / 2);
    if (glu) {
        // (a wavefront needs the gate and the up block of a column pair: even TN only.)  2 x 6912 x 2560, tokens: 27:
        // 5.5 / 6.2 for four column blocks; 128: 10 / 15 for 128 x 128 tiles; 256: 14.5 / 15.5; 700: 28.9 / 30.9.  A wide
        // tile per compute unit on nearly all of them is better than either: 512 tokens (216 tiles) 20.2 / 21.5, 900
        // tokens (432) 34.8 / 36.6; on 63 % of them (700 tokens) 33.
        const long cus = device_cus();
        const long t_wide = (long)((g.nmb + 3) / 4) * ((g.nnb + 7) / 8);
        const bool wide_even = 5 * t_wide >= 4 * ((t_wide + cus - 1) / cus) * cus;
        if (n32x64 <= 512) return launch_direct<1, 2, 4, 2, 4, false>(g, s);
        if (wide_even) return launch_lds<2, 2, 2, 4, false>(g, s);
        if (n32x64 <= 6000) return launch_direct<1, 4, 4, 1, 4, false>(g, s);
    } else {
        // tokens x N x K: 27 x 2560 x 6912 7.1 / 7.7 for 32 x 64; 128 x 2560 x 2560 6.1 (32 x 64) / 6.8; 512 x 2560 x 6912
        // 15.1 / 17.7 for 64 x 32; 900: 22 / 32 and 1750: 37 / 44 for 128 x 128, 2560: 52.6 / 48.4.  Four wavefronts
        // instead of eight once there are enough workgroups and k is short: 1750 x 2560 x 2560 20.1 / 21.6 (22.6 for 128 x
        // 128), 1300 x 3840 x 2560 21.5 / 23.5 (22.9), 1750 x 3840 x 2560 26.3 / 29 (24.8).
        // (k short: 1300 x 2560 of K = 1024 16.4 with four / 19.2 with eight, 2560 22.6 / 24.9, 4096 30.2 / 31.9; from 5120 on
        // eight is level or ahead: 37.4 / 37.8, 1000 x 4096 of 5120 37.0 / 36.5, of 9216 59.2 / 57.0)
        // (ragged columns finish element by element: one per thread there, 817 x 606 x 3200 13.4 / 15.9)
        if (n32 <= (g.fast_epilogue ? 256 : 512)) return launch_direct<1, 1, 16, 1, 4, false>(g, s);
        if (n32x64 <= (g.nsb >= 40 ? 2500 : 960)) return launch_direct<1, 2, 8, 1, 4, false>(g, s);
        if (n32x64 <= 2500) return launch_direct<1, 2, 4, 1, 4, false>(g, s);
        // up to 450 tiles of 128 x 128: eight wavefronts of 64 x 32 on a tile (two per SIMD from one workgroup) instead of
        // four of 64 x 64: 1750 x 3840 x 2560 (420 tiles) 24.8 / 26.4, 2560 x 2560 x 2560 (400) 25.0 / 27.0; 600 tiles 38 / 34
        if (t_narrow <= 450) return launch_lds<2, 1, 2, 4, false>(g, s);
    }
    // 128 x 256 workgroup tiles (8 wavefronts of 64 x 64, two workgroups per CU) or 128 x 128 tiles
    // (4 wavefronts, four per CU).  The wide tile does about 5 % more work per unit time; the narrow
    // one wins when it spreads the tiles more evenly over the compute units.
    if (wide_tile_chosen(g.nmb, g.nnb)) return launch_lds<2, 2, 2, 4, false>(g, s);
    return launch_lds<2, 2, 2, 2, false>(g, s);
}

}  // namespace brl
