// The part that the two weight quantisers share: reading 32 rows x 512 columns of fp32 masters coalesced and
// leaving the codes in the order of the packed blobs, through LDS.
//
// A workgroup of four wavefronts takes one 32-row block and four super-blocks of 128 columns.  A wavefront's load
// covers two rows x 128 columns (32 lanes x 16 bytes of a row), sixteen of them in flight; the codes are turned
// through LDS into the blob's order and leave as whole 1 KB pieces.  Reading one 16-column word per thread instead
// (64 rows of a wavefront, four bytes at a time) took 65 us for 6912 x 2560; this takes 19 us, 70.8 MB out of the
// last-level cache that the preceding statistics pass has filled.
// Of matrices narrower than four super-blocks (NARROW) a workgroup takes the next four of the blob wherever they lie, so
// that it is full: 200000 x 16 38 us with the statistics pass, 60 without, 50000 x 128 29 and 37.  The same for every width
// costs a wavefront per SIMD (four places to keep instead of one): 6912 x 2560 and its like 1 us.
#pragma once

#include "common.hpp"

namespace brl {

constexpr int PACK_THREADS = 256;
constexpr int PACK_SB = 4;                       // super-blocks per workgroup, one per wavefront on the way out
typedef float pack_f4 __attribute__((ext_vector_type(4), aligned(4)));      // rows start anywhere

inline bool pack_narrow(int K) { return K <= (PACK_SB - 1) * SBK; }
// one dimension: a matrix may have more row blocks than a second one has room for
inline dim3 pack_grid(int N, int K) {
    const long nsb = round_up(K, SBK) / SBK, blocks = (N - 1) / NB + 1;
    return dim3((unsigned)(pack_narrow(K) ? (blocks * nsb + PACK_SB - 1) / PACK_SB : blocks * ((nsb + PACK_SB - 1) / PACK_SB)));
}

// Where the workgroup's super-blocks lie: first row and column, and place in the blob of the one a wavefront writes.
template <bool NARROW>
struct PackPlace {
    int n0[NARROW ? PACK_SB : 1], k0[NARROW ? PACK_SB : 1], nsb;
    __device__ explicit PackPlace(int nsb_) : nsb(nsb_) {
        if constexpr (NARROW) {
#pragma unroll
            for (int s = 0; s < PACK_SB; ++s) {
                const int u = (int)blockIdx.x * PACK_SB + s;
                n0[s] = u / nsb * NB;
                k0[s] = u % nsb * SBK;
            }
        } else {
            const int per_row = (nsb + PACK_SB - 1) / PACK_SB;
            n0[0] = (int)blockIdx.x / per_row * NB;
            k0[0] = (int)blockIdx.x % per_row * (PACK_SB * SBK);
        }
    }
    __device__ int row0(int s) const { return n0[NARROW ? s : 0]; }
    __device__ int col0(int s) const { return NARROW ? k0[NARROW ? s : 0] : k0[0] + s * SBK; }
    // (those past the last one lie below the last row or right of the last column)
    __device__ bool wave_writes(int wave, int N) const {
        if constexpr (NARROW) return (int)blockIdx.x * PACK_SB + wave < (N + NB - 1) / NB * nsb;
        else return k0[0] / SBK + wave < nsb;
    }
    __device__ size_t blob(int wave) const {
        if constexpr (NARROW) return (size_t)blockIdx.x * PACK_SB + wave;
        else return (size_t)(n0[0] / NB) * nsb + k0[0] / SBK + wave;
    }
};

// v[s][p]: columns k .. k + 3 of super-block s, row p of this lane (pack_row, pack_col); zeros outside the matrix
__device__ inline int pack_row(int p) { return (int)(threadIdx.x >> 6) * 8 + 2 * p + (int)((threadIdx.x & 63) >> 5); }
__device__ inline int pack_col() { return 4 * (int)(threadIdx.x & 31); }
template <bool NARROW>
__device__ inline void pack_load(const float* __restrict__ W, int N, int K, const PackPlace<NARROW>& at, pack_f4 (&v)[PACK_SB][4]) {
#pragma unroll
    for (int s = 0; s < PACK_SB; ++s)
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int n = at.row0(s) + pack_row(p), k = at.col0(s) + pack_col();
            pack_f4 x = {0.f, 0.f, 0.f, 0.f};
            if (n < N && k + 4 <= K) {
                x = *reinterpret_cast<const pack_f4*>(W + (size_t)n * K + k);
            } else if (n < N) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (k + e < K) x[e] = W[(size_t)n * K + k + e];
            }
            v[s][p] = x;
        }
}

// optional tap: four plain codes of one row
__device__ inline void pack_tap(int8_t* __restrict__ codes, int n, int k, int N, int K, const int (&c)[4]) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (n < N && k + e < K) codes[(size_t)n * K + k + e] = (int8_t)c[e];
}

}  // namespace brl
