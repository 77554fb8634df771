// The part that the two weight quantisers share: reading 32 rows x 512 columns of fp32 masters coalesced and
// leaving the codes in the order of the packed blobs, through LDS.
//
// A workgroup of four wavefronts takes one 32-row block and four super-blocks of 128 columns.  A wavefront's load
// covers two rows x 128 columns (32 lanes x 16 bytes of a row), sixteen of them in flight; the codes are turned
// through LDS into the blob's order and leave as whole 1 KB pieces.  Reading one 16-column word per thread instead
// (64 rows of a wavefront, four bytes at a time) took 65 us for 6912 x 2560; this takes 19 us, 70.8 MB out of the
// last-level cache that the preceding statistics pass has filled.
#pragma once

#include "common.hpp"

namespace brl {

constexpr int PACK_THREADS = 256;
constexpr int PACK_SB = 4;                       // super-blocks per workgroup, one per wavefront on the way out
typedef float pack_f4 __attribute__((ext_vector_type(4), aligned(4)));      // rows start anywhere

inline dim3 pack_grid(int N, int K) {
    const int nsb = round_up(K, SBK) / SBK;
    return dim3((unsigned)((nsb + PACK_SB - 1) / PACK_SB), (unsigned)(round_up(N, NB) / NB));
}

// v[s][p]: columns k .. k + 3 of super-block s, row p of this lane (pack_row, pack_col); zeros outside the matrix
__device__ inline int pack_row(int p) { return (int)(threadIdx.x >> 6) * 8 + 2 * p + (int)((threadIdx.x & 63) >> 5); }
__device__ inline int pack_col() { return 4 * (int)(threadIdx.x & 31); }
__device__ inline void pack_load(const float* __restrict__ W, int N, int K, pack_f4 (&v)[PACK_SB][4]) {
    const int nb = blockIdx.y, sb0 = blockIdx.x * PACK_SB;
#pragma unroll
    for (int s = 0; s < PACK_SB; ++s)
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int n = nb * NB + pack_row(p), k = (sb0 + s) * SBK + pack_col();
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
