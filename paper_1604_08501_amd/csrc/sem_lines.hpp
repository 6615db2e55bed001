// Line transforms on the matrix cores.
//
// Applying D along a direction node by node costs every output Nq reads of
// the staged fluxes and Nq reads of D.  Here the staged flux arrays of a tile
// are transformed line by line instead, in place: a wave reads a line's Nq
// values once, multiplies them by D on the matrix cores (D sits in a few
// registers per lane) and writes the Nq results over them.  Per node and flux
// that is one read and one write, whatever Nq, and D takes no LDS bandwidth.
// On gfx950 an LDS read moves 256 bytes a cycle and a write 128, so a
// transformed flux costs an LDS cycle count of about 12 per 64 nodes and
// direction in FP64 against 20 and the reads of D (Nq = 8).
#pragma once
#include "sem_device.hpp"

namespace semk {

// LDS layout of one staged array (one field of one element) at Nq = 8 in
// FP64: the word of node (i, j, k).  The low bits are permuted by an XOR of
// index bits (pos is linear over bits), so that every access of a wave
// touches each bank once: nodes in order, and 16 lines by 4 nodes along r, s
// or t, reads in groups of 32 lanes (64 banks) and writes in groups of 16
// (32 banks).  In node order the r lines' writes take eight times as long.
struct LineLds {
    static constexpr int WORDS = 512;
    static __device__ __forceinline__ constexpr int pos(int i, int j, int k)
    {
        return 64 * k + 8 * (j ^ (3 * (k & 1))) + (i ^ ((j >> 1) & 3) ^ (4 * (k & 1)));
    }
};

// Applies D along t to NARR consecutive staged arrays, in place; the caller's
// wave takes the arrays first, first + STEP, ...
// v_mfma_f64_4x4x4 multiplies four 4x4 blocks at once.  Lane l holds row l % 4,
// column l / 16 of the left operand, and row l / 16 of column l % 16 (16 lines
// side by side) of the right operand and of the result.
template <int NARR, int STEP>
__device__ __forceinline__ void transform_t_lines(const double* __restrict__ sD,
                                                  double* __restrict__ sF, int first)
{
    constexpr int NG = 4;   // groups of 16 lines per array
    const int l = threadIdx.x & 63;
    const int c = l & 15, kk = l >> 4;
    double a[2][2];
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
            a[rt][kt] = sD[(4 * rt + (l & 3)) * 8 + 4 * kt + kk];
    int off[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g)
        off[g] = LineLds::pos(c & 7, 2 * g + (c >> 3), kk);
    constexpr int HALF = LineLds::pos(0, 0, 4);   // from node kk to node 4 + kk of a line
#pragma unroll 1
    for (int x = first; x < NARR; x += STEP) {
        double* __restrict__ F = sF + x * LineLds::WORDS;
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const double b0 = F[off[g]], b1 = F[off[g] ^ HALF];
            double r[2];
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) {
                r[rt] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[rt][0], b0, 0.0, 0, 0, 0);
                r[rt] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[rt][1], b1, r[rt], 0, 0, 0);
            }
            F[off[g]] = r[0];
            F[off[g] ^ HALF] = r[1];
        }
    }
}

}  // namespace semk
