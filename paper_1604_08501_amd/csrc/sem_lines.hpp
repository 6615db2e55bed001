// Line transforms on the matrix cores.
//
// Applying D along a direction node by node costs every output Nq reads of
// the staged fluxes and Nq reads of D.  Here the staged flux arrays of a tile
// are transformed line by line instead, in place: a wave reads a line's Nq
// values once, multiplies them by D on the matrix cores (D sits in a few
// registers per lane) and writes the Nq results over them.  Per node and flux
// that is one read and one write, whatever Nq, and D takes no LDS bandwidth.
// FP64 products run on the FP64 vector units' hardware, at their rate (64
// TFLOP/s measured for the 4x4x4 shape), so they save LDS traffic and
// instructions, not multiplications; FP32 ones run at twice the scalar rate.
#pragma once
#include "sem_device.hpp"
#include "sem_pow.hpp"

namespace semk {

typedef float float4_t __attribute__((ext_vector_type(4)));

// LDS layout of one staged array (one field of one element): the word of
// node (i, j, k), and the number of words.
//   FP64, Nq = 8: the low bits are permuted by an XOR of index bits (pos is
//   linear over bits), so that every access of a wave touches each bank once:
//   nodes in order, and 16 lines by 4 nodes along r, s or t, reads in groups of
//   32 lanes (64 banks) and writes in groups of 16 (32 banks).  In node order
//   the r lines' writes take eight times as long.
//   FP64, otherwise: node order.
//   FP32: rows padded to an odd length, so that lanes on consecutive rows (the
//   r lines) start in different banks, and at Nq = 8 those of the s lines too.
//   64 lanes on consecutive nodes then span more than the 64 banks, so accesses
//   in node order and of the t lines take twice their cycles at Nq = 6 and 8 (the
//   s lines at 6 and 9): most of the conflict cycles that the counters show for
//   the FP32 line and v + s tiles.  Unpadded, the r lines of Nq = 8 would take
//   eight times theirs.
// The v + s and surface tiles also conflict where boundary nodes stage and
// gather face values: at Nq = 8 the nodes of faces r- and r+ (s- and s+) at the
// same place of either face lie in the same banks, two lanes to each.
template <typename T, int NQ>
struct LineLds {
    static constexpr bool XOR = sizeof(T) == 8 && NQ == 8;
    static constexpr int P1 = sizeof(T) == 4 ? (NQ | 1) : NQ;
    static constexpr int P2 = P1 * NQ;
    static constexpr int WORDS = P2 * NQ;
    static __device__ __forceinline__ constexpr int pos(int i, int j, int k)
    {
        if constexpr (XOR)
            return 64 * k + 8 * (j ^ (3 * (k & 1))) + (i ^ ((j >> 1) & 3) ^ (4 * (k & 1)));
        else
            return i + P1 * j + P2 * k;
    }
    // word of position n of line (u, v) along direction d: r lines (j, k),
    // s lines (i, k), t lines (i, j)
    static __device__ __forceinline__ constexpr int line_pos(int d, int u, int v, int n)
    {
        return d == 0 ? pos(n, u, v) : (d == 1 ? pos(u, n, v) : pos(u, v, n));
    }
};

// D in the operand layout of the matrix product, one copy per wave.
template <typename T, int NQ>
struct LineD;

// FP64: v_mfma_f64_4x4x4 multiplies four 4x4 blocks at once.  Lane l holds
// row l % 4, column l / 16 of the left operand (D, padded by zeros to whole
// blocks), and row l / 16 of column l % 16 (16 lines side by side) of the
// right operand and of the result.
template <int NQ>
struct LineD<double, NQ> {
    static constexpr int KT = (NQ + 3) / 4;
    static constexpr int PER = 16;   // lines at a time
    double a[KT][KT];
    __device__ __forceinline__ void load(const double* __restrict__ D)
    {
        const int l = threadIdx.x & 63;
#pragma unroll
        for (int rt = 0; rt < KT; ++rt)
#pragma unroll
            for (int kt = 0; kt < KT; ++kt) {
                const int row = 4 * rt + (l & 3), col = 4 * kt + (l >> 4);
                a[rt][kt] = row < NQ && col < NQ ? D[row * NQ + col] : 0.0;
            }
    }
    // D applied to this lane's line, whose node n is F[n * STEP], in place
    template <int STEP>
    __device__ __forceinline__ void apply(double* __restrict__ F, bool live) const
    {
        const int kk = (threadIdx.x & 63) >> 4;
        double b[KT], r[KT];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)   // nodes past the line enter as zeros
            b[kt] = 4 * kt + 3 < NQ || 4 * kt + kk < NQ ? F[(4 * kt + kk) * STEP] : 0.0;
#pragma unroll
        for (int rt = 0; rt < KT; ++rt) {
            r[rt] = 0.0;
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
                r[rt] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[rt][kt], b[kt], r[rt], 0, 0, 0);
        }
        if (live) {
#pragma unroll
            for (int rt = 0; rt < KT; ++rt)
                if (4 * rt + 3 < NQ || 4 * rt + kk < NQ)
                    F[(4 * rt + kk) * STEP] = r[rt];
        }
    }
};

// FP32, lines of up to nine nodes: v_mfma_f32_4x4x1 multiplies 16 blocks at
// once: lane l holds row l % 4 of the left operand (a column of D), the value
// of line l of the right one, and four consecutive outputs of line l.  Longer
// lines: v_mfma_f32_16x16x4, operands as in FP64 with 16 rows, results in rows
// 4 (l / 16) .. + 3 of line l % 16; D then takes a register per four columns
// instead of one per column and four rows.
template <int NQ>
struct LineD<float, NQ> {
    static constexpr bool WIDE = NQ > 9;
    static constexpr int RT = (NQ + 3) / 4;
    static constexpr int PER = WIDE ? 16 : 64;
    float a[WIDE ? 1 : RT][WIDE ? RT : NQ];
    __device__ __forceinline__ void load(const float* __restrict__ D)
    {
        const int l = threadIdx.x & 63;
        if constexpr (WIDE) {
#pragma unroll
            for (int kt = 0; kt < RT; ++kt) {
                const int row = l & 15, col = 4 * kt + (l >> 4);
                a[0][kt] = row < NQ && col < NQ ? D[row * NQ + col] : 0.0f;
            }
        } else {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                const int row = 4 * rt + (l & 3);
#pragma unroll
                for (int n = 0; n < NQ; ++n)
                    a[rt][n] = row < NQ ? D[row * NQ + n] : 0.0f;
            }
        }
    }
    template <int STEP>
    __device__ __forceinline__ void apply(float* __restrict__ F, bool live) const
    {
        if constexpr (WIDE) {
            const int kk = (threadIdx.x & 63) >> 4;
            float b[RT];
#pragma unroll
            for (int kt = 0; kt < RT; ++kt)
                b[kt] = 4 * kt + 3 < NQ || 4 * kt + kk < NQ ? F[(4 * kt + kk) * STEP] : 0.0f;
            float4_t o = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int kt = 0; kt < RT; ++kt)
                o = __builtin_amdgcn_mfma_f32_16x16x4f32(a[0][kt], b[kt], o, 0, 0, 0);
            if (live) {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (4 * kk + v < NQ)
                        F[(4 * kk + v) * STEP] = o[v];
            }
        } else {
            float4_t o[RT];
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
                o[rt] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
            float b[NQ];
#pragma unroll
            for (int n = 0; n < NQ; ++n)
                b[n] = F[n * STEP];
#pragma unroll
            for (int n = 0; n < NQ; ++n)
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
                    o[rt] = __builtin_amdgcn_mfma_f32_4x4x1f32(a[rt][n], b[n], o[rt], 0, 0, 0);
            if (live) {
#pragma unroll
                for (int n = 0; n < NQ; ++n)
                    F[n * STEP] = o[n / 4][n % 4];
            }
        }
    }
};

// Applies D along direction DIR to NARR consecutive staged arrays, in place, a
// group of lines at a time; the groups first, first + NW, ... are this wave's.
// Lanes past the last line repeat it and write nothing.
template <typename T, int NQ, int DIR, int NARR, int NW>
__device__ __forceinline__ void transform_lines(const LineD<T, NQ>& A, T* __restrict__ sF,
                                                int first)
{
    using L = LineLds<T, NQ>;
    static_assert(!L::XOR, "additive layouts");
    constexpr int NQ2 = NQ * NQ;
    constexpr int PER = LineD<T, NQ>::PER;
    constexpr int LINES = NARR * NQ2;
#pragma unroll 2
    for (int g = first; g < (LINES + PER - 1) / PER; g += NW) {
        const int q = PER * g + ((int)threadIdx.x & (PER - 1));
        const bool live = LINES % PER == 0 || q < LINES;
        const int line = live ? q : LINES - 1;
        const int a = line / NQ2, r = line - a * NQ2;
        A.template apply<L::line_pos(DIR, 0, 0, 1)>(
            sF + a * L::WORDS + L::line_pos(DIR, r % NQ, r / NQ, 0), live);
    }
}

// Wave that starts the transform of the staged direction at slot s: the groups
// follow one another over the waves, across the directions.
template <typename T, int NQ, int NARR, int NW>
__device__ __forceinline__ int first_group(int s)
{
    constexpr int PER = LineD<T, NQ>::PER;
    const int w = (int)threadIdx.x >> 6;
    const int at = (s * ((NARR * NQ * NQ + PER - 1) / PER)) % NW;
    return w >= at ? w - at : w - at + NW;
}

// Physical constants and pressure of a tile: FP64 takes x^gamma from tables in
// LDS.
template <typename T>
using LinePhys = std::conditional_t<sizeof(T) == 8, PowPhys, Phys>;

template <typename T>
constexpr int pow_table_values()
{
    return sizeof(T) == 8 ? kPowTableValues : 0;
}

template <typename T>
__device__ __forceinline__ void line_pressure(T Th, bool has_ref, double thr, const LinePhys<T>& ph,
                                              T& pflux, T& pfull)
{
    if constexpr (sizeof(T) == 8)
        table_pressure(Th, has_ref, thr, ph, pflux, pfull);
    else
        Pressure<T>::eval_full(Th, has_ref, thr, ph, pflux, pfull);
}

// One workgroup's volume term: EPB elements from e0 (ne of them in the mesh),
// NT lanes, RES = all directions staged at once (two barriers), or 1 at a time
// (two barriers each).  A node's results are read and its next fluxes written
// by the same lane, so the next direction needs no barrier of its own.
template <typename T, int NQ, int EPB, int NF, int RES>
constexpr int line_tile_tables()
{
    return pow_tables_at(RES * EPB * NF * LineLds<T, NQ>::WORDS);
}

template <typename T, int NQ, int EPB, int NF, int RES>
constexpr int line_tile_values()
{
    return line_tile_tables<T, NQ, EPB, NF, RES>() + pow_table_values<T>();
}

template <typename T, int NQ, int EPB, int NT, int RES, bool ACC, int NF, int DIRS, bool GEOE>
__device__ __forceinline__ void line_tile(const BlockPtrs<T>& B, int64_t e0, int ne,
                                          const Phys& phys, T* __restrict__ sF)
{
    using L = LineLds<T, NQ>;
    constexpr int M = NQ * NQ * NQ;
    constexpr int NPT = (EPB * M + NT - 1) / NT;
    constexpr int ND = ndirs<DIRS>();
    constexpr int NARR = EPB * NF;
    constexpr int NW = NT / 64;
    constexpr bool STREAM = Shape<NQ>::template stream_loads<T>();
    static_assert(NT % 64 == 0 && (RES == ND || RES == 1), "whole waves; all directions or one");
    const int tid = threadIdx.x;
    const bool has_ref = B.theta_ref != nullptr;
    LinePhys<T> ph;
    static_cast<Phys&>(ph) = phys;
    if constexpr (sizeof(T) == 8) {
        constexpr int TABLES = line_tile_tables<T, NQ, EPB, NF, RES>();
        ph.tab = sF + TABLES;
        stage_pow_tables<NT, TABLES>(sF);
    }
    auto ld = [](const auto* p) { return STREAM ? ld_stream(p) : *p; };
    NodeState<T, NF> st[NPT];
    double thr[NPT];
    bool live[NPT];
    int at[NPT];   // the node's word in the staged arrays
#pragma unroll
    for (int p = 0; p < NPT; ++p) {
        const int t = tid + p * NT;
        live[p] = t < EPB * M && t / M < ne;
        at[p] = (t / M) * (NF * L::WORDS) + L::pos(t % NQ, (t / NQ) % NQ, (t / (NQ * NQ)) % NQ);
        if (live[p]) {
            const int64_t e = e0 + (EPB == 1 ? 0 : t / M);
            const int m = EPB == 1 ? t : t % M;
            const T* __restrict__ qe = B.q + e * (NF * M) + m;
            st[p].rho = ld(qe);
            st[p].U1 = ld(qe + M);
            st[p].U2 = ld(qe + 2 * M);
            st[p].U3 = ld(qe + 3 * M);
            st[p].Th = ld(qe + 4 * M);
#pragma unroll
            for (int b = 5; b < NF; ++b)
                st[p].Q[b - 5] = ld(qe + b * M);
            const T* __restrict__ ge = GEOE ? B.geo + e * 10 : B.geo + e * (10 * M) + m;
#pragma unroll
            for (int s = 0; s < 9; ++s)
                if ((DIRS >> (s / 3)) & 1)
                    st[p].g[s] = GEOE ? ge[s] : ld(ge + s * M);
            st[p].jinv = GEOE ? ge[9] : ld(ge + 9 * M);
            st[p].src = (T)0;
            thr[p] = 0.0;
            if (has_ref) {
                st[p].src = ld(B.rho_ref + e * M + m);
                thr[p] = ld(B.theta_ref + e * M + m);
            }
        }
    }
    LineD<T, NQ> A;
    A.load(B.D);
    if constexpr (sizeof(T) == 8)
        __syncthreads();   // the tables are staged
    T acc[NPT][NF];
#pragma unroll
    for (int p = 0; p < NPT; ++p)
        if (live[p]) {
            NodeState<T, NF>& s = st[p];
            s.src = -(T)ph.grav * (s.rho - s.src);
            T pfull;
            line_pressure<T>(s.Th, has_ref, thr[p], ph, s.pp, pfull);
            s.rinv = recip(s.rho);
            if constexpr (RES == ND)
#pragma unroll
                for (int d = 0; d < 3; ++d)
                    if ((DIRS >> d) & 1)
                        put_flux<T, L::WORDS, NF>(
                            s, d, sF + dir_slot<DIRS>(d) * (NARR * L::WORDS) + at[p]);
        }
    if constexpr (RES == ND) {
        __syncthreads();
        if constexpr (DIRS & 1)
            transform_lines<T, NQ, 0, NARR, NW>(A, sF, first_group<T, NQ, NARR, NW>(0));
        if constexpr (DIRS & 2)
            transform_lines<T, NQ, 1, NARR, NW>(A, sF + dir_slot<DIRS>(1) * (NARR * L::WORDS),
                                             first_group<T, NQ, NARR, NW>(dir_slot<DIRS>(1)));
        if constexpr (DIRS & 4)
            transform_lines<T, NQ, 2, NARR, NW>(A, sF + dir_slot<DIRS>(2) * (NARR * L::WORDS),
                                             first_group<T, NQ, NARR, NW>(dir_slot<DIRS>(2)));
        __syncthreads();
#pragma unroll
        for (int p = 0; p < NPT; ++p)
            if (live[p])
#pragma unroll
                for (int b = 0; b < NF; ++b) {
                    T a = sF[at[p] + b * L::WORDS];
#pragma unroll
                    for (int d = 1; d < ND; ++d)
                        a += sF[d * (NARR * L::WORDS) + at[p] + b * L::WORDS];
                    acc[p][b] = a;
                }
    } else {
        auto pass = [&](auto dir) {
            constexpr int d = decltype(dir)::value;
            if constexpr ((DIRS >> d) & 1) {
#pragma unroll
                for (int p = 0; p < NPT; ++p)
                    if (live[p])
                        put_flux<T, L::WORDS, NF>(st[p], d, sF + at[p]);
                __syncthreads();
                transform_lines<T, NQ, d, NARR, NW>(A, sF, first_group<T, NQ, NARR, NW>(0));
                __syncthreads();
#pragma unroll
                for (int p = 0; p < NPT; ++p)
                    if (live[p])
#pragma unroll
                        for (int b = 0; b < NF; ++b) {
                            const T v = sF[at[p] + b * L::WORDS];
                            acc[p][b] = dir_slot<DIRS>(d) == 0 ? v : acc[p][b] + v;
                        }
            }
        };
        pass(std::integral_constant<int, 0>{});
        pass(std::integral_constant<int, 1>{});
        pass(std::integral_constant<int, 2>{});
    }
    const RkStage no_rk{0.0, 0.0, 0.0};
    const RkNode<T, false> no_rn{};
#pragma unroll
    for (int p = 0; p < NPT; ++p)
        if (live[p]) {
            const int t = tid + p * NT;
            store_node<T, M, NF, ACC, false, Shape<NQ>::template stream_stores<T>()>(
                B, no_rk, e0 + (EPB == 1 ? 0 : t / M), EPB == 1 ? t : t % M, acc[p], st[p].jinv,
                st[p].src, no_rn);
        }
}

}  // namespace semk
