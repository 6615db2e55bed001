// FP64 tile at Nq = 8 on wave-private slices: one element per workgroup of
// eight waves, wave k holding slice k, lane i + 8 j the node (i, j, k).
//
// The r and s lines of a node lie in its own wave, so those contractions go
// through LDS without a workgroup barrier, one after the other through the
// slice's share of the flux buffer, which then takes the t fluxes: 20 KB of
// staged fluxes instead of 41 to 61, and no node state held across a barrier
// (55 to 64 registers for the volume term of five fields, 64 to 76 for eight and
// 78 for v + s, instead of 101 and more).  What that buys is occupancy: these
// kernels wait on HBM latency, VALU, LDS and matrix units each well under their
// limits, so their time is set by how many workgroups a CU holds.  Five fields
// run four workgroups (32 waves) per CU, eight fields and v + s three; see the
// kernels for what each measured.
#pragma once
#include "sem_lines.hpp"
#include "sem_pow.hpp"

namespace semk {

// Keeps the compiler from moving LDS accesses of a wave across; the hardware
// runs one wave's in order.
__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// acc[b] = or += D along r (DIR = 0) or s (1) of the NF fluxes f held one
// node per lane of slice k.  sF: the element's NF flux arrays; at: the node's
// word in them.  The 16 columns of the matrix product are the slice's eight
// lines twice, for the two halves of the rows: rows 4 h + kk along r, 2 kk + h
// along s (h is bit 3 of the lane, kk the lane's sixteenth), so that a
// 16-lane write touches every bank once in either direction.  (D's rows of 64
// bytes do not: the operand loads here and in transform_t_lines, two of 24 and
// two of 8 extra cycles per wave, are the volume tile's only bank conflicts, 64
// cycles beside some 150 of LDS work.)
template <int DIR, int NF, bool FIRST>
__device__ __forceinline__ void contract_slice(const double* __restrict__ sD,
                                               const double (&f)[NF], int at, int k,
                                               double* __restrict__ sF, double (&acc)[NF])
{
    using L = LineLds<double, 8>;
    const int l = threadIdx.x & 63;
    const int line = l & 7, h = (l >> 3) & 1, kk = l >> 4;
    const int row_in = DIR == 0 ? 4 * h + (l & 3) : 2 * (l & 3) + h;
    const double a0 = sD[row_in * 8 + kk], a1 = sD[row_in * 8 + 4 + kk];
    const int row = DIR == 0 ? 4 * h + kk : 2 * kk + h;
    const int b0 = DIR == 0 ? L::pos(kk, line, k) : L::pos(line, kk, k);
    const int b1 = b0 ^ (DIR == 0 ? L::pos(4, 0, 0) : L::pos(0, 4, 0));
    const int o = DIR == 0 ? L::pos(row, line, k) : L::pos(line, row, k);
    if (!FIRST)
        wave_fence();   // the previous direction's results are read
    // three fields at a time: enough independent products, few registers
    constexpr int G = 3;
#pragma unroll
    for (int g = 0; g < NF; g += G) {
#pragma unroll
        for (int b = g; b < g + G && b < NF; ++b)
            sF[b * L::WORDS + at] = f[b];
        wave_fence();
        double r[G];
#pragma unroll
        for (int b = g; b < g + G && b < NF; ++b) {
            r[b - g] = __builtin_amdgcn_mfma_f64_4x4x4f64(a0, sF[b * L::WORDS + b0], 0.0, 0, 0, 0);
            r[b - g] =
                __builtin_amdgcn_mfma_f64_4x4x4f64(a1, sF[b * L::WORDS + b1], r[b - g], 0, 0, 0);
        }
        wave_fence();
#pragma unroll
        for (int b = g; b < g + G && b < NF; ++b)
            sF[b * L::WORDS + o] = r[b - g];
        wave_fence();
#pragma unroll
        for (int b = g; b < g + G && b < NF; ++b) {
            const double v = sF[b * L::WORDS + at];
            acc[b] = FIRST ? v : acc[b] + v;
        }
    }
}

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
        off[g] = LineLds<double, 8>::pos(c & 7, 2 * g + (c >> 3), kk);
    constexpr int HALF = LineLds<double, 8>::pos(0, 0, 4);   // from node kk to node 4 + kk of a line
#pragma unroll 1
    for (int x = first; x < NARR; x += STEP) {
        double* __restrict__ F = sF + x * LineLds<double, 8>::WORDS;
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

// Own face values the v + s tile stages per face node: the state, the flux
// pressure, the sound speed and the outward normal times its area factor.
constexpr int kSliceOwnVals = 10;

template <int NF, bool SURF>
constexpr int slice_lds_values()
{
    return NF * LineLds<double, 8>::WORDS + kPowTableValues + 64 + (SURF ? 6 * kSliceOwnVals * 64 : 0);
}

// Element e: the volume term of NF fields over DIRS, or v + s (SURF).
template <bool ACC, int NF, int DIRS, bool GEOE, bool SURF>
__device__ __forceinline__ void slice_tile(const BlockPtrs<double>& B, const int32_t* nbr,
                                           double lift, int64_t e, const Phys& phys,
                                           double* __restrict__ smem)
{
    static_assert(!SURF || (NF == 5 && DIRS == 7 && !GEOE), "v + s is for the full volume term");
    using L = LineLds<double, 8>;
    constexpr int M = 512, N = 7;
    double* __restrict__ sF = smem;
    constexpr int TABLES = NF * L::WORDS;
    double* __restrict__ sTab = smem + TABLES;
    double* __restrict__ sD = sTab + kPowTableValues;
    double* __restrict__ sOwn = sD + 64;   // [face][value][64]
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = tid & 7, j = (tid >> 3) & 7, k = w;
    const bool has_ref = B.theta_ref != nullptr;
    stage_pow_tables<512, TABLES>(smem);
    if (w == 7)
        sD[tid & 63] = B.D[tid & 63];

    // every array at a workgroup-uniform address plus the lane's node; v + s
    // reads the state through the cache (the neighbours read it again)
    NodeState<double, NF> st;
    double rr = 0.0, thr = 0.0;
    {
        const unsigned m = tid;
        auto ldq = [](const double* p) { return SURF ? *p : ld_stream(p); };
        st.rho = ldq(B.q + e * NF * M + m);
        st.U1 = ldq(B.q + (e * NF + 1) * M + m);
        st.U2 = ldq(B.q + (e * NF + 2) * M + m);
        st.U3 = ldq(B.q + (e * NF + 3) * M + m);
        st.Th = ldq(B.q + (e * NF + 4) * M + m);
#pragma unroll
        for (int b = 5; b < NF; ++b)
            st.Q[b - 5] = ldq(B.q + (e * NF + b) * M + m);
#pragma unroll
        for (int x = 0; x < 9; ++x)
            st.g[x] = !((DIRS >> (x / 3)) & 1) ? 0.0
                      : GEOE                   ? B.geo[e * 10 + x]
                                               : ld_stream(B.geo + (e * 10 + x) * M + m);
        st.jinv = GEOE ? B.geo[e * 10 + 9] : ld_stream(B.geo + (e * 10 + 9) * M + m);
        if (has_ref) {
            rr = ld_stream(B.rho_ref + e * M + m);
            thr = ldq(B.theta_ref + e * M + m);
        }
    }
    // waves 0 .. 5 take one face each
    int64_t en = SURF && w < 6 ? nbr[e * 6 + w] : -1;
    if (en >= B.Ne)
        en = -1;
    double nq[5], nth = 0.0, np, nc;
    PowPhys ph;
    static_cast<Phys&>(ph) = phys;
    ph.tab = sTab;
    __syncthreads();   // the tables and D are staged
    st.src = -ph.grav * (st.rho - rr);
    table_pressure(st.Th, has_ref, thr, ph, st.pp, st.pfull);
    st.rinv = recip(st.rho);
    if constexpr (SURF) {
        if (i == 0 || i == N || j == 0 || j == N || k == 0 || k == N) {
            const double c = root(ph.gamma * st.pfull * st.rinv);
            const int ijk[3] = {i, j, k};
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                if (ijk[d] != 0 && ijk[d] != N)
                    continue;
                const int side = ijk[d] == N ? 1 : 0;
                const int a = d == 0 ? j + 8 * k : (d == 1 ? i + 8 * k : i + 8 * j);
                const double sg = side ? 1.0 : -1.0;
                const double v[kSliceOwnVals] = {st.rho, st.U1, st.U2, st.U3, st.Th, st.pp, c,
                                                 sg * st.g[3 * d], sg * st.g[3 * d + 1],
                                                 sg * st.g[3 * d + 2]};
                double* __restrict__ o = sOwn + (2 * d + side) * (kSliceOwnVals * 64) + a;
#pragma unroll
                for (int b = 0; b < kSliceOwnVals; ++b)
                    o[b * 64] = v[b];
            }
        }
    }
    const int at = L::pos(i, j, k);
    double acc[NF], f[NF];
    put_flux<double, 1, NF>(st, 0, f);
    contract_slice<0, NF, true>(sD, f, at, k, sF, acc);
    if constexpr (SURF) {
        // the neighbour's facing nodes, in flight during the s contraction
        // (not before: their registers would cost the third workgroup)
        __builtin_amdgcn_sched_barrier(0);
        if (en >= 0) {
            const unsigned mp = face_node<8>(w >> 1, 1 - (w & 1), i, j);
#pragma unroll
            for (int b = 0; b < 5; ++b)
                nq[b] = (B.q + (en * 5 + b) * M)[mp];
            if (has_ref)
                nth = (B.theta_ref + en * M)[mp];
        }
    }
    put_flux<double, 1, NF>(st, 1, f);
    contract_slice<1, NF, false>(sD, f, at, k, sF, acc);
    if constexpr (DIRS & 4) {
        wave_fence();   // the s results are read
        put_flux<double, L::WORDS, NF>(st, 2, sF + at);
    }
    const double jinv = st.jinv, src = st.src;
    if constexpr (SURF) {
        if (en >= 0) {
            double pfull;
            table_pressure(nq[4], has_ref, nth, ph, np, pfull);
            nc = root(ph.gamma * pfull / nq[0]);
        }
    }
    if constexpr (DIRS & 4) {
        __syncthreads();   // the t fluxes (and the own face values) are staged
        if constexpr (SURF) {
            if (w < 6) {
                double* __restrict__ o = sOwn + w * (kSliceOwnVals * 64) + (tid & 63);
                if (en < 0) {
#pragma unroll
                    for (int b = 0; b < 5; ++b)
                        o[b * 64] = 0.0;   // boundary face: exterior state = interior state
                } else {
                    double qm[5];
#pragma unroll
                    for (int b = 0; b < 5; ++b)
                        qm[b] = o[b * 64];
                    const double pm = o[5 * 64], cm = o[6 * 64];
                    const double n[3] = {o[7 * 64], o[8 * 64], o[9 * 64]};
                    // the node's sums wait in the slots just read, out of the
                    // registers (ten would spill to scratch memory, which ran
                    // 706 instead of 580 us)
#pragma unroll
                    for (int b = 0; b < 5; ++b)
                        o[(5 + b) * 64] = acc[b];
                    asm volatile("" ::: "memory");
                    double jump[5];
                    face_flux(qm, nq, pm, np, cm, nc, recip(qm[0]), recip(nq[0]), n, jump);
#pragma unroll
                    for (int b = 0; b < 5; ++b)
                        o[b * 64] = jump[b];
                    asm volatile("" ::: "memory");
#pragma unroll
                    for (int b = 0; b < 5; ++b)
                        acc[b] = o[(5 + b) * 64];
                }
            }
            // t lines on the waves without a face and, for the fifth field, wave 0
            if (w >= 6 || w == 0)
                transform_t_lines<5, 3>(sD, sF, w >= 6 ? w - 6 : 2);
        } else {
            transform_t_lines<NF, 8>(sD, sF, w);
        }
        __syncthreads();
#pragma unroll
        for (int b = 0; b < NF; ++b)
            acc[b] += sF[b * L::WORDS + at];
    }
    if constexpr (SURF)
        gather_face_terms<double, 8, kSliceOwnVals>(i, j, k, sOwn, lift, acc);
    const RkStage no_rk{0.0, 0.0, 0.0};
    const RkNode<double, false> no_rn{};
    store_node<double, M, NF, ACC, false>(B, no_rk, e, tid, acc, jinv, src, no_rn);
}

}  // namespace semk
