// Internal host-side interface between the C-ABI layer (sem_api.cpp) and the
// kernel translation units.  Not installed; not part of the public ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sem_device.hpp"

// Compiled tile shapes (Nq, elements per workgroup, layout).  The
// single-order kernels use ceil64(EPB * Nq^3) threads (one node per thread;
// 512 threads with two nodes each for aliased tiles of more than 512 nodes);
// the mixed-order batch kernel runs every shape with a fixed workgroup size.
// Layout 0 keeps all three directions' fluxes in LDS, layout 1 one direction
// at a time.
#define SEM_VARIANTS(X)                                                        \
    X(2, 8, 0) X(2, 16, 0) X(2, 32, 0) X(2, 64, 0) X(2, 128, 0)                \
    X(3, 4, 0) X(3, 8, 0) X(3, 16, 0) X(3, 32, 0)                              \
    X(4, 1, 0) X(4, 2, 0) X(4, 4, 0) X(4, 8, 0) X(4, 16, 0)                    \
    X(5, 1, 0) X(5, 2, 0) X(5, 4, 0) X(5, 8, 0)                                \
    X(6, 1, 0) X(6, 2, 0) X(6, 4, 0) X(6, 2, 1) X(6, 4, 1)                     \
    X(7, 1, 0) X(7, 2, 0) X(7, 1, 1) X(7, 2, 1)                                \
    X(8, 1, 0) X(8, 2, 0) X(8, 1, 1) X(8, 2, 1)                                \
    X(9, 1, 0) X(9, 1, 1)                                                      \
    X(10, 1, 0) X(10, 1, 1)

constexpr int kMinNq = 2, kMaxNq = 10;   // orders of SEM_VARIANTS

namespace semh {

// A dispatch's work-item count (workgroups x lanes) is a 32-bit field of the
// dispatch packet: launches beyond it fail with this error instead.
constexpr bool dispatch_fits(int64_t groups, int threads)
{
    return groups >= 1 && groups * (int64_t)threads <= (int64_t)UINT32_MAX;
}

struct VariantDef {
    int nq, epb, lay;
};
#define SEM_X_DEF(NQ_, EPB_, LAY_) VariantDef{NQ_, EPB_, LAY_},
inline constexpr VariantDef kVariants[] = {SEM_VARIANTS(SEM_X_DEF)};
#undef SEM_X_DEF
inline constexpr int kNumVariants = (int)(sizeof(kVariants) / sizeof(kVariants[0]));

constexpr int variant_index(int nq, int epb, int lay)
{
    for (int i = 0; i < kNumVariants; ++i)
        if (kVariants[i].nq == nq && kVariants[i].epb == epb && kVariants[i].lay == lay)
            return i;
    return -1;
}

constexpr int kMaxLdsBytes = 160 * 1024;   // LDS per CU on gfx950
constexpr int kBatchThreads[] = {256, 512, 1024};

// Single-order forward/adjoint launchers (defined per dtype in kernels_*.hip).
template <typename T>
hipError_t launch_volume(int nq, int epb, int lay, const semk::BlockPtrs<T>& B,
                         const semk::Phys& ph, int accumulate, hipStream_t s);
template <typename T>
hipError_t launch_adjoint(int nq, int epb, const semk::AdjPtrs<T>& B, const semk::Phys& ph,
                          int accumulate, hipStream_t s);
template <typename T>
hipError_t launch_axpby(int64_t n, double a, const T* x, double b, const T* y, double c,
                        const T* z, T* out, hipStream_t s);

// Extended volume term (defined per dtype in ext_*.hip): nf = 5 or 8 fields,
// dirs = 3 (r+s) or 7 (r+s+t), Nq in 2..10, 12, 16 where the LDS allows.
template <typename T>
bool ext_supported(int nq, int nf, int dirs);
template <typename T>
hipError_t launch_volume_ext(int nq, int nf, int dirs, const semk::BlockPtrs<T>& B,
                             const semk::Phys& ph, int accumulate, hipStream_t s);
// Volume term with per-element metric terms (affine elements; geo [Ne][10]),
// five fields, r+s+t, Nq in 2..10, 12, 16 where the LDS allows.
template <typename T>
bool affine_supported(int nq);
template <typename T>
hipError_t launch_volume_affine(int nq, const semk::BlockPtrs<T>& B, const semk::Phys& ph,
                                int accumulate, hipStream_t s);

// Surface term (surface_*.hip): Nq 2..10, 12, 16.
template <typename T>
bool surface_supported(int nq);
template <typename T>
hipError_t launch_surface(int nq, const semk::SurfPtrs<T>& B, const semk::Phys& ph, int accumulate,
                          hipStream_t s);

// Volume + surface term in one launch (rhs_*.hip): Nq 2..10.
template <typename T>
bool rhs_supported(int nq);
template <typename T>
hipError_t launch_volume_surface(int nq, const semk::BlockPtrs<T>& B, const int32_t* nbr,
                                 const semk::Phys& ph, int accumulate, hipStream_t s);

// FP64 at Nq = 8 on wave-private slices (slice_f64.hip): the volume term of nf
// fields over dirs (per_element_geo: five fields, r+s+t, metric terms per
// element), and v + s.  The only tile of the calls that name no tile shape:
// it measured faster than the shapes of SEM_VARIANTS from 1 element to 32768.
template <typename T>
constexpr bool use_slice(int nq)
{
    return sizeof(T) == 8 && nq == 8;
}
template <typename T>
hipError_t launch_volume_slice(int nf, int dirs, bool per_element_geo,
                               const semk::BlockPtrs<T>& B, const semk::Phys& ph, int accumulate,
                               hipStream_t s);
template <typename T>
hipError_t launch_rhs_slice(const semk::BlockPtrs<T>& B, const int32_t* nbr, const semk::Phys& ph,
                            int accumulate, hipStream_t s);

// Volume tiles on line transforms (sem_lines.hpp): elements of up to `nodes`
// nodes together per workgroup (at least one element), up to `lanes` lanes,
// all directions' fluxes staged at once or one direction's at a time.  Up to
// `few` elements (`few_add` when adding to rhs), and at any number where lanes =
// 0, the tile that contracts node by node stays.
struct LinePick {
    int nodes, lanes;
    bool all = false;
    int few = 0, few_add = few;
};

// The faster of both tiles, and among the line tiles of 64-1024 lanes and
// nodes, on 3.5 million nodes (per-element metric terms and five fields r+s+t
// up to Nq = 10: 8 million), where it gained some 3% or more.  The line tile wins
// where the other one is held by its LDS reads or its few workgroups per CU:
// orders that are no power of two, eight fields, metric terms that cost no
// bandwidth.  us, node by node -> lines:
//   per-element metric terms, FP64, Nq = 2, 4, 5, 6, 7, 9, 10, 12: 178 -> 166,
//     157 -> 131, 182 -> 167, 187 -> 164, 219 -> 164, 224 -> 174, 209 -> 180,
//     293 -> 232 (3: 174, lines 184)
//   FP32, Nq = 3..9, 12: 98 -> 93, 74 -> 70, 91 -> 74, 101 -> 79, 110 -> 85,
//     81 -> 72, 122 -> 90, 131 -> 96 (2: 92, lines 92; 10: 110, lines 104, but
//     1000 elements 16.9, lines 19.7)
//   five fields, r+s+t, FP64, Nq = 6, 7, 9, 12: 241 -> 230, 266 -> 245,
//     279 -> 271, 183 -> 168; FP32, Nq = 6, 9, 12: 130 -> 121, 148 -> 130,
//     79 -> 65
//   five fields, r+s, FP64, Nq = 10: 132 -> 110; FP32, Nq = 6: 52.6 -> 51.0
//   eight fields, r+s+t, FP64, Nq = 3, 5, 6, 7, 10, 12: 176 -> 159, 175 -> 159,
//     172 -> 157, 262 -> 174, 215 -> 183, 277 -> 237; FP32, Nq = 5, 6, 7, 9, 12:
//     87 -> 82, 85 -> 77, 95 -> 89, 98.9 -> 95.8, 103 -> 98
//   eight fields, r+s, FP64, Nq = 3, 5, 10: 160 -> 149, 158 -> 145, 162 -> 154;
//     FP32, Nq = 5, 6, 9: 81 -> 77, 75 -> 70, 85 -> 82
// Few elements, of which a CU holds two or three: the launch takes as long as a
// workgroup or two, and line transforms are the longer chain (fluxes to lines
// and back, a barrier on either side, in FP64 the power's tables before all of
// it; several nodes per lane where lanes are fewer than nodes).  Captured
// launches on the same arrays, us, node by node -> lines on either side of
// `few`:
//   per-element metric terms, FP64, Nq = 2: 1000 elements 4.4 -> 5.6, 127000
//     25.6 -> 23.2; 5: 720 6.0 -> 6.9, 3000 12.2 -> 11.5; 6: 990
//     7.9 -> 8.7, 1152 10.5 -> 9.7; 7: 450 8.0 -> 9.4, 720 11.4 -> 10.8; 9: 512 13.3 -> 15.3; 12: 256
//     16.8 -> 17.8
//   FP32, Nq = 3: 1000 3.9 -> 5.4, 31000 13.5 -> 13.5, 50000 19.4 -> 17.9; 4: 1000
//     3.8 -> 4.6, 12000 10.2 -> 9.3; 6: 450 4.3 -> 5.7, 1844 8.2 -> 7.5; 7: 175
//     4.8 -> 5.1, 720 6.8 -> 6.5; 8: 720 6.4 -> 7.1, 4700 25.5 -> 25.0; 9: 175
//     5.9 -> 7.0, 720 11.7 -> 10.6
//   five fields, r+s, FP64, Nq = 10: 256 11.3 -> 13.3; FP32, Nq = 6: 281 3.8 -> 4.1,
//     720 5.2 -> 4.7 (adding 6.0 -> 5.2, and 281 5.0 -> 4.5)
//   five fields, r+s+t, FP64, Nq = 6: 1 4.7 -> 5.2, 2 5.8 -> 5.3; 7: 1024 16.2 -> 16.7
//   eight fields, r+s, FP64, Nq = 3: 2951 6.3 -> 6.8, 4722 8.8 -> 8.1 (adding 4
//     3.7 -> 5.0, 42 5.7 -> 5.2); 5: 1844 10.3 -> 10.9, 2951 16.6 -> 16.3 (adding
//     175 7.2 -> 6.0)
//   eight fields, r+s+t, FP64, Nq = 3: 2951 8.1 -> 8.4, 4722 10.7 -> 9.8 (adding 4
//     4.1 -> 6.1, 42 6.8 -> 6.3); 5: 281 7.4 -> 8.2, 1152 12.2 -> 10.8 (adding 2
//     5.5 -> 7.1, 42 8.3 -> 7.3); 6: 1 5.1 -> 6.2, 2 6.9 -> 6.4; 7: 175 6.8 -> 8.1,
//     281 11.9 -> 10.9; FP32, Nq = 6: 1 3.7 -> 4.2, 4 4.5 -> 4.4
// (Left as they are, since both signs alternate: FP64 Nq = 4 per-element terms,
// 450 4.7 -> 4.4, 1844 5.5 -> 6.1, 4722 9.7 -> 8.2; FP64 Nq = 6 eight fields
// r+s+t, 175 7.5 -> 7.0, 281 8.0 -> 8.7, 720 11.7 -> 10.5.)
template <typename T>
constexpr LinePick line_pick(int nq, int nf, int dirs, bool per_element_geo)
{
    constexpr LinePick none{0, 0};
    constexpr bool f64 = sizeof(T) == 8;
    if (nq > 12)
        return none;
    if (per_element_geo) {
        if (nq == 12)
            return {256, 512, false, f64 ? 320 : 0};
        if (f64)
            return nq == 3 || nq == 8 ? none
                   : nq == 2          ? LinePick{128, 128, false, 80000}
                   : nq == 4          ? LinePick{64, 64}
                   : nq == 5          ? LinePick{128, 128, false, 2200}
                   : nq == 10         ? LinePick{256, 512}
                                      : LinePick{256, 256, false, nq == 9 ? 640 : nq == 6 ? 1024 : 600};
        return nq == 2 || nq == 10 ? none
               : nq < 5            ? LinePick{512, 256, false, nq == 3 ? 30000 : 9500}
               : nq == 5           ? LinePick{128, 128, true}
               : nq == 6           ? LinePick{256, 128, false, 1200}
               : nq == 8           ? LinePick{512, 256, false, 3500}
                                   : LinePick{256, 256, false, nq == 7 ? 700 : 600};
    }
    if (dirs == 3) {
        if (f64)
            return nq == 10              ? LinePick{256, 512, false, 384}
                   : nf == 8 && nq == 3  ? LinePick{64, 64, false, 3500, 12}
                   : nf == 8 && nq == 5  ? LinePick{128, 128, true, 2200, 3}
                                         : none;
        return nq == 6              ? LinePick{256, 256, false, nf == 5 ? 512 : 0, nf == 5 ? 2 : 0}
               : nf == 8 && nq == 5 ? LinePick{128, 128, true}
               : nf == 8 && nq == 9 ? LinePick{256, 768}
                                    : none;
    }
    if (nq == 12)
        return {256, 1024};
    if (nf == 5)
        return nq == 6          ? LinePick{256, 256, false, f64 ? 1 : 0}
               : f64 && nq == 7 ? LinePick{256, 192, false, 1280}
               : nq == 9        ? LinePick{256, f64 ? 512 : 256}
                                : none;
    return nq == 5           ? LinePick{128, 128, !f64, f64 ? 600 : 0, f64 ? 3 : 0}
           : nq == 6         ? LinePick{256, 256, false, 1}
           : nq == 7         ? LinePick{256, 384, false, f64 ? 256 : 0}
           : f64 && nq == 3  ? LinePick{64, 64, false, 3500, 8}
           : f64 && nq == 10 ? LinePick{256, 512}
           : !f64 && nq == 9 ? LinePick{256, 768}
                             : none;
}

// Elements and lanes of a picked tile's workgroup.
constexpr int line_elements(const LinePick& p, int nq)
{
    int e = 1;
    while (2 * e * nq * nq * nq <= p.nodes)
        e *= 2;
    return e;
}
constexpr int line_lanes(const LinePick& p, int nq)
{
    const int lanes = (line_elements(p, nq) * nq * nq * nq + 63) / 64 * 64;
    return lanes < p.lanes ? lanes : p.lanes;
}

// Whether Ne elements take the picked line tile.  It may need more lanes per
// element than the other one, which then takes the largest launches (Nq = 6,
// 256 lanes instead of 224 or, FP32 volume term, 128: 2^24 elements and more,
// which FP32 arrays and per-element FP64 metric terms can still hold).
constexpr bool takes_lines(const LinePick& p, int nq, int64_t Ne, bool accumulate)
{
    if (p.lanes == 0 || Ne <= (accumulate ? p.few_add : p.few))
        return false;
    const int per = line_elements(p, nq);
    return dispatch_fits((Ne + per - 1) / per, line_lanes(p, nq));
}

// Whether the volume term of five fields, r+s+t, of Ne elements has a tile of
// its own for the calls that name no tile shape (launch_volume_ext).
template <typename T>
constexpr bool volume_own_tile(int nq, int64_t Ne, bool accumulate)
{
    return use_slice<T>(nq) || takes_lines(line_pick<T>(nq, 5, 7, false), nq, Ne, accumulate);
}

// Workgroup cap of the strided k-slice and t-column launches set by
// sem_set_max_workgroups (0 = none); one relaxed atomic load.
int64_t max_workgroups_cap();

// Optimisation ladder of the fused r+s, 8-field FP32 kernel (ladder.hip):
// levels 1..5, Nq 2..10, 12, 16.
bool ladder_supported(int nq);
hipError_t launch_ladder(int level, int nq, int64_t Ne, const float* D, const float* geo,
                         const float* q, float* rhs, const semk::Phys& ph, hipStream_t s);

// Mixed-order batch kernel (defined per dtype in batch_*.hip): one tile per
// workgroup.
struct Tile {
    int32_t block;
    int32_t variant;
    int32_t ne;
    int32_t pad;
    int64_t e0;
};
// rk: the shape must also run a fused Runge-Kutta stage (one node per thread
// for FULL, at most two for ALIAS)
template <typename T>
bool batch_variant_ok(int nt, int nq, int epb, int lay, bool rk);
template <typename T>
int batch_lds_bytes(int nt, int nq, int epb, int lay);
// rk = false: rhs = v(q); rk = true: every block runs the fused stage
// out = a x + b (q + dt v) with the coefficients of its descriptor.
template <typename T>
hipError_t launch_batch(int nt, const Tile* d_tiles, int ntiles,
                        const semk::BatchBlock<T>* d_blocks, bool rk, int lds_bytes,
                        hipStream_t s);
template <typename T>
hipError_t batch_blocks_per_cu(int nt, int lds_bytes, bool rk, int* out);

// Must run once per process before occupancy queries or launches (sets the
// dynamic-LDS limit of the batch kernels).
template <typename T>
hipError_t batch_prepare();

}  // namespace semh
