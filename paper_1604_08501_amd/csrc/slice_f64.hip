// FP64 kernels at Nq = 8 on wave-private slices (sem_slice.hpp): the volume
// term with per-node or per-element metric terms, 5 or 8 fields, r+s or
// r+s+t, and the whole rate v + s.
#include "sem_internal.hpp"
#include "sem_slice.hpp"

namespace semk {

// Waves per SIMD: the five-field tiles fit 64 registers and 23 KB of LDS, so
// four workgroups (32 waves) share a CU; eight fields need 78 registers, and
// at 64 they spill (0.194 instead of 0.153 ms on the 6912-element shape).
// Against the aliased tile of two elements, two nodes per lane (16 waves per
// CU): 32768 elements 473 -> 468 us (6.3 TB/s, the rate of HBM), 4722 elements on
// cached arrays 74.9 -> 67.7, 450 11.1 -> 9.2, 64 8.8 -> 5.6; per-element metric
// terms, 32768 elements, 350 -> 296 us (5.5 TB/s; the other arrays stream at 6.3
// TB/s in 257 us); 8 fields r+s+t 158 -> 153 us.
template <int NF, int DIRS, bool GEOE, bool ACC>
__global__ __attribute__((amdgpu_flat_work_group_size(512, 512),
                          amdgpu_waves_per_eu(NF == 5 ? 8 : 6))) void
volume_slice_kernel(BlockPtrs<double> B, Phys ph)
{
    __shared__ __align__(16) double smem[slice_lds_values<NF, false>()];
    slice_tile<ACC, NF, DIRS, GEOE, false>(B, nullptr, 0.0, (int64_t)blockIdx.x, ph, smem);
}

// v + s on 32768 elements: 732 us in the aliased tile (two workgroups per CU,
// 76 KB of LDS), 580 us here with three (78 registers, 53,760 bytes of LDS,
// the most that lets three share a CU), 662 us with two.  Above the volume
// term's 468 us: the neighbours' face values (64 separate 64-byte pieces per
// value on an r face: 26 us) and the longer chain of each element's phases.
template <bool ACC>
__global__ __attribute__((amdgpu_flat_work_group_size(512, 512), amdgpu_waves_per_eu(6))) void
rhs_slice_kernel(BlockPtrs<double> B, const int32_t* __restrict__ nbr, Phys ph, double lift)
{
    __shared__ __align__(16) double smem[slice_lds_values<5, true>()];
    slice_tile<ACC, 5, 7, false, true>(B, nbr, lift, xcd_contiguous_block(blockIdx.x, gridDim.x),
                                       ph, smem);
}

}  // namespace semk

namespace semh {

template <int NF, int DIRS, bool GEOE>
static void launch_one(const semk::BlockPtrs<double>& B, const semk::Phys& ph, int accumulate,
                       hipStream_t s)
{
    if (accumulate)
        hipLaunchKernelGGL((semk::volume_slice_kernel<NF, DIRS, GEOE, true>), dim3((unsigned)B.Ne),
                           dim3(512), 0, s, B, ph);
    else
        hipLaunchKernelGGL((semk::volume_slice_kernel<NF, DIRS, GEOE, false>),
                           dim3((unsigned)B.Ne), dim3(512), 0, s, B, ph);
}

template <>
hipError_t launch_volume_slice<double>(int nf, int dirs, bool per_element_geo,
                                       const semk::BlockPtrs<double>& B, const semk::Phys& ph,
                                       int accumulate, hipStream_t s)
{
    if (!dispatch_fits(B.Ne, 512))
        return hipErrorInvalidConfiguration;
    if (per_element_geo)
        launch_one<5, 7, true>(B, ph, accumulate, s);
    else if (nf == 5 && dirs == 7)
        launch_one<5, 7, false>(B, ph, accumulate, s);
    else if (nf == 5)
        launch_one<5, 3, false>(B, ph, accumulate, s);
    else if (dirs == 7)
        launch_one<8, 7, false>(B, ph, accumulate, s);
    else
        launch_one<8, 3, false>(B, ph, accumulate, s);
    return hipGetLastError();
}

template <>
hipError_t launch_rhs_slice<double>(const semk::BlockPtrs<double>& B, const int32_t* nbr,
                                    const semk::Phys& ph, int accumulate, hipStream_t s)
{
    if (!dispatch_fits(B.Ne, 512))
        return hipErrorInvalidConfiguration;
    const double lift = 28.0;   // 1 / w_N = N (N + 1) / 2
    if (accumulate)
        hipLaunchKernelGGL((semk::rhs_slice_kernel<true>), dim3((unsigned)B.Ne), dim3(512), 0, s, B,
                           nbr, ph, lift);
    else
        hipLaunchKernelGGL((semk::rhs_slice_kernel<false>), dim3((unsigned)B.Ne), dim3(512), 0, s,
                           B, nbr, ph, lift);
    return hipGetLastError();
}

}  // namespace semh
