// rom_scan_f32_many.hip -- the FP32 row-scan sweep for full GPUs: ensembles and batches, whose problems
// may differ in width, several ordinates per wavefront and four wavefronts per SIMD.
#include "rom_scan.h"

namespace rom {

// The shape of each task follows its problem's width (scan_class).  One kernel holds every shape, so
// a batch of uneven problems is one launch; 128 VGPRs, the values of a few (up to six, with inflow
// tables 39) kept in scratch memory, in the widest shapes.
template <int W, bool INF>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(4))) void scan_many_kernel(ScanArgs A)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const __attribute__((address_space(4))) ScanTaskDev& TK = *scalar_ptr(A.tasks + blockIdx.x);
    switch (TK.cls) {
    case 0: scan_group<float, 16, 4, 4, 2, W, 1, 0, false, INF>(A, TK, (float*)smem); break;
    case 1: scan_group<float, 16, 8, 2, 2, W, 1, 0, false, INF>(A, TK, (float*)smem); break;
    case 2: scan_group<float, 32, 8, 2, 2, W, 1, 0, false, INF>(A, TK, (float*)smem); break;
    case 3: scan_group<float, 64, 6, 2, 2, W, 1, 0, false, INF>(A, TK, (float*)smem); break;
    case 4: scan_group<float, 64, 8, 2, 2, W, 1, 0, false, INF>(A, TK, (float*)smem); break;
    case 5: scan_group<float, 64, 6, 2, 2, W, 2, 0, false, INF>(A, TK, (float*)smem); break;
    default: scan_group<float, 64, 8, 2, 2, W, 2, 0, false, INF>(A, TK, (float*)smem); break;
    }
}

template <int W, bool INF>
static hipError_t launch_many(const ScanArgs& a, int ntasks, hipStream_t s)
{
    // two buffers of a batch's rows, 2 U W 64 RC floats (U RC <= 16 in every shape), and the values
    // handed between strips, 2 U (W / 2) K
    constexpr size_t lds = sizeof(float) * (2 * W * 64 * 16 + 2 * 2 * (W / 2) * 2);
    auto kern = scan_many_kernel<W, INF>;
    const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(ntasks), dim3(64 * W), lds, s, a);
    return hipGetLastError();
}

hipError_t launch_scan_f32_many(const ScanArgs& a, int ntasks, int waves, bool inf, hipStream_t s)
{
    if (ntasks < 1) return hipErrorInvalidValue;
    if (waves == 8) return inf ? launch_many<8, true>(a, ntasks, s) : launch_many<8, false>(a, ntasks, s);
    if (waves == 16) return inf ? launch_many<16, true>(a, ntasks, s) : launch_many<16, false>(a, ntasks, s);
    return hipErrorInvalidValue;
}

}  // namespace rom
