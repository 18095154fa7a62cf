// Root plane pass: the signed n-th root of every channel sample, eq. (4),
// stored beside the sample for the beamformer's staging step.
#include "dmas_kernel.hpp"

namespace dmas {

namespace {

template <int N, int J>
hipError_t launch_roots_n(int dtype, const void *x, float2 *plane, int M, int T, int pad0, int pad1,
                          hipStream_t stream)
{
    const int stride = pad0 + T + pad1;
    unsigned gx = 0, gy = 0;
    root_grid(M, stride, &gx, &gy, J * kRootThreads);
    const dim3 grid(gx, gy), threads(kRootThreads);
    auto kern = dtype == 0   ? root_plane_kernel<N, 0, J>
                : dtype == 1 ? root_plane_kernel<N, 1, J>
                             : root_plane_kernel<N, 2, J>;
    hipLaunchKernelGGL(kern, grid, threads, 0, stream, x, plane, M, T, pad0, stride);
    return hipGetLastError();
}

template <int N>
hipError_t launch_roots_n(int dtype, const void *x, float2 *plane, int M, int T, int pad0, int pad1,
                          hipStream_t stream)
{
    if ((int64_t)M * (pad0 + T + pad1) <= kRootWide)
        return launch_roots_n<N, 1>(dtype, x, plane, M, T, pad0, pad1, stream);
    return launch_roots_n<N, kRootBlock / kRootThreads>(dtype, x, plane, M, T, pad0, pad1, stream);
}

}  // namespace

hipError_t launch_roots(int order, int dtype, const void *x, float2 *plane, int M, int T, int pad0, int pad1,
                        hipStream_t stream)
{
    switch (order) {
    case 2: return launch_roots_n<2>(dtype, x, plane, M, T, pad0, pad1, stream);
    case 3: return launch_roots_n<3>(dtype, x, plane, M, T, pad0, pad1, stream);
    case 4: return launch_roots_n<4>(dtype, x, plane, M, T, pad0, pad1, stream);
    case 5: return launch_roots_n<5>(dtype, x, plane, M, T, pad0, pad1, stream);
    case 6: return launch_roots_n<6>(dtype, x, plane, M, T, pad0, pad1, stream);
    case 7: return launch_roots_n<7>(dtype, x, plane, M, T, pad0, pad1, stream);
    case 8: return launch_roots_n<8>(dtype, x, plane, M, T, pad0, pad1, stream);
    default: return hipErrorNotSupported;
    }
}

}  // namespace dmas
