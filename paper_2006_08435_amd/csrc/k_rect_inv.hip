// Rectangular xy-plane pass (Nx != Ny, both up to 128): instances of sign 1.
#include "kernels_rect.hpp"
#include "registry.hpp"

namespace fft3d {

hipError_t rect_inv(int cls, const RectArgs& a, unsigned grid, size_t lds, hipStream_t st)
{
    switch (cls) {
    case 0: hipLaunchKernelGGL((k_plane_rect<1, 0>), dim3(grid), dim3(kRectClasses[0].threads), lds, st, a); break;
    case 1: hipLaunchKernelGGL((k_plane_rect<1, 1>), dim3(grid), dim3(kRectClasses[1].threads), lds, st, a); break;
    case 2: hipLaunchKernelGGL((k_plane_rect<1, 2>), dim3(grid), dim3(kRectClasses[2].threads), lds, st, a); break;
    case 3: hipLaunchKernelGGL((k_plane_rect<1, 3>), dim3(grid), dim3(kRectClasses[3].threads), lds, st, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

const void* rect_inv_kernel(int cls)
{
    switch (cls) {
    case 0: return reinterpret_cast<const void*>(&k_plane_rect<1, 0>);
    case 1: return reinterpret_cast<const void*>(&k_plane_rect<1, 1>);
    case 2: return reinterpret_cast<const void*>(&k_plane_rect<1, 2>);
    case 3: return reinterpret_cast<const void*>(&k_plane_rect<1, 3>);
    default: return nullptr;
    }
}

}  // namespace fft3d
