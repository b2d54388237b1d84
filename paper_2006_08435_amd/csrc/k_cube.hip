// Whole-grid kernel instances: radix stages in LDS (cubic N <= 16) and a line
// a thread (cubic 8 <= N <= 32).
#include "kernels_fp32.hpp"
#include "registry.hpp"

namespace fft3d {

template <int N, int S>
static hipError_t launch_cube(const float2* in, float2* out, const float2* tw, long grids, hipStream_t st)
{
    return launch_blocks(grids, [&](long first, unsigned n) {
        hipLaunchKernelGGL((k_cube<N, S>), dim3(n), dim3(CubeGeom<N>::T), 0, st, in + first * (N * N * N),
                           out + first * (N * N * N), tw);
    });
}

template <int N, int S>
static hipError_t launch_cube_lines(const float2* in, float2* out, const float2*, long grids, hipStream_t st)
{
    return launch_blocks(grids, [&](long first, unsigned n) {
        hipLaunchKernelGGL((k_cube_lines<N, S>), dim3(n), dim3(CubeLines<N>::T), 0, st, in + first * (N * N * N),
                           out + first * (N * N * N));
    });
}

#define FFT3D_CUBE_CASE(n)                                                     \
    case n:                                                                    \
        return sign < 0 ? &launch_cube<n, -1> : &launch_cube<n, 1>;
#define FFT3D_CUBE_INFO(n)                                                     \
    case n:                                                                    \
        return {CubeGeom<n>::T, (int)(CubeGeom<n>::WORDS * sizeof(float2))};
#define FFT3D_FOR_EACH_CUBE(X) X(1) X(2) X(3) X(4) X(5) X(6) X(8) X(9) X(10) X(12) X(15) X(16)
#define FFT3D_CUBE_LINES_CASE(n)                                               \
    case n:                                                                    \
        return sign < 0 ? &launch_cube_lines<n, -1> : &launch_cube_lines<n, 1>;
#define FFT3D_CUBE_LINES_INFO(n)                                               \
    case n:                                                                    \
        return {CubeLines<n>::T, (int)sizeof(CubeLines<n>::W) * CubeLines<n>::WORDS};
#define FFT3D_FOR_EACH_CUBE_LINES(X)                                           \
    X(8) X(9) X(10) X(12) X(15) X(16) X(18) X(20) X(24) X(25) X(27) X(30) X(32)

CubeFn cube_fn(int n, int sign)
{
    switch (n) {
        FFT3D_FOR_EACH_CUBE(FFT3D_CUBE_CASE)
    default: return nullptr;
    }
}

CubeFn cube_lines_fn(int n, int sign)
{
    switch (n) {
        FFT3D_FOR_EACH_CUBE_LINES(FFT3D_CUBE_LINES_CASE)
    default: return nullptr;
    }
}

KernelInfo cube_info(int n)
{
    switch (n) {
        FFT3D_FOR_EACH_CUBE(FFT3D_CUBE_INFO)
    default: return {0, 0};
    }
}

KernelInfo cube_lines_info(int n)
{
    switch (n) {
        FFT3D_FOR_EACH_CUBE_LINES(FFT3D_CUBE_LINES_INFO)
    default: return {0, 0};
    }
}

}  // namespace fft3d
