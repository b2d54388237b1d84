// Two-pass form of cubic grids of 129 to 256 points a side: instances.
#include "kernels_split.hpp"
#include "registry.hpp"

namespace fft3d {

template <int N, int S>
static hipError_t launch_split_plane(const float2* in, float2* out, const float2* tw_x, const float2* tw_y, long planes,
                                     int cus, hipStream_t st)
{
    using G = SplitGeom<N>;
    if (in == out) {   // this pass alone: its rows move, so whole columns instead
        hipError_t e = axis_row_fn(N, S)(in, out, tw_x, planes * N, st);
        if (e == hipSuccess) {
            const long tiles = planes * split_y_tiles(N);
            hipLaunchKernelGGL((k_split_y<N, S>), dim3((unsigned)(tiles < kMaxBlocks ? tiles : kMaxBlocks)), dim3(G::T),
                               0, st, out, tw_y, tiles);
            e = hipGetLastError();
        }
        return e;
    }
    const long items = planes * G::R;
    const dim3 grid((unsigned)(items < cus ? items : cus));
    if (planes * N * N * (long)sizeof(float2) >= kStreamMinBytes)
        hipLaunchKernelGGL((k_split_plane<N, S, true>), grid, dim3(G::T), 0, st, in, out, tw_x, tw_y, items);
    else
        hipLaunchKernelGGL((k_split_plane<N, S, false>), grid, dim3(G::T), 0, st, in, out, tw_x, tw_y, items);
    return hipGetLastError();
}

template <int N, int S>
static hipError_t launch_split_z(const float2* in, float2* out, const float2* tw_z, const float2* root, long grids,
                                 int cus, hipStream_t st)
{
    using G = SplitGeom<N>;
    const long tiles = grids * G::N1 * G::XT;
    hipLaunchKernelGGL((k_split_z<N, S>), dim3((unsigned)(tiles < cus ? tiles : cus)), dim3(G::T), 0, st, in, out,
                       tw_z, root, tiles);
    return hipGetLastError();
}

template <int N, int S>
static hipError_t launch_split_cols(const float2* in, float2* out, const float2* tw, const AxisMap& m, hipStream_t st)
{
    constexpr int L = 32;   // as the strided passes of these lengths (k_axis_large.hip)
    const long blocks = (m.lines + L - 1) / L;
    return launch_tiles(in_runs(m, blocks, L, false), blocks, [&](const AxisMap& map, unsigned grid) {
        hipLaunchKernelGGL((k_axis_str<N, S, L, false, 0, 4>), dim3(grid), dim3(AxisGeom<N, L, 4>::T), 0, st, in, out,
                           tw, map, nullptr, nullptr, 0L, 0.0, nullptr, 0L);
    });
}

#define FFT3D_SPLIT_PLANE_CASE(n)                                              \
    case n:                                                                    \
        return sign < 0 ? &launch_split_plane<n, -1> : &launch_split_plane<n, 1>;
#define FFT3D_SPLIT_Z_CASE(n)                                                  \
    case n:                                                                    \
        return sign < 0 ? &launch_split_z<n, -1> : &launch_split_z<n, 1>;
#define FFT3D_SPLIT_COLS_CASE(n)                                               \
    case n:                                                                    \
        return sign < 0 ? &launch_split_cols<n, -1> : &launch_split_cols<n, 1>;
#define FFT3D_SPLIT_PARTS_CASE(n)                                              \
    case n:                                                                    \
        return SplitGeom<n>::R;

SplitPlaneFn split_plane_fn(int n, int sign)
{
    switch (n) {
        FFT3D_FOR_EACH_SPLIT_SIZE(FFT3D_SPLIT_PLANE_CASE)
    default: return nullptr;
    }
}

SplitZFn split_z_fn(int n, int sign)
{
    switch (n) {
        FFT3D_FOR_EACH_SPLIT_SIZE(FFT3D_SPLIT_Z_CASE)
    default: return nullptr;
    }
}

AxisVarFn split_cols_fn(int n, int sign)
{
    switch (n) {
        FFT3D_FOR_EACH_SPLIT_SIZE(FFT3D_SPLIT_COLS_CASE)
    default: return nullptr;
    }
}

#define FFT3D_SPLIT_INFO_PLANE(n)                                              \
    case n:                                                                    \
        return {SplitGeom<n>::T, (int)sizeof(float2) * SplitGeom<n>::PLANE_WORDS};
#define FFT3D_SPLIT_INFO_Z(n)                                                  \
    case n:                                                                    \
        return {SplitGeom<n>::T, (int)sizeof(float2) * SplitGeom<n>::Z_WORDS};
#define FFT3D_SPLIT_INFO_COLS(n)                                               \
    case n:                                                                    \
        return {AxisGeom<n, 32, 4>::T, (int)sizeof(float2) * AxisGeom<n, 32, 4>::WORDS};

KernelInfo split_plane_info(int n)
{
    switch (n) {
        FFT3D_FOR_EACH_SPLIT_SIZE(FFT3D_SPLIT_INFO_PLANE)
    default: return {0, 0};
    }
}

KernelInfo split_z_info(int n)
{
    switch (n) {
        FFT3D_FOR_EACH_SPLIT_SIZE(FFT3D_SPLIT_INFO_Z)
    default: return {0, 0};
    }
}

KernelInfo split_cols_info(int n)
{
    switch (n) {
        FFT3D_FOR_EACH_SPLIT_SIZE(FFT3D_SPLIT_INFO_COLS)
    default: return {0, 0};
    }
}

// A tile above 12300 points that is not whole turns (240) spills registers in
// the plane pass: it pays only where input and output are twice the 256 MB Infinity
// Cache and the third pass costs HBM traffic (240^3, inverse + forward: one
// grid 214 -> 231 us, four 975 -> 850).
bool split_batch_ok(int n, int batch)
{
    const int r = split_parts_of(n);
    if (r == 0) return false;
    return n / r * n <= 12300 || n % 64 == 0 || 16L * n * n * n * batch > (512L << 20);
}

int split_parts_of(int n)
{
    switch (n) {
        FFT3D_FOR_EACH_SPLIT_SIZE(FFT3D_SPLIT_PARTS_CASE)
    default: return 0;
    }
}

}  // namespace fft3d
