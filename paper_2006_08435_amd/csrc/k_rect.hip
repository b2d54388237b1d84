// Rectangular xy-plane pass (Nx != Ny, both up to 128): class choice and launch.
#include "kernels_rect.hpp"
#include "registry.hpp"

namespace fft3d {

static int rect_tile(int nx, int ny)
{
    const int a = ny * odd_stride(nx), b = nx * odd_stride(ny);
    return a > b ? a : b;
}

static int rect_lds_bytes(int nx, int ny)
{
    return (int)sizeof(float2) *
           (rect_tile(nx, ny) + sched_tw_len(make_sched(nx)) + sched_tw_len(make_sched(ny)));
}

// The smallest class that has room for the plane; 512 threads only where two
// such workgroups fit the 160 KB of a compute unit (just above, at 81 x 125 and
// 100 x 100, one alone waits for its barriers: 209 -> 218 us against the row
// and y passes, 206 with 1024 threads).  Up to a plane a compute unit nothing
// shares one, and twice the threads halve every stage (us a plane pass replayed
// from a graph, this class / the next: 100 x 72 x 32 9.0 / 8.2, x 256 12.1 /
// 11.4; 125 x 75 x 32 12.9 / 12.1; 60 x 48 x 32 7.1 / 6.4; but 24 x 20 x 32, of the
// smallest class, 4.7 / 4.9).
constexpr long kRectOneTurn = 256;
static int rect_class(int nx, int ny, long planes)
{
    for (int c = 0; c < 4; ++c)
        if (nx * ny <= kRectClasses[c].points && (c != 2 || rect_lds_bytes(nx, ny) <= 80 * 1024))
            return (c == 1 || c == 2) && planes <= kRectOneTurn ? c + 1 : c;
    return -1;
}

// Small planes keep the row and y passes once there are many: a workgroup of
// 128 threads waits for its barriers with next to no work (400 x (8, 9, 128),
// inverse + forward, 67 -> 116 us; 2000 x (12, 20, 18) 138 -> 142; 300 x (15,
// 18, 100) even; 900 x (32, 16, 8) 61 -> 52).  Where one turn of the device
// takes all planes, a launch less decides (one (20, 24, 18) 32 -> 26 us).
// A few large planes lose on the device what the launch saves the host (row and
// y passes / this one: 125 x 75 x 1 8.7 / 11.2, x 64 13.9 / 12.4; 128 x 125 x 1 9.8 /
// 13.5, x 128 17.8 / 17.2; 128 x 96 x 1 8.6 / 9.9, x 32 11.5 / 10.6).
constexpr int kRectMinPoints = 300;
constexpr long kRectFewPlanes = 2048;

bool rect_init(int nx, int ny, long planes, int sign)
{
    constexpr int kMaxLds = 160 * 1024;
    if (nx > 128 || ny > 128 || nx < 2 || ny < 2) return false;
    if (nx * ny < kRectMinPoints && planes > kRectFewPlanes) return false;
    const int c = rect_class(nx, ny, planes);
    if (c < 0 || rect_lds_bytes(nx, ny) > kMaxLds) return false;
    if (hipFuncSetAttribute(sign < 0 ? rect_fwd_kernel(c) : rect_inv_kernel(c),
                            hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return true;
}

KernelInfo rect_info(int nx, int ny, long planes)
{
    return {kRectClasses[rect_class(nx, ny, planes)].threads, rect_lds_bytes(nx, ny)};   // of a plane that rect_init took
}

hipError_t launch_plane_rect(const float2* in, float2* out, const float2* tw_x, const float2* tw_y, int nx, int ny,
                             long planes, int sign, hipStream_t st)
{
    auto magic = [](int d) { return (unsigned)(((1ull << 32) + d - 1) / d); };
    const RectArgs a{in,         out,       tw_x,      tw_y,     sched_tw_len(make_sched(nx)),
                     sched_tw_len(make_sched(ny)),     planes,   nx,   ny,   rect_tile(nx, ny),
                     magic(nx),  magic(ny), nx % 2 ? magic(nx) : (nx > 2 ? magic(nx / 2) : 0u)};
    const unsigned grid = (unsigned)(planes < kMaxBlocks ? planes : kMaxBlocks);
    return (sign < 0 ? rect_fwd : rect_inv)(rect_class(nx, ny, planes), a, grid, (size_t)rect_lds_bytes(nx, ny), st);
}

}  // namespace fft3d
