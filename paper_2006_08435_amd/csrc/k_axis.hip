// Single-axis pass kernel instances: strided (y, z) and row (x) forms.
#include "kernels_fp32.hpp"
#include "registry.hpp"

namespace fft3d {

// Sum of n FP64 partials in a fixed order, by one workgroup.  It is bound by
// the latency of its loads, so every thread keeps four running sums over
// loads that do not wait for each other, and 1024 threads share the list: the
// 18432 partials of 128 x 96^3 took 19 us with 256 threads and one sum each.
constexpr int kSumThreads = 1024;
__global__ void __launch_bounds__(kSumThreads)
k_sum_partials(const double* __restrict__ p, long n, double* __restrict__ out)
{
    __shared__ double red[kSumThreads / 64];
    const int tid = threadIdx.x;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    long i = tid;
    for (; i + 3 * kSumThreads < n; i += 4 * kSumThreads) {
        s0 += p[i];
        s1 += p[i + kSumThreads];
        s2 += p[i + 2 * kSumThreads];
        s3 += p[i + 3 * kSumThreads];
    }
    for (; i < n; i += kSumThreads) s0 += p[i];
    const double t = block_sum<kSumThreads>((s0 + s1) + (s2 + s3), red, tid);
    if (tid == 0) out[0] = t;
}

long axis_str_blocks(long lines) { return (lines + kAxisLines - 1) / kAxisLines; }

hipError_t launch_sum_partials(const double* partials, long n, double* out, hipStream_t st)
{
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(kSumThreads), 0, st, partials, n, out);
    return hipGetLastError();
}

template <int N, int S>
static hipError_t launch_axis_str(const float2* in, float2* out, const float2* tw, const AxisMap& m, int energy,
                                  const float* V, double* partials, long vol, hipStream_t st)
{
    const long blocks = axis_str_blocks(m.lines);
    constexpr int T = AxisGeom<N, kAxisLines>::T;
    return launch_tiles(in_runs(m, blocks, kAxisLines, energy != 0), blocks, [&](const AxisMap& map, unsigned grid) {
        if (energy == 2)
            hipLaunchKernelGGL((k_axis_energy<N, S, kAxisLines>), dim3(grid), dim3(T), 0, st, in, tw, map, V, partials,
                               vol);
        else if (energy)
            hipLaunchKernelGGL((k_axis_str<N, S, kAxisLines, true>), dim3(grid), dim3(T), 0, st, in, out, tw, map, V,
                               partials, vol, 0.0);
        else
            hipLaunchKernelGGL((k_axis_str<N, S, kAxisLines, false>), dim3(grid), dim3(T), 0, st, in, out, tw, map, V,
                               partials, vol, 0.0);
    });
}

template <int N, int S>
static hipError_t launch_axis_str_pruned(const float2* in, float2* out, const float2* tw, const AxisMap& map,
                                         double R2, const SphereRow* rows, long npts, hipStream_t st)
{
    const long blocks = axis_str_blocks(map.lines);
    constexpr int T = AxisGeom<N, kAxisLines>::T;
    if (S > 0 && rows) return hipErrorInvalidValue;
    // inverse plans prune the loads (sphere-limited input), forward plans
    // lines and stores (optionally scattering into a packed sphere).  Forward
    // tiles keep launch order: their lines outside the sphere are skipped, and
    // runs of an eighth of a grid would leave the XCDs of the middle ones idle
    // (forward to a packed sphere, us, launch order / runs: 92 x 75^3 169 / 203,
    // 32 x 90^3 98 / 114, 20 x 81^3 55 / 64; inverse 32 x 90^3 87 / 82).
    const AxisMap order = S > 0 ? in_runs(map, blocks, kAxisLines, false) : map;
    return launch_tiles(order, blocks, [&](const AxisMap& m, unsigned grid) {
        if constexpr (S < 0) {
            if (rows) {
                hipLaunchKernelGGL((k_axis_str<N, S, kAxisLines, false, 3>), dim3(grid), dim3(T), 0, st, in, out, tw, m,
                                   nullptr, nullptr, 0L, R2, rows, npts);
                return;
            }
        }
        hipLaunchKernelGGL((k_axis_str<N, S, kAxisLines, false, (S > 0 ? 1 : 2)>), dim3(grid), dim3(T), 0, st, in, out,
                           tw, m, nullptr, nullptr, 0L, R2, nullptr, 0L);
    });
}

#define FFT3D_STR_PRUNED_CASE(n)                                               \
    case n:                                                                    \
        return sign < 0 ? &launch_axis_str_pruned<n, -1> : &launch_axis_str_pruned<n, 1>;

AxisStrPrunedFn axis_str_pruned_fn(int n, int sign)
{
    switch (n) {
        FFT3D_FOR_EACH_SIZE(FFT3D_STR_PRUNED_CASE)
    default: return nullptr;
    }
}

template <int N>
static hipError_t launch_hloc(float2* buf, const float2* tw_inv, const float2* tw_fwd, const AxisMap& map,
                              const float* V, const double* scale, float mult, double* partials, long vol, double R2,
                              int mode, hipStream_t st)
{
    const long blocks = axis_str_blocks(map.lines);
    // the pruned form gains from whole cache lines only (64 x 80^3 249 us, in runs 251)
    constexpr int T = AxisGeom<N, kAxisLines>::T;
    return launch_tiles(in_runs(map, blocks, kAxisLines, mode == 0), blocks, [&](const AxisMap& m, unsigned grid) {
        if (mode)
            hipLaunchKernelGGL((k_axis_hloc<N, kAxisLines, 1>), dim3(grid), dim3(T), 0, st, buf, tw_inv, tw_fwd, m, V,
                               scale, mult, partials, vol, R2);
        else
            hipLaunchKernelGGL((k_axis_hloc<N, kAxisLines, 0>), dim3(grid), dim3(T), 0, st, buf, tw_inv, tw_fwd, m, V,
                               scale, mult, partials, vol, R2);
    });
}

#define FFT3D_HLOC_CASE(n)                                                     \
    case n:                                                                    \
        return &launch_hloc<n>;

HlocFn axis_hloc_fn(int n)
{
    switch (n) {
        FFT3D_FOR_EACH_SIZE(FFT3D_HLOC_CASE)
    default: return nullptr;
    }
}

constexpr int kDensityLines = 32;

// Orbital ranges of the density's z pass, from sweeps of both limits below.
// Fewer tiles than compute units need more workgroups at any price (ranges of
// four orbitals or more: 30 orbitals at 64^3 47 -> 29 us, 256 at 32^3 250 ->
// 31).  From 200 tiles on (80^2 lines) the split only evens out the last turn
// and hides latency, and the partial sums cost: ranges of 16 orbitals or more
// (128 at 96^3 342 -> 252 us; 40 at 90^3 143 -> 139, with ranges of ten 151).
// 512 tiles (128^2 lines) are two for every compute unit and gain nothing (32
// orbitals at 128^3 147 us in one range, 157 in two).
static int density_splits(long tiles, int batch)
{
    if (tiles >= 512) return 1;
    const long want = (tiles >= 200 ? 1536 : 1024) / tiles, most = batch / (tiles >= 200 ? 16 : 4);
    const long s = want < most ? want : most;
    return (int)(s < 1 ? 1 : s);
}

template <int N>
static hipError_t launch_density(float2* buf, const float2* tw, const AxisMap& m, int batch, long vol,
                                 const float* occ, float* rho, double R2, int mode, hipStream_t st)
{
    const int tiles = (int)((m.lines + kDensityLines - 1) / kDensityLines), splits = density_splits(tiles, batch);
    const OrbitalRanges ranges{splits, batch / splits, batch % splits};
    const dim3 grid((unsigned)tiles, (unsigned)splits), block(AxisGeom<N, kDensityLines>::T);
    if (mode)
        hipLaunchKernelGGL((k_axis_density<N, kDensityLines, 1>), grid, block, 0, st, buf, tw, m, vol, occ, rho, R2,
                           ranges);
    else
        hipLaunchKernelGGL((k_axis_density<N, kDensityLines, 0>), grid, block, 0, st, buf, tw, m, vol, occ, rho, R2,
                           ranges);
    if (splits > 1)
        hipLaunchKernelGGL((k_density_sum<kDensityLines>), dim3((unsigned)((vol + 255) / 256)), dim3(256), 0, st, buf,
                           rho, vol, (int)m.lines, ranges);
    return hipGetLastError();
}

#define FFT3D_DENSITY_CASE(n)                                                  \
    case n:                                                                    \
        return &launch_density<n>;

DensityFn axis_density_fn(int n)
{
    switch (n) {
        FFT3D_FOR_EACH_SIZE(FFT3D_DENSITY_CASE)
    default: return nullptr;
    }
}

// Workgroups of the packed-sphere copies: one per plane (grid-stride beyond
// 2^20) of four waves, or of one for up to 128 points.  Where planes fill the
// device several times over, one wave serves up to 320 points better, as four
// have little to do each (unpack / pack us, replayed, four waves -> one: 587 x 15^3
// 9.4 / 4.7 -> 7.5 / 4.7, 873 x 18^3 14.1 -> 10.1, 300 x 24^3 10.5 -> 9.2, 200 x 25^3
// pack 6.1 -> 4.1; but 111 x 30^3, 450 pairs, 7.2 -> 8.2).
static dim3 sphere_grid(long planes) { return dim3((unsigned)(planes < (1L << 20) ? planes : (1L << 20))); }
static dim3 sphere_block(long planes, long points) { return dim3(points > (planes >= 2048 ? 320 : 128) ? 256 : 64); }
// Workgroups that share a plane of `units` units: as many as make 2048 of them
// in all, eight a compute unit, with a unit or more a thread.  With one a plane
// two grids of 125^3 took 30.4 us and one of 128^3 17.4, so 10.6 and 7.6 (one
// point of all grids a thread: 10.6 and 8.7); from 2048 planes on it is one.
static unsigned sphere_parts(long planes, long units)
{
    const long want = (2047 + planes) / planes, most = (units + 255) / 256;
    return (unsigned)(want < most ? want : most);
}

hipError_t launch_sphere_pack(const float2* src, float2* dst, const SphereRow* rows, long npts, const int* zlist,
                              int nzp, int nz, const SphereAxis& ax, const SphereAxis& ay, long batch, hipStream_t st)
{
    const long planes = batch * nzp;
    if (planes <= 0) return hipSuccess;
    const dim3 block = sphere_block(planes, (long)ax.count() * ay.count());
    hipLaunchKernelGGL(k_sphere_pack, sphere_grid(planes), block, 0, st, src, dst, rows, npts, zlist, nzp, nz, ax, ay,
                       planes);
    return hipGetLastError();
}

hipError_t launch_sphere_unpack(const float2* src, float2* dst, const SphereRow* rows, long npts, int nz, int ny,
                                int nx, double R2, long batch, hipStream_t st)
{
    const long planes = batch * nz, units = (long)ny * nx / (nx % 2 == 0 ? 2 : 1);
    const dim3 block = sphere_block(planes, units);
    dim3 grid = sphere_grid(planes);
    grid.y = sphere_parts(planes, units);
    if (nx % 2 == 0)   // every row, so every plane, starts on 16 bytes
        hipLaunchKernelGGL(k_sphere_unpack<2>, grid, block, 0, st, src, dst, rows, npts, nz, ny, nx, R2, planes);
    else
        hipLaunchKernelGGL(k_sphere_unpack<1>, grid, block, 0, st, src, dst, rows, npts, nz, ny, nx, R2, planes);
    return hipGetLastError();
}

template <int N, int S>
static hipError_t launch_axis_row(const float2* in, float2* out, const float2* tw, long rows, hipStream_t st)
{
    const long blocks = (rows + kRowLines - 1) / kRowLines;
    return launch_blocks(blocks, [&](long first, unsigned grid) {
        const long r0 = first * kRowLines;
        hipLaunchKernelGGL((k_axis_row<N, S, kRowLines>), dim3(grid), dim3(RowGeom<N, kRowLines>::T), 0, st,
                           in + r0 * N, out + r0 * N, tw, rows - r0);
    });
}

#define FFT3D_STR_CASE(n)                                                      \
    case n:                                                                    \
        return sign < 0 ? &launch_axis_str<n, -1> : &launch_axis_str<n, 1>;
#define FFT3D_ROW_CASE(n)                                                      \
    case n:                                                                    \
        return sign < 0 ? &launch_axis_row<n, -1> : &launch_axis_row<n, 1>;
#define FFT3D_STR_INFO(n)                                                      \
    case n:                                                                    \
        return {AxisGeom<n, kAxisLines>::T,                                    \
                (int)((Plan1D<n>::stages > 1 ? AxisGeom<n, kAxisLines>::WORDS : 1) * sizeof(float2))};
#define FFT3D_ROW_INFO(n)                                                      \
    case n:                                                                    \
        return {RowGeom<n, kRowLines>::T, (int)(RowGeom<n, kRowLines>::WORDS * sizeof(float2))};

AxisStrFn axis_str_fn(int n, int sign)
{
    if (n > 128) return axis_str_large_fn(n, sign);
    switch (n) {
        FFT3D_FOR_EACH_SIZE(FFT3D_STR_CASE)
    default: return nullptr;
    }
}

AxisRowFn axis_row_fn(int n, int sign)
{
    if (n > 128) return axis_row_large_fn(n, sign);
    switch (n) {
        FFT3D_FOR_EACH_SIZE(FFT3D_ROW_CASE)
    default: return nullptr;
    }
}

KernelInfo axis_str_info(int n)
{
    if (n > 128) return axis_str_large_info(n);
    switch (n) {
        FFT3D_FOR_EACH_SIZE(FFT3D_STR_INFO)
    default: return {0, 0};
    }
}

KernelInfo axis_row_info(int n)
{
    if (n > 128) return axis_row_large_info(n);
    switch (n) {
        FFT3D_FOR_EACH_SIZE(FFT3D_ROW_INFO)
    default: return {0, 0};
    }
}

}  // namespace fft3d
