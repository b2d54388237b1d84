// xy-plane pass of grids whose x and y lengths differ: one plane per workgroup
// in LDS, x lines, then y lines, so that the grid takes two passes (this one
// and the strided z pass) instead of three.
//
// A kernel for every pair of lengths would be 1400 of them for each sign.  Here
// one kernel calls two out-of-line functions, one for the x length and one
// for the y length, each compiled for its length and any number of lines:
// the number of lines is a runtime value, the radix stages, twiddle offsets,
// register arrays and nearly all LDS offsets are not.  The x lines lie in the
// tile as rows of x (pitch odd(nx)); their last stage writes rows of y (pitch
// odd(ny)) for the y lines.  Nothing is prefetched: but for the largest planes
// two workgroups or more share a compute unit and overlap.  Inverse + forward
// in us, row and y passes -> this one, on buffers that change from call to call:
// 16 x (100, 72, 90) 180 -> 145 (100 for two sweeps at the copy rate), 200 x
// (24, 40, 30) 100 -> 76, 4 x (128, 125, 128) 140 -> 127, 64 x (128, 8, 64) 70 ->
// 57, one (20, 24, 18) 28 -> 17 (a launch less, and less host time a call).
#pragma once
#include <hip/hip_runtime.h>

#include "kernels_fp32.hpp"

namespace fft3d {

// Threads a plane and the points it may have, one class of planes each: 8 to 20
// points a thread, and ten, four, two and one workgroups on a compute unit:
// registers leave 20, 16, 16 and 16 waves, the largest planes take 9, 34, 80
// and 131 KB of LDS.
struct RectClass {
    int threads, points;
};
constexpr RectClass kRectClasses[4] = {{128, 1024}, {256, 4096}, {512, 10240}, {1024, 16384}};

// A scalar argument of an out-of-line function, which arrives in a vector
// register.
__device__ __forceinline__ unsigned rect_uniform(unsigned v) { return __builtin_amdgcn_readfirstlane(v); }

// LDS at byte offset `off`, as a pointer whose address space the compiler sees.
__device__ __forceinline__ float2* rect_lds(unsigned off)
{
    return (float2*)(reinterpret_cast<__attribute__((address_space(3))) float2*>(off));
}

// The stages from ST on of `lines` transforms of length N in the LDS tile:
// element e of line l at tile[l * odd(N) + e].  Consecutive lanes take
// consecutive lines (a butterfly's line and index by multiplication with
// magic = ceil(2^32 / lines), exact below 2^32 / lines butterflies).  The last
// stage writes element e of line l to dst[e * pitch + l]: OUT: in global
// memory; otherwise in the tile itself, whose reads it waits for.  C: the
// class of planes, lines * N <= its points.
template <int N, int S, int C, int ST, bool OUT>
__device__ __forceinline__ void rect_stages(float2* tile, const float2* tw, int lines, unsigned magic, float2* dst,
                                            int pitch, int tid)
{
    using P = Plan1D<N>;
    constexpr int T = kRectClasses[C].threads, LS = odd_stride(N);
    constexpr int R = P::radix(ST), NS = P::ns(ST), M = N / R, IT = (kRectClasses[C].points / R + T - 1) / T;
    constexpr bool LAST = ST == P::stages - 1;
    const int nb = lines * M;
    float2 v[IT][R];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const int b = tid + it * T;
        if (b < nb) {
            const int j = (int)__umulhi((unsigned)b, magic), line = b - j * lines;
            const float2* src = tile + line * LS + j;
#pragma unroll
            for (int q = 0; q < R; ++q) v[it][q] = src[q * M];
            if constexpr (NS > 1) {
                const float2* w = tw + P::tw_off(ST) + (j % NS) * (R - 1);
#pragma unroll
                for (int q = 1; q < R; ++q) v[it][q] = cmul(v[it][q], w[q - 1]);
            }
            dft<R, S>(v[it]);
        }
    }
    if constexpr (!LAST || !OUT) __syncthreads();
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const int b = tid + it * T;
        if (b < nb) {
            const int j = (int)__umulhi((unsigned)b, magic), line = b - j * lines;
            const int base = (j / NS) * NS * R + (j % NS);
            if constexpr (LAST) {
                float2* d = dst + base * pitch + line;
#pragma unroll
                for (int q = 0; q < R; ++q) d[q * NS * pitch] = v[it][q];
            } else {
                float2* d = tile + line * LS + base;
#pragma unroll
                for (int q = 0; q < R; ++q) d[q * NS] = v[it][q];
            }
        }
    }
    if constexpr (!LAST) {
        __syncthreads();
        rect_stages<N, S, C, ST + 1, OUT>(tile, tw, lines, magic, dst, pitch, tid);
    }
}

// All stages of the x lines (OUT = false: the result in the tile, rows of y of
// pitch `pitch`) or of the y lines (OUT: the result at out, rows of `pitch` = nx).
template <int N, int S, int C, bool OUT>
__device__ __noinline__ void rect_lines(unsigned tile_, unsigned tw_, int lines_, unsigned magic_, float2* out_,
                                        int pitch_)
{
    const unsigned long long o = reinterpret_cast<unsigned long long>(out_);
    const unsigned long long ou = ((unsigned long long)rect_uniform((unsigned)(o >> 32)) << 32) | rect_uniform((unsigned)o);
    float2* tile = rect_lds(rect_uniform(tile_));
    float2* dst = OUT ? (float2*)(reinterpret_cast<__attribute__((address_space(1))) float2*>(ou)) : tile;
    rect_stages<N, S, C, 0, OUT>(tile, rect_lds(rect_uniform(tw_)), (int)rect_uniform((unsigned)lines_),
                                 rect_uniform(magic_), dst, (int)rect_uniform((unsigned)pitch_), (int)threadIdx.x);
}

// Geometry of a rectangular plane pass, filled by the host.
struct RectArgs {
    const float2* in;
    float2* out;
    const float2 *tw_x, *tw_y;   // twiddle tables of the two lengths
    int ntw_x, ntw_y;            // their lengths
    long planes;
    int nx, ny;
    int tile;                    // points of the LDS tile: max(ny odd(nx), nx odd(ny))
    unsigned magic_nx, magic_ny; // ceil(2^32 / nx), ceil(2^32 / ny)
    unsigned magic_row;          // ceil(2^32 / units a row), a unit = 16 bytes (nx even) or 8
};

template <int S, int C>
__global__ void __launch_bounds__(kRectClasses[C].threads, 4) k_plane_rect(RectArgs a)
{
    constexpr int T = kRectClasses[C].threads;
    extern __shared__ float2 lds[];
    const int tid = threadIdx.x;
    const int rs = odd_stride(a.nx);
    float2* twx = lds + a.tile;
    float2* twy = twx + a.ntw_x;
    const unsigned tile_off = (unsigned)(size_t)(__attribute__((address_space(3))) float2*)lds;
    const unsigned twx_off = tile_off + (unsigned)a.tile * sizeof(float2);
    const unsigned twy_off = twx_off + (unsigned)a.ntw_x * sizeof(float2);
    for (int i = tid; i < a.ntw_x; i += T) twx[i] = a.tw_x[i];   // visible after the first barrier below
    for (int i = tid; i < a.ntw_y; i += T) twy[i] = a.tw_y[i];
    const long pts = (long)a.nx * a.ny;
    for (long p = blockIdx.x; p < a.planes; p += gridDim.x) {
        constexpr int U = 4;   // loads in flight a lane
        if (a.nx % 2 == 0) {
            const float4* src = reinterpret_cast<const float4*>(a.in + p * pts);
            const int w = a.nx / 2, n = a.ny * w;
            for (int i0 = tid; i0 < n; i0 += U * T) {
                float4 r[U];
#pragma unroll
                for (int k = 0; k < U; ++k)
                    if (i0 + k * T < n) r[k] = src[i0 + k * T];
#pragma unroll
                for (int k = 0; k < U; ++k) {
                    const int i = i0 + k * T;
                    if (i < n) {
                        const int y = w == 1 ? i : (int)__umulhi((unsigned)i, a.magic_row);
                        float2* d = lds + y * rs + 2 * (i - y * w);
                        d[0] = make_float2(r[k].x, r[k].y);
                        d[1] = make_float2(r[k].z, r[k].w);
                    }
                }
            }
        } else {
            const float2* src = a.in + p * pts;
            const int n = a.ny * a.nx;
            for (int i0 = tid; i0 < n; i0 += U * T) {
                float2 r[U];
#pragma unroll
                for (int k = 0; k < U; ++k)
                    if (i0 + k * T < n) r[k] = src[i0 + k * T];
#pragma unroll
                for (int k = 0; k < U; ++k) {
                    const int i = i0 + k * T;
                    if (i < n) {
                        const int y = (int)__umulhi((unsigned)i, a.magic_row);
                        lds[y * rs + (i - y * a.nx)] = r[k];
                    }
                }
            }
        }
        __syncthreads();
        switch (a.nx) {
#define FFT3D_RECT_X(m)                                                                                        \
    case m: rect_lines<m, S, C, false>(tile_off, twx_off, a.ny, a.magic_ny, nullptr, odd_stride(a.ny)); break;
            FFT3D_FOR_EACH_SIZE(FFT3D_RECT_X)
#undef FFT3D_RECT_X
        default: break;
        }
        __syncthreads();
        switch (a.ny) {
#define FFT3D_RECT_Y(m)                                                                                        \
    case m: rect_lines<m, S, C, true>(tile_off, twy_off, a.nx, a.magic_nx, a.out + p * pts, a.nx); break;
            FFT3D_FOR_EACH_SIZE(FFT3D_RECT_Y)
#undef FFT3D_RECT_Y
        default: break;
        }
        __syncthreads();   // the tile is free for the next plane
    }
}

}  // namespace fft3d
