// Cubic grids above 128 points a side in two passes.
//
// An N x N plane above 128^2 does not fit a compute unit, but R interleaved
// parts of it do: with y = y0 + R y1 and ky = k1 + N1 k2 (N = R N1),
//   Y[k1 + N1 k2] = sum_y0 W_R^(y0 k2) W_N^(y0 k1) A_y0[k1],
//   A_y0[k1]      = sum_y1 y[y0 + R y1] W_N1^(y1 k1).
// Pass one (k_split_plane) takes the rows y0 + R y1 of a plane as one LDS
// tile: x lines, then the length-N1 transforms along y1; A_y0 goes to the rows
// N1 y0 + k1.  Pass two (k_split_z) takes, for one k1, the R rows k1 + N1 y0
// of every plane, L points of x at a time: twiddle and R-point DFT across y0 in
// registers (the factors are the same for the whole tile), then the z lines in
// LDS, stored to the rows k1 + N1 k2.  Its tile reads and writes the same
// points, so it runs in place; pass one moves rows, so a transform with in ==
// out takes three passes: rows, whole y columns with the same butterflies
// (k_axis_str of schedule kind 4), and the plain z pass.  They leave the same
// bits.  Whole columns also serve a caller who runs pass one alone in place
// (k_split_y).  In place, copy of the input included, us, the three passes with
// default radices -> these: 16 x 150^3 670 -> 623, 8 x 162^3 417 -> 375,
// 12 x 160^3 557 -> 557, 4 x 256^3 761 -> 763, one 256^3 166.1 -> 168.5, one
// 144^3 38.0 -> 38.9 (a third stage along y; worst is one 180^3, alone and
// replayed from a graph 54.2 -> 57.2), one 135^3 44.1 -> 40.0; rows,
// k_split_y and k_split_z instead: 794, 500, 588, 820, 173.5, 43.6, 50.1.
// Both passes hold one tile of up to 16384 points a compute unit, bound by HBM
// and their barriers as k_plane_pf is.  Inverse + forward in us, three passes
// -> two: 4 x 256^3 1161 -> 776 (322 at the copy rate for one sweep each way),
// 8 x 192^3 995 -> 627, 8 x 200^3 1237 -> 841, 12 x 160^3 861 -> 540, 16 x 150^3
// 1067 -> 798, one 256^3 254 -> 195, one 150^3 or 144^3 unchanged.
#pragma once
#include <hip/hip_runtime.h>

#include "kernels_fp32.hpp"

namespace fft3d {

#define FFT3D_FOR_EACH_SPLIT_SIZE(X)                                           \
    X(135) X(144) X(150) X(160) X(162) X(180) X(192) X(200) X(216) X(240)      \
    X(256)

// The list holds exactly the lengths that the rule accepts.
constexpr bool split_listed(int n)
{
#define FFT3D_SPLIT_LISTED(m) if (n == m) return true;
    FFT3D_FOR_EACH_SPLIT_SIZE(FFT3D_SPLIT_LISTED)
#undef FFT3D_SPLIT_LISTED
    return false;
}
constexpr bool split_list_is_rule()
{
    for (int n = 129; n <= 256; ++n) {
        int m = n;
        while (m % 2 == 0) m /= 2;
        while (m % 3 == 0) m /= 3;
        while (m % 5 == 0) m /= 5;
        if (m == 1 && split_ok(n) != split_listed(n)) return false;
    }
    return true;
}
static_assert(split_list_is_rule(), "FFT3D_FOR_EACH_SPLIT_SIZE and split_ok");

template <int N>
struct SplitGeom {
    static_assert(split_ok(N), "a length of the two-pass form");
    static constexpr int R = split_parts(N), N1 = N / R, L = split_lines(N, R);
    static constexpr int T = 1024;
    // plane tile: N1 rows of N points
    static constexpr int RS = odd_stride(N), PLANE_WORDS = N1 * RS;
    // z tile: N rows of R * L lines (the x points of k2 = 0, of k2 = 1, ...)
    static constexpr int LINES = R * L, LP = odd_stride(LINES), Z_WORDS = N * LP;
    static constexpr int XT = (N + L - 1) / L;   // tiles along x, the last one ragged
    static constexpr int VEC = N % 2 == 0 ? 2 : 1;
};

// Rows base + i * stride (i < ROWS) of ROW points in registers, as 16-byte
// pairs for even rows.
template <int ROWS, int ROW, int T, bool NT>
struct RowRegs {
    static constexpr bool PAIRS = ROW % 2 == 0;
    static constexpr int W = PAIRS ? ROW / 2 : ROW, UNITS = ROWS * W, IT = (UNITS + T - 1) / T;
    typedef float f4v __attribute__((ext_vector_type(4)));
    typedef float f2v __attribute__((ext_vector_type(2)));
    using U = typename std::conditional<PAIRS, f4v, f2v>::type;
    U r[IT];

    __device__ __forceinline__ void load(const float2* base, int stride, int tid)
    {
#pragma unroll
        for (int k = 0; k < IT; ++k) {
            const int i = tid + k * T;
            if (UNITS % T == 0 || i < UNITS) {
                const int row = i / W, c = i - row * W;
                const U* p = reinterpret_cast<const U*>(base + (long)row * stride) + c;
                if constexpr (NT) r[k] = __builtin_nontemporal_load(p);
                else r[k] = *p;
            }
        }
    }
    template <int RS>
    __device__ __forceinline__ void store_lds(float2* lds, int tid) const
    {
#pragma unroll
        for (int k = 0; k < IT; ++k) {
            const int i = tid + k * T;
            if (UNITS % T == 0 || i < UNITS) {
                const int row = i / W, c = i - row * W;
                if constexpr (PAIRS) {
                    lds[row * RS + 2 * c] = make_float2(r[k].x, r[k].y);
                    lds[row * RS + 2 * c + 1] = make_float2(r[k].z, r[k].w);
                } else {
                    lds[row * RS + c] = make_float2(r[k].x, r[k].y);
                }
            }
        }
    }
};

// Pass one: item i = (plane, y0), persistent, the next item's rows in flight
// while this one is transformed (as k_plane_pf).  in != out.
template <int N, int S, bool NT>
__global__ void __launch_bounds__(SplitGeom<N>::T)
k_split_plane(const float2* in, float2* out, const float2* __restrict__ tw_x, const float2* __restrict__ tw_y, long items)
{
    using G = SplitGeom<N>;
    constexpr int R = G::R, N1 = G::N1, T = G::T, RS = G::RS;
    __shared__ float2 lds[G::PLANE_WORDS];
    // lines not a multiple of 64: a wave's butterflies span two twiddle groups
    // and read them per lane, from an LDS copy
    constexpr bool TWX = N1 % 64 != 0, TWY = N % 64 != 0;
    constexpr int NX = Plan1D<N>::tw_len, NY = Plan1D<N1>::tw_len;
    __shared__ float2 twx_lds[TWX && NX > 0 ? NX : 1];
    __shared__ float2 twy_lds[TWY && NY > 0 ? NY : 1];
    const int tid = threadIdx.x;
    if constexpr (TWX && NX > 0) {
        for (int i = tid; i < NX; i += T) twx_lds[i] = tw_x[i];   // visible after the first barrier below
        tw_x = twx_lds;
    }
    if constexpr (TWY && NY > 0) {
        for (int i = tid; i < NY; i += T) twy_lds[i] = tw_y[i];
        tw_y = twy_lds;
    }
    RowRegs<N1, N, T, NT> regs;
    auto load = [&](long i) {
        const long p = i / R;
        regs.load(in + p * (N * N) + (int)(i - p * R) * N, R * N, tid);
    };
    long i = blockIdx.x;
    if (i < items) load(i);
    for (; i < items; i += gridDim.x) {
        regs.template store_lds<RS>(lds, tid);
        __syncthreads();
        if (i + gridDim.x < items) load(i + gridDim.x);
        fft_lds_all<N, S, N1, T, RS, 1>(lds, tw_x, tid);
        // the y1 lines: part y0 fills the rows N1 y0 .. of the plane, and the
        // parts of a plane follow each other, so item i starts at row N1 i
        float2* dst = out + i * (N1 * N);
        if constexpr (pairs_ok<N1, N, 0>(T)) {
            tail_pairs<N1, S, N, T, 0, 0>(LdsAcc<1, RS>{lds}, dst, (long)N, tw_y, tid);
        } else {
            const LdsAcc<1, RS> col{lds};
            const PlaneColOut<N> o{dst};
            run_tail<N1, S, N, T, 0, false>(col, o, tw_y, tid);
        }
        __syncthreads();
    }
}

// The length-N1 transforms of pass one on whole columns, for pass one run
// alone in place: the rows already transformed along x.  A workgroup takes L
// adjacent columns of a plane.
constexpr int kSplitYLines = 16;
constexpr int split_y_tiles(int n) { return (n + kSplitYLines - 1) / kSplitYLines; }   // of a plane

template <int N, int S>
__global__ void __launch_bounds__(SplitGeom<N>::T)
k_split_y(float2* buf, const float2* __restrict__ tw_y, long tiles)
{
    using G = SplitGeom<N>;
    constexpr int R = G::R, N1 = G::N1, T = G::T, L = kSplitYLines, LP = odd_stride(L), XT = split_y_tiles(N);
    __shared__ float2 lds[N * LP];
    const int tid = threadIdx.x;
    for (long t = blockIdx.x; t < tiles; t += gridDim.x) {
        const long p = t / XT;
        const int x0 = (int)(t - p * XT) * L;
        float2* plane = buf + p * (N * N) + x0;
        for (int i = tid; i < N * L; i += T) {
            const int y = i / L, x = i - y * L;
            lds[y * LP + x] = x0 + x < N ? plane[(long)y * N + x] : make_float2(0.f, 0.f);
        }
        __syncthreads();
        // line (y0, x): element y1 is the tile's row y0 + R y1, the result row N1 y0 + k1
        struct Out {
            float2* p;
            int valid;
            __device__ __forceinline__ void store(int line, int e, float2 v) const
            {
                const int y0 = line / L, x = line - y0 * L;
                if (x < valid) p[(long)(N1 * y0 + e) * N + x] = v;
            }
        };
        const LdsAcc2<L, LP, 1, R * LP> a{lds};
        const Out o{plane, N - x0};
        run_tail<N1, S, R * L, T, 0, false>(a, o, tw_y, tid);
        __syncthreads();   // the tile is free for the next one
    }
}

// Pass two: tile t = (grid, k1, x tile), persistent with the next tile's points
// in flight; in == out allowed.  root[m] = W_N^m.
template <int N, int S>
__global__ void __launch_bounds__(SplitGeom<N>::T)
k_split_z(const float2* in, float2* out, const float2* __restrict__ tw_z, const float2* __restrict__ root, long tiles)
{
    using G = SplitGeom<N>;
    constexpr int R = G::R, N1 = G::N1, T = G::T, L = G::L, LINES = G::LINES, LP = G::LP, XT = G::XT, VEC = G::VEC;
    __shared__ float2 lds[G::Z_WORDS];
    constexpr bool TWZ = LINES % 64 != 0;
    constexpr int NZ = Plan1D<N>::tw_len;
    __shared__ float2 tw_lds[TWZ && NZ > 0 ? NZ : 1];
    const int tid = threadIdx.x;
    if constexpr (TWZ && NZ > 0) {
        for (int i = tid; i < NZ; i += T) tw_lds[i] = tw_z[i];   // visible after the first barrier below
        tw_z = tw_lds;
    }
    // the tiles of the grid written last come first (still in the caches)
    struct Where {
        long base;    // of its grid
        int k1, x0;
    };
    auto where = [&](long t) {
        const long u = tiles - 1 - t, g = u / (N1 * XT);
        const int r = (int)(u - g * (N1 * XT)), k1 = r / XT;
        return Where{g * ((long)N * N * N), k1, (r - k1 * XT) * L};
    };
    // units of VEC points along x: LV a run, N runs (z), R rows each
    constexpr int LV = L / VEC, UNITS = N * LV, IT = (UNITS + T - 1) / T;
    typedef float fv __attribute__((ext_vector_type(2 * VEC)));
    fv r[IT][R];
    auto load = [&](const Where& w) {
        const float2* src = in + w.base + w.k1 * N + w.x0;
#pragma unroll
        for (int k = 0; k < IT; ++k) {
            const int i = tid + k * T, z = i / LV, x = (i - z * LV) * VEC;
            if ((UNITS % T == 0 || i < UNITS) && w.x0 + x < N) {
#pragma unroll
                for (int q = 0; q < R; ++q)
                    r[k][q] = *reinterpret_cast<const fv*>(src + (long)z * (N * N) + q * (N1 * N) + x);
            }
        }
    };
    long t = blockIdx.x;
    Where w = where(t < tiles ? t : 0);
    if (t < tiles) load(w);
    for (; t < tiles; t += gridDim.x) {
        float2 f[R];
#pragma unroll
        for (int q = 1; q < R; ++q) f[q] = root[q * w.k1];   // uniform
#pragma unroll
        for (int k = 0; k < IT; ++k) {
            const int i = tid + k * T, z = i / LV, x = (i - z * LV) * VEC;
            if (UNITS % T == 0 || i < UNITS) {
#pragma unroll
                for (int c = 0; c < VEC; ++c) {
                    float2 v[R];
#pragma unroll
                    for (int q = 0; q < R; ++q) v[q] = make_float2(r[k][q][2 * c], r[k][q][2 * c + 1]);
#pragma unroll
                    for (int q = 1; q < R; ++q) v[q] = cmul(v[q], f[q]);
                    dft<R, S>(v);
#pragma unroll
                    for (int q = 0; q < R; ++q) lds[z * LP + q * L + x + c] = v[q];
                }
            }
        }
        __syncthreads();
        const Where here = w;
        if (t + gridDim.x < tiles) {
            w = where(t + gridDim.x);
            load(w);
        }
        struct Out {
            float2* p;
            int valid;
            __device__ __forceinline__ void store(int line, int e, float2 v) const
            {
                const int k2 = line / L, x = line - k2 * L;
                if (N % L == 0 || x < valid) p[(long)e * (N * N) + k2 * (N1 * N) + x] = v;
            }
        };
        const LdsAcc<1, LP> a{lds};
        const Out o{out + here.base + here.k1 * N + here.x0, N - here.x0};
        run_tail<N, S, LINES, T, 0, false>(a, o, tw_z, tid);
        __syncthreads();
    }
}

}  // namespace fft3d
