// Separable Gaussian smoothing of a count map, shared by the log-magnification
// histogram and the source maps of light curves.
//
// A source of finite size sees the magnification map convolved with its
// profile (arXiv:1703.09707, Sec. 1).  For a circular Gaussian of width sigma
// the profile is sampled at pixel offsets |k| <= r = ceil(3 sigma / P),
// normalised per axis, and applied rows first, then columns, in FP64 with
// every product and sum rounded on its own.  Only pixels at least r from
// every edge are kept.
#pragma once

#include <cmath>

#include <hip/hip_runtime.h>

#include "launch_rules.h"

namespace {

constexpr int kSmoothThreads = 256;

// taps[0..2r] of one axis: exp(-0.5 ((k - r) P / sigma)^2), then divided by
// their sum (one workgroup).
__global__ __launch_bounds__(kSmoothThreads) void taps_kernel(double sigma, double pixel, int r,
                                                            double *taps) {
    __shared__ double part[kSmoothThreads];
    const int n = 2 * r + 1;
    double s = 0.0;
    for (int k = threadIdx.x; k < n; k += kSmoothThreads) {
        const double d = ((double)(k - r) * pixel) / sigma;
        const double g = exp(-0.5 * (d * d));
        taps[k] = g;
    }
    __syncthreads();
    if (threadIdx.x == 0) {   // sum in index order, as a plain loop does
        for (int k = 0; k < n; ++k) s += taps[k];
        part[0] = s;
    }
    __syncthreads();
    const double total = part[0];
    for (int k = threadIdx.x; k < n; k += kSmoothThreads) taps[k] = taps[k] / total;
}

// tmp[j][i] = sum_k gx[k] * (counts[j][i + k] * norm), i < wx, taps in order.
__global__ __launch_bounds__(kSmoothThreads) void smooth_rows_kernel(const int32_t *__restrict__ counts,
                                                                   int nx, int ny, double norm,
                                                                   const double *__restrict__ gx,
                                                                   int rx, int wx, double *__restrict__ tmp) {
#pragma clang fp contract(off)
    const int64_t idx = (int64_t)blockIdx.x * kSmoothThreads + threadIdx.x;
    if (idx >= (int64_t)wx * ny) return;
    const int j = (int)(idx / wx), i = (int)(idx % wx);
    const int32_t *row = counts + (int64_t)j * nx + i;
    double acc = 0.0;
    for (int k = 0; k <= 2 * rx; ++k) acc = acc + gx[k] * ((double)row[k] * norm);
    tmp[idx] = acc;
}

// out[j][i] = sum_l gy[l] * tmp[j + l][i] over the valid interior.
__global__ __launch_bounds__(kSmoothThreads) void smooth_cols_kernel(const double *__restrict__ tmp, int wx,
                                                                     int wy, const double *__restrict__ gy,
                                                                     int ry, double *__restrict__ out) {
#pragma clang fp contract(off)
    const int64_t idx = (int64_t)blockIdx.x * kSmoothThreads + threadIdx.x;
    if (idx >= (int64_t)wx * wy) return;
    const int j = (int)(idx / wx), i = (int)(idx % wx);
    const double *col = tmp + (int64_t)j * wx + i;
    double acc = 0.0;
    for (int k = 0; k <= 2 * ry; ++k) acc = acc + gy[k] * col[(int64_t)k * wx];
    out[idx] = acc;
}

// ---- Radii up to kTapsMaxRadius: two launches in all, each workgroup forming
// the taps itself.
//
// A pass over a map of this size is a few microseconds, so launches of their
// own for the taps (two, with a sum over global memory one load after the
// other) cost as much as the passes.  Each output's sum keeps its order, so
// the values are those of the kernels above, bit for bit; what changes is
// that a thread takes several neighbouring outputs and slides over their
// common inputs, one load for 4 (rows) or R (columns) multiplies and adds.
// A 1024^2 map with radius 6: rows 9.1 -> 7.4 us, columns 11.7 -> 6.5, and the
// two launches for the taps (4.6 each) gone; four histograms of a 512^2 map
// (radii 3 to 87): 207 -> 82 us, six launches each -> two.

constexpr int kTapsMaxRadius = 512;
constexpr int kTapsLds = 2 * kTapsMaxRadius + 1;

// The taps of taps_kernel, in LDS (every thread of the workgroup calls it;
// ends at a barrier).
__device__ __forceinline__ void taps_to_lds(double sigma, double pixel, int r, double *taps, double *total) {
    const int n = 2 * r + 1;
    for (int k = threadIdx.x; k < n; k += kSmoothThreads) {
        const double d = ((double)(k - r) * pixel) / sigma;
        taps[k] = exp(-0.5 * (d * d));
    }
    __syncthreads();
    if (threadIdx.x == 0) {   // in index order; eight loads ahead of their additions
        double s = 0.0;
        int k = 0;
        for (; k + 8 <= n; k += 8) {
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = taps[k + u];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; k < n; ++k) s += taps[k];
        *total = s;
    }
    __syncthreads();
    const double t = *total;
    for (int k = threadIdx.x; k < n; k += kSmoothThreads) taps[k] = taps[k] / t;
    __syncthreads();
}

// Rows: each wave takes 256 outputs of one row, 4 consecutive ones a lane.
// The row's counts are staged as magnifications, kRowChunk taps' worth at a
// time, element e at [e % 4][e / 4]: lane l then reads element 4 l + k from
// consecutive words.  zero[0 .. n_zero) is cleared for the pass after it.
constexpr int kRowSpan = 256, kRowChunk = 256;

__global__ __launch_bounds__(kSmoothThreads) void smooth_rows_slide_kernel(
    const int32_t *__restrict__ counts, int nx, int ny, double norm, double sigma, double pixel, int rx, int wx,
    double *__restrict__ tmp, unsigned *__restrict__ zero, int n_zero, unsigned *__restrict__ done) {
#pragma clang fp contract(off)
    constexpr int kPart = (kRowSpan + kRowChunk) / 4 + 1;
    __shared__ double taps[kTapsLds], total;
    __shared__ double seg[kSmoothThreads / 64][4][kPart];
    if (zero && blockIdx.x == 0) {
        for (int b = threadIdx.x; b < n_zero; b += kSmoothThreads) zero[b] = 0;
        if (threadIdx.x == 0) *done = 0;
    }
    taps_to_lds(sigma, pixel, rx, taps, &total);
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int across = (wx + kRowSpan - 1) / kRowSpan;   // workgroups along a row
    const int i0 = (blockIdx.x % across) * kRowSpan, j = (blockIdx.x / across) * (kSmoothThreads / 64) + wave;
    const int32_t *row = counts + (int64_t)(j < ny ? j : 0) * nx;
    double(*s)[kPart] = seg[wave];
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int k0 = 0; k0 <= 2 * rx; k0 += kRowChunk) {   // uniform
        const int kn = min(kRowChunk, 2 * rx + 1 - k0);
        __syncthreads();   // the chunk before has been read
        for (int e = lane; e < kRowSpan + kn; e += 64) {
            const int i = i0 + k0 + e;
            s[e % 4][e / 4] = (double)(i < nx ? row[i] : 0) * norm;
        }
        __syncthreads();
        double x0 = s[0][lane], x1 = s[1][lane], x2 = s[2][lane];
        int k = 0;
        for (; k + 4 <= kn; k += 4) {
            const int q = lane + k / 4;
            const double x3 = s[3][q], x4 = s[0][q + 1], x5 = s[1][q + 1], x6 = s[2][q + 1];
            const double g0 = taps[k0 + k], g1 = taps[k0 + k + 1], g2 = taps[k0 + k + 2], g3 = taps[k0 + k + 3];
            acc[0] = (((acc[0] + g0 * x0) + g1 * x1) + g2 * x2) + g3 * x3;
            acc[1] = (((acc[1] + g0 * x1) + g1 * x2) + g2 * x3) + g3 * x4;
            acc[2] = (((acc[2] + g0 * x2) + g1 * x3) + g2 * x4) + g3 * x5;
            acc[3] = (((acc[3] + g0 * x3) + g1 * x4) + g2 * x5) + g3 * x6;
            x0 = x4;
            x1 = x5;
            x2 = x6;
        }
        for (; k < kn; ++k) {
            const int e = 4 * lane + k + 3;
            const double x3 = s[e % 4][e / 4], g = taps[k0 + k];
            acc[0] = acc[0] + g * x0;
            acc[1] = acc[1] + g * x1;
            acc[2] = acc[2] + g * x2;
            acc[3] = acc[3] + g * x3;
            x0 = x1;
            x1 = x2;
            x2 = x3;
        }
    }
    if (j >= ny) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int i = i0 + 4 * lane + q;
        if (i < wx) tmp[(int64_t)j * wx + i] = acc[q];
    }
}

// Columns: R outputs (i, j0 ... j0 + R - 1) of one thread, acc[r] = sum_l
// taps[l] tmp[j0 + r + l][i] in order of l.  Inputs past row `last` belong to
// outputs the caller drops; the last row is read in their place.
template <int R>
__device__ __forceinline__ void slide_columns(const double *__restrict__ tmp, int wx, int i, int j0, int last,
                                              const double *taps, int ry, double (&acc)[R]) {
#pragma clang fp contract(off)
    constexpr int U = 8;   // taps a step: that many loads in flight
    double win[R - 1 + U];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = 0.0;
#pragma unroll
    for (int r = 0; r < R - 1; ++r) win[r] = tmp[(int64_t)min(j0 + r, last) * wx + i];
    int l = 0;
    for (; l + U <= 2 * ry + 1; l += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) win[R - 1 + u] = tmp[(int64_t)min(j0 + R - 1 + l + u, last) * wx + i];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const double g = taps[l + u];
#pragma unroll
            for (int r = 0; r < R; ++r) acc[r] = acc[r] + g * win[r + u];
        }
#pragma unroll
        for (int r = 0; r < R - 1; ++r) win[r] = win[r + U];
    }
    const int rest = 2 * ry + 1 - l;   // fewer than U
#pragma unroll
    for (int u = 0; u < U - 1; ++u)
        if (u < rest) win[R - 1 + u] = tmp[(int64_t)min(j0 + R - 1 + l + u, last) * wx + i];
#pragma unroll
    for (int u = 0; u < U - 1; ++u)
        if (u < rest) {
            const double g = taps[l + u];
#pragma unroll
            for (int r = 0; r < R; ++r) acc[r] = acc[r] + g * win[r + u];
        }
}

template <int R>
__global__ __launch_bounds__(kSmoothThreads) void smooth_cols_slide_kernel(const double *__restrict__ tmp, int wx,
                                                                           int wy, double sigma, double pixel, int ry,
                                                                           double *__restrict__ out) {
    __shared__ double taps[kTapsLds], total;
    taps_to_lds(sigma, pixel, ry, taps, &total);
    const int idx = blockIdx.x * kSmoothThreads + threadIdx.x;
    const int j0 = (idx / wx) * R, i = idx % wx;
    if (j0 >= wy) return;
    double acc[R];
    slide_columns<R>(tmp, wx, i, j0, wy + 2 * ry - 1, taps, ry, acc);
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (j0 + r < wy) out[(int64_t)(j0 + r) * wx + i] = acc[r];
}

// Outputs a thread takes in the column pass: 8 when that still leaves every
// SIMD of the device a wave (1024 of 64 threads), else 4 (four histograms of
// a 512^2 map: 82 us; with 2 or 8 outputs 85, with 1 where fewer waves than
// SIMDs are left 88).
inline int slide_rows_per_thread(int64_t n_out) { return n_out >= 8 * 65536 ? 8 : 4; }

// Workgroups of a column pass of wx x wy outputs, R rows a thread.
inline unsigned slide_blocks(int wx, int wy, int R) {
    const int64_t threads = (int64_t)wx * ((wy + R - 1) / R);
    return (unsigned)((threads + kSmoothThreads - 1) / kSmoothThreads);
}

// Whether the two sliding passes serve these radii and this map.
inline bool slides(int rx, int ry, int wx, int ny) {
    return rx <= kTapsMaxRadius && ry <= kTapsMaxRadius &&
           raysh::grid_fits(raysh::smooth_row_blocks(wx, ny), kSmoothThreads);
}

inline void launch_smooth_rows(hipStream_t s, const int32_t *counts, int nx, int ny, double norm, double sigma,
                               double pixel, int rx, int wx, double *tmp, unsigned *zero = nullptr, int n_zero = 0,
                               unsigned *done = nullptr) {
    static_assert(kRowSpan == 256 && kSmoothThreads == 256, "smooth_row_blocks");
    const unsigned blocks = (unsigned)raysh::smooth_row_blocks(wx, ny);
    hipLaunchKernelGGL(smooth_rows_slide_kernel, dim3(blocks), dim3(kSmoothThreads), 0, s, counts, nx, ny, norm,
                       sigma, pixel, rx, wx, tmp, zero, n_zero, done);
}

inline int taps_radius(double sigma, double pixel) { return (int)std::ceil(3.0 * sigma / pixel); }

}  // namespace
