// Sweeps of the smallest problems (n <= kSmallMaxN, float64): one kernel per call.  What bounds such a call is the number of
// launches and the latency of each, not arithmetic, so a workgroup makes the coefficients itself, in LDS (at most 496 angles, two
// per thread, four in the reverse sweep), instead of reading a table that a launch before it wrote; a thread owns one arc and one
// column of the workgroup's strip, so a block is one rotation deep; and the reverse sweep keeps every rotation's contribution in
// LDS and sums over the columns at the end, writing dtheta itself where one workgroup holds all columns.
// Forward and backward calls in us, back to back, tables and sweeps of their own before and now: n = 8, B = 4 9.9 / 13.4 and
// 7.9 / 8.5; n = 16, B = 64 10.1 / 13.1 and 8.2 / 11.4, 1024 10.0 / 13.4 and 8.0 / 11.3.
#pragma once
#include <hip/hip_runtime.h>
#include "coef_kernels.hpp"
#include "rr_index.h"

namespace givens {

constexpr int kSmallMaxN = 32;
constexpr int kSmallMaxAngles = kSmallMaxN * (kSmallMaxN - 1) / 2;
// threads that rotate (the strip's width is what they leave per arc); the reverse sweep's are fewer, so that the contributions,
// (n - 1) of 8 bytes for each of them, fit 64 KB beside the strips
constexpr int kSmallFwdThreads = 256, kSmallBwdThreads = 128;
inline int small_width(int n, long long B, bool backward)
{
    const int fit = (backward ? kSmallBwdThreads : kSmallFwdThreads) / (n / 2);
    return (int)(B < fit ? B : fit);
}
// enough threads for the strip, and for the coefficients at two or so each
inline int small_threads(int n, int w, bool backward)
{
    const int most = backward ? kSmallBwdThreads : kSmallFwdThreads, angles = n * (n - 1) / 2, cells = n / 2 * w;
    const int want = cells > angles ? cells : angles;
    return want >= most ? most : (want + 63) / 64 * 64;
}
// What a workgroup makes of the angles before it sweeps: the entries of coef_table_kernel's standard form, and which pairs are
// bypassed (those neither rotate nor have a gradient).
struct SmallTable {
    double2 cs[kSmallMaxAngles];
    unsigned char bypass[kSmallMaxAngles];
    __device__ __forceinline__ void fill(int n, const double *theta, const int *map, int mirror)
    {
        const int H = n >> 1, N = (n - 1) * H;
        for (int e = threadIdx.x; e < N; e += blockDim.x) {
            const int k = e / H, p = e - k * H;
            const double orient = rr_label(n, k, p) < rr_label(n, k, n - 1 - p) ? 1.0 : -1.0;
            double s, c;
            sincos(theta_at(theta, map, mirror, n, e), &s, &c);
            cs[e] = make_double2(c, orient * s);
            bypass[e] = map && map[mirror ? (n - 2 - k) * H + p : e] < 0;
        }
    }
};

// Y = U X, or U^T X with `mirror` (as lds_forward_kernel); strips of w columns, one per workgroup.  Y may be X.
__global__ __launch_bounds__(kSmallFwdThreads) void small_forward_kernel(int n, int rows, long long B, int w, const double *theta,
                                                                         const int *__restrict__ map, const double *X, double *Y,
                                                                         int identity, int mirror)
{
    __shared__ SmallTable table;
    __shared__ double strip[2 * kSmallFwdThreads];   // [column][row] (rows first: two- to sixteenfold bank conflicts), n w <= 2 kSmallFwdThreads
    const int H = n >> 1;
    const long long b0 = (long long)blockIdx.x * w;
    for (int idx = threadIdx.x; idx < n * w; idx += blockDim.x) {
        const int q = idx / w, c = idx - q * w;
        const int r = mirror && q ? n - q : q;
        double v = 0.0;
        if (b0 + c < B && r < rows) v = identity ? (r == b0 + c ? 1.0 : 0.0) : X[(long long)r * B + b0 + c];
        strip[c * n + q] = v;
    }
    table.fill(n, theta, map, mirror);
    __syncthreads();
    const int c = threadIdx.x / H, p = threadIdx.x - c * H;
    for (int k = n - 2; k >= 0; --k) {
        if (c < w && !table.bypass[k * H + p]) {
            const double2 cs = table.cs[k * H + p];
            double &top = strip[c * n + rr_label(n, k, p)], &bot = strip[c * n + rr_label(n, k, n - 1 - p)];
            const double a = top, b = bot;
            top = cs.x * a - cs.y * b;
            bot = cs.y * a + cs.x * b;
        }
        __syncthreads();   // the next block pairs these rows differently
    }
    for (int idx = threadIdx.x; idx < n * w; idx += blockDim.x) {
        const int q = idx / w, col = idx - q * w;
        const int r = mirror && q ? n - q : q;
        if (b0 + col < B && r < rows) Y[(long long)r * B + b0 + col] = strip[col * n + q];
    }
}

// Reverse sweep of one strip per workgroup.  One workgroup: its sums are dtheta.  Several: each leaves a row of them in
// `partial`, signs applied, and reduce_partials_kernel adds the rows.  dX (may be null) may be G.
__global__ __launch_bounds__(kSmallBwdThreads) void small_backward_kernel(int n, int rows, long long B, int w, const double *theta,
                                                                          const int *__restrict__ map, const double *Y,
                                                                          const double *G, double *dX, double *partial,
                                                                          double *dtheta)
{
    __shared__ SmallTable table;
    __shared__ double z[2 * kSmallBwdThreads], g[2 * kSmallBwdThreads];      // [column][row]
    __shared__ double share[(kSmallMaxN - 1) * kSmallBwdThreads];            // [column][angle], w N <= (n - 1) kSmallBwdThreads
    const int H = n >> 1, N = (n - 1) * H;
    const long long b0 = (long long)blockIdx.x * w;
    for (int idx = threadIdx.x; idx < n * w; idx += blockDim.x) {
        const int r = idx / w, c = idx - r * w;
        const bool held = b0 + c < B && r < rows;
        z[c * n + r] = held ? Y[(long long)r * B + b0 + c] : 0.0;
        g[c * n + r] = held ? G[(long long)r * B + b0 + c] : 0.0;
    }
    table.fill(n, theta, map, 0);
    __syncthreads();
    const int c = threadIdx.x / H, p = threadIdx.x - c * H;
    for (int k = 0; k <= n - 2; ++k) {
        if (c < w && !table.bypass[k * H + p]) {
            const double2 cs = table.cs[k * H + p];
            const int top = c * n + rr_label(n, k, p), bot = c * n + rr_label(n, k, n - 1 - p);
            const double va = z[top], vb = z[bot], ua = g[top], ub = g[bot];
            share[c * N + k * H + p] = ub * va - ua * vb;
            z[top] = cs.x * va + cs.y * vb;
            z[bot] = cs.x * vb - cs.y * va;
            g[top] = cs.x * ua + cs.y * ub;
            g[bot] = cs.x * ub - cs.y * ua;
        }
        __syncthreads();
    }
    if (dX)
        for (int idx = threadIdx.x; idx < n * w; idx += blockDim.x) {
            const int r = idx / w, col = idx - r * w;
            if (b0 + col < B && r < rows) dX[(long long)r * B + b0 + col] = g[col * n + r];
        }
    for (int e = threadIdx.x; e < N; e += blockDim.x) {
        if (table.bypass[e]) continue;
        double sum = 0.0;
        for (int col = 0; col < w; ++col) sum += share[col * N + e];
        const int k = e / H, q = e - k * H;
        if (rr_label(n, k, q) > rr_label(n, k, n - 1 - q)) sum = -sum;
        if (gridDim.x > 1) partial[(long long)blockIdx.x * N + e] = sum;
        else dtheta[map ? map[e] : e] = sum;
    }
}

} // namespace givens
