// One-wavefront sweeps in float64: the carousel of carousel_kernels.hpp (a strip in circle-method position order, folded in
// two, M slots per lane) with the exchange inside the wavefront, standard rotation form.  n = 2 M L, L <= 64 lanes.
//
// Why.  The LDS kernels spend a block on two LDS round trips and a barrier whatever the batch; here a block is M rotations
// per lane and column and one move between lanes, and its coefficients are on their way kWave64Depth - 1 blocks ahead.
// Bound by the chain of blocks for narrow batches and by float64 arithmetic for wide ones.  Measured, LDS kernels against
// these in us: see wave64_supported.
#pragma once
#include <hip/hip_runtime.h>

#include <utility>

#include "rr_index.h"

namespace givens {

constexpr int kWave64Depth = 4;   // ring of coefficients, in blocks
constexpr int wave64_unroll(int M) { return M > kWave64Depth ? M : kWave64Depth; }   // a multiple of both (powers of two)

template <int CTRL>
__device__ __forceinline__ double wave64_shift(double incoming, double v)
{
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(incoming), __double2loint(v), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(incoming), __double2hiint(v), CTRL, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}
// lane l receives the value of lane l + 1 / l - 1; the lane without a source keeps `incoming`
__device__ __forceinline__ double wave64_from_next(double incoming, double v) { return wave64_shift<0x130>(incoming, v); }
__device__ __forceinline__ double wave64_from_prev(double incoming, double v) { return wave64_shift<0x138>(incoming, v); }

template <int M>
struct Wave64Coefs {
    double2 cs[kWave64Depth][M];
    const double2 *lane;   // table + slots of this lane
    int H;
    __device__ __forceinline__ void load(int k, int slot)
    {
        const double2 *src = lane + (long long)k * H;
#pragma unroll
        for (int r = 0; r < M; ++r) cs[slot][r] = src[r];
    }
};

template <int M, int W>
struct Wave64Fwd {
    static constexpr int kUnroll = wave64_unroll(M);
    double top[M][W], bot[M][W];
    Wave64Coefs<M> co;
    int lane, lanes;
    // unrolled copy C of a block: register map C mod M, ring slot C mod depth; AHEAD: a block depth - 1 further on exists
    template <int C, bool LAST, bool AHEAD>
    __device__ __forceinline__ void step(int k)
    {
        constexpr int U = C % M, D = kWave64Depth;
        if constexpr (AHEAD) co.load(k - (D - 1), (C + D - 1) % D);
#pragma unroll
        for (int r = 0; r < M; ++r) {
            const int it = (r + U) % M, ib = (r - U + M) % M;
            const double c = co.cs[C % D][r].x, s = co.cs[C % D][r].y;
#pragma unroll
            for (int x = 0; x < W; ++x) {
                const double a = top[it][x], b = bot[ib][x];
                top[it][x] = fma(c, a, -(s * b));
                bot[ib][x] = fma(c, b, s * a);
            }
        }
        if constexpr (!LAST) {
            constexpr int q = U % M, qb = (M - 1 - U + M) % M, q1 = (1 + U) % M;
            const bool far = lane == lanes - 1;
#pragma unroll
            for (int x = 0; x < W; ++x) {
                const double t_out = top[q][x], b_out = bot[qb][x], t_one = top[q1][x];
                const double t_in = wave64_from_next(b_out, t_out);
                if constexpr (M == 1) {
                    bot[0][x] = wave64_from_prev(t_in, b_out);
                    top[0][x] = lane == 0 ? t_out : (far ? b_out : t_in);
                } else {
                    bot[qb][x] = wave64_from_prev(t_one, b_out);
                    top[q][x] = far ? b_out : t_in;
                    top[q1][x] = lane == 0 ? t_out : top[q1][x];
                }
            }
        }
    }
    template <int... Cs>
    __device__ __forceinline__ void group(int k, std::integer_sequence<int, Cs...>)
    {
        (step<Cs, false, true>(k - Cs), ...);
    }
    template <int... Cs>
    __device__ __forceinline__ void tail(std::integer_sequence<int, Cs...>)
    {
        (step<Cs, Cs == kUnroll - 2, (kUnroll - 2 - Cs >= kWave64Depth - 1)>(kUnroll - 2 - Cs), ...);
    }
    __device__ __forceinline__ void sweep(int n)
    {
        int k = n - 2;
        for (; k > n - 2 - n % kUnroll; --k) {   // (one slot per lane only)
            co.load(k, 0);
            step<0, false, false>(k);
        }
#pragma unroll
        for (int d = 0; d < kWave64Depth - 1; ++d)
            if (k - d >= 0) co.load(k - d, d);
        for (; k >= kUnroll - 1; k -= kUnroll) group(k, std::make_integer_sequence<int, kUnroll>{});
        tail(std::make_integer_sequence<int, kUnroll - 1>{});
    }
};

// rows: the operand's row count (n, or n - 1 when n pads an odd problem); mirror: rows relabelled r -> n - r, with mirrored
// tables the launch applies U^T (carousel_kernels.hpp)
template <int M, int W>
__global__ __launch_bounds__(64, 1) void wave64_forward_kernel(int n, int rows, long long B, const double2 *__restrict__ table,
                                                               const double *X, double *Y, int identity, int mirror)
{
    using State = Wave64Fwd<M, W>;
    State st;
    const int l = threadIdx.x, L = n / (2 * M);
    const bool idle = l >= L;
    st.lane = l;
    st.lanes = L;
    st.co.H = n >> 1;
    st.co.lane = table + (idle ? 0 : l * M);
    const long long b0 = (long long)blockIdx.x * W;
    auto place = [&](int label) { return (mirror && label) ? n - label : label; };
    auto bring = [&](double(&v)[W], int row) {
#pragma unroll
        for (int x = 0; x < W; ++x) {
            v[x] = 0.0;
            if (!idle && row < rows && b0 + x < B) v[x] = identity ? (row == b0 + x ? 1.0 : 0.0) : X[(long long)row * B + b0 + x];
        }
    };
#pragma unroll
    for (int r = 0; r < M; ++r) {
        const int p = l * M + r;
        bring(st.top[r], idle ? 0 : place(rr_label(n, n - 2, p)));
        bring(st.bot[r], idle ? 0 : place(rr_label(n, n - 2, n - 1 - p)));
    }
    st.sweep(n);
    constexpr int UL = (2 * M - 2) % M;
#pragma unroll
    for (int r = 0; r < M; ++r) {
        const int p = l * M + r, rt = place(p), rb = place(n - 1 - p);
        if (idle) continue;
#pragma unroll
        for (int x = 0; x < W; ++x) {
            if (b0 + x >= B) continue;
            if (rt < rows) Y[(long long)rt * B + b0 + x] = st.top[(r + UL) % M][x];
            if (rb < rows) Y[(long long)rb * B + b0 + x] = st.bot[(r - UL + M) % M][x];
        }
    }
}

template <int M, int W>
struct Wave64Bwd {
    static constexpr int kUnroll = wave64_unroll(M);
    double zt[M][W], zb[M][W], gt[M][W], gb[M][W];
    Wave64Coefs<M> co;
    int lane, lanes;
    bool idle;
    double *part;   // this strip's row of partial sums + slots of this lane
    template <int U>
    __device__ __forceinline__ void move(double (&t)[M][W], double (&b)[M][W])
    {
        constexpr int qt = (M - 1 - U + M) % M, qb = U % M, pf = (M - U) % M;
        const bool far = lane == lanes - 1;
#pragma unroll
        for (int x = 0; x < W; ++x) {
            const double t_out = t[qt][x], b_out = b[qb][x], held = t[pf][x];
            const double b_in = wave64_from_next(t_out, b_out);
            if constexpr (M == 1) {
                t[0][x] = wave64_from_prev(t_out, lane == 0 ? b_out : t_out);
                b[0][x] = far ? t_out : b_in;
            } else {
                t[qt][x] = wave64_from_prev(held, t_out);
                b[qb][x] = far ? t_out : b_in;
                t[pf][x] = lane == 0 ? b_out : held;
            }
        }
    }
    template <int C, bool LAST, bool AHEAD>
    __device__ __forceinline__ void step(int k)
    {
        constexpr int U = C % M, D = kWave64Depth;
        if constexpr (AHEAD) co.load(k + (D - 1), (C + D - 1) % D);
        double sums[M];
#pragma unroll
        for (int r = 0; r < M; ++r) {
            const int it = (r - U + M) % M, ib = (r + U) % M;
            const double c = co.cs[C % D][r].x, s = co.cs[C % D][r].y;
            double sum = 0.0;
#pragma unroll
            for (int x = 0; x < W; ++x) {
                const double za = zt[it][x], zv = zb[ib][x], ga = gt[it][x], gv = gb[ib][x];
                sum = fma(gv, za, sum);
                sum = fma(-ga, zv, sum);
                zt[it][x] = fma(c, za, s * zv);
                zb[ib][x] = fma(c, zv, -(s * za));
                gt[it][x] = fma(c, ga, s * gv);
                gb[ib][x] = fma(c, gv, -(s * ga));
            }
            sums[r] = sum;
        }
        if (!idle) {
            double *dst = part + (long long)k * co.H;
#pragma unroll
            for (int r = 0; r < M; ++r) dst[r] = sums[r];
        }
        if constexpr (!LAST) {
            move<U>(zt, zb);
            move<U>(gt, gb);
        }
    }
    template <int... Cs>
    __device__ __forceinline__ void group(int k, std::integer_sequence<int, Cs...>)
    {
        (step<Cs, false, true>(k + Cs), ...);
    }
    template <int... Cs>
    __device__ __forceinline__ void tail(int k, std::integer_sequence<int, Cs...>)
    {
        (step<Cs, Cs == kUnroll - 2, (kUnroll - 2 - Cs >= kWave64Depth - 1)>(k + Cs), ...);
    }
    __device__ __forceinline__ void sweep(int n)
    {
        int k = 0;
        for (; k < n % kUnroll; ++k) {
            co.load(k, 0);
            step<0, false, false>(k);
        }
#pragma unroll
        for (int d = 0; d < kWave64Depth - 1; ++d)
            if (k + d <= n - 2) co.load(k + d, d);
        for (; k + kUnroll <= n - 1; k += kUnroll) group(k, std::make_integer_sequence<int, kUnroll>{});
        tail(k, std::make_integer_sequence<int, kUnroll - 1>{});
    }
};

// strips strip0 + blockIdx.x of W columns; partial: [gridDim.x][N]
template <int M, int W>
__global__ __launch_bounds__(64, 1) void wave64_backward_kernel(int n, int rows, long long B, long long strip0,
                                                                const double2 *__restrict__ table, const double *Yin,
                                                                const double *G, double *dX, double *__restrict__ partial)
{
    using State = Wave64Bwd<M, W>;
    State st;
    const int l = threadIdx.x, L = n / (2 * M);
    const bool idle = l >= L;
    st.lane = l;
    st.lanes = L;
    st.idle = idle;
    st.co.H = n >> 1;
    st.co.lane = table + (idle ? 0 : l * M);
    st.part = partial + (long long)blockIdx.x * (n - 1) * (n >> 1) + (idle ? 0 : l * M);
    const long long b0 = (strip0 + blockIdx.x) * W;
    auto bring = [&](double(&v)[W], const double *src, int row) {
#pragma unroll
        for (int x = 0; x < W; ++x) v[x] = !idle && row < rows && b0 + x < B ? src[(long long)row * B + b0 + x] : 0.0;
    };
#pragma unroll
    for (int r = 0; r < M; ++r) {
        const int p = l * M + r;
        bring(st.zt[r], Yin, p);
        bring(st.zb[r], Yin, n - 1 - p);
        bring(st.gt[r], G, p);
        bring(st.gb[r], G, n - 1 - p);
    }
    st.sweep(n);
    if (!dX || idle) return;
    constexpr int UL = (2 * M - 2) % M;
#pragma unroll
    for (int r = 0; r < M; ++r) {
        const int p = l * M + r, rt = rr_label(n, n - 2, p), rb = rr_label(n, n - 2, n - 1 - p);
#pragma unroll
        for (int x = 0; x < W; ++x) {
            if (b0 + x >= B) continue;
            if (rt < rows) dX[(long long)rt * B + b0 + x] = st.gt[(r - UL + M) % M][x];
            if (rb < rows) dX[(long long)rb * B + b0 + x] = st.gb[(r + UL) % M][x];
        }
    }
}

} // namespace givens
