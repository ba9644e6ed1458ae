// One-wavefront sweeps in float64: the carousel of carousel_kernels.hpp (a strip in circle-method position order, folded in
// two, M slots per lane) with the exchange inside the wavefront, standard rotation form.  n = 2 M L, L <= 64 lanes.
//
// Why.  The LDS kernels spend a block on two LDS round trips and a barrier whatever the batch; here a block is M rotations
// per lane and column and one move between lanes, and its coefficients are on their way kWave64Depth - 1 blocks ahead.
// Bound by the chain of blocks for narrow batches and by float64 arithmetic for wide ones.  Measured, LDS kernels against
// these in us: see wave64_supported.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "carousel_host.hpp"
#include "rr_index.h"

namespace givens {

constexpr int kWave64Depth = 4;   // ring of coefficients, in blocks
// Strips of a workgroup, one wavefront each, where there are many.  They read the same coefficients within a few blocks of each
// other, so most come from the compute unit's L1, and in the reverse sweep they share a row of partial sums.  Where there are no
// more strips than places for them each has a compute unit's L1 to itself (wave64_fwd_strips, wave64_bwd_strips).
// Whether the first loads of the ring stand under a condition, which always holds (n >= 10).  Where the compiler does not know
// how many loads are on their way it waits for all of them in every fourth block: n = 448, B = 15 forward and backward 65 and 109 us
// with the condition, 57 and 89 without, n = 512, B = 1024 90 and 198, 77 and 175.  Only the shortest blocks, which end before
// their loads come back, are better off with that wait than with one in every block: one slot and four columns, n = 18, B = 2541
// 11.0 and 16.0 us, 11.0 and 16.4, n = 28, B = 2204 11.1 and 18.1, 11.4 and 18.4.
constexpr bool wave64_asks(int M, int W) { return M == 1 && W == 4; }
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

// A row of the table lists the first slots of 64 lanes, then the second ones, and so on: a load of a wavefront is 1 KB of
// consecutive memory (with a lane's slots side by side each load of eight-slot lanes touched 64 lines, and four wavefronts of a
// compute unit had no use of its L1: n = 1024, B = 256 forward 904 us).
template <int M>
struct Wave64Coefs {
    double2 cs[kWave64Depth][M];
    const double2 *lane;   // table + first slot of this lane
    __device__ __forceinline__ void load(int k, int slot)
    {
        const double2 *src = lane + (long long)k * (64 * M);
#pragma unroll
        for (int r = 0; r < M; ++r) cs[slot][r] = src[64 * r];
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
            if (!wave64_asks(M, W) || k - d >= 0) co.load(k - d, d);
        for (; k >= kUnroll - 1; k -= kUnroll) group(k, std::make_integer_sequence<int, kUnroll>{});
        tail(std::make_integer_sequence<int, kUnroll - 1>{});
    }
};

// rows: the operand's row count (n, or n - 1 when n pads an odd problem); mirror: rows relabelled r -> n - r, with mirrored
// tables the launch applies U^T (carousel_kernels.hpp)
template <int M, int W>
__global__ __launch_bounds__(64 * kWave64Strips, 1) void wave64_forward_kernel(int n, int rows, long long B, const double2 *__restrict__ table,
                                                               const double *X, double *Y, int identity, int mirror)
{
    using State = Wave64Fwd<M, W>;
    State st;
    const int l = threadIdx.x & 63, L = n / (2 * M);
    const bool idle = l >= L;
    st.lane = l;
    st.lanes = L;
    st.co.lane = table + (idle ? 0 : l);
    const long long b0 = ((long long)blockIdx.x * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * W;
    if (b0 >= B) return;
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

// Reverse sweep.  With several strips in a workgroup their sums of four blocks go to LDS, and after a barrier each wavefront adds
// those of one block, in strip order, and stores them.  So a row of partial sums stands for 4 W columns, while a wavefront's
// block has the arithmetic of W: n = 512, B = 1024 with the second stage 219 us, 645 with a wavefront of one column per row;
// n = 1024, B = 1024 871 and 2667.
template <int M, int W, int STRIPS>
struct Wave64Bwd {
    static constexpr int kUnroll = wave64_unroll(M);
    double zt[M][W], zb[M][W], gt[M][W], gb[M][W];
    Wave64Coefs<M> co;
    int lane, lanes, wave, H;
    bool idle;
    double *part;   // this workgroup's row of partial sums + slots of this lane
    struct Sums {
        double of[kWave64Depth][STRIPS][M][64];
    };
    Sums *sums_of;  // two of them, which take turns
    int turn;
    // sums of the `count` blocks from k0 on are in LDS
    __device__ __forceinline__ void flush(int k0, int count)
    {
        if constexpr (STRIPS == 1) return;   // (stored by the blocks themselves)
        __syncthreads();
        const auto &s = sums_of[turn].of;
        turn ^= 1;
        if (wave >= count || idle) return;
        double *dst = part + (long long)(k0 + wave) * H;
#pragma unroll
        for (int r = 0; r < M; ++r) {
            double v = s[wave][0][r][lane];
#pragma unroll
            for (int w = 1; w < STRIPS; ++w) v += s[wave][w][r][lane];
            dst[r] = v;
        }
    }
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
    // `place`: of this block's sums in LDS
    template <int C, bool LAST, bool AHEAD>
    __device__ __forceinline__ void step(int k, int place = C % kWave64Depth)
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
        if constexpr (STRIPS == 1) {
            if (!idle)
#pragma unroll
                for (int r = 0; r < M; ++r) part[(long long)k * H + r] = sums[r];
        } else {
#pragma unroll
            for (int r = 0; r < M; ++r) sums_of[turn].of[place][wave][r][lane] = sums[r];
        }
        if constexpr (!LAST) {
            move<U>(zt, zb);
            move<U>(gt, gb);
        }
    }
    template <int C, bool LAST, bool AHEAD>
    __device__ __forceinline__ void step_and_flush(int k)
    {
        step<C, LAST, AHEAD>(k);
        if constexpr (C % kWave64Depth == kWave64Depth - 1 || LAST) flush(k - C % kWave64Depth, C % kWave64Depth + 1);
    }
    template <int... Cs>
    __device__ __forceinline__ void group(int k, std::integer_sequence<int, Cs...>)
    {
        (step_and_flush<Cs, false, true>(k + Cs), ...);
    }
    template <int... Cs>
    __device__ __forceinline__ void tail(int k, std::integer_sequence<int, Cs...>)
    {
        (step_and_flush<Cs, Cs == kUnroll - 2, (kUnroll - 2 - Cs >= kWave64Depth - 1)>(k + Cs), ...);
    }
    __device__ __forceinline__ void sweep(int n)
    {
        int k = 0;
        for (; k < n % kUnroll; ++k) {   // (one slot per lane only, three blocks at most)
            co.load(k, 0);
            step<0, false, false>(k, k);
        }
        if (k) flush(0, k);
#pragma unroll
        for (int d = 0; d < kWave64Depth - 1; ++d)
            if (!wave64_asks(M, W) || k + d <= n - 2) co.load(k + d, d);
        for (; k + kUnroll <= n - 1; k += kUnroll) group(k, std::make_integer_sequence<int, kUnroll>{});
        tail(k, std::make_integer_sequence<int, kUnroll - 1>{});
    }
};

// strips of W columns, STRIPS of them per workgroup, from group group0 + blockIdx.x on; partial: [gridDim.x][N]
template <int M, int W, int STRIPS>
__global__ __launch_bounds__(64 * STRIPS, 1) void wave64_backward_kernel(int n, int rows, long long B, long long group0,
                                                                const double2 *__restrict__ table, const double *Yin,
                                                                const double *G, double *dX, double *__restrict__ partial)
{
    using State = Wave64Bwd<M, W, STRIPS>;
    __shared__ std::conditional_t<STRIPS == 1, char, typename State::Sums> sums[2];
    State st;
    if constexpr (STRIPS > 1) st.sums_of = sums;
    st.turn = 0;
    st.wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l = threadIdx.x & 63, L = n / (2 * M);
    const bool idle = l >= L;
    st.lane = l;
    st.lanes = L;
    st.idle = idle;
    st.H = n >> 1;
    st.co.lane = table + (idle ? 0 : l);
    st.part = partial + (long long)blockIdx.x * (n - 1) * (n >> 1) + (idle ? 0 : l * M);
    const long long b0 = ((group0 + blockIdx.x) * STRIPS + st.wave) * W;   // (past the end: zeros)
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
