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
#include "carousel_kernels.hpp"
#include "rr_index.h"

namespace givens {

constexpr int kWave64Depth = 4;   // ring of coefficients, in blocks, and blocks whose sums are added up together
// Strips of a workgroup, one wavefront each, where there are many.  They read the same coefficients within a few blocks of each
// other, so most come from the compute unit's L1, and in the reverse sweep they share a row of partial sums.  Where there are no
// more strips than places for them each has a compute unit's L1 to itself (wave64_fwd_strips, wave64_bwd_strips).
// Whether the first loads of the ring stand under a condition, which always holds (n >= 10).  Where the compiler does not know
// how many loads are on their way it waits for all of them in every fourth block: n = 448, B = 15 forward and backward 65 and 109 us
// with the condition, 57 and 89 without, n = 512, B = 1024 90 and 198, 77 and 175.  Only the shortest blocks, which end before
// their loads come back, are better off with that wait than with one in every block: one slot and four columns, n = 18, B = 2541
// 11.0 and 16.0 us, 11.0 and 16.4, n = 28, B = 2204 11.1 and 18.1, 11.4 and 18.4.
constexpr bool wave64_asks(int M, int W) { return M == 1 && W == 4; }
constexpr int wave64_unroll(int M, int depth) { return M > depth ? M : depth; }   // a multiple of both (powers of two)
// Where a strip of one column has a compute unit's L1 nearly to itself a block takes as long as its wavefront needs to issue it: rows by a
// scalar offset (RowBuffer), a deeper ring, and forward the rotations in phases (keep_phases).  n = 512, B = 64 forward and backward
// 63 and 105 us before, 48 and 91 now, n = 1024, B = 64 177 and 335, 152 and 313.  The same in the four strips of a workgroup makes them read
// the L1 more than it gives (n = 512, B = 1024 forward 73 us with a ring of 4 and pointers, 78 with RowBuffer, 85 with a ring of 8 too), so those keep
// pointers, and for each number of slots and columns what was the fastest (n = 256, B = 4000 forward 53 and 50 us, RowBuffer 60; n = 512,
// B = 2000 81 and 75 in phases, 84 without; n = 1024, B = 2000 280 and 257, 295).  With one slot per lane rows are short: n = 64, B = 65536 118 and
// 313 us, 95 and 256.
constexpr bool wave64_alone(int M, int W, bool shared) { return M == 1 || (!shared && W == 1); }
constexpr int wave64_depth_fwd(int M, int W, bool shared)
{
    return wave64_alone(M, W, shared) && M <= 4 && W <= 2 ? 8 : kWave64Depth;
}
constexpr int wave64_depth_bwd(int M, bool shared) { return M == 4 && !shared ? 8 : kWave64Depth; }
constexpr bool wave64_in_phases(int M, int W, bool shared)
{
    return W <= 2 && !(M == 2 && W == 2) && !(M == 4 && W == 1 && shared);
}
// Slots in phases together: as many as there are registers for.
constexpr int wave64_together(int M, int W) { return M * W > 4 ? 4 / W : M; }
// Whether a select by VCC, the slow one in its short form, is kept out of the moves.  (Not worth it: n = 512, B = 1024 forward 73 us without
// and 91 with it, n = 256, B = 64 backward 44.8 and 47.3.)
constexpr bool wave64_spares_vcc_fwd(int M, int W, bool shared) { return !(M == 4 && W == 1 && shared); }
constexpr bool wave64_spares_vcc_bwd(int M, bool shared) { return !(M == 2 && !shared); }

template <int CTRL>
__device__ __forceinline__ double wave64_shift(double incoming, double v)
{
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(incoming), __double2loint(v), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(incoming), __double2hiint(v), CTRL, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}
// lane l receives the value of lane l + 1 / l - 1; the lane without a source, or whose source is switched off, keeps `incoming`
__device__ __forceinline__ double wave64_from_next(double incoming, double v) { return wave64_shift<0x130>(incoming, v); }
__device__ __forceinline__ double wave64_from_prev(double incoming, double v) { return wave64_shift<0x138>(incoming, v); }

// A row of the table lists the first slots of 64 lanes, then the second ones, and so on: a load of a wavefront is 1 KB of
// consecutive memory (with a lane's slots side by side each load of eight-slot lanes touched 64 lines, and four wavefronts of a
// compute unit had no use of its L1: n = 1024, B = 256 forward 904 us).
template <int M, int DEPTH, bool ALONE>
struct Wave64Coefs {
    double2 cs[DEPTH][M];
    RowBuffer table;
    const double2 *first;   // of this lane's slots
    __device__ __forceinline__ void init(const double2 *base, int n, int lane)
    {
        table = RowBuffer::of(base, (long long)(n - 1) * (1024 * M));
        first = base + lane;
    }
    __device__ __forceinline__ void load(int k, int lane, int slot)
    {
        const double2 *src = first + (long long)k * (64 * M);
#pragma unroll
        for (int r = 0; r < M; ++r) {
            if constexpr (ALONE) {
                const auto v = __builtin_amdgcn_raw_buffer_load_b128(table.r, lane * 16 + 1024 * r, k * (1024 * M), 0);
                cs[slot][r] = make_double2(__hiloint2double((int)v[1], (int)v[0]), __hiloint2double((int)v[3], (int)v[2]));
            } else {
                cs[slot][r] = src[64 * r];
            }
        }
    }
};

// Lanes without slots are switched off before the sweep (lane_is_off).  Those that are not bring zeros and read what stands in their places of
// the table's rows, which are 64 lanes wide; nothing of theirs reaches a lane with slots or is stored.
template <int M, int W, bool SHARED>
struct Wave64Fwd {
    static constexpr bool kPhases = wave64_in_phases(M, W, SHARED);
    static constexpr int kDepth = wave64_depth_fwd(M, W, SHARED), kUnroll = wave64_unroll(M, kDepth), kTogether = kPhases ? wave64_together(M, W) : 1;
    double top[M][W], bot[M][W];
    Wave64Coefs<M, kDepth, wave64_alone(M, W, SHARED)> co;
    int lane;
    // slots FIRST + Rs, those with the same phase after each other (the same arithmetic in any order)
    template <int C, int FIRST, int... Rs>
    __device__ __forceinline__ void rotate(std::integer_sequence<int, Rs...>)
    {
        constexpr int U = C % M;
        double p[M][W], q[M][W];
        auto products = [&](int r) {
            const int it = (r + U) % M, ib = (r - U + M) % M;
            const double s = co.cs[C % kDepth][r].y;
#pragma unroll
            for (int x = 0; x < W; ++x) {
                p[r][x] = -(s * bot[ib][x]);
                q[r][x] = s * top[it][x];
            }
        };
        auto sums = [&](int r) {
            const int it = (r + U) % M, ib = (r - U + M) % M;
            const double c = co.cs[C % kDepth][r].x;
#pragma unroll
            for (int x = 0; x < W; ++x) {
                top[it][x] = fma(c, top[it][x], p[r][x]);
                bot[ib][x] = fma(c, bot[ib][x], q[r][x]);
            }
        };
        (products(FIRST + Rs), ...);
        if constexpr (kPhases) keep_phases<>();
        (sums(FIRST + Rs), ...);
        if constexpr (kPhases) keep_phases<>();
    }
    template <int C, int... Gs>
    __device__ __forceinline__ void rotate_groups(std::integer_sequence<int, Gs...>)
    {
        (rotate<C, Gs * kTogether>(std::make_integer_sequence<int, kTogether>{}), ...);
    }
    // unrolled copy C of a block: register map C mod M, ring slot C mod depth; AHEAD: a block depth - 1 further on exists
    template <int C, bool LAST, bool AHEAD>
    __device__ __forceinline__ void step(int k)
    {
        constexpr int U = C % M;
        if constexpr (AHEAD) co.load(k - (kDepth - 1), lane, (C + kDepth - 1) % kDepth);
        rotate_groups<C>(std::make_integer_sequence<int, M / kTogether>{});
        if constexpr (!LAST) {
            constexpr int q = U % M, qb = (M - 1 - U + M) % M, q1 = (1 + U) % M;
            if constexpr (wave64_spares_vcc_fwd(M, W, SHARED)) asm volatile("" ::: "vcc");   // (the mask of lane 0 lives elsewhere)
#pragma unroll
            for (int x = 0; x < W; ++x) {
                const double t_out = top[q][x], b_out = bot[qb][x], t_one = top[q1][x];
                const double t_in = wave64_from_next(b_out, t_out);
                if constexpr (M == 1) {
                    bot[0][x] = wave64_from_prev(t_in, b_out);
                    top[0][x] = lane == 0 ? t_out : t_in;
                } else {
                    bot[qb][x] = wave64_from_prev(t_one, b_out);
                    top[q][x] = t_in;
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
        (step<Cs, Cs == kUnroll - 2, (kUnroll - 2 - Cs >= kDepth - 1)>(kUnroll - 2 - Cs), ...);
    }
    // the first `count` blocks, a multiple of M, fetched together: what n mod kUnroll leaves over
    template <int... Cs>
    __device__ __forceinline__ void lead(int k, int count, std::integer_sequence<int, Cs...>)
    {
        ((Cs < count ? co.load(k - Cs, lane, Cs) : (void)0), ...);
        ((Cs < count ? step<Cs, false, false>(k - Cs) : (void)0), ...);
    }
    __device__ __forceinline__ void sweep(int n)
    {
        int k = n - 2;
        if constexpr (2 * M % kUnroll != 0) {   // (n is a multiple of 2 M)
            const int first = n % kUnroll;
            if (first) lead(k, first, std::make_integer_sequence<int, kUnroll - 1>{});
            k -= first;
        }
#pragma unroll
        for (int d = 0; d < kDepth - 1; ++d)
            if (!wave64_asks(M, W) || k - d >= 0) co.load(k - d, lane, d);
        for (; k >= kUnroll - 1; k -= kUnroll) group(k, std::make_integer_sequence<int, kUnroll>{});
        tail(std::make_integer_sequence<int, kUnroll - 1>{});
    }
};

// rows: the operand's row count (n, or n - 1 when n pads an odd problem); mirror: rows relabelled r -> n - r, with mirrored
// tables the launch applies U^T (carousel_kernels.hpp)
template <int M, int W, bool SHARED>
__global__ __launch_bounds__(64 * kWave64Strips, 1) void wave64_forward_kernel(int n, int rows, long long B, const double2 *__restrict__ table,
                                                               const double *X, double *Y, int identity, int mirror)
{
    using State = Wave64Fwd<M, W, SHARED>;
    State st;
    const int l = threadIdx.x & 63, L = n / (2 * M);
    const bool idle = M == 1 && l >= L;
    st.lane = l;
    st.co.init(table, n, l);
    const long long b0 = ((long long)blockIdx.x * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * W;
    if (b0 >= B || lane_is_off<M>(l, L)) return;
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
        bring(st.top[r], place(rr_label(n, n - 2, p)));
        bring(st.bot[r], place(rr_label(n, n - 2, n - 1 - p)));
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
    static constexpr int kDepth = wave64_depth_bwd(M, STRIPS > 1), kUnroll = wave64_unroll(M, kDepth);
    double zt[M][W], zb[M][W], gt[M][W], gb[M][W];
    Wave64Coefs<M, kDepth, wave64_alone(M, W, STRIPS > 1)> co;
    int lane, wave, H;
    bool idle;        // (one slot per lane: no slot)
    RowBuffer part;   // this workgroup's row of partial sums
    double *sums_row; // ... and this lane's slots in it
    // Whether a sum is stored before the next one is read.  Eight slots and single columns: all sums and then the stores n = 784, B = 300, 512
    // and 768 317, 382 and 427 us, one by one 316, 350 and 374; n = 1024 457, 531 and 593, 433, 483 and 532.  Others are the slower for it: four
    // slots and two columns n = 512, B = 2000 187 and 198, eight and two n = 784, B = 1024 468 and 485.
    static constexpr bool kOneByOne = M == 8 && W == 1 && STRIPS > 1;
    struct Sums {
        double of[kWave64Depth][STRIPS][M][64];
    };
    Sums *sums_of;  // two of them, which take turns
    int turn;
    __device__ __forceinline__ void store(const double (&v)[M], int k)
    {
        typedef unsigned Two __attribute__((ext_vector_type(2)));
        typedef unsigned Four __attribute__((ext_vector_type(4)));
        const int at = lane * (M * 8), row = k * H * 8;
        auto lo = [](double d) { return (unsigned)__double2loint(d); };
        auto hi = [](double d) { return (unsigned)__double2hiint(d); };
        if constexpr (M == 1) {
            const Two w = {lo(v[0]), hi(v[0])};
            __builtin_amdgcn_raw_buffer_store_b64(w, part.r, at, row, 0);
        } else {
#pragma unroll
            for (int r = 0; r < M; r += 2) {
                const Four w = {lo(v[r]), hi(v[r]), lo(v[r + 1]), hi(v[r + 1])};
                __builtin_amdgcn_raw_buffer_store_b128(w, part.r, at + 8 * r, row, 0);
            }
        }
    }
    // sums of the `count` blocks from k0 on are in LDS
    __device__ __forceinline__ void flush(int k0, int count)
    {
        if constexpr (STRIPS == 1) return;   // (stored by the blocks themselves)
        __syncthreads();
        const auto &s = sums_of[turn].of;
        turn ^= 1;
        if (wave >= count || (M == 1 && idle)) return;
        if constexpr (kOneByOne) {
            double *dst = sums_row + (long long)(k0 + wave) * H;
#pragma unroll
            for (int r = 0; r < M; ++r) {
                double v = s[wave][0][r][lane];
#pragma unroll
                for (int w = 1; w < STRIPS; ++w) v += s[wave][w][r][lane];
                dst[r] = v;
            }
        } else {
            double v[M];
#pragma unroll
            for (int r = 0; r < M; ++r) {
                v[r] = s[wave][0][r][lane];
#pragma unroll
                for (int w = 1; w < STRIPS; ++w) v[r] += s[wave][w][r][lane];
            }
            store(v, k0 + wave);
        }
    }
    template <int U>
    __device__ __forceinline__ void move(double (&t)[M][W], double (&b)[M][W])
    {
        constexpr int qt = (M - 1 - U + M) % M, qb = U % M, pf = (M - U) % M;
#pragma unroll
        for (int x = 0; x < W; ++x) {
            const double t_out = t[qt][x], b_out = b[qb][x], held = t[pf][x];
            const double b_in = wave64_from_next(t_out, b_out);
            if constexpr (M == 1) {
                t[0][x] = wave64_from_prev(t_out, lane == 0 ? b_out : t_out);
                b[0][x] = b_in;
            } else {
                t[qt][x] = wave64_from_prev(held, t_out);
                b[qb][x] = b_in;
                t[pf][x] = lane == 0 ? b_out : held;
            }
        }
    }
    // `place`: of this block's sums in LDS
    template <int C, bool LAST, bool AHEAD>
    __device__ __forceinline__ void step(int k, int place = C % kWave64Depth)
    {
        constexpr int U = C % M;
        if constexpr (AHEAD) co.load(k + (kDepth - 1), lane, (C + kDepth - 1) % kDepth);
        double sums[M];
#pragma unroll
        for (int r = 0; r < M; ++r) {
            const int it = (r - U + M) % M, ib = (r + U) % M;
            const double c = co.cs[C % kDepth][r].x, s = co.cs[C % kDepth][r].y;
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
            if (M > 1 || !idle) store(sums, k);
        } else {
#pragma unroll
            for (int r = 0; r < M; ++r) sums_of[turn].of[place][wave][r][lane] = sums[r];
        }
        if constexpr (!LAST) {
            if constexpr (wave64_spares_vcc_bwd(M, STRIPS > 1)) asm volatile("" ::: "vcc");
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
        (step_and_flush<Cs, Cs == kUnroll - 2, (kUnroll - 2 - Cs >= kDepth - 1)>(k + Cs), ...);
    }
    __device__ __forceinline__ void sweep(int n)
    {
        static_assert(M == 1 ? kUnroll <= kWave64Depth : 2 * M % kUnroll == 0, "blocks before the groups, and the place of their sums");
        int k = 0;
        if constexpr (M == 1) {
            for (; k < n % kUnroll; ++k) {   // (three blocks at most)
                co.load(k, lane, 0);
                step<0, false, false>(k, k);
            }
            if (k) flush(0, k);
        }
#pragma unroll
        for (int d = 0; d < kDepth - 1; ++d)
            if (!wave64_asks(M, W) || k + d <= n - 2) co.load(k + d, lane, d);
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
    if (lane_is_off<M>(l, L)) return;
    const bool idle = M == 1 && l >= L;
    st.lane = l;
    st.idle = idle;
    st.H = n >> 1;
    st.co.init(table, n, l);
    const long long sums_of_all = (long long)(n - 1) * (n >> 1);
    st.part = RowBuffer::of(partial + blockIdx.x * sums_of_all, sums_of_all * 8);
    if constexpr (State::kOneByOne) st.sums_row = partial + blockIdx.x * sums_of_all + l * M;
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
