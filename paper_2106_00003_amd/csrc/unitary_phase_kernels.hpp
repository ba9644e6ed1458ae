// Coefficients of the unitary carousel kernels (unitary_carousel_kernels.hpp explains the carried phases):
// the parallel conversion of phi to fixed point, the pass over the blocks that produces the phase
// every pair's top row is turned by, and the parallel kernel that writes the coefficient tables.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "rr_index.h"

namespace givens {

constexpr int kUnitaryCarouselMaxN = 4096;   // phases of all rows in LDS, two buffers of 4 bytes each: 32 KB
constexpr int kPhaseScanThreads = 1024;

// x = r + m * pi with |r| <= pi/2; returns m's parity.  Two-piece pi, like the lifted form's reduction.
__device__ __forceinline__ int reduce_by_pi(double x, double *r)
{
    const double m = rint(x * 0.31830988618379067154);
    *r = fma(-m, 1.2246467991473532e-16, fma(-m, 3.141592653589793116, x));
    return (int)((long long)m & 1);
}

// Phases in the pass are fixed-point numbers: an unsigned 32-bit integer x stands for the angle
// 2 pi x / 2^32, so that sums and differences wrap round modulo 2 pi by themselves and the pass needs integer
// additions only.  Rounding phi to 2 pi / 2^32 = 1.5e-9 rad is a perturbation of the parameter far below
// float32's resolution of the result.
//
// The pass is bound by the latency of its blocks, so everything that does not depend on the carried phases is prepared here.  With f = phi in fixed
// point, F2 = pi if reducing the rotation angle by a multiple of pi negates both rows (rint(theta / pi) odd)
// and "i on top" = the top position holds the pair's smaller label, per pair (see the pass for their use):
//   forward:  q.x = (i on top ? f : -f) + pi/2,   q.y = (i on top ? 0 : f) + F2
//   reverse:  q.x = (i on top ? -f : 0) + F2,     q.y = (i on top ? 0 : -f) + F2
constexpr unsigned kFixedQuarterTurn = 1u << 30, kFixedHalfTurn = 1u << 31;

template <bool REVERSE>
__global__ void unitary_phase_input_kernel(int n, const float *__restrict__ theta, const float *__restrict__ phi,
                                           uint2 *__restrict__ q)
{
    const int H = n >> 1;
    const long long N = (long long)(n - 1) * H;
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < N;
         e += (long long)gridDim.x * blockDim.x) {
        double x = (double)phi[e] * 0.31830988618379067154;     // in units of pi
        x -= 2.0 * rint(0.5 * x);                                 // [-1, 1]
        const unsigned f = (unsigned)(long long)llrint(x * 2147483648.0);   // pi = 2^31; +-pi wrap to one value
        double unused;
        const unsigned f2 = reduce_by_pi((double)theta[e], &unused) ? kFixedHalfTurn : 0u;
        const int k = (int)(e / H), p = (int)(e % H);
        const bool i_on_top = rr_label(n, k, p) < rr_label(n, k, n - 1 - p);
        if (!REVERSE)
            q[e] = make_uint2((i_on_top ? f : 0u - f) + kFixedQuarterTurn, (i_on_top ? 0u : f) + f2);
        else
            q[e] = make_uint2((i_on_top ? 0u - f : 0u) + f2, (i_on_top ? 0u : 0u - f) + f2);
    }
}

// The pass over the blocks.  REVERSE = false: blocks n-2 .. 0 (forward sweep); true: blocks 0 .. n-2 (reverse sweep).
// blockDim.x * PER >= n/2.  q: unitary_phase_input_kernel<REVERSE>'s output.
// The carried phases live in LDS indexed by circle-method *position*, in two buffers that take turns: thread p
// owns the pair of positions (p, n-1-p) in every block, reads its two phases from one buffer and writes the
// new ones to the places the two rows take in the next block of the pass, in the other buffer -- all four
// addresses are fixed per thread.  One barrier per block and five or six integer operations per pair:
//   forward (r_i = w c y_i - s y_j, r_j = w s y_i + c y_j: row i enters with w, both rows leave with the bottom
//   row's phase, plus phi when the bottom row is row i):
//       u = top - bottom + q.x        new bottom = bottom + q.y       new top = new bottom + (u's top bit)
//   reverse (z_i' = conj(w) (c z_i + s z_j), z_j' = -s z_i + c z_j: the rows meet at the bottom row's phase and
//   row i leaves with -phi on top of it):
//       u = top - bottom + pi/2       new bottom = bottom + q.y       new top = bottom + q.x + (u's top bit)
// u - pi/2 is the angle the top row is short of; written as r + flip * pi with r in [-pi/2, pi/2), the top bit of
// u is flip (the turned top row counts as negated) and its low 31 bits are r + pi/2.  turn[e] = u is all the pass
// stores; the table kernel takes it apart.
// Inputs are fetched kDepth blocks ahead (a block of the pass is far shorter than a trip to memory).
//
// A block takes 0.16 to 0.45 us whatever runs beside it, so the blocks are cut into chunks that run at once, and the result
// is put together from two facts, both exact.  The low 31 bits of a row's phase are those of some row before (the bottom one's)
// plus a constant, so a chunk is a map from rows to rows with a constant each: the first kernel (MAP) finds the chunks' maps,
// and a workgroup of the second one goes through the maps before its chunk to know the low bits it starts from.  And a row's
// top bit before a chunk turns its top bits in that chunk, and those of the u it takes part in, without further effect: the
// second kernel starts a chunk from zeros, notes which rows' bits it turns (`flips`, a bit per chunk), and the table kernel
// turns u where the chunks before have turned an odd number of times.  n = 1024: 182 us for the pass in one workgroup,
// 25 us for both kernels in 32 chunks (a step of B = 4096 2520 and 2237).
constexpr int kPhaseChunksMost = 32;   // a bit each of a word of `flips`
inline int phase_chunks(int n) { return n >= 1024 ? kPhaseChunksMost : n >= 256 ? 16 : 8; }
__host__ __device__ inline int phase_chunk_steps(int n, int chunks) { return (n - 1 + chunks - 1) / chunks; }
struct PhaseScan {
    int chunks;
    uint2 *maps;       // [chunks][n]: source row and constant
    unsigned *flips;   // [n]
    unsigned *last;    // [n]: phases the rows end with, but for the flips before the last chunk
};
// label of position `pos` in the block of step `step` of the pass (step n-1: one move past the last block)
template <bool REVERSE>
__device__ __forceinline__ int phase_label(int n, int step, int pos)
{
    if (!REVERSE) {   // block 1's order is the identity; one move further position x holds row x+1
        if (step < n - 1) return rr_label(n, n - 2 - step, pos);
        return pos == 0 ? 0 : (pos == n - 1 ? 1 : pos + 1);
    }
    if (step < n - 1) return rr_label(n, step, pos);
    return rr_label(n, n - 2, pos == 0 ? 0 : (pos == 1 ? n - 1 : pos - 1));
}
template <bool REVERSE, int PER, bool MAP>
__global__ __launch_bounds__(kPhaseScanThreads) void unitary_phase_scan_kernel(int n, const uint2 *__restrict__ q,
                                                                               unsigned *__restrict__ turn, PhaseScan scan)
{
    using State = std::conditional_t<MAP, uint2, unsigned>;
    __shared__ State a[2][kUnitaryCarouselMaxN];
    constexpr int kDepth = 16 / PER;
    constexpr unsigned kLow = kFixedHalfTurn - 1;
    static_assert(kDepth % 2 == 0, "the buffer a block reads is its index modulo 2");
    const int H = n >> 1;
    const int tid = threadIdx.x, threads = blockDim.x, chunk = blockIdx.x, steps = phase_chunk_steps(n, scan.chunks);
    const int from = chunk * steps, to = from + steps < n - 1 ? from + steps : n - 1;

    // fixed places: read (top, bottom), write (where the two rows sit in the next block of the pass)
    int rt[PER], rb[PER], wt[PER], wb[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int p = tid + i * threads, b = n - 1 - p;
        rt[i] = p;
        rb[i] = b;
        if (!REVERSE) {   // towards block k-1: position x -> x-1, position 1 -> n-1, position 0 held
            wt[i] = p == 0 ? 0 : (p == 1 ? n - 1 : p - 1);
            wb[i] = b - 1;
        } else {          // towards block k+1: position x -> x+1, position n-1 -> 1, position 0 held
            wt[i] = p == 0 ? 0 : p + 1;
            wb[i] = b == n - 1 ? 1 : b + 1;
        }
    }
    uint2 ring[kDepth][PER];
    auto fetch = [&](int step, uint2 (&dst)[PER]) {
        const int k = REVERSE ? step : n - 2 - step;
        const uint2 *row = q + (long long)k * H;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const unsigned p = tid + i * threads;
            dst[i] = (step < to && p < (unsigned)H) ? row[p] : make_uint2(0u, 0u);
        }
    };
#pragma unroll
    for (int d = 0; d < kDepth; ++d) fetch(from + d, ring[d]);

    if constexpr (MAP) {
        if (chunk == 0)
            for (int r = tid; r < n; r += threads) scan.flips[r] = 0u;
        for (int pos = tid; pos < n; pos += threads) a[0][pos] = make_uint2((unsigned)phase_label<REVERSE>(n, from, pos), 0u);
    } else {
        // low bits at the start of this chunk, by row in a[1], from those of the chunks before
        constexpr int ROWS = 2 * PER;
        unsigned x[ROWS];
        uint2 m[2][ROWS];
        auto read = [&](int c, uint2 (&v)[ROWS]) {
#pragma unroll
            for (int i = 0; i < ROWS; ++i) {
                const int r = tid + i * threads;
                v[i] = c < chunk && r < n ? scan.maps[(long long)c * n + r] : make_uint2(0u, 0u);
            }
        };
        read(0, m[0]);
#pragma unroll
        for (int i = 0; i < ROWS; ++i) x[i] = 0u;
        for (int c0 = 0; c0 < chunk; c0 += 2)
#pragma unroll
            for (int d = 0; d < 2; ++d) {
                const int c = c0 + d;
                if (c >= chunk) break;
                read(c + 1, m[d ^ 1]);
#pragma unroll
                for (int i = 0; i < ROWS; ++i)
                    if (tid + i * threads < n) a[d][tid + i * threads] = x[i];
                __syncthreads();
#pragma unroll
                for (int i = 0; i < ROWS; ++i) x[i] = (a[d][m[d][i].x] + m[d][i].y) & kLow;
            }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ROWS; ++i)
            if (tid + i * threads < n) a[1][tid + i * threads] = x[i];
        __syncthreads();
        for (int pos = tid; pos < n; pos += threads) a[0][pos] = a[1][phase_label<REVERSE>(n, from, pos)];
    }
    __syncthreads();

    for (int step0 = from; step0 < to; step0 += kDepth) {
#pragma unroll
        for (int d = 0; d < kDepth; ++d) {
            const int step = step0 + d;
            if (step < to) {                                      // uniform over the workgroup
                const int k = REVERSE ? step : n - 2 - step;
                const State *cur = a[d & 1];
                State *nxt = a[(d & 1) ^ 1];
                unsigned *out = turn + (long long)k * H;
#pragma unroll
                for (int i = 0; i < PER; ++i) {
                    const unsigned p = tid + i * threads;
                    if (p < (unsigned)H) {
                        if constexpr (MAP) {
                            const uint2 ab = cur[rb[i]];
                            const unsigned nb = ab.y + ring[d][i].y;
                            nxt[wt[i]] = make_uint2(ab.x, REVERSE ? ab.y + ring[d][i].x : nb);
                            nxt[wb[i]] = make_uint2(ab.x, nb);
                        } else {
                            const unsigned at = cur[rt[i]], ab = cur[rb[i]];
                            unsigned u, nt, nb;
                            if (!REVERSE) {
                                u = at - ab + ring[d][i].x;
                                nb = ab + ring[d][i].y;
                                nt = nb ^ (u & kFixedHalfTurn);
                            } else {
                                u = at - ab + kFixedQuarterTurn;
                                nb = ab + ring[d][i].y;
                                nt = (ab + ring[d][i].x) ^ (u & kFixedHalfTurn);
                            }
                            nxt[wt[i]] = nt;
                            nxt[wb[i]] = nb;
                            out[p] = u;
                        }
                    }
                }
                fetch(step + kDepth, ring[d]);
                __syncthreads();
            }
        }
    }
    // the phases are in the buffer the last block wrote, in the position order of the block after it
    const State *final_phase = a[(to > from ? to - from : 0) & 1];
    for (int pos = tid; pos < n; pos += threads) {
        const int row = phase_label<REVERSE>(n, to, pos);
        if constexpr (MAP) {
            scan.maps[(long long)chunk * n + row] = final_phase[pos];
        } else {
            if (final_phase[pos] >> 31) atomicOr(scan.flips + row, 1u << chunk);
            if (chunk == scan.chunks - 1) scan.last[row] = final_phase[pos];
        }
    }
}
// whether the chunks before `chunk` have turned the top bit of row `row` an odd number of times, as that bit
__device__ __forceinline__ unsigned phase_flip(const PhaseScan &scan, int row, int chunk)
{
    return (unsigned)__popc(scan.flips[row] & ((1u << chunk) - 1u)) << 31;
}

// rot[e] = (tan(theta'/2), sin theta') and phs[e] = (tan(psi'/2), sin psi') from the pass's turn[e]; sgn[e] = +-1:
// the real rotation uses the angle sgn[e] * theta[e], reduced by a multiple of pi to theta' (and in the reverse
// sweep sgn[e] is also the sign of the pair's dL/dtheta sum); with ORIENT, orient[e] = 1 when the top position of
// the pair holds its smaller label (reverse sweep).
// shift: log2 of the slots per lane of a sweep that reads rot and phs in the order of turned_place, or 0.
// The first threads write fin[r], (cos, sin) of the phase row r ends with.
template <bool ORIENT>
__global__ void unitary_carousel_table_kernel(int n, const float *__restrict__ theta, const unsigned *__restrict__ turn,
                                              PhaseScan scan, float *__restrict__ sgn, float2 *__restrict__ rot,
                                              float2 *__restrict__ phs, float *__restrict__ orient, float2 *__restrict__ fin,
                                              int shift)
{
    const int H = n >> 1, steps = phase_chunk_steps(n, scan.chunks);
    const long long N = (long long)(n - 1) * H;
    for (int row = blockIdx.x * blockDim.x + threadIdx.x; row < n; row += gridDim.x * blockDim.x) {
        double s, c;
        sincos((double)(int)(scan.last[row] ^ phase_flip(scan, row, scan.chunks - 1)) * 1.4629180792671596e-09, &s, &c);
        fin[row] = make_float2((float)c, (float)s);   // (2 pi / 2^32)
    }
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < N;
         e += (long long)gridDim.x * blockDim.x) {
        const int k = (int)(e / H), p = (int)(e % H);
        const int top = rr_label(n, k, p), bottom = rr_label(n, k, n - 1 - p), chunk = (ORIENT ? k : n - 2 - k) / steps;
        const bool i_on_top = top < bottom;
        const unsigned u = turn[e] ^ phase_flip(scan, top, chunk) ^ phase_flip(scan, bottom, chunk);
        const bool flip = (u >> 31) != 0;
        const double psi = (double)((int)(u & (kFixedHalfTurn - 1)) - (int)kFixedQuarterTurn) * 1.4629180792671596e-09;
        const float sg = (i_on_top != flip) ? 1.f : -1.f;
        double r;
        reduce_by_pi((double)sg * (double)theta[e], &r);
        double s, c;
        sincos(0.5 * r, &s, &c);
        const long long at = shift ? (long long)k * H + turned_place(p, shift, H >> shift) : e;
        rot[at] = make_float2((float)(s / c), (float)(2.0 * s * c));
        sincos(0.5 * psi, &s, &c);
        phs[at] = make_float2((float)(s / c), (float)(2.0 * s * c));
        sgn[e] = sg;
        if constexpr (ORIENT) orient[e] = i_on_top ? 1.f : 0.f;
    }
}

} // namespace givens
