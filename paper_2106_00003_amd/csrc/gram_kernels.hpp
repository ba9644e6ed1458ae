// Gram matrix of the reverse sweep for wide batches: C = Y G^T (rows x rows, contraction over the B columns).
//
// Why it is on the path.  The reverse sweep's per-pair sums (paper Section 4.1/4.2: the row sums of the matrix A,
// the only step of the method that reduces across data) are entries of z gbar^T = A_k (Y G^T) A_k^T, where A_k is
// the product of the transposed blocks undone so far.  For B >= 2n it is cheaper to contract over B once, here,
// and to run the sweep on the rows x rows operand C instead of on all B columns.
//
// Kernel.  Both operands are row-major rows x B, i.e. contiguous along the contraction index.  A workgroup computes
// one tile of C for one slice of the contraction range.  Per step of 16 columns every thread brings octets of one
// row (32 bytes) into registers one step ahead, cuts them into three bf16 pieces (product_kernels.hpp: float32
// operands and sums, six bf16 matrix instructions for a product) and puts them into the LDS buffer of the step's
// parity, in the order in which the matrix instructions take their operands: a lane writes and reads 16 consecutive
// bytes and a wavefront 1 KB, so neither side has bank conflicts.  One barrier per step.
//
// Bound by the matrix cores.  Tile of 256 x 128, four wavefronts of 128 x 64 (128 accumulator registers), two
// workgroups per compute unit, one staging while the other multiplies: n = 2048, B = 65536 in 2.77 ms = 198 TFLOP/s
// of float32 product, 1190 of bf16 (with the float32 matrix instructions the same contraction took 4.25 ms,
// 129 TFLOP/s); 256 x 256 with eight wavefronts 2.87 ms, 128 x 128 3.13 ms.  Few rows give too few tiles of that
// size, and B is then cut into more slices of 64 x 64 tiles: n = 64, B = 65536 in 10 us (256 slices), where the
// 128 x 128 tile takes 36.  Rows of any length and alignment take the same 16-byte loads: n = 1002, B = 65536 in 0.76 ms
// = 172 TFLOP/s (1.76 ms with element-by-element loads), B = 3001 in 58 us (166).
//
// Complex operands (interleaved): C = Y G^H has the real parts Y G^T and the imaginary parts Y (i G)^T of the real
// rows x 2B arrays, where i G swaps the two columns of a complex number and negates the first: one contraction with
// 2 rows result columns.
//
// Split-K: B is cut into slices, each slice writes its own rows x rows matrix and sum_slices_kernel adds them in slice
// order, so the result does not depend on scheduling.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "product_kernels.hpp"

namespace givens {

typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

struct GramArgs {
    int rows;
    long long B, slice_cols;
    const float *Y, *G;
    float *C;                    // [slices][rows][cols]
    int tiles_m, tiles_n;
    int cols;                    // rows, or for complex operands (B counts real columns) 2 rows
};

// MW x NW wavefronts of (32 MF) x (32 NF) results each.  GUARD: the tiles or the last
// slice are not full; rows past the end repeat the last one, and only the step that reaches past the slice's end goes
// element by element.
template <int MW, int NW, int MF, int NF, bool GUARD, bool CPLX>
__device__ __forceinline__ void gram_tile(const GramArgs &args, unsigned block, unsigned blocks)
{
    // (values: a choice between two members would be one between their addresses)
    const GramArgs a = args;
    const float *const Y = a.Y, *const G = a.G;
    const int y_rows = a.rows, g_rows = a.cols;
    constexpr int T = 64 * MW * NW, BM = 32 * MF * MW, BN = 32 * NF * NW, BOTH = BM + BN;
    constexpr int PER = BOTH * 2 / T;                  // octets per thread and step
    static_assert(BOTH * 2 % T == 0, "whole octets per thread");
    __shared__ u32x4 panel[2][3][2][BOTH];             // [buffer][piece][octet of the step][row of Y, then of G]
    __shared__ float tops[BOTH][2];                    // largest magnitude of every row in this slice, by its two threads
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave % MW, wn = wave / MW;
    // The list of (slice, tile row, tile column) is cut into eight consecutive parts, one per XCD, so that the workgroups
    // that share an L2 at any time work on neighbouring tiles of one slice and reuse each other's panels (64 x 64 tiles, handed
    // out in turn and so, in us: n = 314, B = 15395 in 60 slices 69 and 37, n = 192, B = 55531 in 170 81 and 41).
    const unsigned id = xcd_order(block, blocks);
    const int tile_j = id % a.tiles_n, tile_i = (id / a.tiles_n) % a.tiles_m;
    const unsigned slice = id / (a.tiles_n * a.tiles_m);
    const long long kbeg = (long long)slice * a.slice_cols;
    const long long kend = (kbeg + a.slice_cols < a.B) ? kbeg + a.slice_cols : a.B;

    float xr[PER][8];
    auto fetch = [&](long long k0) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int c = (int)threadIdx.x + T * i;
            const int pr = c >> 1;                     // panel row
            const bool of_y = pr < BM;
            int r = of_y ? tile_i * BM + pr : tile_j * BN + (pr - BM);
            const float *src = of_y ? Y : G;
            const long long k = k0 + 8 * (c & 1);
            if constexpr (GUARD) {                     // past the end: its results are not stored
                const int end = of_y || !CPLX ? y_rows : g_rows;
                r = r < end ? r : end - 1;
            }
            const bool turned = CPLX && !of_y && r >= a.rows;
            if (turned) r -= a.rows;
            const float *p = src + (long long)r * a.B + k;
            if (!GUARD || k0 + kGramK <= kend) {
                // (a row may start at any multiple of four bytes: the loads take that)
                const f32x4_any u = *reinterpret_cast<const f32x4_any *>(p), w = *reinterpret_cast<const f32x4_any *>(p + 4);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    xr[i][j] = u[j];
                    xr[i][4 + j] = w[j];
                }
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float v = k + j < kend ? p[j] : src[(long long)r * a.B];
                    xr[i][j] = k + j < kend ? v : 0.f;
                }
            }
            if constexpr (CPLX)
#pragma unroll
                for (int j = 0; j < 8; j += 2) {
                    const float re = xr[i][j], im = xr[i][j + 1];
                    xr[i][j] = turned ? -im : re;
                    xr[i][j + 1] = turned ? re : im;
                }
        }
    };
    float top[PER], scale[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) top[i] = 0.f;
    // SCALED: the second run, of rows out of the middle range
    auto stash = [&](auto scaled, int buf) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int c = (int)threadIdx.x + T * i;
            if constexpr (scaled()) {
#pragma unroll
                for (int j = 0; j < 8; ++j) xr[i][j] *= scale[i];
            } else {
                top[i] = range_top(top[i], xr[i]);
            }
            const Split8 s = split8(xr[i]);
            panel[buf][0][c & 1][c >> 1] = s.h;
            panel[buf][1][c & 1][c >> 1] = s.m;
            panel[buf][2][c & 1][c >> 1] = s.l;
        }
    };

    // results in IB groups of rows, a group's operands at a time in registers
    constexpr int IB = MF == 4 ? 2 : 1;
    f32x16 acc[IB][MF / IB][NF];
    auto run = [&](auto scaled) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < MF; ++i)
#pragma unroll
            for (int j = 0; j < NF; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i / (MF / IB)][i % (MF / IB)][j][v] = 0.f;
        auto note = [&](long long k0) {   // with the last panel, whose barrier is the last one
            if constexpr (!scaled())
                if (k0 + kGramK >= kend)
#pragma unroll
                    for (int i = 0; i < PER; ++i) {
                        const int c = (int)threadIdx.x + T * i;
                        tops[c >> 1][c & 1] = top[i];
                    }
        };
        if (kbeg < kend) {
            fetch(kbeg);
            stash(scaled, 0);
            note(kbeg);
        }
        int buf = 0;
        for (long long k0 = kbeg; k0 < kend; k0 += kGramK, buf ^= 1) {
            __syncthreads();   // this step's panels are whole; the other buffer is free (its readers passed this barrier)
            const bool more = k0 + kGramK < kend;
            if (more) fetch(k0 + kGramK);
            u32x4 fb[NF][3];
#pragma unroll
            for (int j = 0; j < NF; ++j)
#pragma unroll
                for (int p = 0; p < 3; ++p) fb[j][p] = panel[buf][p][lane >> 5][BM + wn * 32 * NF + 32 * j + (lane & 31)];
#pragma unroll
            for (int i = 0; i < IB; ++i) {
                u32x4 fa[MF / IB][3];
#pragma unroll
                for (int q = 0; q < MF / IB; ++q)
#pragma unroll
                    for (int p = 0; p < 3; ++p)
                        fa[q][p] = panel[buf][p][lane >> 5][wm * 32 * MF + 32 * (i * (MF / IB) + q) + (lane & 31)];
                mfma_split(fa, fb, acc[i]);
            }
            if (more) {
                stash(scaled, buf ^ 1);
                note(k0 + kGramK);
            }
        }
    };
    run(std::false_type{});

    // the rows' largest magnitudes: every wavefront looks at all of them and comes to the same result
    auto scale_of = [&](int r) { return range_scale(tops[r][0] > tops[r][1] ? tops[r][0] : tops[r][1]); };
    bool odd = false;
    if (kbeg < kend)                       // (an empty slice has none)
#pragma unroll
        for (int r = 0; r < BOTH; r += 64) odd = odd || scale_of(r + lane) != 1.f;
    const bool again = __any(odd);
    if (again) {
        __syncthreads();                   // the last step's panels have been read
#pragma unroll
        for (int i = 0; i < PER; ++i) scale[i] = scale_of(((int)threadIdx.x + T * i) >> 1);
        run(std::true_type{});
    }

    // accumulator layout of the 32 x 32 matrix instructions: register v of lane l is row 8 (v / 4) + 4 (l / 32) + v % 4,
    // column l % 32 of the fragment
    const int cols = CPLX ? a.cols : a.rows;
    float *out = a.C + (long long)slice * a.rows * cols;
#pragma unroll
    for (int j = 0; j < NF; ++j) {
        const int col = tile_j * BN + wn * 32 * NF + 32 * j + (lane & 31);
        const int at = !CPLX ? col : (col < a.rows ? 2 * col : 2 * (col - a.rows) + 1);
        if (again) {
            const float undo = range_unscale(scale_of(BM + wn * 32 * NF + 32 * j + (lane & 31)));
#pragma unroll
            for (int i = 0; i < MF; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int r = wm * 32 * MF + 32 * i + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
                    const float x = acc[i / (MF / IB)][i % (MF / IB)][j][v] * undo;
                    acc[i / (MF / IB)][i % (MF / IB)][j][v] = x * range_unscale(scale_of(r));
                }
        }
#pragma unroll
        for (int i = 0; i < MF; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = tile_i * BM + wm * 32 * MF + 32 * i + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
                if (row < a.rows && col < cols) out[(long long)row * cols + at] = acc[i / (MF / IB)][i % (MF / IB)][j][v];
            }
    }
}
template <int MW, int NW, int MF, int NF, bool GUARD, bool CPLX>
__global__ __launch_bounds__(64 * MW * NW, 2) void gram_tile_kernel(GramArgs a)
{
    gram_tile<MW, NW, MF, NF, GUARD, CPLX>(a, blockIdx.x, gridDim.x);
}

// c[0] += c[1] + ... + c[slices-1] element by element: 64 elements at a time per workgroup, kSumGroups threads for each,
// thread g adding the slices g, g + kSumGroups, ... and the first one the sums, in that order (a single thread per element
// leaves most of the chip idle for small matrices and waits for one load after the other).  Workgroups take turns: one
// for every 64 elements would be more threads than a launch may have for the largest matrices.
constexpr int kSumGroups = 8, kSumBlocks = 16384;
__global__ __launch_bounds__(64 * kSumGroups) void sum_slices_kernel(long long count, int slices, float *__restrict__ c)
{
    __shared__ float part[kSumGroups][64];
    const int g = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (long long i0 = (long long)blockIdx.x * 64; i0 < count; i0 += (long long)gridDim.x * 64) {
        const long long i = i0 + lane;
        float acc = 0.f;
        if (i < count) {
#pragma unroll 4
            for (int s = g; s < slices; s += kSumGroups) acc += c[(long long)s * count + i];
        }
        part[g][lane] = acc;
        __syncthreads();
        if (g == 0 && i < count) {
            for (int q = 1; q < kSumGroups; ++q) acc += part[q][lane];
            c[i] = acc;
        }
        __syncthreads();
    }
}

template <int MW, int NW, int MF, int NF, bool CPLX>
inline void launch_gram(GramArgs a, int slices, hipStream_t stream)
{
    constexpr int BM = 32 * MF * MW, BN = 32 * NF * NW;
    a.tiles_m = (a.rows + BM - 1) / BM;
    a.tiles_n = (a.cols + BN - 1) / BN;
    const bool full = a.B % kGramK == 0 && a.rows % BM == 0 && a.cols % BN == 0;
    const dim3 grid((unsigned)(a.tiles_m * a.tiles_n * slices)), block(64 * MW * NW);
    if (full)
        hipLaunchKernelGGL((gram_tile_kernel<MW, NW, MF, NF, false, CPLX>), grid, block, 0, stream, a);
    else
        hipLaunchKernelGGL((gram_tile_kernel<MW, NW, MF, NF, true, CPLX>), grid, block, 0, stream, a);
}

// Launches the slices of C = Y G^T, plan.slices arrays of rows * rows floats.
// CPLX: C = Y G^H, interleaved, with B counting real columns and twice the floats.
template <bool CPLX = false>
inline void gram_slices(int rows, long long B, const GramPlan &plan, const float *Y, const float *G, float *C,
                        hipStream_t stream)
{
    const int cols = CPLX ? 2 * rows : rows;
    const GramArgs a{rows, B, plan.cols, Y, G, C, 0, 0, cols};
    if (plan.tile == 2)
        launch_gram<2, 2, 4, 2, CPLX>(a, plan.slices, stream);
    else if (plan.tile == 1)
        launch_gram<2, 2, 2, 2, CPLX>(a, plan.slices, stream);
    else
        launch_gram<2, 2, 1, 1, CPLX>(a, plan.slices, stream);
}
// ... and their sum, into the first of them
inline void sum_gram(int rows, const GramPlan &plan, float *C, hipStream_t stream, bool cplx = false)
{
    if (plan.slices <= 1) return;
    const long long count = (long long)rows * (cplx ? 2 * rows : rows);
    const unsigned blocks = (unsigned)((count + 63) / 64 < kSumBlocks ? (count + 63) / 64 : kSumBlocks);
    hipLaunchKernelGGL(sum_slices_kernel, dim3(blocks), dim3(64 * kSumGroups), 0, stream, count, plan.slices, C);
}
template <bool CPLX = false>
inline void gram_matrix(int rows, long long B, const GramPlan &plan, const float *Y, const float *G, float *C,
                        hipStream_t stream)
{
    gram_slices<CPLX>(rows, B, plan, Y, G, C, stream);
    sum_gram(rows, plan, C, stream, CPLX);
}

} // namespace givens
