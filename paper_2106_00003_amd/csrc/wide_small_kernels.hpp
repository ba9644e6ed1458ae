// Smallest matrices on wide batches (float32, even n from 16 to kWideSmallMaxN in the column family): the chain of small kernels
// around the products and the contraction in fewer launches.
//
// Why.  With n = 64, B = 65536 the three kernels that read the batch take 10 to 13 us each; the table, the sweep over n columns and
// the split of its result took 11 us more in a forward call and, with the sums, 23 in a backward one, eight launches of 3 to 8
// us that leave the chip empty.  Here a workgroup makes the coefficients in LDS, sweeps eight columns of the identity and cuts
// them into pieces, as a kernel of its own in the forward call and beside the contraction in the backward one, whose own sweep
// runs beside the product.  n = 64, B = 65536, both calls: 48.5 us, 60.7 with a launch for each part.  Entries of the table and the
// arithmetic of a column and of a sum are those of the kernels that this stands for: the calls that keep them (prepared, not
// allocating, dX not wanted or in the place of G) give the same bits.
#pragma once
#include "carousel_kernels.hpp"
#include "coef_kernels.hpp"
#include "gram_kernels.hpp"
#include "product_kernels.hpp"

namespace givens {

// The contraction's result and a column block of the product are one tile of 64 x 64 each, and the table takes 16 KB of LDS beside the
// contraction's 26; at n = 128 it would be four tiles and 65 KB, which leaves one workgroup per compute unit (not tried).
constexpr int kWideSmallMaxN = 64;
constexpr int kWideSmallCols = 8;      // of a workgroup: four wavefronts of two, an octet of the split matrix

struct SmallMatrixArgs {
    int n, rows, mirror;               // mirror: U^T instead of U
    int k16s;                          // fragments in a row of the split matrix
    const float *theta;
    const int *map;
    u32x4 *pieces;
};
inline unsigned small_matrix_blocks(int rows) { return (unsigned)product_k16(rows) * 2; }

// Entry e of the table in the standard form; orient: the sign in its sine.
__device__ __forceinline__ float2 small_coefs(const SmallMatrixArgs &a, int mirror, int e, float *orient)
{
    const int H = a.n >> 1, k = e / H, p = e - k * H;
    *orient = rr_label(a.n, k, p) < rr_label(a.n, k, a.n - 1 - p) ? 1.f : -1.f;
    return standard_entry<float>((double)theta_at(a.theta, a.map, mirror, a.n, (long long)e), *orient);
}
// Columns 8 block + 2 wave and the next one into `cols`.
typedef float SmallColumns[kWideSmallMaxN][kWideSmallCols + 1];
__device__ __forceinline__ void small_columns(const SmallMatrixArgs &a, int block, int wave, int lane, const float2 *table,
                                              SmallColumns &cols)
{
    constexpr int W = 2;
    using State = CarouselFwd<1, W, 1, kFormStandard, kExchangeWave, false, kTableLds>;
    State st;
    const int n = a.n, L = n / 2;
    const bool idle = lane >= L;
    st.n = n;
    st.H = L;
    st.lanes = L;
    st.lane = st.tid = lane;
    st.wave = 0;
    st.table_of_lane(table, idle ? 0 : lane);
    const int c0 = block * kWideSmallCols + wave * W;
    auto unit = [&](float(&v)[W], int label) {
        const int row = mirrored_row(n, label, a.mirror);
#pragma unroll
        for (int x = 0; x < W; ++x) v[x] = !idle && row == c0 + x && row < a.rows ? 1.f : 0.f;
    };
    unit(st.top[0], idle ? 0 : rr_label(n, n - 2, lane));
    unit(st.bot[0], idle ? 0 : rr_label(n, n - 2, n - 1 - lane));
    if (!lane_is_off<1>(lane, L)) {
        st.lead_in();
#pragma unroll
        for (int d = 0; d < State::kDepth - 1; ++d) st.load_coefs(n - 2 - st.leading_blocks() - d, st.cs[d]);
        st.sweep();
        const int rt = mirrored_row(n, lane, a.mirror), rb = mirrored_row(n, n - 1 - lane, a.mirror);
#pragma unroll
        for (int x = 0; x < W; ++x) {
            if (idle) break;
            cols[rt][wave * W + x] = st.top[0][x];
            cols[rb][wave * W + x] = st.bot[0][x];
        }
    }
}
// Columns 8 block .. + 7 of U or U^T in operand order (split_matrix_kernel), those past the end zeros.
template <int THREADS>
__device__ __forceinline__ void small_matrix(const SmallMatrixArgs &a, int block)
{
    __shared__ float2 table[kWideSmallMaxN * (kWideSmallMaxN - 1) / 2];
    __shared__ SmallColumns cols;
    const int n = a.n, N = n * (n - 1) / 2;
    for (int e = threadIdx.x; e < N; e += THREADS) {
        float orient;
        table[e] = small_coefs(a, a.mirror, e, &orient);
    }
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (wave < kWideSmallCols / 2) small_columns(a, block, wave, lane, table, cols);
    __syncthreads();
    // a thread cuts a row's octet; the split matrix has 256 rows
    const int row = threadIdx.x, k0 = block * kWideSmallCols;
    if (row >= 256) return;
    float x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = row < a.rows && k0 + j < a.rows ? cols[row < n ? row : 0][j] : 0.f;
    const Split8 s = split8<true>(x);
    u32x4 *o = a.pieces + ((size_t)(row / 32) * a.k16s + block / 2) * 192 + (row & 31) + 32 * (block & 1);
    o[0] = s.h;
    o[64] = s.m;
    o[128] = s.l;
}
constexpr int kSmallMatrixThreads = 1024;   // two angles each at n = 64
__global__ __launch_bounds__(kSmallMatrixThreads) void small_matrix_kernel(SmallMatrixArgs a)
{
    small_matrix<kSmallMatrixThreads>(a, blockIdx.x);
}

// The contraction's slices, with the pieces of U^T and the reverse sweep's table beside them.  A multiple of eight workgroups
// stands before those of the contraction, whose order by XCD stays.
constexpr unsigned kSmallTableBlocks = 8;
inline unsigned wide_small_extra(int rows) { return (small_matrix_blocks(rows) + kSmallTableBlocks + 7) / 8 * 8; }
template <bool GUARD>
__global__ __launch_bounds__(256, 2) void wide_small_gram_kernel(GramArgs g, SmallMatrixArgs m, unsigned matrix_blocks, unsigned extra,
                                                                 float2 *__restrict__ table, float *__restrict__ factor)
{
    if (blockIdx.x >= extra) {
        gram_tile<2, 2, 1, 1, GUARD, false>(g, blockIdx.x - extra, gridDim.x - extra);
    } else if (blockIdx.x < matrix_blocks) {
        small_matrix<256>(m, blockIdx.x);
    } else if (blockIdx.x < matrix_blocks + kSmallTableBlocks) {
        const int N = m.n * (m.n - 1) / 2;
        for (int e = (int)(blockIdx.x - matrix_blocks) * 256 + threadIdx.x; e < N; e += 256 * kSmallTableBlocks) {
            float orient;
            table[e] = small_coefs(m, 0, e, &orient);
            factor[e] = orient;
        }
    }
}

// The product with U^T, and before it (in workgroups of which one wavefront works) the reverse sweep over the contraction's
// `rows` columns.
struct SmallSweepArgs {
    int n, rows;
    const float2 *table;
    const float *C;
    float *partial;
    const float *zeros;
    float *sink;
};
__device__ __forceinline__ void small_sweep(const SmallSweepArgs &a)
{
    if (threadIdx.x >= 64 || (int)blockIdx.x >= a.rows) return;
    NoExchange none;
    const CarouselChainArgs chain{};
    carousel_backward_body<1, 1, 1, kFormStandard, kExchangeWave, 0>(none, a.n, a.rows, a.rows, 0, a.rows, a.table, nullptr, a.C,
                                                                     nullptr, nullptr, a.partial, a.zeros, a.sink, 0, 1, chain);
}
__global__ __launch_bounds__(256, 2) void wide_small_product_kernel(ProductArgs p, SmallSweepArgs s, unsigned sweeps)
{
    if (blockIdx.x < sweeps)
        small_sweep(s);
    else
        product_tiled<2, 2, 1, 1, 1, false>(p, blockIdx.x - sweeps);
}
__global__ __launch_bounds__(64 * kNarrowWaves, 1) void wide_small_narrow_kernel(ProductArgs p, SmallSweepArgs s, unsigned sweeps)
{
    __shared__ NarrowShared sh;
    if (blockIdx.x < sweeps)
        small_sweep(s);
    else
        product_narrow<false>(p, sh, blockIdx.x - sweeps);
}

} // namespace givens
