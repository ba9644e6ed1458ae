// Launches of the tiled sweeps (tile_kernels.hpp).
#include "tile_kernels.hpp"

#include <utility>

namespace givens {
namespace {

inline void tile_build(const TilePlan &g, const float *theta, const int *map, int free_rows, double2 *table, float *matrices,
                       u32x4 *pieces, int *range, const TileTops &tops, bool transposed, hipStream_t stream)
{
    const long long tiles = tile_count(g), entries = tile_coef_entries(g);
    hipLaunchKernelGGL(tile_coef_kernel, dim3((unsigned)((entries + 255) / 256)), dim3(256), 0, stream, g, theta, map,
                       free_rows, entries, table, range, tops.X ? tops.B : 0LL, tops.tops);
    hipLaunchKernelGGL(tile_build_kernel, dim3((unsigned)(g.P * (kTilePad / 64) + tiles)), dim3(128), 0, stream, g, table,
                       free_rows, matrices);
    const long long frags = (tiles + 1) * (kTilePad / 32) * (kTilePad / 16);
    const unsigned split_blocks = (unsigned)((frags + 3) / 4);
    hipLaunchKernelGGL(tile_split_kernel, dim3(split_blocks + (unsigned)tile_top_blocks(tops)), dim3(256), 0, stream, g,
                       free_rows, matrices, pieces, transposed ? 1 : 0, split_blocks, tops);
}
// Y <- U X (forward, pieces of the transposed matrices) or U^T X; X may be Y, nullptr means I
inline void tile_apply(const TilePlan &g, int compute_units, int rows, int free_rows, long long B, const u32x4 *pieces,
                       const unsigned *tops, const float *X, float *Y, bool forward, hipStream_t stream)
{
    // at most what the chip holds at once (eight wavefronts per compute unit)
    const long long resident = (long long)compute_units * 8 / (kTilePad / 32), steps = (B + kTileCols - 1) / kTileCols;
    for (int i = 0; i < g.stages; ++i) {
        const int st = forward ? g.stages - 1 - i : i;
        const bool copies = i == 0 && X != Y;          // the first stage writes every row
        int active = g.P;
        if (!copies && free_rows < g.n - 1) {
            active = 0;
            for (int u = 0; u < g.P; ++u) active += tile_is_identity(g, tile_at(g, st, u), free_rows) ? 0 : 1;
            if (active == 0) continue;
        }
        long long runs = resident / active > 1 ? resident / active : 1;
        const long long per = (steps + runs - 1) / runs;
        runs = (steps + per - 1) / per;
        const TileApplyArgs a{g, st, rows, free_rows, B, pieces, i ? Y : X, Y, per * kTileCols, X ? tops : nullptr};
        hipLaunchKernelGGL(tile_apply_kernel, dim3((unsigned)(runs * g.P)), dim3(2 * kTilePad), 0, stream, a);
    }
}
inline void tile_gradient(const TilePlan &g, int rows, int free_rows, const double2 *table, const int *map, const u32x4 *pieces,
                          const float *C, float *S, float *blocks, int *range, float *dtheta, hipStream_t stream)
{
    const int t = tile_ld(g) / 32;
    const unsigned pairs = (unsigned)(g.P * (g.P + 1) / 2);
    float *second = tile_gradient_narrow(g, free_rows) ? S + tile_s_floats(g) : nullptr;
    hipLaunchKernelGGL(tile_antisym_kernel, dim3(t, t), dim3(256), 0, stream, g, rows, C, S, second, range);
    float *in = S, *out = second ? second : S;
    for (int st = 0; st < g.stages; ++st) {
        const TileTwoSidedArgs a{g, st, free_rows, pieces, in, out, blocks, range};
        if (second)
            hipLaunchKernelGGL(tile_two_sided_narrow_kernel, dim3(pairs * (kTilePad / 32)), dim3(2 * kTilePad), 0, stream, a);
        else
            hipLaunchKernelGGL(tile_two_sided_kernel, dim3(pairs), dim3(2 * kTilePad), 0, stream, a);
        if (second) std::swap(in, out);
    }
    hipLaunchKernelGGL(tile_gradient_kernel, dim3((unsigned)(g.P + (tile_count(g) + 1) / 2)), dim3(2 * kTilePad), 0, stream, g,
                       table, map, free_rows, blocks, dtheta);
}
} // namespace

void tiles_build(const TilePlan &g, const float *theta, const int *map, int free_rows, const TileBuffers &b, bool forward,
                 int rows, long long B, const float *X, hipStream_t stream)
{
    tile_build(g, theta, map, free_rows, b.table, b.matrices, static_cast<u32x4 *>(b.pieces), b.range,
               TileTops{rows, B, X, b.tops}, forward, stream);
}
void tiles_apply(const TilePlan &g, int compute_units, int rows, int free_rows, long long B, const TileBuffers &b,
                 const float *X, float *Y, bool forward, hipStream_t stream)
{
    tile_apply(g, compute_units, rows, free_rows, B, static_cast<const u32x4 *>(b.pieces), b.tops, X, Y, forward,
               stream);
}
void tiles_gradient(const TilePlan &g, int rows, int free_rows, const int *map, const TileBuffers &b, const float *C,
                    float *dtheta, hipStream_t stream)
{
    tile_gradient(g, rows, free_rows, b.table, map, static_cast<const u32x4 *>(b.pieces), C, b.S, b.matrices, b.range, dtheta,
                            stream);
}

} // namespace givens
