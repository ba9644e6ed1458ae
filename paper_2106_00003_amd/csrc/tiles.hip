// Launches of the tiled sweeps (tile_kernels.hpp).
#include "tile_kernels.hpp"

#include <algorithm>
#include <utility>

namespace givens {
namespace {

// Stage st of Y <- U X or U^T X, the `first` one from X (nullptr: I), the others in place.  `runs` of column blocks for each
// tile; 0: no tile of the stage has a free pair.  `resident`: workgroups to aim at.
inline int tile_active(const TilePlan &g, int st, int free_rows)
{
    if (free_rows >= g.n - 1) return g.P;
    int active = 0;
    for (int u = 0; u < g.P; ++u) active += tile_is_identity(g, tile_at(g, st, u), free_rows) ? 0 : 1;
    return active;
}
inline long long tile_apply_stage(const TilePlan &g, long long resident, int st, bool first, int rows,
                                  int free_rows, const TileOperand &op, const u32x4 *pieces, const unsigned *tops,
                                  TileApplyArgs *out)
{
    const int active = first && op.X != op.Y ? g.P : tile_active(g, st, free_rows);   // the first stage writes every row
    if (active == 0) return 0;
    const long long steps = (op.B + kTileCols - 1) / kTileCols;
    const long long most = std::max(1LL, resident / active);
    const long long per = (steps + most - 1) / most;
    *out = TileApplyArgs{g, st, rows, free_rows, op.B, pieces, first ? op.X : op.Y, op.Y, per * kTileCols,
                         op.X ? tops : nullptr};
    return (steps + per - 1) / per;
}
// Y <- U X (forward, pieces of the transposed matrices) or U^T X
inline void tile_apply(const TilePlan &g, int compute_units, int rows, int free_rows, const TileOperand &op,
                       const u32x4 *pieces, const unsigned *tops, bool forward, hipStream_t stream)
{
    // at most what the chip holds at once (eight wavefronts per compute unit)
    const long long resident = (long long)compute_units * 8 / (kTilePad / 32);
    for (int i = 0; i < g.stages; ++i) {
        TileApplyArgs a;
        const long long runs = tile_apply_stage(g, resident, forward ? g.stages - 1 - i : i, i == 0, rows, free_rows,
                                                op, pieces, tops, &a);
        if (runs)
            hipLaunchKernelGGL(tile_apply_kernel, dim3((unsigned)(runs * g.P)), dim3(2 * kTilePad), 0, stream, a);
    }
}
inline void tile_gradient(const TilePlan &g, int compute_units, int rows, int free_rows, const float *theta, const int *map,
                          const u32x4 *pieces, const float *C, int slices, float *S, float *blocks, int *range, float *halves,
                          const unsigned *tops, float *dtheta, const TileOperand &op, hipStream_t stream)
{
    const bool narrow = tile_gradient_narrow(g, free_rows);
    const unsigned pairs = (unsigned)(g.P * (g.P + 1) / 2) * (narrow ? kTilePad / 32 : 1);
    float *second = narrow ? S + tile_s_floats(g) : nullptr;
    hipLaunchKernelGGL(tile_antisym_kernel, dim3(tile_antisym_blocks(g)), dim3(256), 0, stream, g, rows, slices, C, S, range);
    const long long slots = (long long)compute_units * 8 / (kTilePad / 32);
    float *in = S, *out = second ? second : S;
    for (int st = 0; st < g.stages; ++st) {
        TileStageArgs a{TileTwoSidedArgs{g, st, free_rows, pieces, in, out, blocks, range}, {}, pairs};
        long long runs = 0;
        if (op.Y) {   // beside the pairs that have something to do
            const long long idle = g.P - tile_active(g, st, free_rows);
            const long long busy = narrow ? pairs : pairs - idle * (idle + 1) / 2, room = slots - busy;
            runs = tile_apply_stage(g, std::max(room, slots / 2), st, st == 0, rows, free_rows, op, pieces, tops,
                                    &a.a);
        }
        const auto kernel = narrow ? (runs ? tile_stage_kernel<true, true> : tile_stage_kernel<true, false>)
                                   : (runs ? tile_stage_kernel<false, true> : tile_stage_kernel<false, false>);
        hipLaunchKernelGGL(kernel, dim3((unsigned)(pairs + runs * g.P)), dim3(2 * kTilePad), 0, stream, a);
        if (second) std::swap(in, out);
    }
    hipLaunchKernelGGL(tile_gradient_kernel, dim3((unsigned)(2 * g.P + tile_count(g))), dim3(kTileThreads), 0, stream, g, theta,
                       map, free_rows, blocks, range + kTileRangeWords, halves, dtheta);
}
} // namespace

void tiles_build(const TilePlan &g, const float *theta, const int *map, int free_rows, const TileBuffers &b, bool forward,
                 int rows, long long B, const float *X, hipStream_t stream)
{
    const TileTops tops{rows, B, X, b.tops};
    const int top_blocks = (int)tile_top_blocks(tops);
    const long long grid = 2 * g.P + top_blocks + tile_count(g) + 1;
    hipLaunchKernelGGL(tile_build_kernel, dim3((unsigned)grid), dim3(kTileThreads), 0, stream, g, theta, map, free_rows,
                       static_cast<u32x4 *>(b.pieces), forward ? 1 : 0, b.range, tops, top_blocks);
}
void tiles_apply(const TilePlan &g, int compute_units, int rows, int free_rows, const TileBuffers &b, const TileOperand &op,
                 bool forward, hipStream_t stream)
{
    tile_apply(g, compute_units, rows, free_rows, op, static_cast<const u32x4 *>(b.pieces), b.tops, forward, stream);
}
void tiles_gradient(const TilePlan &g, int compute_units, int rows, int free_rows, const float *theta, const int *map,
                    const TileBuffers &b, const float *C, int slices, float *dtheta, const TileOperand &op, hipStream_t stream)
{
    tile_gradient(g, compute_units, rows, free_rows, theta, map, static_cast<const u32x4 *>(b.pieces), C, slices, b.S, b.blocks, b.range,
                  b.halves, b.tops, dtheta, op, stream);
}

} // namespace givens
