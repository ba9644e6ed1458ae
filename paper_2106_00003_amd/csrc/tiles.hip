// Launches of the tiled sweeps (tile_kernels.hpp).
#include "tile_choice.hpp"
#include "tile_kernels.hpp"

#include <algorithm>
#include <utility>

namespace givens {
namespace {

inline bool tile_restricted(const TilePlan &g, int free_rows) { return free_rows < g.n - 1; }
inline TileList tile_list(const TilePlan &g, int st, int free_rows)
{
    TileList l;
    l.active = 0;
    for (int pass = 0, at = 0; pass < 2; ++pass)
        for (int u = 0; u < g.P; ++u) {
            const bool idle = tile_is_identity(g, tile_at(g, st, u), free_rows);
            if (idle != (pass == 1)) continue;
            l.tile[at++] = (unsigned char)u;
            l.active = idle ? l.active : at;
        }
    return l;
}
// Stage st of Y <- U X or U^T X: the `first` one takes X, the last one leaves Y.  Returns the runs of column blocks for each tile
// (0: no tile of the stage has a free pair).  A tile's matrix is worth loading for three steps where there are workgroups
// enough, for one where the chip holds all of those, and beside `pairs` workgroups of the gradient for two where it holds all,
// or three where each has a compute unit of its own.  Measured in us, alone with 1, 2, 3, 4, 8 steps: n = 1002 5.4, 6.6, 7.9, 9.2,
// 15.1, n = 1700 10.1, 9.4, 9.2, 10.4, 15.9, n = 2050 13.3, 13.4, 11.8, 13.4, 16.4, n = 4098, m = 512 17.6, 15.0, 13.8, 14.3, 20.0;
// beside pairs: n = 1002 10.0, 9.9, 9.2, 10.2, 15.8, n = 1024 10.8, 10.5, 11.2, 10.5, 16.0, n = 4098 36.6, 33.0, 32.2, 32.9, 37.1.
inline long long tile_apply_stage(const TilePlan &g, int compute_units, long long pairs, int st, int active, bool first, bool last,
                                  int rows, int free_rows, const TileOperand &op, const TileBuffers &b, TileApplyArgs *out)
{
    if (active == 0) return 0;
    const long long steps = (op.B + kTileCols - 1) / kTileCols;
    auto groups = [&](long long per) { return pairs + active * ((steps + per - 1) / per); };
    long long per = 3;
    if (!pairs && groups(1) <= 2LL * compute_units) per = 1;
    if (pairs && groups(3) > compute_units && groups(2) <= 2LL * compute_units) per = 2;
    *out = TileApplyArgs{g, st, rows, free_rows, op.B, static_cast<const u32x4 *>(b.pieces), first, last, op.X, b.operand, op.Y,
                         (unsigned)(per * kTileCols), op.X ? b.tops : nullptr};
    return (steps + per - 1) / per;
}
// Y <- U X (forward, pieces of the transposed matrices) or U^T X
inline void tile_apply(const TilePlan &g, int compute_units, int rows, int free_rows, const TileOperand &op, const TileBuffers &b,
                       bool forward, hipStream_t stream)
{
    for (int i = 0; i < g.stages; ++i) {
        const int st = forward ? g.stages - 1 - i : i;
        const bool first = i == 0, last = i == g.stages - 1;
        TileList list{};
        list.active = g.P;
        const bool idle = tile_restricted(g, free_rows) && !first && !last;   // (those two take every tile)
        if (idle) list = tile_list(g, st, free_rows);
        TileApplyArgs a;
        const long long runs = tile_apply_stage(g, compute_units, 0, st, list.active, first, last, rows, free_rows, op, b, &a);
        const bool listed = idle && runs && tile_apply_listed(g.P, compute_units, runs, a.chunk / kTileCols, list.active);
        const dim3 grid((unsigned)(runs * (listed ? list.active : g.P)));
        if (listed)
            hipLaunchKernelGGL(tile_apply_kernel<TileList>, grid, dim3(2 * kTilePad), 0, stream, a, list);
        else if (runs)
            hipLaunchKernelGGL(tile_apply_kernel<TileAll>, grid, dim3(2 * kTilePad), 0, stream, a, TileAll{});
    }
}
inline void tile_gradient(const TilePlan &g, int compute_units, int rows, int free_rows, const float *theta, const int *map,
                          const TileBuffers &b, const float *C, int slices, float *dtheta, const TileOperand &op,
                          hipStream_t stream)
{
    const u32x4 *pieces = static_cast<const u32x4 *>(b.pieces);
    const bool narrow = tile_gradient_narrow(g, compute_units, free_rows);
    float *second = narrow ? b.S + tile_s_floats(g) : nullptr;
    hipLaunchKernelGGL(tile_antisym_kernel, dim3(tile_antisym_blocks(g)), dim3(256), 0, stream, g, rows, slices, C, b.S, b.range);
    float *in = b.S, *out = second ? second : b.S;
    for (int st = 0; st < g.stages; ++st) {
        // (the narrow kernel leaves no pair out, since its result is another array, and the first and last stage of an operand no tile)
        const bool first = st == 0, last = st == g.stages - 1, restricted = tile_restricted(g, free_rows);
        const bool listed = restricted && !narrow && !((first || last) && op.Y) && tile_pairs_listed(g.P, compute_units);
        TileList list{};
        list.active = g.P;
        if (restricted) list = tile_list(g, st, free_rows);
        const int active = first || last ? g.P : list.active, c = listed ? list.active : g.P;
        const unsigned pairs = (unsigned)(c * (c + 1) / 2 + c * (g.P - c)) * (narrow ? kTilePad / 32 : 1);
        TileStageArgs a{TileTwoSidedArgs{g, st, free_rows, pieces, in, out, b.blocks, b.range}, {}, pairs};
        long long runs = 0;
        if (op.Y) runs = tile_apply_stage(g, compute_units, pairs, st, active, first, last, rows, free_rows, op, b, &a.a);
        const dim3 grid((unsigned)(pairs + runs * c)), block(2 * kTilePad);
        if (listed && c) {
            const auto kernel = runs ? tile_stage_kernel<false, true, TileList> : tile_stage_kernel<false, false, TileList>;
            hipLaunchKernelGGL(kernel, grid, block, 0, stream, a, list);
        } else if (!listed) {
            const auto kernel = narrow ? (runs ? tile_stage_kernel<true, true, TileAll> : tile_stage_kernel<true, false, TileAll>)
                                       : (runs ? tile_stage_kernel<false, true, TileAll> : tile_stage_kernel<false, false, TileAll>);
            hipLaunchKernelGGL(kernel, grid, block, 0, stream, a, TileAll{});
        }
        if (second) std::swap(in, out);
    }
    hipLaunchKernelGGL(tile_gradient_kernel, dim3((unsigned)(2 * g.P + tile_count(g))), dim3(kTileThreads), 0, stream, g, theta,
                       map, free_rows, b.blocks, b.range + kTileRangeWords, b.halves, dtheta);
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
    tile_apply(g, compute_units, rows, free_rows, op, b, forward, stream);
}
void tiles_gradient(const TilePlan &g, int compute_units, int rows, int free_rows, const float *theta, const int *map,
                    const TileBuffers &b, const float *C, int slices, float *dtheta, const TileOperand &op, hipStream_t stream)
{
    tile_gradient(g, compute_units, rows, free_rows, theta, map, b, C, slices, dtheta, op, stream);
}

} // namespace givens
