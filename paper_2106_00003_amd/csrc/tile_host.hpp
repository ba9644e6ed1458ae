// Host side of the tiled sweeps (tile_kernels.hpp): the plan of a problem, sizes of its buffers, entry points of tiles.hip.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>

namespace givens {

struct TilePlan {
    int n, h, m;         // h = n / 2, m = n - 1
    int s, P;            // indices per piece, pieces per half
    int first, stages;   // first stage (-2 or -1), number of stages
};
constexpr int kTilePad = 128;                 // rows of a tile's matrix (64: n = 4096 applied in 4.6 ms against 2.7)
constexpr int kTileSlots = kTilePad / 2 - 1;  // longest piece: 2 s + 1 <= kTilePad
constexpr int kTileMinN = 8, kTileMaxN = 8192;
constexpr TilePlan tile_plan(int n)
{
    TilePlan p{};
    p.n = n;
    p.h = n / 2;
    p.m = n - 1;
    p.P = (p.h + kTileSlots - 1) / kTileSlots;
    p.s = (p.h + p.P - 1) / p.P;
    p.P = (p.h + p.s - 1) / p.s;
    p.first = p.P * p.s == p.h ? -1 : -2;
    p.stages = 2 * p.P - p.first;
    return p;
}
constexpr long long tile_count(const TilePlan &p) { return (long long)p.stages * p.P; }
constexpr int kTilePieceWords = kTilePad * kTilePad * 3 / 8;   // u32x4 per tile

// The gradient's matrix S: a row and column for every one of the kTileHalf slots of each of the 2P pieces (those past a piece's end
// are zeros), as blocks of piece by piece in the order of tile_block_at, and behind the blocks row 0 (S is antisymmetric, so its
// column is not kept).
constexpr int kTileHalf = kTilePad / 2;
constexpr int kTileBlock = kTileHalf * kTileHalf;
inline __host__ __device__ size_t tile_held_offset(const TilePlan &g) { return (size_t)4 * g.P * g.P * kTileBlock; }
inline __host__ __device__ size_t tile_s_floats(const TilePlan &g) { return tile_held_offset(g) + (size_t)2 * g.P * kTileHalf; }
// What the stages of an operand of B columns work on: 64 x 32 blocks, those of a piece one after the other, and row 0 behind them
constexpr int kTileCols = 32;   // columns per step of the apply kernel
constexpr size_t tile_operand_floats(const TilePlan &g, long long B)
{
    return (size_t)((B + kTileCols - 1) / kTileCols) * kTileCols * (2 * g.P * kTileHalf + 1);
}
// Whether the gradient's stages run with 32 columns of a pair of tiles per workgroup (tile_two_sided_narrow): where that gives at
// most two workgroups per compute unit (measured on 256 of them, 32 columns against a pair per workgroup: P = 8 8.0 and 14.9 us,
// P = 17 20.6 and 17.7, P = 24 33.9 and 26.6).  With restricted parametrisations most pairs have nothing to do, which only the
// other kernel leaves alone.
inline bool tile_gradient_narrow(const TilePlan &g, int compute_units, int free_rows)
{
    return free_rows >= g.n - 2 && (kTilePad / 32) * (g.P * (g.P + 1) / 2) <= 2 * compute_units;
}

// What the calls on one problem need: bytes of each buffer.
struct TileBuffers {
    void *pieces;        // the tiles' matrices, cut into bf16 pieces, in operand order
    float *blocks;       // gradient only (forward: null): the tiles' own blocks of S, which its stages leave
    float *S;            // the same
    int *range;          // the same: the range of S's elements and counts of the gradient kernel, behind it
    float *halves;       // the same: sums of special tiles, behind those
    float *operand;      // null: there is none
    unsigned *tops;      // of its columns, one word each; null where the tiles are applied to I only
};
constexpr size_t tile_blocks_bytes(const TilePlan &g) { return (size_t)tile_count(g) * kTilePad * kTilePad * sizeof(float); }
constexpr size_t tile_pieces_bytes(const TilePlan &g) { return (size_t)(tile_count(g) + 1) * kTilePieceWords * 16; }
inline size_t tile_range_offset(const TilePlan &g) { return 2 * tile_s_floats(g) * sizeof(float); }
// behind S: its range and the counts (one page), and the sums of the special tiles' two halves
inline size_t tile_halves_offset(const TilePlan &g) { return tile_range_offset(g) + 1024; }
inline size_t tile_s_bytes(const TilePlan &g)
{
    return tile_halves_offset(g) + (size_t)g.P * 4 * kTileSlots * (kTilePad / 2) * sizeof(float);
}

// free_rows: pairs (i, j) with i < free_rows rotate (n - 1: all of them); rows: of the operand, n or n - 1.
// Matrices of all tiles, cut into pieces: of U's side (forward) or of U^T's, which the gradient takes too.
// X (may be null): the rows x B operand that tiles_apply is going to take, whose columns' range is looked at beside.
void tiles_build(const TilePlan &g, const float *theta, const int *map, int free_rows, const TileBuffers &b, bool forward,
                 int rows, long long B, const float *X, hipStream_t stream);
// What the tiles are applied to: Y <- U X or U^T X on B columns; X may be Y, nullptr means I
struct TileOperand {
    long long B;
    const float *X;
    float *Y;            // null: nothing to apply to
};
void tiles_apply(const TilePlan &g, int compute_units, int rows, int free_rows, const TileBuffers &b, const TileOperand &op,
                 bool forward, hipStream_t stream);
// dtheta from the slices of C = Y G^T (leading dimension `rows`), whose sum it is; the pieces are U^T's.  Beside it, U^T is applied to `op`.
void tiles_gradient(const TilePlan &g, int compute_units, int rows, int free_rows, const float *theta, const int *map,
                    const TileBuffers &b, const float *C, int slices, float *dtheta, const TileOperand &op, hipStream_t stream);

} // namespace givens
