// Tiled sweeps (float): the blocks of rotations regrouped into tiles that run on the matrix cores.
//
// Order.  Let m = n - 1 (odd).  Give ring label L >= 1 the index a with label(a) = n - 1 - 2a for a < n/2 and
// 2m - 2a from there on (so the low half runs through the odd labels, the high half through the even ones).  Block k
// of the circle method then pairs a and b with a + b = k (mod m), and row 0, which the circle method holds, with the a
// of 2a = k (mod m).  Rotations that share no row commute, so any order in which every row meets its partners in block
// order gives the same product.  Cut both halves into P pieces of s indices: the rotations between piece i and piece j
// (i < j) are a tile, a + b <= m - 1 its late and a + b >= m its early part, and stage t = -2 (or -1) ... 2P - 1 holds
// the late parts with i + j = t and the early parts with i + j = t + 2P: P tiles that share no row.  The pairs inside
// piece i and inside piece i + P, whose rotations with row 0 alternate, are one special tile of stage 2i.
//
// A tile's rotations act on at most 2s + 1 <= kTilePad rows, so they are one kTilePad x kTilePad orthogonal matrix: built here
// in float64, column by column, and applied to any number of columns as a product of bf16 pieces (split_bf16.hpp).  A rotation
// then costs 8 operations per column on the matrix cores instead of 2 to 4 vector instructions, and the chain of n - 1
// dependent blocks becomes one of about n / s products.
//
// Gradient.  With S = Z G^T - G Z^T (antisymmetric) of the strips z and gbar before a tile, the share of a pair (i, j),
// i < j, is S_ij in the frame of its rotation, and a rotation takes S to R S R^T.  So the reverse sweep needs neither
// strip: it starts from S = C - C^T, C = Y G^T, takes S through the stages (S <- A S A^T, two products per pair of
// tiles, half of them by antisymmetry) and leaves every tile's own kTilePad x kTilePad block behind; the sums of all tiles then
// come from those blocks in one launch.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "rr_index.h"
#include "small_trig.hpp"
#include "split_bf16.hpp"
#include "tile_host.hpp"
#include "wave_order.hpp"

namespace givens {

enum { kTileLate = 0, kTileEarly = 1, kTileSpecial = 2, kTileNone = 3 };
// The rows of a tile's matrix: those of piece i from 0, of piece j from kTilePad / 2, and at kTilePad - 1 row 0, which goes with
// tile 0 of every stage (an identity row unless the tile is special).
struct Tile {
    int i, j, kind;
    int a0, na, b0, nb;   // indices of the two pieces
};
__host__ __device__ inline void tile_piece(const TilePlan &g, int i, int *start, int *count)
{
    const int lo = i < g.P ? i * g.s : g.h + (i - g.P) * g.s, end = i < g.P ? g.h : g.m;
    const int c = end - lo;
    *start = lo;
    *count = c < 0 ? 0 : (c < g.s ? c : g.s);
}
__host__ __device__ inline int tile_label(const TilePlan &g, int a) { return a < g.h ? g.n - 1 - 2 * a : 2 * g.m - 2 * a; }
// tile u of stage number st (0-based).  kTileNone: the pieces P - 1 and 2P - 1, which stage -2 leaves alone.
__host__ __device__ inline Tile tile_at(const TilePlan &g, int st, int u)
{
    Tile x;
    const int t = st + g.first, I = 2 * g.P;
    if (t < 0) {
        x.i = u;
        x.j = t + I - u;
        x.kind = kTileEarly;
        if (t == -2 && u == g.P - 1) {
            x.j = I - 1;
            x.kind = kTileNone;
        }
    } else if (!(t & 1) && u == 0) {
        x.i = t / 2;
        x.j = t / 2 + g.P;
        x.kind = kTileSpecial;
    } else {
        const int v = (t & 1) ? u : u - 1, late = (t + 1) / 2;
        x.kind = v < late ? kTileLate : kTileEarly;
        x.i = v < late ? v : t + 1 + (v - late);
        x.j = v < late ? t - v : I - 1 - (v - late);
    }
    tile_piece(g, x.i, &x.a0, &x.na);
    tile_piece(g, x.j, &x.b0, &x.nb);
    return x;
}
// Restricted parametrisation (pairs (i, j), i < free_rows): does the tile hold no free pair?  (labels go down by 2 along
// a piece)
__host__ __device__ inline bool tile_is_identity(const TilePlan &g, const Tile &x, int free_rows)
{
    if (x.kind == kTileNone) return true;
    if (x.kind == kTileSpecial) return false;
    const int la = x.na ? tile_label(g, x.a0 + x.na - 1) : g.n, lb = x.nb ? tile_label(g, x.b0 + x.nb - 1) : g.n;
    return la >= free_rows && lb >= free_rows;
}

// The tiles of a stage, those that hold a free pair first, for launches that take only those (tile_apply_listed, tile_pairs_listed).
constexpr int kTileMaxP = (kTileMaxN / 2 + kTileSlots - 1) / kTileSlots;
struct TileList {
    int active;
    unsigned char tile[kTileMaxP];
};
struct TileAll {};
static_assert(kTileMaxP <= 256, "a tile's number in its stage is a byte");
__device__ __forceinline__ int tile_listed(const TileList &l, int i) { return l.tile[i]; }
__device__ __forceinline__ int tile_listed(const TileAll &, int i) { return i; }
__device__ __forceinline__ int tiles_listed(const TilePlan &, const TileList &l) { return l.active; }
__device__ __forceinline__ int tiles_listed(const TilePlan &g, const TileAll &) { return g.P; }

// index in E of the pair (a, b), and of the pair of a with row 0
__device__ __forceinline__ long long tile_pair_entry(const TilePlan &g, int a, int b)
{
    int k = a + b;
    if (k >= g.m) k -= g.m;
    const int d = a < b ? b - a : a - b, p = d < g.m - d ? d : g.m - d;
    return (long long)k * g.h + p;
}
__device__ __forceinline__ long long tile_held_entry(const TilePlan &g, int a)
{
    int k = 2 * a;
    if (k >= g.m) k -= g.m;
    return (long long)k * g.h;
}
__device__ __forceinline__ bool tile_has_pair(const TilePlan &g, const Tile &x, int a, int b)
{
    return x.kind == kTileSpecial || (a + b >= g.m) == (x.kind == kTileEarly);
}
// The range (split_bf16.hpp) of the gradient's matrix S, one for all of it: the stages keep its norm.  Words that the build kernel clears
// and the antisymmetric part's sets, 1 each: an element other than zero, one of the middle range or above, one above it.
// Behind them, cleared with them, a count for every special tile (tile_gradient_kernel).
enum { kTileAny = 0, kTileMiddle = 1, kTileLarge = 2, kTileRangeWords = 3 };
__device__ __forceinline__ float tile_scale(const int *range)
{
    return range[kTileLarge] ? range_scale(kRangeLarge) : range[kTileMiddle] || !range[kTileAny] ? 1.f : range_scale(kRangeSmall / 2);
}

// A tile's rotations as a table of s x 64 entries, row by row in order.  Row r of an ordinary tile: row r of piece i with every
// row of piece j.  Row r of a special tile, for piece i and for piece i + P: with the rows before it, oldest first, and in the
// last entry with row 0.  Places without a rotation: -1.
constexpr int kTileTable = kTilePad / 2;   // entries in a row of the table
constexpr int kTileThreads = 512;          // of the kernels that go rotation by rotation
struct TileEntry {
    int e;            // in E
    bool ordered;     // the first row has the smaller label
};
__device__ __forceinline__ TileEntry tile_entry(const TilePlan &g, const Tile &x, bool special, int which, int r, int slot)
{
    TileEntry t{-1, false};
    if (special) {
        const int start = which ? x.b0 : x.a0, a = start + r;
        if (r >= (which ? x.nb : x.na)) return t;
        if (slot == kTileTable - 1) {
            t.e = (int)tile_held_entry(g, a);
        } else if (slot < r) {
            t.e = (int)tile_pair_entry(g, a, start + slot);
            t.ordered = tile_label(g, a) < tile_label(g, start + slot);
        }
    } else if (r < x.na && slot < x.nb) {
        const int a = x.a0 + r, b = x.b0 + slot;
        if (tile_has_pair(g, x, a, b)) {
            t.e = (int)tile_pair_entry(g, a, b);
            t.ordered = tile_label(g, a) < tile_label(g, b);
        }
    }
    return t;
}
constexpr int kTilePlaces = kTileTable * kTileTable;
// Piece, row and slot of place `id` < kTilePlaces.  The lanes of a wavefront run along r + slot, that is along a block, whose
// angles are neighbours in memory.  The two triangles of a special tile share the places (row 63, which no piece has, stands
// for the entries with row 0 of piece i + P).
__device__ __forceinline__ void tile_table_place(bool special, int id, int *which, int *r, int *slot)
{
    const int row = id % kTileTable, col = (id / kTileTable - id) & (kTileTable - 1), last = kTileTable - 1;
    *which = special && (col > row || row == last) ? 1 : 0;
    *r = special && (col > row || row == last) ? col : row;
    *slot = !special || (col < row && row != last) ? col : (col > row ? row : last);
}
// Cosines and sines (the sine negated when the first row has the larger label; (1, 0) for a pair that is bypassed or not in the
// tile) into the table `out`, [piece][rows][64].
template <typename R2, typename R>
__device__ __forceinline__ void tile_coefs(const TilePlan &g, const Tile &x, bool special, int rows,
                                           const float *__restrict__ theta, const int *__restrict__ map, R2 *out)
{
    auto place = [&](int id, int *which, int *r, int *slot) {
        tile_table_place(special, id, which, r, slot);
        return out + ((size_t)*which * rows + *r) * kTileTable + *slot;
    };
    if (special)   // (the rows' ends: rotations are taken eight at a time)
        for (int id = threadIdx.x; id < 2 * rows * kTileTable; id += kTileThreads) {
            const int r = id / kTileTable % rows, slot = id % kTileTable;
            if (slot >= r && slot != kTileTable - 1) {
                out[id].x = (R)1;
                out[id].y = (R)0;
            }
        }
    // angles first, eight loads at a time, then their cosines and sines
    static_assert(kTilePlaces == 8 * kTileThreads, "eight places per thread");
    float th[8], sign[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        int which, r, slot;
        tile_table_place(special, threadIdx.x + q * kTileThreads, &which, &r, &slot);
        const TileEntry t = tile_entry(g, x, special, which, r, slot);
        const int e = t.e >= 0 && map ? map[t.e] : t.e;
        th[q] = e >= 0 ? theta[e] : 0.f;
        sign[q] = e < 0 ? 0.f : (t.ordered ? 1.f : -1.f);
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        int which, r, slot;
        R2 *to = place(threadIdx.x + q * kTileThreads, &which, &r, &slot);
        if (r < rows) {
            to->x = (R)th[q];
            to->y = (R)sign[q];
        }
    }
#pragma unroll 1
    for (int id = threadIdx.x; id < kTilePlaces; id += kTileThreads) {
        int which, r, slot;
        R2 *to = place(id, &which, &r, &slot);
        if (r >= rows) continue;
        const R2 v = *to;
        const double2 cs = tile_sincos((double)v.x);
        R2 w;
        w.x = v.y != (R)0 ? (R)cs.x : (R)1;
        w.y = v.y != (R)0 ? (R)(v.y > (R)0 ? cs.y : -cs.y) : (R)0;
        *to = w;
    }
}

// the transposed rotation of rows p, q: p' = c p + s q, q' = c q - s p
template <typename T, typename R2>
__device__ __forceinline__ void tile_rotate(T &p, T &q, const R2 &cs)
{
    const T a = p, b = q;
    p = fma(cs.x, a, cs.y * b);
    q = fma(cs.x, b, -(cs.y * a));
}

// address spaces of the loads that go from memory to LDS
typedef __attribute__((address_space(3))) void *lds_ptr;
typedef __attribute__((address_space(1))) const void *global_ptr;
constexpr int kWaitForLoads = 0x0f70;   // s_waitcnt vmcnt(0): this wavefront's loads into LDS are there

// A fragment of a tile's matrix: rows 32 f .. + 31, contraction indices 16 k .. + 15, as in product_kernels.hpp but with
// the indices of a half wavefront in the order in which the matrix instructions leave their results in registers, so that
// a result can be the next product's operand without a move between lanes.
__device__ __forceinline__ int tile_k(int half, int j) { return (j & 3) + 4 * half + 8 * (j >> 2); }
// Place of element (row, col) in a block of float32 fragments of such an order, `columns` / 16 of them beside one another: a lane's
// eight values of a fragment are consecutive, a wavefront loads or stores one as 2 KB.
__device__ __forceinline__ int tile_block_at(int columns, int row, int col)
{
    return ((row >> 5) * (columns / 16) + (col >> 4)) * 512 + ((row & 31) + 32 * ((col >> 2) & 1)) * 8 + (col & 3) +
           4 * ((col >> 3) & 1);
}
// a b over 16 contraction indices added to large + small, operands given as pieces: the largest products in one accumulator,
// those below 2^-16 of them in the other.  The two take turns, since a matrix instruction has to wait for the one before it on
// its accumulator; and half of the roundings are those of small sums.
__device__ __forceinline__ void tile_mfma(const u32x4 (&a)[3], const u32x4 (&b)[3], f32x16 &large, f32x16 &small)
{
    constexpr int pa[6] = {2, 1, 0, 0, 1, 0}, pb[6] = {0, 0, 2, 1, 1, 0};
#pragma unroll
    for (int p = 0; p < 6; ++p) {
        f32x16 &acc = p & 1 ? large : small;
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[pa[p]]), __builtin_bit_cast(bf16x8, b[pb[p]]),
                                                      acc, 0, 0, 0);
    }
}

// What the apply stages have to know of their operand's columns: tops, the bits of their largest magnitudes.  A workgroup takes
// 64 columns, a wavefront an eighth of the rows.
struct TileTops {
    int rows;
    long long B;
    const float *X;      // null: nothing to do
    unsigned *tops;
};
inline long long tile_top_blocks(const TileTops &t) { return t.X ? (t.B + 63) / 64 : 0; }
__device__ __forceinline__ void tile_tops(const TileTops &t, long long block, float (*part)[64])
{
    constexpr int WAVES = kTileThreads / 64, ONCE = 32;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long long mine = block * 64 + lane, col = mine < t.B ? mine : t.B - 1;
    const int per = (t.rows + WAVES - 1) / WAVES, from = wave * per, to = from + per < t.rows ? from + per : t.rows;
    float top = 0.f;
    for (int r0 = from; r0 < to; r0 += ONCE) {
        float x[ONCE];
#pragma unroll
        for (int r = 0; r < ONCE; ++r) x[r] = t.X[(long long)(r0 + r < to ? r0 + r : to - 1) * t.B + col];
#pragma unroll
        for (int r = 0; r < ONCE; r += 2) top = range_top(top, x[r], x[r + 1]);
    }
    part[wave][lane] = top;
    __syncthreads();
    if (wave == 0 && mine < t.B) {
        for (int w = 1; w < WAVES; ++w) top = range_top(top, part[w][lane], 0.f);
        t.tops[mine] = __float_as_uint(top);
    }
}

// Matrices of the tiles: A = the tile's transposed rotations in block order (the reverse sweep's matrix; its transpose is
// the forward sweep's), float64, rounded once at the end and cut into pieces in operand order.
//
// A workgroup makes one tile, a lane two columns of it, a wavefront the rotations with some of the rows that stay in registers:
// 8 rows of piece j (ordinary tile), or 16 rows of one piece (special tile: of the rows that are finished).  A row of piece i is
// fresh in the first wavefront and handed from one to the next through LDS, so the wavefronts work on different rows at once:
// s / 2 + 7 steps of twice 8 rotations where one wavefront with all rows takes s steps of s.  A special tile's row stays with the
// wavefront it belongs to, after its rotation with row 0, which the two pieces take in turn; that chain makes its steps longer,
// so two workgroups share it, 64 columns each.
//
// Bound by the float64 rotations (four instructions of eight cycles each; 81000 cycles for an ordinary tile's loop, which is
// what they take), a compute unit holding one tile.  All matrices in pieces: n = 1002 53 us, n = 4097 with m = 512 238 us
// (a table kernel, one lane per column of a tile and a kernel that cuts into pieces: 78 and 279 us).
constexpr int kTilePart = 8, kTileParts = (kTileSlots + kTilePart - 1) / kTilePart;   // ordinary tiles
constexpr int kTileSpecialPart = 16;
struct TileBuildShared {
    union {
        double2 special[2][kTileSlots][kTileTable];
        struct {
            double2 coef[kTileTable][kTileTable];
            float A[kTilePad][kTilePad + 1];
        } ordinary;
        float A[kTilePad][kTilePad + 1];     // of a special tile: when its coefficients are done with
        float tops[kTileThreads / 64][64];
    };
    double hand[2][kTileParts - 1][2][kTilePad];   // rows on their way to the next wavefront, by the parity of the step
    double row0[kTilePad];
};
// A wavefront of an ordinary tile takes row r (or pair of rows) in step r + its number: `row(r, t)`; all make the same number
// of steps.
template <typename F>
__device__ __forceinline__ void tile_steps(int s, int parts, int wave, F &&row)
{
    const int before = wave < parts ? wave : s + parts - 1;
    for (int t = 0; t < before; ++t) __syncthreads();
    if (wave >= parts) return;
    for (int r = 0; r < s; ++r) {
        row(r, r + wave);
        __syncthreads();
    }
    for (int t = wave + s; t < s + parts - 1; ++t) __syncthreads();
}
__global__ __launch_bounds__(kTileThreads, 1) void tile_build_kernel(TilePlan g, const float *__restrict__ theta,
                                                                     const int *__restrict__ map, int free_rows,
                                                                     u32x4 *__restrict__ out, int transposed,
                                                                     int *__restrict__ range, TileTops tops, int top_blocks)
{
    __shared__ TileBuildShared sh;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tiles = g.stages * g.P;
    const bool special = (int)blockIdx.x < 2 * g.P;
    const int id = (int)blockIdx.x - 2 * g.P - top_blocks, half = special ? blockIdx.x & 1 : 0;
    if (range && blockIdx.x == 0 && threadIdx.x < kTileRangeWords + g.P) range[threadIdx.x] = 0;
    if (!special && id < 0) {
        tile_tops(tops, id + top_blocks, sh.tops);
        return;
    }
    const int st = special ? 2 * ((int)blockIdx.x / 2) - g.first : id / g.P, u = special ? 0 : id % g.P;
    const bool identity = !special && id == tiles;   // shared by all tiles without a free pair, behind the last tile
    float(*A)[kTilePad + 1] = special ? sh.A : sh.ordinary.A;
    if (identity) {
        for (int i = threadIdx.x; i < kTilePad * kTilePad; i += kTileThreads)
            A[i / kTilePad][i % kTilePad] = i / kTilePad == i % kTilePad ? 1.f : 0.f;
    } else {
        const Tile x = tile_at(g, st, u);
        if (!special && (x.kind == kTileSpecial || tile_is_identity(g, x, free_rows))) return;
        tile_coefs<double2, double>(g, x, special, special ? g.s : kTileTable, theta, map, special ? &sh.special[0][0][0] : &sh.ordinary.coef[0][0]);
        if (special && threadIdx.x < 64) sh.row0[threadIdx.x] = threadIdx.x + 64 * half == kTilePad - 1 ? 1.0 : 0.0;
        __syncthreads();
        auto unit = [&](int row, double(&v)[2]) {
            v[0] = row == lane ? 1.0 : 0.0;
            v[1] = row == lane + 64 ? 1.0 : 0.0;
        };
        if (special) {
            constexpr int ROWS = kTileSpecialPart;
            const int which = wave & 1, part = wave >> 1, base = which * (kTilePad / 2);   // (the two on different SIMDs)
            const int col = lane + 64 * half;
            const double2 *table = &sh.special[0][0][0] + (size_t)which * g.s * kTileTable;
            double q[ROWS];
#pragma unroll
            for (int b = 0; b < ROWS; ++b) q[b] = 0.0;
            for (int t = 0; t < g.s + 3; ++t) {
                const int r = t - part, place = r - ROWS * part;      // (row r ends in part r / 16)
                const bool mine = r < g.s && place >= 0, own = mine && place < ROWS;
                double cur = 0.0;
                double2 held{};
                if (mine) {
                    const double2 *coef = table + (size_t)r * kTileTable;
                    held = coef[kTileTable - 1];
                    cur = part ? sh.hand[(t + 1) & 1][part - 1][which][lane] : (base + r == col ? 1.0 : 0.0);
#pragma unroll
                    for (int b0 = 0; b0 < ROWS; b0 += 8)
                        if (b0 < place) {
                            double2 cs[8];   // read together: one LDS latency for eight rotations
#pragma unroll
                            for (int v = 0; v < 8; ++v) cs[v] = coef[ROWS * part + b0 + v];
                            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                            for (int v = 0; v < 8; ++v)
                                if (b0 + v < ROWS - 1 || !own) tile_rotate(cur, q[b0 + v], cs[v]);   // (its last entry may be row 0's)
                        }
                    if (!own) sh.hand[t & 1][part][which][lane] = cur;
                }
                for (int turn = 0; turn < 2; ++turn) {                // row 0: piece i, then piece i + P
                    if (own && turn == which) {
                        double zero = sh.row0[lane];
                        tile_rotate(cur, zero, held);
                        sh.row0[lane] = zero;
                    }
                    __syncthreads();
                }
                if (own)
#pragma unroll
                    for (int b0 = 0; b0 < ROWS; b0 += 8)
                        if (place / 8 == b0 / 8)
#pragma unroll
                            for (int v = 0; v < 8; ++v) q[b0 + v] = place % 8 == v ? cur : q[b0 + v];
            }
#pragma unroll
            for (int b = 0; b < ROWS; ++b) {
                const int row = base + ROWS * part + b;
                if (row != kTilePad - 1) A[row][col] = (float)q[b];
            }
            if (threadIdx.x < 64) A[kTilePad - 1][threadIdx.x + 64 * half] = (float)sh.row0[threadIdx.x];
        } else {
            const int parts = (g.s + kTilePart - 1) / kTilePart, first = kTilePart * wave;
            const double2(*coef)[kTileTable] = sh.ordinary.coef;
            double q[kTilePart][2];
#pragma unroll
            for (int b = 0; b < kTilePart; ++b) {
                unit(first + b < g.s ? kTilePad / 2 + first + b : -1, q[b]);
            }
            double2 cs[2][kTilePart];   // a row's coefficients are read while the row before it is turned
            auto read = [&](int set, int r) {
#pragma unroll
                for (int v = 0; v < kTilePart; ++v) cs[set][v] = coef[r < kTileTable ? r : 0][first + v];
            };
            read(0, 0);
            // (two rows a step; the row after an odd number of them is zeros)
            tile_steps((g.s + 1) / 2, parts, wave, [&](int pair, int t) __attribute__((always_inline)) {
                double cur[2][2];
                if (wave) {
#pragma unroll
                    for (int w = 0; w < 2; ++w)
#pragma unroll
                        for (int i = 0; i < 2; ++i) cur[w][i] = sh.hand[(t + 1) & 1][wave - 1][w][lane + 64 * i];
                } else {
                    unit(2 * pair, cur[0]);
                    unit(2 * pair + 1 < g.s ? 2 * pair + 1 : -1, cur[1]);
                }
                read(1, 2 * pair + 1);
#pragma unroll
                for (int w = 0; w < 2; ++w) {
#pragma unroll
                    for (int v = 0; v < kTilePart; ++v)
#pragma unroll
                        for (int i = 0; i < 2; ++i) tile_rotate(cur[w][i], q[v][i], cs[w][v]);
                    if (w == 0) read(0, 2 * pair + 2);
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        if (wave + 1 < parts)
                            sh.hand[t & 1][wave][w][lane + 64 * i] = cur[w][i];
                        else
                            A[2 * pair + w][lane + 64 * i] = (float)cur[w][i];
                }
            });
#pragma unroll
            for (int b = 0; b < kTilePart; ++b) {
                const int row = kTilePad / 2 + first + b;
                const bool last = row == kTilePad - 1;                // row 0, where it is this tile's
                A[row][lane] = last ? 0.f : (float)q[b][0];
                A[row][lane + 64] = last ? (u == 0 && lane == 63 ? 1.f : 0.f) : (float)q[b][1];
            }
            for (int row = (g.s + 1) / 2 * 2 + wave; row < kTilePad / 2; row += kTileThreads / 64) A[row][lane] = A[row][lane + 64] = 0.f;
        }
    }
    __syncthreads();
    const long long tile = identity ? tiles : (long long)st * g.P + u;
    u32x4 *o = out + tile * kTilePieceWords + lane;
    constexpr int FRAGMENTS = (kTilePad / 32) * (kTilePad / 16);
    for (int i = wave; i < (special ? FRAGMENTS / 2 : FRAGMENTS); i += kTileThreads / 64) {
        // (of a special tile those of its half of the columns, which are rows of the transposed matrix)
        const int f = !special ? i : transposed ? half * (FRAGMENTS / 2) + i : i / 4 * 8 + half * 4 + i % 4;
        const int row = (f / (kTilePad / 16)) * 32 + (lane & 31), k0 = (f % (kTilePad / 16)) * 16;
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int k = k0 + tile_k(lane >> 5, j);
            v[j] = transposed ? A[k][row] : A[row][k];
        }
        const Split8 sp = split8(v);
        o[f * 192] = sp.h;
        o[f * 192 + 64] = sp.m;
        o[f * 192 + 128] = sp.l;
    }
}

// where a tile's pieces are (in tiles)
__device__ __forceinline__ size_t tile_piece_index(const TilePlan &g, int st, int u, bool identity)
{
    return identity ? (size_t)g.stages * g.P : (size_t)st * g.P + u;
}

struct TileApplyArgs {
    TilePlan g;
    int stage, rows, free_rows;
    long long B;
    const u32x4 *pieces;
    bool from_rows, to_rows;   // first and last stage of a sweep, which take every row
    const float *X;      // the first stage's operand, row by row; nullptr: the identity
    float *W;            // what the stages work on (tile_operand_floats)
    float *Y;            // the last stage's result, row by row
    unsigned chunk;      // columns per workgroup
    const unsigned *tops;   // largest magnitude of every column at the sweep's start, as bits (its stages keep a column's
                            // norm: split_bf16.hpp, "Range"); null: all of the middle range
};

// One stage on B columns: rows of each tile <- matrix * rows.  A workgroup takes one tile and a run of columns, a wavefront
// 32 rows of the result with its part of the matrix in registers throughout.  Per step of kTileCols columns a wavefront brings
// 32 of the tile's rows (a lane has its values of a column, so cutting them into pieces needs no exchange) and puts the pieces
// into LDS as fragments, into the buffer of the step's parity: while a step's products run, the next one's rows are cut and the
// rows after that are on their way.  Between a sweep's first and last stage the rows lie in the order in which the wavefronts
// take and leave them, 32 consecutive bytes a lane: as rows, 16 loads of 4 bytes a lane took a wavefront 1800 cycles to issue
// and its stores 1000, the 48 matrix instructions of a step 1770.  (An operand of the tiles has fewer than max(2n, 2048)
// columns, less than 4 GiB.)
struct TileApplyShared {
    u32x4 panel[2][kTilePad / 16][3][64];
};
template <typename List>
__device__ __forceinline__ void tile_apply(const TileApplyArgs &a, const List &list, unsigned block, TileApplyShared &sh)
{
    constexpr int KF = kTilePad / 16;
    const TilePlan &g = a.g;
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tiles = tiles_listed(g, list), u = tile_listed(list, block % tiles);
    const unsigned B = (unsigned)a.B, n0 = block / tiles * a.chunk, n1 = n0 + a.chunk < B ? n0 + a.chunk : B;
    const Tile x = tile_at(g, a.stage, u);
    const bool identity = tile_is_identity(g, x, a.free_rows);
    if (n0 >= B || (!a.from_rows && !a.to_rows && identity)) return;
    // this wavefront's 32 rows: labels first, first - 2, ...; `count` of them are there, row 0 may stand at the end
    const int local = 32 * wave, in_piece = local % kTileHalf;
    const bool second = local >= kTileHalf;
    const int count = (second ? x.nb : x.na) - in_piece;
    const int first = tile_label(g, (second ? x.b0 : x.a0)) - 2 * in_piece;
    const bool has_held = u == 0 && local == kTilePad - 32;
    const int skip = first >= a.rows ? 1 : 0;          // the added row of an odd problem is the first of its piece
    // byte offset of row first - 2 (4 half); the rows below it are 8 B bytes apart
    const unsigned row_of_half = (unsigned)(first - 8 * half) * B;
    // ... and where they are in W
    const unsigned blocks = (B + kTileCols - 1) / kTileCols;
    float *const mine = a.W + (size_t)((second ? x.j : x.i) * blocks) * (kTileHalf * kTileCols) + (wave & 1) * 1024;
    float *const held_row = a.W + (size_t)(2 * g.P) * blocks * (kTileHalf * kTileCols);

    // a lane brings 16 rows of one column, those of its half of the fragments
    float xr[16];
    unsigned top = 0u;
    auto fetch = [&](unsigned c0) {
        const unsigned col = c0 + l32 < n1 ? c0 + l32 : n1 - 1;
        if (a.tops) top = a.tops[col];
        if (a.from_rows) {
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const int r = 16 * (q >> 3) + tile_k(half, q & 7), below = 16 * (q >> 3) + tile_k(0, q & 7);
                const bool there = r < count && r >= skip, held = has_held && r == 31;
                const unsigned at = there ? (row_of_half - 2 * below * B + col) * 4u : col * 4u;
                const float v = a.X ? *reinterpret_cast<const float *>(reinterpret_cast<const char *>(a.X) + at)
                                    : ((int)col == (there ? first - 2 * r : 0) ? 1.f : 0.f);
                xr[q] = there || held ? v : 0.f;
            }
        } else {
            const float *src = mine + c0 / kTileCols * (kTileHalf * kTileCols) + lane * 8;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 v = *reinterpret_cast<const f32x4 *>(src + (q >> 1) * 512 + (q & 1) * 4);
#pragma unroll
                for (int w = 0; w < 4; ++w) xr[4 * q + w] = v[w];
            }
            if (has_held) {                            // (its place in the block is nobody's)
                const float v = held_row[c0 + l32];
                xr[15] = half ? v : xr[15];
            }
        }
    };
    float undo[2] = {1.f, 1.f};   // of the columns in the panels
    auto stash = [&](int buf) {
        const float scale = range_scale(__uint_as_float(top));
        undo[buf] = range_unscale(scale);
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            float v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = xr[8 * f + q] * scale;
            const Split8 sp = split8(v);
            sh.panel[buf][2 * wave + f][0][lane] = sp.h;
            sh.panel[buf][2 * wave + f][1][lane] = sp.m;
            sh.panel[buf][2 * wave + f][2][lane] = sp.l;
        }
    };
    fetch(n0);
    u32x4 fa[KF][3];
    const u32x4 *ap = a.pieces + tile_piece_index(g, a.stage, u, identity) * kTilePieceWords + (size_t)wave * KF * 192 + lane;
#pragma unroll
    for (int kf = 0; kf < KF; ++kf)
#pragma unroll
        for (int p = 0; p < 3; ++p) fa[kf][p] = ap[kf * 192 + 64 * p];
    stash(0);
    if (n0 + kTileCols < n1) fetch(n0 + kTileCols);
    for (unsigned at = n0; at < n1; at += 2 * kTileCols)
#pragma unroll
        for (int buf = 0; buf < 2; ++buf) {
            const unsigned c0 = at + buf * kTileCols;
            if (buf && c0 >= n1) break;
            __syncthreads();   // this step's panel is whole; the other one is free (its readers passed this barrier)
            f32x16 acc, small;
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] = small[v] = 0.f;
#pragma unroll
            for (int kf = 0; kf < KF; ++kf) {
                const u32x4 fb[3] = {sh.panel[buf][kf][0][lane], sh.panel[buf][kf][1][lane], sh.panel[buf][kf][2][lane]};
                tile_mfma(fa[kf], fb, acc, small);
            }
            if (c0 + kTileCols < n1) {
                stash(buf ^ 1);
                if (c0 + 2 * kTileCols < n1) fetch(c0 + 2 * kTileCols);
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] = (acc[v] + small[v]) * undo[buf];
            const unsigned col = c0 + l32;
            if (!a.to_rows) {
                float *to = mine + c0 / kTileCols * (kTileHalf * kTileCols) + lane * 8;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    f32x4 v;
#pragma unroll
                    for (int w = 0; w < 4; ++w) v[w] = acc[4 * q + w];
                    *reinterpret_cast<f32x4 *>(to + (q >> 1) * 512 + (q & 1) * 4) = v;
                }
                if (has_held && half) held_row[col] = acc[15];
            } else if (col < n1) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int r = 8 * (v >> 2) + 4 * half + (v & 3), below = 8 * (v >> 2) + (v & 3);
                    char *const to = reinterpret_cast<char *>(a.Y);
                    if (r < count && r >= skip)
                        *reinterpret_cast<float *>(to + (row_of_half - 2 * below * B + col) * 4u) = acc[v];
                    else if (has_held && r == 31)
                        a.Y[col] = acc[v];
                }
            }
        }
}
template <typename List>
__global__ __launch_bounds__(2 * kTilePad, 2) void tile_apply_kernel(TileApplyArgs a, List list)
{
    __shared__ TileApplyShared sh;
    tile_apply(a, list, blockIdx.x, sh);
}

// ---- the gradient's matrix S (tile_s_floats).
// S[p][q] = C[row p][row q] - C[row q][row p] for C the sum of its slices.  A workgroup takes two 32 x 32 blocks that mirror each
// other and reads each slice of them once; the last ones take row 0.  Bound by memory (labels go by two, so half of a line is
// another block's): n = 1002 with 7 slices 18 us, n = 4097
// 50 us (a kernel that summed the slices first, and one that read C twice: 15 + 10 us with 4 slices, 83 us).
inline unsigned tile_antisym_blocks(const TilePlan &g)
{
    const int t = 2 * g.P * (kTileHalf / 32);
    return (unsigned)(t * (t + 1) / 2 + (2 * g.P * kTileHalf + 255) / 256);
}
__global__ __launch_bounds__(256) void tile_antisym_kernel(TilePlan g, int rows, int slices, const float *__restrict__ C,
                                                           float *__restrict__ S, int *__restrict__ range)
{
    __shared__ float block[2][32][33];
    const int t = 2 * g.P * (kTileHalf / 32), pairs = t * (t + 1) / 2;
    auto label = [&](int p) {
        int start, count;
        tile_piece(g, p / kTileHalf, &start, &count);
        const int r = p % kTileHalf;
        if (r >= count) return -1;
        const int l = tile_label(g, start + r);
        return l < rows ? l : -1;
    };
    const size_t slice = (size_t)rows * rows;
    float top = 0.f;
    if ((int)blockIdx.x < pairs) {
        int bi = 0, bj = blockIdx.x;
        while (bj >= t - bi) bj -= t - bi++;
        bj += bi;
        const int p0 = bi * 32, q0 = bj * 32, tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
        const int lp = label(p0 + tx), lq = label(q0 + tx);
        size_t at[8];          // rows ty, ty + 8, ... of block (p, q), then of block (q, p)
        bool there[8];
        float sum[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int lr = label((i < 4 ? p0 : q0) + ty + 8 * (i & 3)), lc = i < 4 ? lq : lp;
            there[i] = lr >= 0 && lc >= 0;
            at[i] = there[i] ? (size_t)lr * rows + lc : 0;
            sum[i] = 0.f;
        }
#pragma unroll 4
        for (int s = 0; s < slices; ++s)
#pragma unroll
            for (int i = 0; i < 8; ++i) sum[i] += C[s * slice + at[i]];
#pragma unroll
        for (int i = 0; i < 8; ++i) block[i >> 2][ty + 8 * (i & 3)][tx] = there[i] ? sum[i] : 0.f;
        __syncthreads();
        // four consecutive columns of a row: half of a lane's values of a fragment
        const int r = threadIdx.x / 2 % 32, c = threadIdx.x / 128 * 16 + threadIdx.x / 64 % 2 * 4 + threadIdx.x % 2 * 8;
#pragma unroll
        for (int which = 0; which < 2; ++which) {
            f32x4 v;
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = block[which][r][c + q] - block[which ^ 1][c + q][r];
            const int row0 = which ? q0 : p0, col0 = which ? p0 : q0;
            float *to = S + (size_t)(row0 / kTileHalf * 2 * g.P + col0 / kTileHalf) * kTileBlock;
            *reinterpret_cast<f32x4 *>(to + tile_block_at(kTileHalf, row0 % kTileHalf + r, col0 % kTileHalf + c)) = v;
            top = range_top(range_top(top, v[0], v[1]), v[2], v[3]);
        }
    } else {
        const int p = ((int)blockIdx.x - pairs) * 256 + threadIdx.x;
        if (p < 2 * g.P * kTileHalf) {
            const int l = label(p);
            float of_row = 0.f, of_col = 0.f;
            if (l >= 0)
                for (int s = 0; s < slices; ++s) {
                    of_row += C[s * slice + l];
                    of_col += C[s * slice + (size_t)l * rows];
                }
            S[tile_held_offset(g) + p] = of_row - of_col;
            top = range_top(top, of_row - of_col, 0.f);
        }
    }
    // (each word is written by the first wavefronts that get there: they all write the same)
    auto set = [&](bool on, int word) {
        if (__any(on) && (threadIdx.x & 63) == 0 && range[word] == 0) range[word] = 1;
    };
    set(top > 0.f, kTileAny);
    set(top >= kRangeSmall, kTileMiddle);
    set(top >= kRangeLarge, kTileLarge);
}

struct TileTwoSidedArgs {
    TilePlan g;
    int stage, free_rows;
    const u32x4 *pieces;   // of A (not transposed)
    const float *in;       // S before the stage
    float *out;            // S after it: the same array, or another one
    float *blocks;         // every tile's own block before its stage, in the order of tile_block_at
    const int *range;      // of S
};
struct TilePair {
    Tile x, y;
    int ux, uy;
    bool idx, idy;         // identities
};
// pairs of the listed tiles, then one of them and another
template <typename List>
__device__ __forceinline__ TilePair tile_pair(const TileTwoSidedArgs &a, const List &list, unsigned id)
{
    const TilePlan &g = a.g;
    TilePair t;
    const int c = tiles_listed(g, list), both = c * (c + 1) / 2;
    int first = 0, second = id;
    if (std::is_same<List, TileAll>::value || second < both) {
        while (second >= c - first) second -= c - first++;
        second += first;
    } else {
        first = (second - both) % c;
        second = c + (second - both) / c;
    }
    const int p = tile_listed(list, first), q = tile_listed(list, second);
    t.ux = p < q ? p : q;
    t.uy = p < q ? q : p;
    t.x = tile_at(g, a.stage, t.ux);
    t.y = tile_at(g, a.stage, t.uy);
    t.idx = tile_is_identity(g, t.x, a.free_rows);
    t.idy = tile_is_identity(g, t.y, a.free_rows);
    return t;
}
__device__ __forceinline__ size_t tile_s_block(const TilePlan &g, int i, int j) { return ((size_t)i * 2 * g.P + j) * kTileBlock; }

// Rows 32 wave .. + 31 of S for the columns of fragment kf, a lane's eight values (S of the pair's two tiles; row 0, which stands in
// the last row of tile 0, from behind the blocks)
__device__ __forceinline__ void tile_load_s(const TileTwoSidedArgs &a, const TilePair &t, int wave, int kf, f32x4 (&v)[2])
{
    const int lane = threadIdx.x & 63;
    const int i = wave < 2 ? t.x.i : t.x.j, j = kf < 4 ? t.y.i : t.y.j;
    const float *src = a.in + tile_s_block(a.g, i, j) + ((wave & 1) * 4 + (kf & 3)) * 512 + lane * 8;
    v[0] = *reinterpret_cast<const f32x4 *>(src);
    v[1] = *reinterpret_cast<const f32x4 *>(src + 4);
}
__device__ __forceinline__ void tile_load_held(const TileTwoSidedArgs &a, const TilePair &t, int wave, int kf, f32x4 (&v)[2])
{
    if (t.ux != 0 || wave != 3) return;
    const int lane = threadIdx.x & 63, half = lane >> 5;
    const float *held = a.in + tile_held_offset(a.g);
    if ((lane & 31) == 31) {
        const float *src = held + (kf < 4 ? t.y.i : t.y.j) * kTileHalf + (kf & 3) * 16 + 4 * half;
        v[0] = *reinterpret_cast<const f32x4 *>(src);
        v[1] = *reinterpret_cast<const f32x4 *>(src + 8);
    }
}
// (the column of row 0, in tile 0's own pair)
__device__ __forceinline__ void tile_load_held_column(const TileTwoSidedArgs &a, const TilePair &t, int wave, f32x4 (&v)[2])
{
    if (t.uy != 0) return;
    const int lane = threadIdx.x & 63, row = (wave & 1) * 32 + (lane & 31);
    if (lane >= 32) {
        const float held = a.in[tile_held_offset(a.g) + (wave < 2 ? t.x.i : t.x.j) * kTileHalf + row];
        v[1][3] = wave == 3 && row == kTileHalf - 1 ? 0.f : -held;
    }
}
// Rows 32 wave .. + 31 and columns 32 part .. + 31 of a result R as the matrix instructions leave it: to (x, y), turned in LDS
// (`turn` is this wavefront's), and as it stands, negated, to (y, x)
typedef float TileTurn[32][36];
__device__ __forceinline__ void tile_store_both(const TileTwoSidedArgs &a, const TilePair &t, f32x16 R, int wave, int part,
                                                TileTurn &turn)
{
    const TilePlan &g = a.g;
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const int i = wave < 2 ? t.x.i : t.x.j, j = part < 2 ? t.y.i : t.y.j;
    const int row0 = (wave & 1) * 32, col = (part & 1) * 32 + l32;
    if (t.ux == 0 && wave == 3 && half == 1) a.out[tile_held_offset(g) + j * kTileHalf + col] = col < g.s ? R[15] : 0.f;
    if (row0 + 31 >= g.s || (part & 1) * 32 + 31 >= g.s)      // places without a row stay zeros
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row = row0 + 8 * (v >> 2) + 4 * half + (v & 3);
            R[v] = row < g.s && col < g.s ? R[v] : 0.f;
        }
    float *mirror = a.out + tile_s_block(g, j, i) + (part & 1) * 2048 + (wave & 1) * 1024 + lane * 8;
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            f32x4 neg;
#pragma unroll
            for (int w = 0; w < 4; ++w) neg[w] = -R[8 * f + 4 * q + w];
            *reinterpret_cast<f32x4 *>(mirror + 512 * f + 4 * q) = neg;
        }
    if (t.ux == t.uy) return;                                 // (its own mirror)
#pragma unroll
    for (int v = 0; v < 16; v += 4) {
        f32x4 four;
#pragma unroll
        for (int w = 0; w < 4; ++w) four[w] = R[v + w];
        *reinterpret_cast<f32x4 *>(&turn[l32][8 * (v >> 2) + 4 * half]) = four;
    }
    wavefront_order();
    float *to = a.out + tile_s_block(g, i, j) + (wave & 1) * 2048 + (part & 1) * 1024 + lane * 8;
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            f32x4 four;
#pragma unroll
            for (int w = 0; w < 4; ++w) four[w] = turn[16 * f + tile_k(half, 4 * q + w)][l32];
            *reinterpret_cast<f32x4 *>(to + 512 * f + 4 * q) = four;
        }
    wavefront_order();   // the next result is turned in the same place
}

// One stage of S <- A S A^T: a workgroup per pair of tiles (x, y), x <= y, in place.  First V = S A_y^T, a wavefront taking
// 32 of its columns (its part of A_y in registers) and all rows, then R = A_x V, a wavefront taking 32 of its rows (its
// part of A_x in registers).  The other operand of both products is cut into pieces once and shared through LDS, half the
// contraction at a time: S as its fragments, V as its accumulators are.  Pairs without a rotation are left alone.
// n = 3002: 26.6 us a stage.
struct TileTwoSidedShared {
    u32x4 panel[kTilePad / 32][kTilePad / 32][3][64];
    TileTurn turn[kTilePad / 32];
};
// The same for a pair of which one tile has no free pair (neither of them tile 0, with which row 0 goes): one product, R = A S of the
// other tile's rows.  S is the operand that goes through LDS; its fragments are, negated, those of the mirrored block.
// n = 4097, m = 512, where that is three pairs of four: 32.5 us a stage beside an operand of 4096 columns (both products, one of them
// with the identity: 35.8).
__device__ __forceinline__ void tile_one_sided(const TileTwoSidedArgs &a, const TilePair &pair, TileTwoSidedShared &sh)
{
    constexpr int MF = kTilePad / 32, KF = kTilePad / 16, KH = KF / 2;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    TilePair t = pair;               // x: the tile that rotates
    if (t.idx) {
        t.x = pair.y;
        t.y = pair.x;
        t.ux = pair.uy;
        t.uy = pair.ux;
    }
    TilePair mirror = t;
    mirror.x = t.y;
    mirror.y = t.x;
    const u32x4 *px = a.pieces + tile_piece_index(a.g, a.stage, t.ux, false) * kTilePieceWords + (size_t)wave * KF * 192 + lane;
    const float scale = -tile_scale(a.range), undo = range_unscale(-scale);
    f32x4 sr[KF][2];
#pragma unroll
    for (int k = 0; k < KF; ++k) tile_load_s(a, mirror, wave, k, sr[k]);
    u32x4 fm[KH][1][3];
    f32x16 R[1][MF];
#pragma unroll
    for (int j = 0; j < MF; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) R[0][j][v] = 0.f;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int k = 0; k < KH; ++k)
#pragma unroll
            for (int q = 0; q < 3; ++q) fm[k][0][q] = px[(KH * h + k) * 192 + 64 * q];
#pragma unroll
        for (int k = 0; k < KH; ++k) {
            float v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = sr[KH * h + k][q >> 2][q & 3] * scale;
            const Split8 sp = split8(v);
            sh.panel[k][wave][0][lane] = sp.h;
            sh.panel[k][wave][1][lane] = sp.m;
            sh.panel[k][wave][2][lane] = sp.l;
        }
        __syncthreads();   // (in the second half: every wavefront has read its part of S)
#pragma unroll
        for (int k = 0; k < KH; ++k) {
            u32x4 fv[MF][3];
#pragma unroll
            for (int j = 0; j < MF; ++j)
#pragma unroll
                for (int q = 0; q < 3; ++q) fv[j][q] = sh.panel[k][j][q][lane];
            mfma_split(fm[k], fv, R);
        }
        if (h == 0) __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < MF; ++j) tile_store_both(a, t, R[0][j] * undo, wave, j, sh.turn[wave]);
}
template <typename List>
__device__ __forceinline__ void tile_two_sided(const TileTwoSidedArgs &a, const List &list, unsigned block_id, TileTwoSidedShared &sh)
{
    constexpr int MF = kTilePad / 32, KF = kTilePad / 16, KH = KF / 2;
    auto &panel = sh.panel;
    const TilePlan &g = a.g;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const TilePair t = tile_pair(a, list, block_id);
    const bool own = t.ux == t.uy;
    if (t.idx && t.idy) return;      // (a tile that stage -2 leaves alone)
    if ((t.idx || t.idy) && t.ux != 0) return tile_one_sided(a, t, sh);
    const u32x4 *px = a.pieces + tile_piece_index(g, a.stage, t.ux, t.idx) * kTilePieceWords + (size_t)wave * KF * 192 + lane;
    const u32x4 *py = a.pieces + tile_piece_index(g, a.stage, t.uy, t.idy) * kTilePieceWords + (size_t)wave * KF * 192 + lane;

    f32x4 sr[KH][2];
    auto fetch = [&](int h) {
#pragma unroll
        for (int k = 0; k < KH; ++k) tile_load_s(a, t, wave, KH * h + k, sr[k]);
#pragma unroll
        for (int k = 0; k < KH; ++k) tile_load_held(a, t, wave, KH * h + k, sr[k]);
        if (h == 1) tile_load_held_column(a, t, wave, sr[KH - 1]);
    };
    auto stash = [&](int k, const float(&v)[8]) {
        const Split8 sp = split8(v);
        panel[k][wave][0][lane] = sp.h;
        panel[k][wave][1][lane] = sp.m;
        panel[k][wave][2][lane] = sp.l;
    };
    u32x4 fm[KH][1][3];
    auto load_matrix = [&](const u32x4 *p, int h) {
#pragma unroll
        for (int k = 0; k < KH; ++k)
#pragma unroll
            for (int q = 0; q < 3; ++q) fm[k][0][q] = p[(KH * h + k) * 192 + 64 * q];
    };
    fetch(0);
    load_matrix(py, 0);
    const float scale = tile_scale(a.range), undo = range_unscale(scale);
    auto stash_s = [&](int h) {
#pragma unroll
        for (int k = 0; k < KH; ++k) {
            if (own) {
                float *o = a.blocks + ((size_t)a.stage * g.P + t.ux) * kTilePad * kTilePad + (wave * KF + KH * h + k) * 512 + lane * 8;
                *reinterpret_cast<f32x4 *>(o) = sr[k][0];
                *reinterpret_cast<f32x4 *>(o + 4) = sr[k][1];
            }
            float v[8];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                v[q] = sr[k][0][q] * scale;
                v[4 + q] = sr[k][1][q] * scale;
            }
            stash(k, v);
        }
    };
    f32x16 V[MF][1], R[1][MF];
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) V[i][0][v] = R[0][i][v] = 0.f;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        if (h) load_matrix(py, h);
        stash_s(h);
        __syncthreads();
        if (h == 0) fetch(1);
#pragma unroll
        for (int k = 0; k < KH; ++k)
#pragma unroll
            for (int i = 0; i < MF; i += 2) {
                u32x4 fs[2][3];
#pragma unroll
                for (int w = 0; w < 2; ++w)
#pragma unroll
                    for (int q = 0; q < 3; ++q) fs[w][q] = panel[k][i + w][q][lane];
                f32x16(&pair)[2][1] = reinterpret_cast<f32x16(&)[2][1]>(V[i]);
                mfma_split(fs, fm[k], pair);
            }
        __syncthreads();
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        load_matrix(px, h);
#pragma unroll
        for (int k = 0; k < KH; ++k) {
            float v[8];
            const int kf = KH * h + k;
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = V[kf / 2][0][8 * (kf & 1) + q];
            stash(k, v);
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < KH; ++k) {
            u32x4 fv[MF][3];
#pragma unroll
            for (int j = 0; j < MF; ++j)
#pragma unroll
                for (int q = 0; q < 3; ++q) fv[j][q] = panel[k][j][q][lane];
            mfma_split(fm[k], fv, R);
        }
        if (h == 0) __syncthreads();
    }
    // (every wavefront has read its part of S by now: the barriers above)
#pragma unroll
    for (int j = 0; j < MF; ++j) tile_store_both(a, t, R[0][j] * undo, wave, j, sh.turn[wave]);
}

// The same for few tiles, where a pair per workgroup leaves compute units idle: a workgroup takes 32 columns of tile y, a
// wavefront 32 rows of tile x, and only V's pieces and the part of A_y, which all wavefronts need, go through LDS.  The other
// workgroups of a pair still read what one writes, so the result goes to another array, all of it.  Bound by latency:
// everything that the first product needs is on its way before it starts, and A_x while it runs.  n = 1024: 10.2 us a
// stage (12.2 with S row by row and one accumulator).
struct TileNarrowShared {
    u32x4 panel[kTilePad / 16][3][64];   // V
    u32x4 matrix[kTilePad / 16][3][64];  // the part of A_y
    TileTurn turn[kTilePad / 32];
};
__device__ __forceinline__ void tile_two_sided_narrow(const TileTwoSidedArgs &a, unsigned block_id, TileNarrowShared &sh)
{
    constexpr int MF = kTilePad / 32, KF = kTilePad / 16;
    auto &panel = sh.panel;
    const TilePlan &g = a.g;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int part = block_id % MF;
    const TilePair t = tile_pair(a, TileAll{}, block_id / MF);
    const u32x4 *py = a.pieces + tile_piece_index(g, a.stage, t.uy, t.idy) * kTilePieceWords + (size_t)part * KF * 192 + lane;
    const u32x4 *px = a.pieces + tile_piece_index(g, a.stage, t.ux, t.idx) * kTilePieceWords + (size_t)wave * KF * 192 + lane;
#pragma unroll
    for (int k = 0; k < KF / 4; ++k)
#pragma unroll
        for (int q = 0; q < 3; ++q)
            __builtin_amdgcn_global_load_lds((global_ptr)(py + (KF / 4 * wave + k) * 192 + 64 * q),
                                             (lds_ptr)(sh.matrix[KF / 4 * wave + k][q]), 16, 0, 0);
    f32x4 sr[KF][2];
#pragma unroll
    for (int k = 0; k < KF; ++k) tile_load_s(a, t, wave, k, sr[k]);
#pragma unroll
    for (int k = 0; k < KF; ++k) tile_load_held(a, t, wave, k, sr[k]);
    tile_load_held_column(a, t, wave, sr[KF - 1]);
    u32x4 fm[KF][3];
    const float scale = tile_scale(a.range), undo = range_unscale(scale);
    __builtin_amdgcn_s_waitcnt(kWaitForLoads);
    __syncthreads();       // the part of A_y is in LDS
#pragma unroll
    for (int k = 0; k < KF; ++k)
#pragma unroll
        for (int q = 0; q < 3; ++q) fm[k][q] = px[k * 192 + 64 * q];
    if (t.ux == t.uy && part == 0) {
        float *block = a.blocks + ((size_t)a.stage * g.P + t.ux) * kTilePad * kTilePad + wave * KF * 512 + lane * 8;
#pragma unroll
        for (int k = 0; k < KF; ++k) {
            *reinterpret_cast<f32x4 *>(block + 512 * k) = sr[k][0];
            *reinterpret_cast<f32x4 *>(block + 512 * k + 4) = sr[k][1];
        }
    }
    f32x16 acc, small;
    auto clear = [&]() {
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = small[v] = 0.f;
    };
    clear();
#pragma unroll
    for (int k = 0; k < KF; ++k) {
        float v[8];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            v[q] = sr[k][0][q] * scale;
            v[4 + q] = sr[k][1][q] * scale;
        }
        const Split8 sp = split8(v);
        const u32x4 fs[3] = {sp.h, sp.m, sp.l}, fy[3] = {sh.matrix[k][0][lane], sh.matrix[k][1][lane], sh.matrix[k][2][lane]};
        tile_mfma(fs, fy, acc, small);
    }
    // V as operand of the second product: these 32 rows are contraction indices 32 wave .. + 31 of it
#pragma unroll
    for (int f = 0; f < 2; ++f) {
        float v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = acc[8 * f + q] + small[8 * f + q];
        const Split8 sp = split8(v);
        panel[2 * wave + f][0][lane] = sp.h;
        panel[2 * wave + f][1][lane] = sp.m;
        panel[2 * wave + f][2][lane] = sp.l;
    }
    __syncthreads();
    clear();
#pragma unroll
    for (int k = 0; k < KF; ++k) {
        const u32x4 fv[3] = {panel[k][0][lane], panel[k][1][lane], panel[k][2][lane]};
        tile_mfma(fm[k], fv, acc, small);
    }
    tile_store_both(a, t, (acc + small) * undo, wave, part, sh.turn[wave]);
}

// One launch per stage of the reverse sweep: the workgroups before `pair_blocks` take S through it, the others (OPERAND) what
// dX comes from (G, or I where U^T is wanted).  Neither reads what the other writes, and alone each leaves compute units
// idle.  Per stage, launches of their own against this one: n = 1002 with I 8.0 + 5.4 and 9.2 us, n = 2050, B = 2050 with G
// 17.7 + 11.8 and 26.8, n = 4097, m = 512, B = 4096 with G 25.3 + 13.8 and 32.
struct TileStageArgs {
    TileTwoSidedArgs s;
    TileApplyArgs a;
    unsigned pair_blocks;
};
template <bool NARROW, bool OPERAND, typename List>
__global__ __launch_bounds__(2 * kTilePad, NARROW && !OPERAND ? 1 : 2) void tile_stage_kernel(TileStageArgs a, List list)
{
    __shared__ union {
        std::conditional_t<NARROW, TileNarrowShared, TileTwoSidedShared> s;
        TileApplyShared a;
    } sh;
    if constexpr (OPERAND)
        if (blockIdx.x >= a.pair_blocks) {
            tile_apply(a.a, list, blockIdx.x - a.pair_blocks, sh.a);
            return;
        }
    if constexpr (NARROW)
        tile_two_sided_narrow(a.s, blockIdx.x, sh.s);
    else
        tile_two_sided(a.s, list, blockIdx.x, sh.s);
}

// N values per lane (8 or 16) -> lane l has the sum over all lanes of value l / (64 / N)
template <int N>
__device__ __forceinline__ float tile_reduce(const float (&v)[N])
{
    const int lane = threadIdx.x & 63;
    float w[N / 2];
#pragma unroll
    for (int r = 0; r < N / 2; ++r) {
        const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[r]), __float_as_uint(v[r + N / 2]), false, false);
        w[r] = __uint_as_float(t[0]) + __uint_as_float(t[1]);
    }
#pragma unroll
    for (int r = 0; r < N / 4; ++r) {
        const auto t = __builtin_amdgcn_permlane16_swap(__float_as_uint(w[r]), __float_as_uint(w[r + N / 4]), false, false);
        w[r] = __uint_as_float(t[0]) + __uint_as_float(t[1]);
    }
    auto moved = [](auto ctrl, float x) {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    // within a row of 16 lanes: keep one value of a pair, hand the other to the lane that keeps it; one value left: add it
    auto step = [&](auto ctrl, int bit, auto left) {
        constexpr int HALF = decltype(left)::value / 2;
        if constexpr (HALF == 0) w[0] += moved(ctrl, w[0]);
#pragma unroll
        for (int r = 0; r < HALF; ++r) {
            const bool up = (lane & bit) != 0;
            const float keep = up ? w[r + HALF] : w[r], give = up ? w[r] : w[r + HALF];
            w[r] = keep + moved(ctrl, give);
        }
    };
    step(std::integral_constant<int, 0x128>{}, 8, std::integral_constant<int, N / 4>{});   // row_ror:8: lane ^ 8
    step(std::integral_constant<int, 0x141>{}, 4, std::integral_constant<int, N / 8>{});   // row_half_mirror: lane ^ 7
    step(std::integral_constant<int, 0x1b>{}, 2, std::integral_constant<int, 1>{});        // quad_perm 3 2 1 0: lane ^ 3
    step(std::integral_constant<int, 0xb1>{}, 1, std::integral_constant<int, 1>{});        // quad_perm 1 0 3 2: lane ^ 1
    return w[0];
}

// The sums of all tiles' pairs from the blocks the stages have left: the reverse sweep of a tile on the strips
// W = A S and A (columns of the block, two per lane); the share of rows a, b is W_a . A_b, summed over the lanes.  A workgroup
// takes a tile, its wavefronts the rotations with some of the rows, as in the build kernel; a wavefront puts the sums of a
// row where the coefficients were that it alone has read.  A special tile's columns are shared by two workgroups: the one that
// is done last adds the two sums, the first half's first.  Bound by the vector instructions, 20 for a rotation of two
// columns.  n = 1002 92 us, n = 4097 with m = 512 247 us (one lane per column with all rows of a tile: 144 and 428 us).
__global__ __launch_bounds__(kTileThreads, 4) void tile_gradient_kernel(TilePlan g, const float *__restrict__ theta,
                                                                        const int *__restrict__ map, int free_rows,
                                                                        const float *__restrict__ blocks,
                                                                        int *__restrict__ counts, float *__restrict__ halves,
                                                                        float *__restrict__ dtheta)
{
    __shared__ float2 table[2 * kTileSlots * kTileTable];   // [piece][s][64]
    __shared__ float hand[2][kTileParts - 1][4][64];
    __shared__ float2 row0[64];
    __shared__ int finished;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool special = (int)blockIdx.x < 2 * g.P;
    const int id = (int)blockIdx.x - 2 * g.P, half = special ? blockIdx.x & 1 : 0;
    const int st = special ? 2 * ((int)blockIdx.x / 2) - g.first : id / g.P, u = special ? 0 : id % g.P;
    const Tile x = tile_at(g, st, u);
    if (!special && (x.kind == kTileSpecial || tile_is_identity(g, x, free_rows))) return;
    const float *blk = blocks + ((size_t)st * g.P + u) * kTilePad * kTilePad;
    auto at = [&](int row, int col) { return blk[tile_block_at(kTilePad, row, col)]; };
    tile_coefs<float2, float>(g, x, special, g.s, theta, map, table);
    if (special && threadIdx.x < 64) {
        const int col = threadIdx.x + 64 * half;
        row0[threadIdx.x] = make_float2(col == kTilePad - 1 ? 1.f : 0.f, at(kTilePad - 1, col));
    }
    __syncthreads();

    if (special) {
        constexpr int ROWS = kTileSpecialPart;
        const int which = wave & 1, part = wave >> 1, base = which * (kTilePad / 2);   // (the two on different SIMDs)
        const int col = lane + 64 * half;
        float fa[ROWS], fw[ROWS], ca = 0.f, cw = 0.f, ahead = at(base, col);
#pragma unroll
        for (int b = 0; b < ROWS; ++b) fa[b] = fw[b] = 0.f;
        for (int t = 0; t < g.s + 3; ++t) {
            const int r = t - part, place = r - ROWS * part;      // (row r ends in part r / 16)
            const bool mine = r < g.s && place >= 0, own = mine && place < ROWS;
            float2 *coef = table + ((size_t)which * g.s + (mine ? r : 0)) * kTileTable;
            float prod[ROWS];
#pragma unroll
            for (int b = 0; b < ROWS; ++b) prod[b] = 0.f;
            const float2 held = coef[kTileTable - 1];
            if (mine) {
                if (part) {
                    ca = hand[(t + 1) & 1][part - 1][2 * which][lane];
                    cw = hand[(t + 1) & 1][part - 1][2 * which + 1][lane];
                } else {
                    ca = base + r == col ? 1.f : 0.f;
                    cw = ahead;
                    ahead = at(base + (r + 1 < g.s ? r + 1 : r), col);
                }
#pragma unroll
                for (int b0 = 0; b0 < ROWS; b0 += 8)
                    if (b0 < place) {
                        float2 cs[8];   // read together: one LDS latency for eight rotations
#pragma unroll
                        for (int v = 0; v < 8; ++v) cs[v] = coef[ROWS * part + b0 + v];
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int v = 0; v < 8; ++v)
                            if (b0 + v < ROWS - 1 || !own) {      // (its last entry may be that of row 0)
                                prod[b0 + v] = cw * fa[b0 + v];
                                tile_rotate(cw, fw[b0 + v], cs[v]);
                                tile_rotate(ca, fa[b0 + v], cs[v]);
                            }
                    }
                if (!own) {
                    hand[t & 1][part][2 * which][lane] = ca;
                    hand[t & 1][part][2 * which + 1][lane] = cw;
                }
            }
            for (int turn = 0; turn < 2; ++turn) {                // row 0: piece i, then piece i + P
                if (own && turn == which) {
                    float2 zero = row0[lane];
                    prod[ROWS - 1] = cw * zero.x;                 // (no row is behind 15 others of its part)
                    tile_rotate(cw, zero.y, held);
                    tile_rotate(ca, zero.x, held);
                    row0[lane] = zero;
                }
                __syncthreads();
            }
            if (mine) {
                const float sum = tile_reduce<ROWS>(prod);
                const int slot = lane >> 2;
                if ((lane & 3) == 0) coef[own && slot == ROWS - 1 ? kTileTable - 1 : ROWS * part + slot].x = sum;
            }
            if (own)
#pragma unroll
                for (int b0 = 0; b0 < ROWS; b0 += 8)
                    if (place / 8 == b0 / 8)
#pragma unroll
                        for (int v = 0; v < 8; ++v) {
                            fa[b0 + v] = place % 8 == v ? ca : fa[b0 + v];
                            fw[b0 + v] = place % 8 == v ? cw : fw[b0 + v];
                        }
        }
    } else {
        const int parts = (g.s + kTilePart - 1) / kTilePart, first = kTilePart * wave;
        float fa[kTilePart][2], fw[kTilePart][2];
#pragma unroll
        for (int b = 0; b < kTilePart; ++b)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int row = kTilePad / 2 + first + b;
                fa[b][i] = row == lane + 64 * i ? 1.f : 0.f;
                fw[b][i] = at(row, lane + 64 * i);
            }
        float ahead[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) ahead[i] = at(0, lane + 64 * i);
        float2 cs[kTilePart];   // a row's coefficients are read while the row before it is turned
#pragma unroll
        for (int v = 0; v < kTilePart; ++v) cs[v] = table[first + v];
        tile_steps(g.s, parts, wave, [&](int r, int t) __attribute__((always_inline)) {
            float2 *coef = table + r * kTileTable + first;
            float ca[2], cw[2];
#pragma unroll
            for (int i = 0; i < 2; ++i)
                if (wave) {
                    ca[i] = hand[(t + 1) & 1][wave - 1][i][lane];
                    cw[i] = hand[(t + 1) & 1][wave - 1][2 + i][lane];
                } else {                                       // a from I, w from the block, one row ahead
                    ca[i] = r == lane + 64 * i ? 1.f : 0.f;
                    cw[i] = ahead[i];
                    ahead[i] = at(r + 1 < g.s ? r + 1 : r, lane + 64 * i);
                }
            const float2 *next = coef + (r + 1 < g.s ? kTileTable : 0);
            float prod[kTilePart];
#pragma unroll
            for (int b = 0; b < kTilePart; ++b) {
                const float2 now = cs[b];
                cs[b] = next[b];
                prod[b] = fmaf(cw[0], fa[b][0], cw[1] * fa[b][1]);
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    tile_rotate(cw[i], fw[b][i], now);
                    tile_rotate(ca[i], fa[b][i], now);
                }
            }
            if (wave + 1 < parts)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    hand[t & 1][wave][i][lane] = ca[i];
                    hand[t & 1][wave][2 + i][lane] = cw[i];
                }
            const float sum = tile_reduce<kTilePart>(prod);
            if ((lane & 7) == 0) coef[lane >> 3].x = sum;
        });
    }
    __syncthreads();
    const float *first_half = nullptr, *second_half = nullptr;
    if (special) {
        const size_t words = 2 * kTileSlots * kTileTable;
        float *const out = halves + (size_t)blockIdx.x * words;
        for (int i = threadIdx.x; i < 2 * g.s * kTileTable; i += kTileThreads) out[i] = table[i].x;
        __threadfence();
        __syncthreads();
        if (threadIdx.x == 0) finished = atomicAdd(counts + blockIdx.x / 2, 1);
        __syncthreads();
        if (finished == 0) return;
        __threadfence();
        first_half = out - half * words;
        second_half = first_half + words;
    }
    for (int i = threadIdx.x; i < kTilePlaces; i += kTileThreads) {
        int which, r, slot;
        tile_table_place(special, i, &which, &r, &slot);
        const TileEntry t = tile_entry(g, x, special, which, r, slot);
        if (t.e < 0) continue;
        const int to = map ? map[t.e] : t.e;
        if (to < 0) continue;
        const int at = (which * g.s + r) * kTileTable + slot;
        const float v = special ? first_half[at] + second_half[at] : table[at].x;
        dtheta[to] = t.ordered ? v : -v;
    }
}

} // namespace givens
