// Host-side choices behind the products and contractions (product_kernels.hpp, gram_kernels.hpp), in plain C++.
#pragma once
#include <algorithm>

#include "rr_index.h"

namespace givens {

// Workgroups are handed to the eight XCDs (each with an L2 of its own) in turn.  Place of workgroup `block` in a list of
// `total` that is cut into eight consecutive parts, one per XCD, the first total % 8 of them one longer.
RR_HD inline unsigned xcd_order(unsigned block, unsigned total)
{
    const unsigned xcd = block % 8, more = total % 8;
    return xcd * (total / 8) + (xcd < more ? xcd : more) + block / 8;
}

// Time in us of a launch of tiles, from the workgroups of the XCD that has most.  What counts is how many its fullest
// compute unit gets: 128 x 128 tiles with a contraction of 1024 take 58 to 62 us for up to 256 workgroups on 256 units, 85
// for 272 and 96 for 512, 139 for 528.
struct TileCost {
    int bm, bn, slots;   // results of a workgroup; workgroups that a compute unit holds
    double ends, full;   // the first loads and last stores; a step where every unit gets `slots` more workgroups
    int known;           // entries of `step`
    double step[6][2];   // a step where the fullest units get 1, 2, ... workgroups: a first unit that many, all of them
};
inline double tile_time(const TileCost &t, long long groups_of_xcd, long long steps, int compute_units)
{
    const long long units = std::max(1, compute_units / 8), most = (groups_of_xcd + units - 1) / units;
    const long long rounds = most > t.known ? (most - t.known + t.slots - 1) / t.slots : 0;
    const double of_units = (double)(groups_of_xcd - (most - 1) * units) / (double)units, *s = t.step[most - rounds * t.slots - 1];
    return t.ends + (double)steps * ((double)rounds * t.full + s[0] + (s[1] - s[0]) * of_units);
}

constexpr int kProductStep = 32;   // contraction indices per step of the product kernel (two fragments)

// The tile of a product, m rows, contraction k, B columns: the one whose launch is shortest by tile_time.  All tiles add in the
// same order.  The figures are fitted to products of n = 36 ... 3000 with every tile, 270 real and 230 complex ones: among them the
// choice is 0.04 % slower than the best tile on average and 3.6 % at most, complex 0.2 % and 6 %.  Times measured in us, 64 x 64 /
// 128 x 64 /
// 128 x 128 / 256 x 128: n = 256, B = 65536 79 / 69 / 60 / 52, n = 1002, B = 3001 46 / 49 / 60 / 96, n = 1024, B = 4096
// 59 / 53 / 61 / 95, n = 512, B = 9856 45 / 48 / 51 / 55, n = 640, B = 6784 51 / 55 / 58 / 65, n = 2048, B = 4096
// 242 / 202 / 176 / 192, n = 4097, B = 4096 974 / 969 / 829 / 901; complex n = 1024, B = 5760 415 / 334 / 305 / 456.
constexpr int kProductTiles = 4, kProductComplexTiles = 3;
constexpr TileCost kProductCost[kProductTiles] = {
    {64, 64, 4, 2.9, 1.79, 4, {{0.62, 0.75}, {0.97, 1.05}, {1.28, 1.47}, {1.67, 1.82}}},
    {128, 64, 2, 3.3, 1.55, 2, {{0.87, 1.07}, {1.43, 1.65}}},
    {128, 128, 2, 4.5, 2.69, 2, {{1.57, 1.81}, {2.55, 2.89}}},
    {256, 128, 2, 5.9, 4.90, 2, {{2.48, 3.15}, {3.99, 4.69}}}};
constexpr TileCost kProductComplexCost[kProductComplexTiles] = {
    {64, 64, 4, 2.7, 1.98, 4, {{0.92, 1.06}, {1.36, 1.53}, {1.84, 2.06}, {2.33, 2.49}}},
    {128, 64, 2, 2.9, 1.69, 4, {{1.19, 1.53}, {1.99, 2.12}, {2.84, 2.84}, {3.61, 3.74}}},
    {128, 128, 2, 4.2, 3.06, 4, {{1.99, 2.71}, {3.28, 3.59}, {4.78, 4.80}, {6.76, 6.76}}}};
inline int product_tile(int m, int k, long long B, int compute_units, bool cplx)
{
    int best = 0;
    double least = 0.0;
    for (int i = 0; i < (cplx ? kProductComplexTiles : kProductTiles); ++i) {
        const TileCost &t = cplx ? kProductComplexCost[i] : kProductCost[i];
        // (an XCD has whole blocks of columns: product_kernel)
        const long long groups = (long long)((m + t.bm - 1) / t.bm) * (((B + t.bn - 1) / t.bn + 7) / 8);
        const double us = tile_time(t, groups, (k + kProductStep - 1) / kProductStep, compute_units);
        if (i == 0 || us < least) {
            best = i;
            least = us;
        }
    }
    return best;
}

constexpr int kGramK = 16;         // contraction columns per step of the contraction kernel

// Tile and number of slices of a contraction: the shortest by tile_time and by the slices' sum, among slices of at least 256
// columns (64 x 64 tiles), 384 or 768, at most 256 of them.  The figures are fitted to 218 contractions of n = 36 ... 4096 with
// every tile in 1 to 256 slices, the complex ones to 140: among these the choice is 0.4 % slower than the best on average and 9 % at
// most, complex 0.6 % and 7 %.  Times measured in us without the sum, 64 x 64 / 128 x 128 / 256 x 128, slices in brackets:
// n = 256, B = 65536 70 (128) / 55 (128) /
// 53 (256), n = 514, B = 2048 17 (8) / 22 (8) / 28 (12), n = 1002, B = 3001 55 (4) / 45 (8) / 51 (12), n = 1024, B = 4096
// 68 (4) / 54 (8) / 50 (16), n = 2048, B = 4096 241 (4) / 173 (2) / 155 (4), n = 4097, B = 4096 1085 (2) / 775 (2) / 881 (2) or
// 1114 (1: 561 workgroups for 512 places).
//
// A result's error grows with the square root of the additions behind it, six for every sixteen columns here, where the
// float32 matrix instructions made eight.  Slices of at most 4096 columns keep it below theirs: n = 2048, B = 65536, normal
// operands 2.5e-6 with slices of 16384, 1.3e-6 with 4096 (float32 instructions 2.3e-6), contraction 2.70 and 2.82 ms;
// n = 1024, B = 131072 2.2e-6 with 8192, 1.6e-6 with 4096 (1.6e-6).  As far as the slices fit 4 GiB (n = 8192: sixteen).
constexpr long long kGramMaxSlice = 4096, kGramSliceBytes = 1LL << 32;
constexpr TileCost kGramCost[2][3] = {
    {{64, 64, 6, 2.5, 1.56, 6, {{0.46, 0.57}, {0.64, 0.74}, {0.86, 0.93}, {1.10, 1.12}, {1.27, 1.40}, {1.52, 1.60}}},
     {128, 128, 3, 6.0, 2.22, 3, {{0.92, 1.02}, {1.24, 1.47}, {1.95, 2.20}}},
     {256, 128, 2, 8.2, 2.90, 2, {{1.55, 1.80}, {2.16, 2.60}}}},
    // complex
    {{64, 64, 6, 2.8, 1.65, 6, {{0.60, 0.69}, {0.77, 0.83}, {0.95, 1.06}, {1.24, 1.24}, {1.46, 1.53}, {1.69, 1.73}}},
     {128, 128, 3, 3.6, 2.37, 3, {{1.19, 1.38}, {1.68, 1.74}, {2.44, 2.44}}},
     {256, 128, 2, 2.5, 3.21, 2, {{2.02, 2.40}, {2.69, 3.06}}}}};
constexpr long long kGramLeastSlice[3] = {256, 384, 768};
constexpr double kGramSumEnds = 2.5, kGramSumRate = 3.5e6;   // of the slices' sum: us, and bytes that are read in a microsecond
struct GramPlan {
    int tile;                            // of kGramCost
    int slices;                          // none of them empty
    long long cols;                      // ... of all but the last one: they start on a step boundary
};
inline GramPlan gram_plan(int rows, long long B, int compute_units, bool cplx = false)
{
    const int result_cols = cplx ? 2 * rows : rows;
    const long long bytes = 4LL * rows * result_cols, fit = std::max(1LL, kGramSliceBytes / bytes);
    const long long least = std::min((B + kGramMaxSlice - 1) / kGramMaxSlice, std::min(fit, 256LL));
    GramPlan plan{0, 0, 0};
    double best = 0.0;
    for (int i = 0; i < 3; ++i) {
        const TileCost &t = kGramCost[cplx][i];
        if (i > 0 && rows <= t.bm / 2) continue;
        const long long tiles = (long long)((rows + t.bm - 1) / t.bm) * ((result_cols + t.bn - 1) / t.bn);
        const long long most = std::max(least, std::min(std::min(B / kGramLeastSlice[i], fit), 256LL));
        // as few as there may be, and as many as give every compute unit one workgroup, two, ... two rounds of them
        for (int held = 0; held <= 2 * t.slots; ++held) {
            const long long want = std::min(most, std::max(least, held * (long long)compute_units / tiles));
            const long long cols = ((B + want - 1) / want + kGramK - 1) / kGramK * kGramK, s = (B + cols - 1) / cols;
            const double us = tile_time(t, (tiles * s + 7) / 8, cols / kGramK, compute_units) +
                              (s > 1 ? kGramSumEnds + (double)(s * bytes) / kGramSumRate : 0.0);
            if (!plan.slices || us < best) {
                plan = GramPlan{i, (int)s, cols};
                best = us;
            }
        }
    }
    return plan;
}

// Restricted tiled sweeps: whether a stage, P tiles in `runs` runs of `per` steps, launches only the `active` ones, which hold a
// free pair.  The others return at once: while the chip holds them all they cost nothing, and a list of the rest was up to 8 % slower
// there (fewer workgroups, on other XCDs, whose tile comes from a load).  Beyond that the list is faster where its workgroups
// have a compute unit each, where they fill most of a second round and others would be in their way, where nearly all launched ones
// are idle, and early where a tile's number is an XCD's, since the few that rotate are then on few XCDs.  Forward calls in us, all
// tiles launched and listed: n = 2050, m = 41, B = 8 219 / 229, m = 256, B = 2000 385 / 403; n = 2561, m = 51, B = 64 262 / 271,
// B = 4500 506 / 427; n = 3001, m = 375, B = 1000 539 / 458; n = 3250, m = 406, B = 4500 928 / 977; n = 4097, m = 512, B = 1000
// 765 / 795, B = 4096 1389 / 1293.
inline bool tile_apply_listed(int P, int compute_units, long long runs, long long per, int active)
{
    const long long all = runs * P, wanted = runs * active, units = compute_units;
    if (P % 8 == 0) return 10 * all >= 9 * units && 3 * wanted <= 2 * all;
    if (10 * all < 11 * units) return false;
    const bool filled = per > 1 ? 3 * wanted >= 5 * units : 8 * wanted >= 15 * units;
    return wanted <= units || (filled && 10 * all >= 13 * wanted) || 3 * all >= 20 * units;
}
// ... and one of the gradient: where there are more pairs of tiles than compute units (time of listed ones, all of them 1: n = 706 to
// 1250 1.007, 1500 to 2561 1.001, 3001 to 6100 0.945).
inline bool tile_pairs_listed(int P, int compute_units) { return P * (P + 1) / 2 > compute_units; }

} // namespace givens
