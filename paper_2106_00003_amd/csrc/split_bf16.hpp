// Float32 products on the bf16 matrix cores.
//
// Precision.  The fastest matrix instructions of the chip take bf16 operands; a float32 value is exactly the sum of
// three bf16 values (8 + 8 + 8 significand bits: x = h + m + l, h = x rounded to bf16, m = x - h rounded to bf16,
// l = x - h - m, which fits).  A product of two float32 values is therefore the sum of nine exact bf16 products, of
// which the six largest are formed (hh, hm, mh, hl, lh, mm).  With x and y at least 2^e and 2^f, m is at most 2^(e-8) and
// l at most 2^(e-17), so what is left out (ml, lm, ll) is at most 2^-24 of the product: what rounding it to float32 may
// cost.  (Were h cut instead, m could be twice, l twice and the error four times as large.)  Sums are float32, sixteen
// products at a time.  So operands keep their 24 bits and the accumulation its float32, and six bf16 instructions of
// 16-deep contraction still take 1/2.7 of the time of the eight float32 ones (2-deep) they replace.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace givens {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Eight float32 values as three rows of eight bf16 values with h + m + l == x (exact for every x whose last bits are
// normal numbers, up to the largest bf16 number, 2^128 - 2^120).
struct Split8 {
    u32x4 h, m, l;
};
__device__ __forceinline__ unsigned pack_bf16(float a, float b)
{
    const bf16x2 v = __builtin_convertvector((f32x2){a, b}, bf16x2);   // round to nearest even
    return __builtin_bit_cast(unsigned, v);
}
// CLAMP: of every finite x (h stays finite)
template <bool CLAMP = false>
__device__ __forceinline__ Split8 split8(const float (&x)[8])
{
    constexpr float kLargest = 0x1.fep127f;
    Split8 s;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float a = x[2 * i], b = x[2 * i + 1];
        const unsigned h = CLAMP ? pack_bf16(__builtin_amdgcn_fmed3f(a, -kLargest, kLargest),
                                             __builtin_amdgcn_fmed3f(b, -kLargest, kLargest))
                                 : pack_bf16(a, b);
        s.h[i] = h;
        const float ra = a - __uint_as_float(h << 16), rb = b - __uint_as_float(h & 0xffff0000u);
        const unsigned m = pack_bf16(ra, rb);
        s.m[i] = m;
        s.l[i] = pack_bf16(ra - __uint_as_float(m << 16), rb - __uint_as_float(m & 0xffff0000u));
    }
    return s;
}

// Range.  The trailing pieces of a value below 2^-110 fall below the smallest bf16 numbers, so an operand whose columns
// (for the contraction: rows) are that small as a whole would be multiplied with fewer bits than it has.  The kernels
// therefore keep the largest magnitude of every column they bring, and where one is far from the middle of float32's range
// (range_scale) they do their work once more with such columns scaled by a power of two, which they take out of the
// results.  Small elements of a column that has larger ones do not count: what they lose is below 2^-134, and 2^-34 of the
// column.  (The upper end leaves room for a column's norm to gather in one element.)
constexpr float kRangeSmall = 0x1p-100f, kRangeLarge = 0x1p120f;
__device__ __forceinline__ float range_scale(float top)
{
    return top >= kRangeLarge ? 0x1p-8f : (top < kRangeSmall && top > 0.f) ? 0x1p100f : 1.f;
}
__device__ __forceinline__ float range_unscale(float scale) { return scale > 1.f ? 0x1p-100f : scale < 1.f ? 0x1p8f : 1.f; }
// the larger of top and |a|, |b| (NaN counts as nothing; the instruction by name: the compiler would quieten every operand
// first)
__device__ __forceinline__ float range_top(float top, float a, float b)
{
    asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(top) : "v"(a), "v"(b));
    return top;
}
__device__ __forceinline__ float range_top(float top, const float (&x)[8])
{
#pragma unroll
    for (int i = 0; i < 8; i += 2) top = range_top(top, x[i], x[i + 1]);
    return top;
}

// acc[i][j] += a[i] b[j] over 16 contraction indices, float32 operands given as their pieces, smallest products first.
// Each of the six instructions of a result needs the one before it, so the results take turns: back to back on one
// accumulator the matrix cores wait.
template <int NA, int NB>
__device__ __forceinline__ void mfma_split(const u32x4 (&a)[NA][3], const u32x4 (&b)[NB][3], f32x16 (&acc)[NA][NB])
{
    constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
    for (int p = 0; p < 6; ++p)
#pragma unroll
        for (int i = 0; i < NA; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[i][pa[p]]),
                                                                    __builtin_bit_cast(bf16x8, b[j][pb[p]]), acc[i][j], 0, 0, 0);
}

} // namespace givens
