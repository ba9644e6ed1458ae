// A matrix kept for angles that may change unseen (givens_keep): beside the matrix lie a copy of the angles it was made
// from and their standard-form table.
#pragma once
#include <hip/hip_runtime.h>

#include "product_kernels.hpp"
#include "rr_index.h"

namespace givens {

struct KeptAngles {
    int n;
    const float *theta;
    const int *map;      // index in theta of every entry of E, or -1 (nullptr: every pair is free)
    float *copy;         // the angles as they were
    float2 *table;
    int *changed;
    long long id, *note; // host memory: takes the id of a kept matrix whose angles have changed
};

// Looks every angle up again; where one has other bits than its copy, *changed is set, the table takes the entry of the
// new angle and *note takes the id.  Once *changed is set, every entry is written anew by every call, so the table is
// that of the present angles whatever they were in between, and calls on several streams write what they read; the copy
// stays.  FIRST: fills both.
template <bool FIRST>
__device__ __forceinline__ void kept_angles(const KeptAngles &a, long long thread, long long threads)
{
    const int H = a.n >> 1;
    const long long N = (long long)(a.n - 1) * H;
    const bool all = FIRST || *a.changed != 0;
    bool differ = false;
    for (long long e = thread; e < N; e += threads) {
        const long long i = a.map ? (long long)a.map[e] : e;
        const float th = i < 0 ? 0.f : a.theta[i];
        const bool other = !FIRST && i >= 0 && __float_as_uint(th) != __float_as_uint(a.copy[i]);
        differ = differ || other;
        if (!all && !other) continue;
        const int k = (int)(e / H), p = (int)(e % H);
        double s, c;
        sincos((double)th, &s, &c);
        a.table[e] = make_float2((float)c, (float)(rr_label(a.n, k, p) < rr_label(a.n, k, a.n - 1 - p) ? s : -s));
        if (FIRST && i >= 0) a.copy[i] = th;
    }
    if (FIRST) {
        if (thread == 0) *a.changed = 0;
        return;
    }
    // one store over the bus: of the first wavefront that sees a change, and later of the first thread (the note may have
    // gone to another matrix since)
    if (__any(differ) && (threadIdx.x & 63) == 0 && atomicExch(a.changed, 1) == 0) *a.note = a.id;
    if (all && thread == 0) *a.note = a.id;
}
// Bound by reading theta and its copy: n = 1024 (4 MB) in 3.2 us.
template <bool FIRST>
__global__ __launch_bounds__(256) void kept_angles_kernel(KeptAngles a)
{
    kept_angles<FIRST>(a, (long long)blockIdx.x * 256 + threadIdx.x, (long long)gridDim.x * 256);
}
// The product of few columns and the look at the angles in one launch: the workgroups from `product_blocks` on look.
// n = 1024, B = 64: a launch less on the host, which is what bounds a call.
__global__ __launch_bounds__(64 * kNarrowWaves, 1) void product_narrow_kept_kernel(ProductArgs a, unsigned product_blocks,
                                                                                  KeptAngles k)
{
    __shared__ NarrowShared sh;
    if (blockIdx.x >= product_blocks)
        kept_angles<false>(k, (long long)(blockIdx.x - product_blocks) * (64 * kNarrowWaves) + threadIdx.x,
                           (long long)(gridDim.x - product_blocks) * (64 * kNarrowWaves));
    else
        product_narrow<false>(a, sh, blockIdx.x);
}

} // namespace givens
