// Forward carousel kernels with eight slots per lane: strips of one column with staged tables, those of several wavefronts with turned ones.
#include "carousel_kernels.hpp"

namespace givens {
namespace {

// Eight slots per lane, one wavefront per strip: the table, turned, by way of LDS (CarouselFwd::staged_sweep).  A wavefront's part of a row is
// 4 KB, so where each strip reads it by itself the loads set the time, 256 cycles of a compute unit's L1 for the four strips of n = B =
// 1024, whose arithmetic takes 190.
template <int FORM>
__device__ __forceinline__ void carousel_staged_body(StagedRows &staged, int n, int rows, long long B, const float2 *__restrict__ table,
                                                     const float2 *__restrict__ renorm, const float *X, float *Y, int identity,
                                                     int mirror, int turned)
{
    constexpr int M = kTurnedSlots, W = 1;
    using State = CarouselFwd<M, W, 1, FORM, kExchangeWave, true, kTableStaged>;
    State st;
    const int L = n / (2 * M), lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (lane_is_off<M>(lane, L)) return;
    st.n = n;
    st.H = n >> 1;
    st.lanes = L;
    st.lane = st.tid = lane;
    st.wave = 0;
    st.table_of_lane(table, lane);
    st.tab_lane = table;
    st.rn_lane = renorm + (long long)lane * M;
    // (a strip that is not there is swept all the same, as zeros, since its wavefront brings a part of the rows)
    const long long b0 = (long long)blockIdx.x * kTurnedStrips + wave;
    const int my_rows = b0 < B ? rows : 0;
#pragma unroll
    for (int r = 0; r < M; ++r) {
        const int p = lane * M + r;
        load_row<W>(st.top[r], X, B, mirrored_row(n, rr_label(n, n - 2, p), mirror), my_rows, b0, W, false, identity);
        load_row<W>(st.bot[r], X, B, mirrored_row(n, rr_label(n, n - 2, n - 1 - p), mirror), my_rows, b0, W, false, identity);
    }
    st.staged_sweep(staged, turned != 0);
    constexpr int UL = State::kLastU;
#pragma unroll
    for (int r = 0; r < M; ++r) {
        const int p = lane * M + r;
        store_row<W>(st.top[(r + UL) % M], Y, B, mirrored_row(n, p, mirror), my_rows, b0, W, false);
        store_row<W>(st.bot[(r - UL + M) % M], Y, B, mirrored_row(n, n - 1 - p, mirror), my_rows, b0, W, false);
    }
}
__global__ __launch_bounds__(64 * kTurnedStrips, 2) void carousel_forward_staged_kernel(
    int n, int rows, long long B, const float2 *__restrict__ table, const float2 *__restrict__ renorm,
    const unsigned *flag, float scaled_max, const float *X, float *Y, int identity, int mirror, int turned)
{
    __shared__ StagedRows staged;
    const int form = __builtin_amdgcn_readfirstlane(selected_form(flag, scaled_max));
    if (form == kFormScaled)
        carousel_staged_body<kFormScaled>(staged, n, rows, B, table, renorm, X, Y, identity, mirror, turned);
    else if (form == kFormLifted)
        carousel_staged_body<kFormLifted>(staged, n, rows, B, table, renorm, X, Y, identity, mirror, turned);
    else
        carousel_staged_body<kFormStandard>(staged, n, rows, B, table, renorm, X, Y, identity, mirror, turned);
}

} // namespace

int carousel_forward_staged(const CarouselFwdArgs &a)
{
    hipLaunchKernelGGL(carousel_forward_staged_kernel, dim3((unsigned)((a.B + kTurnedStrips - 1) / kTurnedStrips)), dim3(64 * kTurnedStrips),
                       0, a.stream, a.n, a.rows, a.B, a.coefs.table, a.coefs.renorm, a.coefs.flag, a.coefs.scaled_max, a.X, a.Y, a.identity,
                       a.mirror, a.coefs.turned ? 1 : 0);
    return GIVENS_OK;
}
int carousel_forward_turned_lds(const CarouselFwdArgs &a, int waves, int W)
{
    if (W > 2) return GIVENS_ERR_UNSUPPORTED;
    switch (waves) {
    case 2: return carousel_forward_turned_widths<2>(a, W);
    case 3: return carousel_forward_turned_widths<3>(a, W);
    case 4: return carousel_forward_turned_widths<4>(a, W);
    case 5: return carousel_forward_turned_widths<5>(a, W);
    case 6: return carousel_forward_turned_widths<6>(a, W);
    case 7: return carousel_forward_turned_widths<7>(a, W);
    case 8: return carousel_forward_turned_widths<8>(a, W);
    default: return GIVENS_ERR_UNSUPPORTED;
    }
}

} // namespace givens
