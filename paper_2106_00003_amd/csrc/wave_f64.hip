// Launches of the one-wavefront float64 sweeps (wave_f64_kernels.hpp): strips of 1, 2 or 4 columns (2 at most with eight
// slots per lane in the reverse sweep, by its registers), one or kWave64Strips of them per workgroup.
#include "wave_f64_kernels.hpp"

#include "carousel_host.hpp"

namespace givens {
namespace {
template <int M, int W>
void forward(int n, int rows, long long B, const double2 *table, const double *X, double *Y, int identity, int mirror,
             hipStream_t stream)
{
    const long long strips = (B + W - 1) / W;
    const int per = wave64_fwd_strips(strips);
    hipLaunchKernelGGL((wave64_forward_kernel<M, W>), dim3((unsigned)((strips + per - 1) / per)), dim3(64 * per), 0, stream, n, rows,
                       B, table, X, Y, identity, mirror);
}
template <int M>
int forward_widths(int W, int n, int rows, long long B, const double2 *table, const double *X, double *Y, int identity,
                   int mirror, hipStream_t stream)
{
    if (W == 4) forward<M, 4>(n, rows, B, table, X, Y, identity, mirror, stream);
    else if (W == 2) forward<M, 2>(n, rows, B, table, X, Y, identity, mirror, stream);
    else forward<M, 1>(n, rows, B, table, X, Y, identity, mirror, stream);
    return GIVENS_OK;
}
template <int M, int W, int STRIPS>
void backward(int n, int rows, long long B, long long group0, long long groups, const double2 *table, const double *Y,
              const double *G, double *dX, double *partial, hipStream_t stream)
{
    hipLaunchKernelGGL((wave64_backward_kernel<M, W, STRIPS>), dim3((unsigned)groups), dim3(64 * STRIPS), 0, stream, n, rows, B,
                       group0, table, Y, G, dX, partial);
}
template <int M>
int backward_widths(int W, int strips, int n, int rows, long long B, long long group0, long long groups, const double2 *table,
                    const double *Y, const double *G, double *dX, double *partial, hipStream_t stream)
{
    constexpr int S = kWave64Strips;
    if constexpr (M < 8)
        if (W == 4) {
            backward<M, 4, S>(n, rows, B, group0, groups, table, Y, G, dX, partial, stream);
            return GIVENS_OK;
        }
    if (strips == 1 && W == 1) backward<M, 1, 1>(n, rows, B, group0, groups, table, Y, G, dX, partial, stream);
    else if (W == 2) backward<M, 2, S>(n, rows, B, group0, groups, table, Y, G, dX, partial, stream);
    else if (W == 1) backward<M, 1, S>(n, rows, B, group0, groups, table, Y, G, dX, partial, stream);
    else return GIVENS_ERR_UNSUPPORTED;
    return GIVENS_OK;
}
} // namespace

int wave64_forward(int n, int rows, long long B, const double2 *table, const double *X, double *Y, int identity, int mirror,
                   hipStream_t stream)
{
    const int M = wave64_slots(n), W = wave64_fwd_width(n, B);
    switch (M) {
    case 1: return forward_widths<1>(W, n, rows, B, table, X, Y, identity, mirror, stream);
    case 2: return forward_widths<2>(W, n, rows, B, table, X, Y, identity, mirror, stream);
    case 4: return forward_widths<4>(W, n, rows, B, table, X, Y, identity, mirror, stream);
    case 8: return forward_widths<8>(W, n, rows, B, table, X, Y, identity, mirror, stream);
    default: return GIVENS_ERR_UNSUPPORTED;
    }
}
int wave64_backward(int n, int rows, long long B, long long group0, long long groups, const double2 *table, const double *Y,
                    const double *G, double *dX, double *partial, hipStream_t stream)
{
    const int M = wave64_slots(n), strips = wave64_bwd_strips(n, B), W = wave64_bwd_width(n, B) / strips;
    switch (M) {
    case 1: return backward_widths<1>(W, strips, n, rows, B, group0, groups, table, Y, G, dX, partial, stream);
    case 2: return backward_widths<2>(W, strips, n, rows, B, group0, groups, table, Y, G, dX, partial, stream);
    case 4: return backward_widths<4>(W, strips, n, rows, B, group0, groups, table, Y, G, dX, partial, stream);
    case 8: return backward_widths<8>(W, strips, n, rows, B, group0, groups, table, Y, G, dX, partial, stream);
    default: return GIVENS_ERR_UNSUPPORTED;
    }
}

} // namespace givens
