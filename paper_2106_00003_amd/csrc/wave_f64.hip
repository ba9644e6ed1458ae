// Launches of the one-wavefront float64 sweeps (wave_f64_kernels.hpp): strips of 1, 2 or 4 columns (2 at most with eight
// slots per lane in the reverse sweep, by its registers).
#include "wave_f64_kernels.hpp"

#include "carousel_host.hpp"

namespace givens {
namespace {
template <int M, int W>
void forward(int n, int rows, long long B, const double2 *table, const double *X, double *Y, int identity, int mirror,
             hipStream_t stream)
{
    hipLaunchKernelGGL((wave64_forward_kernel<M, W>), dim3((unsigned)((B + W - 1) / W)), dim3(64), 0, stream, n, rows, B, table,
                       X, Y, identity, mirror);
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
template <int M, int W>
void backward(int n, int rows, long long B, long long strip0, long long strips, const double2 *table, const double *Y,
              const double *G, double *dX, double *partial, hipStream_t stream)
{
    hipLaunchKernelGGL((wave64_backward_kernel<M, W>), dim3((unsigned)strips), dim3(64), 0, stream, n, rows, B, strip0, table, Y,
                       G, dX, partial);
}
template <int M>
int backward_widths(int W, int n, int rows, long long B, long long strip0, long long strips, const double2 *table,
                    const double *Y, const double *G, double *dX, double *partial, hipStream_t stream)
{
    if constexpr (M < 8)
        if (W == 4) {
            backward<M, 4>(n, rows, B, strip0, strips, table, Y, G, dX, partial, stream);
            return GIVENS_OK;
        }
    if (W == 2) backward<M, 2>(n, rows, B, strip0, strips, table, Y, G, dX, partial, stream);
    else if (W == 1) backward<M, 1>(n, rows, B, strip0, strips, table, Y, G, dX, partial, stream);
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
int wave64_backward(int n, int rows, long long B, long long strip0, long long strips, const double2 *table, const double *Y,
                    const double *G, double *dX, double *partial, hipStream_t stream)
{
    const int M = wave64_slots(n), W = wave64_bwd_width(n, B);
    switch (M) {
    case 1: return backward_widths<1>(W, n, rows, B, strip0, strips, table, Y, G, dX, partial, stream);
    case 2: return backward_widths<2>(W, n, rows, B, strip0, strips, table, Y, G, dX, partial, stream);
    case 4: return backward_widths<4>(W, n, rows, B, strip0, strips, table, Y, G, dX, partial, stream);
    case 8: return backward_widths<8>(W, n, rows, B, strip0, strips, table, Y, G, dX, partial, stream);
    default: return GIVENS_ERR_UNSUPPORTED;
    }
}

} // namespace givens
