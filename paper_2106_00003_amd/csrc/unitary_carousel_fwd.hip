// Unitary carousel kernels: the phase pass, the coefficient tables and the forward sweep (8 slots per lane).
#include "unitary_carousel_kernels.hpp"
#include "unitary_phase_kernels.hpp"

namespace givens {

template <bool REVERSE, int PER>
static void launch_phase_scan(int n, int threads, const uint2 *q, unsigned *turn, const PhaseScan &scan, hipStream_t stream)
{
    hipLaunchKernelGGL((unitary_phase_scan_kernel<REVERSE, PER, true>), dim3(scan.chunks), dim3(threads), 0, stream, n, q, turn,
                       scan);
    hipLaunchKernelGGL((unitary_phase_scan_kernel<REVERSE, PER, false>), dim3(scan.chunks), dim3(threads), 0, stream, n, q, turn,
                       scan);
}

size_t unitary_scan_bytes(int n) { return (size_t)n * (2 * sizeof(unsigned) + phase_chunks(n) * sizeof(uint2)); }

template <bool REVERSE>
static void coefficients(int n, const float *theta, const float *phi, uint2 *q, unsigned *turn, void *scratch, float *sgn,
                         float2 *rot, float2 *phs, float *orient, float2 *fin, hipStream_t stream)
{
    const long long N = (long long)n * (n - 1) / 2;
    const int threads = 256, H = n / 2, chunks = phase_chunks(n);
    const unsigned blocks = (unsigned)((N + threads - 1) / threads < 8192 ? (N + threads - 1) / threads : 8192);
    uint2 *const maps = static_cast<uint2 *>(scratch);
    unsigned *const flips = reinterpret_cast<unsigned *>(maps + (size_t)chunks * n);
    const PhaseScan scan{chunks, maps, flips, flips + n};
    hipLaunchKernelGGL(unitary_phase_input_kernel<REVERSE>, dim3(blocks), dim3(threads), 0, stream, n, theta, phi, q);
    // one thread per pair up to 1024 threads, then two pairs per thread
    if (H <= kPhaseScanThreads)
        launch_phase_scan<REVERSE, 1>(n, (H + 63) / 64 * 64, q, turn, scan, stream);
    else
        launch_phase_scan<REVERSE, 2>(n, kPhaseScanThreads, q, turn, scan, stream);
    hipLaunchKernelGGL(unitary_carousel_table_kernel<REVERSE>, dim3(blocks), dim3(threads), 0, stream, n, theta, turn, scan, sgn,
                       rot, phs, orient, fin, !REVERSE && n / 16 <= 64 ? 3 : 0);   // (forward sweeps of one wavefront: eight slots)
}
int unitary_carousel_coefficients(int n, const float *theta, const float *phi, int reverse, uint2 *q, unsigned *turn, void *scratch,
                                  float *sgn, float2 *rot, float2 *phs, float *orient, float2 *fin, hipStream_t stream)
{
    if (!unitary_carousel_supported(n) || n / 2 > 2 * kPhaseScanThreads) return GIVENS_ERR_UNSUPPORTED;
    (reverse ? coefficients<true> : coefficients<false>)(n, theta, phi, q, turn, scratch, sgn, rot, phs, orient, fin, stream);
    return GIVENS_OK;
}

int unitary_carousel_forward_m8(const UnitaryCarouselFwdArgs &a, int waves, int W)
{
    return unitary_carousel_forward_slots<8>(a, waves, W);
}

} // namespace givens
