// Forward carousel kernels with eight slots per lane and a turned coefficient table: strips of one or two columns.
#include "carousel_kernels.hpp"

namespace givens {

int carousel_forward_turned(const CarouselFwdArgs &a, int W, int strips)
{
    if (W == 1)
        carousel_launch_fwd_turned<1, 1, kExchangeWave>(a, strips);
    else
        carousel_launch_fwd_turned<2, 1, kExchangeWave>(a, strips);
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
