// Host-side choices behind the products and contractions (product_kernels.hpp, gram_kernels.hpp), in plain C++.
#pragma once
#include "rr_index.h"

namespace givens {

// Workgroups are handed to the eight XCDs (each with an L2 of its own) in turn.  Place of workgroup `block` in a list of
// `total` that is cut into eight consecutive parts, one per XCD, the first total % 8 of them one longer.
RR_HD inline unsigned xcd_order(unsigned block, unsigned total)
{
    const unsigned xcd = block % 8, more = total % 8;
    return xcd * (total / 8) + (xcd < more ? xcd : more) + block / 8;
}

} // namespace givens
