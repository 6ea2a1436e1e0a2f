// tap_block.h -- a number for the block of 4x4x4 voxels in which a query's
// taps begin.
#pragma once

#include <stdint.h>

namespace stf {

// The same for queries of one block, hardly ever so for neighbouring blocks.
// In unsigned arithmetic: a coordinate with a cell lies within 2^24, and the
// products of coordinates that far out wrap.
constexpr uint32_t tap_block(int x, int y, int z)
{
    return (uint32_t)(x >> 2) + (uint32_t)(y >> 2) * 1021u + (uint32_t)(z >> 2) * 31397u;
}

}  // namespace stf
