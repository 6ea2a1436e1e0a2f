// shade_grid.h -- how the deterministic shading modes divide a call into
// launches (host code only).
#pragma once

#include <stdint.h>

namespace stf {

// HIP launches fewer than 2^32 work-items in a dimension.  With `lanes`
// work-items a query that is reached by fewer queries than a call may have
// (2^31 - 1), so a call is launched in parts of at most this many; its results
// do not depend on the split (no query takes its number into account).
constexpr int64_t SHADE_PART = (int64_t)1 << 29;

inline int64_t shade_part(int64_t n, int64_t first)
{
    return n - first < SHADE_PART ? n - first : SHADE_PART;
}

// Blocks of `block` threads for m queries of `lanes` lanes each.
inline uint32_t shade_blocks(int64_t m, int lanes, int block)
{
    return (uint32_t)((m * lanes + block - 1) / block);
}

}  // namespace stf
