// Block-to-tile mapping shared by the tiled kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace twg {

// Blocks are dispatched round-robin over the 8 XCDs; give each XCD a
// contiguous range of tiles so that its L2 sees a compact band of the grid.
__device__ __forceinline__ int xcd_remap(int b, int nb)
{
    constexpr int X = 8;
    int per = nb / X, rem = nb % X;
    int xcd = b % X, local = b / X;
    return xcd < rem ? xcd * (per + 1) + local : rem * (per + 1) + (xcd - rem) * per + local;
}

}  // namespace twg
