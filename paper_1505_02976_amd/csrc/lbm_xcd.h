// Block order over the XCDs, shared by the two- and the three-dimensional kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace lbm {

// Logical block of dispatched block b out of nb: blocks are dealt round-robin to the eight
// XCDs, each with its own L2; this hands every XCD one contiguous range of logical blocks,
// so that the neighbouring wavefronts whose halo columns and rows overlap share an L2.
__device__ __forceinline__ int xcd_block(int b, int nb)
{
    constexpr int X = 8;
    const int per = nb / X, rem = nb % X;
    const int x = b % X, i = b / X;
    return x * per + min(x, rem) + i;
}

}  // namespace lbm
