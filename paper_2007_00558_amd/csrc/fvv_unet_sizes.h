// fvv_unet_sizes.h -- grid and buffer sizes of the network's training kernels
// that have to agree (host arithmetic only, no HIP).
#pragma once

#include <algorithm>
#include <cstddef>

// Blocks of a convolution launch that writes bias partials: a row of M floats
// per `mgroups` blocks (the blocks of a row share its columns), in a buffer of
// `floats`.  The kernels walk their work in steps of the grid, so any multiple
// of 8 computes the same; `mgroups` divides 8 and `grid` is a multiple of 8,
// and the buffer holds at least the rows of 8 blocks.
inline int unet_bias_grid(int grid, int mgroups, int M, size_t floats)
{
    const size_t blocks = floats / (size_t)M * (size_t)mgroups;
    return std::max(8, (int)std::min<size_t>((size_t)grid, blocks / 8 * 8));
}
