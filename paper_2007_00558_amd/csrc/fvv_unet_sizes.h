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

// Floats of the bias partials of a training step on `px` full-resolution pixels
// (multiples of 8 x 8 per image): no level has more than px / 64 patches, each a
// row of up to 256 channels, rounded up to 8 blocks; 2,048 rows of 128 channels
// at most (the pool gradient's).  Grows with px.
inline size_t unet_bias_floats(size_t px) { return std::min<size_t>(4 * px + 512, (size_t)2048 * 128); }

// Blocks of the head's training kernel (256 pixels per block and step).
inline int unet_head_blocks(size_t px) { return (int)std::min<size_t>(1024, (px + 255) / 256); }

// Floats of the weight gradients' partials where memory is short: one partial of
// the widest layer (256 x 9 x 256) and what the other buffers of a training set
// leave of 1.2 kB per pixel.  The layers then take fewer pixel chunks.
inline size_t unet_lean_partials(size_t px) { return (size_t)256 * 9 * 256 + 80 * px; }
