// Launch geometry of the kernels that render a frame tile by tile: which block renders what, shared by
// the kernels, the launchers and host tests.
#pragma once
#include <stdint.h>

namespace amr {

// One-wave blocks along a grid's x axis at most: HIP takes fewer than 2^32 threads there.
constexpr int64_t kSliceBlocks = 1 << 25;

// The x and z extents of a launch of `blocks` blocks (a multiple of 8, which keeps block i on XCD i mod
// 8): one slice as a rule, else slices of kSliceBlocks along z, the last of which may hold blocks
// beyond the count.  Block i = z * x extent + x.  A 32768 x 32768 image with four blocks per 8x8 tile
// takes two.
struct Slices {
    uint32_t x, z;
};
constexpr Slices slices_of(int64_t blocks) {
    return blocks <= kSliceBlocks ? Slices{(uint32_t)blocks, 1u}
                                  : Slices{(uint32_t)kSliceBlocks, (uint32_t)((blocks + kSliceBlocks - 1) / kSliceBlocks)};
}

// Sides of an image that the tile numbering serves without a schedule, and tiles of a launch with one.
constexpr int32_t kMaxSide = 32768;
constexpr int64_t kMaxSchedTiles = (int64_t)1 << 26;

}  // namespace amr
