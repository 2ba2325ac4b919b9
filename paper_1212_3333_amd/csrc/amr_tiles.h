// Launch geometry of the kernels that render a frame tile by tile: which block renders what, shared by
// the kernels, the launchers and host tests.
#pragma once
#include <stdint.h>

namespace amr {

// A frame's super-tiles (4x4 tiles) in launch order: squares of 2^sq super-tiles a side, nx to a row, row by
// row, each along a Morton curve, so that the super-tiles in flight on an XCD, which takes every eighth,
// stay close together.  The squares are the largest with which the order has at most slack / 2 times
// as many places as the frame has super-tiles.  A launch (kLaunchSlack) keeps one square over the
// frame until three places in four are empty: an empty place is 64 blocks that return at once.  A
// 16384x16 frame has 512 super-tiles and the square over it 262144: lit 5.7 -> 0.9 ms, unlit 3.95 -> 0.54
// (3.5 and 1.48 ms with one lane per ray and a quarter of the blocks).  Tighter launches gain on some
// frames and lose on others, by what their order is worth on the XCDs (27 sizes from 63x70 to 1100x1000
// in two scenes: 0.85 to 1.15 of the time at kQueueSlack, 0.99 on average; 0.96 to 1.04 at this).  A
// queue (kQueueSlack) hands out its empty places by an atomic each: four images of 100 to 384 pixels a
// side, unlit, 2.53 -> 1.77 ms.
struct Cover {
    int32_t sq, nx;
    int64_t n;                         // places
};
constexpr int kLaunchSlack = 8, kQueueSlack = 3;
constexpr Cover cover_of(int64_t tiles_x, int64_t tiles_y, int slack) {
    const int64_t w = (tiles_x + 3) / 4, h = (tiles_y + 3) / 4;
    int32_t sq = 0;
    while (((int64_t)1 << sq) < w || ((int64_t)1 << sq) < h) sq++;
    for (;; sq--) {
        const int64_t nx = (w + ((int64_t)1 << sq) - 1) >> sq, ny = (h + ((int64_t)1 << sq) - 1) >> sq;
        const int64_t n = (nx * ny) << (2 * sq);
        if (sq == 0 || 2 * n <= slack * w * h) return Cover{sq, (int32_t)nx, n};
    }
}

// Super-tile i of the order; beyond the cover, one below the frame.
struct SuperTile {
    int32_t x, y;
};
constexpr SuperTile super_tile(int32_t sq, int32_t nx, uint32_t i) {
    const uint32_t q = i >> (2 * sq);
    int32_t x = (int32_t)(q % (uint32_t)nx) << sq, y = (int32_t)(q / (uint32_t)nx) << sq;
    for (int32_t bit = 0; bit < sq; bit++) {
        x |= (int32_t)((i >> (2 * bit)) & 1u) << bit;
        y |= (int32_t)((i >> (2 * bit + 1)) & 1u) << bit;
    }
    return SuperTile{x, y};
}

// Lanes that march a ray of an unlit image, of `pixels` pixels on average in its launch.  Four while a ray's
// chain of dependent reads is what the image waits for; one when there are rays enough to cover it:
// then the walk from leaf to leaf, which four lanes pay four times, and the part of a segment's last
// step that is empty count, and neighbouring rays share bricks as a ray's samples do.  In a deep tree a ray's
// segments are more, and its chain longer, so that the line lies further up.  Four lanes, one lane and
// (before four were tried) one that restarted its walks, in ms: 300 patches, 1024^2 2.21, 1.94, 2.38;
// 1536^2 4.41, 3.35, 4.10; 2048^2 7.34, 5.32, 6.54; 4096^2 27.0, 17.2, 21.3.  2000 patches, 1024^2 3.12,
// 3.79, 4.41; 1280^2 4.60, 4.68, 5.70; 1536^2 5.90, 5.55, 6.74; 4096^2 32.1, 24.0, 29.7.  20 levels
// (depth 82), 1024^2 1.02, 1.47, 2.42; 1536^2 1.49, 1.73, 2.91; 2048^2 2.54, 2.54, 4.28; 4096^2 9.5, 6.2,
// 8.7.  Views of 512^2 and 768^2, eight to a launch, are better off with four lanes in both scenes,
// or as well.  With checkpoints the line lies further up in shallow trees too: 300 patches, 1280^2 3.50,
// 3.44, 3.43; 2048^2 7.78, 6.67, 6.71; 4096^2 28.4, 20.4, 21.4.  2000 patches, 1280^2 4.86, 6.52, 6.33;
// 1536^2 6.36, 7.74, 7.53; 2048^2 10.2, 10.7, 10.3; 4096^2 34.0, 30.3, 30.3.
constexpr int lanes_per_ray(int64_t pixels, int32_t depth, bool ckpt = false) {
    return pixels < (depth < 48 && !ckpt ? (int64_t)3 << 19 : (int64_t)1 << 22) ? 4 : 1;
}

// Blocks of a launch over n super-tiles, dealt to the 8 XCDs in turn (block i on XCD i mod 8), with `per`
// blocks to a tile; block i renders part (i / 8) % per of tile (i / (8 per)) % 16 of super-tile
// (i / (128 per)) * 8 + i % 8.
constexpr int64_t cover_blocks(int64_t n, int per) { return (n + 7) / 8 * 8 * 16 * per; }

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
