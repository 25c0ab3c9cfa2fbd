// Tile edge of a per-sample reslice (dare_literal.hip).  Plain C++: the launch and its host test use it.
#pragma once

#include <cmath>
#include <cstdint>

namespace dare {

constexpr int kTileBox = 1536;            // voxels whose sums a tiled reslice workgroup keeps in LDS

// Workgroups of a W x H slice in tiles of 1 << shift pixels square, one each.
inline int64_t sample_tiles(int W, int H, int shift) {
    const int64_t edge = (int64_t)1 << shift;
    return ((W + edge - 1) >> shift) * ((H + edge - 1) >> shift);
}

// log2 of the tile edge: the largest of 16, 8 and 4 pixels whose box of voxels (its extent and the
// reading's reach R; `step`: voxels per pixel and axis, |i step| + |j step|) has at most kTileBox
// wherever it falls.  16, whose tiles may then sum per pixel, where none has, or where the smaller
// tiles' workgroups of 256 threads would be more than a launch takes (2^32 - 1 threads; 16384 x
// 16384 pixels in tiles of 4).  Two 489 x 137 slices at R = 2, 0.6 voxels per pixel, box reading: 599
// us with 16 x 16 tiles that sum per pixel, 69 us with 8 x 8 tiles; 300 x 300 at R = 1, 0.8 voxels
// 180 and 37 us.
inline int sample_tile_shift(const double step[3], int R, int W, int H) {
    for (int shift = 4; shift >= 2; --shift) {
        double box = 1.0;
        for (int a = 0; a < 3; ++a) box *= std::floor(((1 << shift) - 1) * step[a] + 1e-6) + 2.0 * R + 2.0;
        if (box <= (double)kTileBox) return sample_tiles(W, H, shift) * 256 <= 0xFFFFFFFFll ? shift : 4;
    }
    return 4;
}

}  // namespace dare
