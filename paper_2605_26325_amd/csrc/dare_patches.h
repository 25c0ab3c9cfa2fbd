// Patches of 1024 pixels that the per-pixel compounding passes take, one per workgroup of 256
// threads (dare_compound.hip).  Plain C++ (constexpr: device code too): the launches, the kernels
// and the host tests use it.
#pragma once

#include <algorithm>
#include <cstdint>

namespace dare {

// A patch is 16 blocks of 64 pixels, `1 << across` side by side; a wave takes four blocks in turn,
// one pixel per lane.  nx x ny patches cover a frame.
struct PatchShape {
    int block;                             // log2 of a block's width
    int across;                            // log2 of the blocks side by side
    int nx, ny;
};

struct PatchPixel {
    int i, j;                              // column and row; may lie past the frame's edges
};
constexpr PatchPixel patch_pixel(const PatchShape& s, int px, int py, int q, int lane) {
    const int bx = (px << s.across) + (q & ((1 << s.across) - 1)), by = (py << (4 - s.across)) + (q >> s.across);
    return PatchPixel{(bx << s.block) + (lane & ((1 << s.block) - 1)), (by << (6 - s.block)) + (lane >> s.block)};
}

// Blocks of 8 x 8 pixels, narrower or flatter only where the frame is, so that a wave's lanes all have
// pixels: 1000 frames of 1 x 512 pixels take 71 us, 183 in 8 x 8 blocks (4 x 512: 102 and 186).  Of
// the ways to lay out 16 blocks the one with the fewest patches, 4 x 4 blocks where that is one of
// them (33 x 33 pixels: 3 patches, not 4, 554 us against 590 for 1000 frames).
inline PatchShape patch_shape(int w, int h) {
    PatchShape best{3, 2, 0, 0};
    while (best.block > 0 && w <= 1 << (best.block - 1)) --best.block;
    if (best.block == 3)
        while (best.block < 6 && h <= 1 << (5 - best.block)) ++best.block;
    const int64_t bw = (int64_t)1 << best.block, bh = 64 / bw;
    const int64_t cols = (w + bw - 1) / bw, rows = (h + bh - 1) / bh;
    for (int across : {2, 1, 3, 0, 4}) {
        const int64_t nx = (cols + (1 << across) - 1) >> across, ny = (rows + (16 >> across) - 1) / (16 >> across);
        if (best.nx == 0 || nx * ny < (int64_t)best.nx * best.ny) best = PatchShape{best.block, across, (int)nx, (int)ny};
    }
    return best;
}

// Frames per launch of the per-pixel passes (flat grids of patches x frames): fewer than 2^24
// workgroups, as a launch takes at most 2^32 - 1 threads.
inline int frames_per_launch(int n, const PatchShape& s) {
    const int64_t fc = (((int64_t)1 << 24) - 1) / ((int64_t)s.nx * s.ny);
    return (int)std::max<int64_t>(1, std::min<int64_t>(n, fc));
}

}  // namespace dare
