// Host test of the per-sample reslice's tile edge: every slice that 16 x 16 tiles can launch (at most
// 2^32 - 1 threads, 256 per tile) can be launched at the edge chosen, at the sizes about the limit,
// and below it the edge is the largest whose box of voxels is staged.
#include <cstdio>

#include "dare_sample_tiles.h"

int main() {
    const int sizes[][2] = {{1 << 15, 1 << 15}, {1 << 14, 1 << 14}, {16385, 16383}, {16380, 16380}, {1 << 20, 1 << 10},
                            {1 << 30, 1}, {1, 1 << 28}, {1 << 24, 16}, {1 << 12, 1 << 12}, {512, 512}, {5, 3}, {1, 1}};
    for (auto& z : sizes)
        for (int R = 1; R <= 8; ++R)
            for (double pitch = 0.02; pitch < 40.0; pitch *= 1.1) {
                const double step[3] = {pitch, 0.3 * pitch, 0.8 * pitch};
                const int shift = dare::sample_tile_shift(step, R, z[0], z[1]);
                const bool ran = dare::sample_tiles(z[0], z[1], 4) * 256 <= 0xFFFFFFFFll;
                const bool runs = dare::sample_tiles(z[0], z[1], shift) * 256 <= 0xFFFFFFFFll;
                const int free = dare::sample_tile_shift(step, R, 64, 64);
                if (shift < 2 || shift > 4 || (ran && !runs) ||
                    (dare::sample_tiles(z[0], z[1], free) * 256 <= 0xFFFFFFFFll && shift != free)) {
                    std::printf("%d x %d R %d pitch %g: shift %d\n", z[0], z[1], R, pitch, shift);
                    return 1;
                }
            }
    std::printf("sample tiles host test ok\n");
    return 0;
}
