// Host test of the compounding passes' patches: every pixel of a frame lies in exactly one lane of one
// patch, thin frames keep their lanes in use, and every frame that the entry points take fits a launch.
#include <cstdio>
#include <random>
#include <vector>

#include "dare_patches.h"

using namespace dare;

#define CHECK(x)                                                      \
    do {                                                              \
        if (!(x)) {                                                   \
            std::printf("line %d, %d x %d: %s\n", __LINE__, w, h, #x); \
            return 1;                                                 \
        }                                                             \
    } while (0)

int main() {
    std::mt19937 g(3);
    for (int trial = 0; trial < 4000; ++trial) {
        const int w = 1 + g() % (trial % 3 ? 40 : 300), h = 1 + g() % (trial % 5 ? 40 : 300);
        const PatchShape s = patch_shape(w, h);
        CHECK(s.block >= 0 && s.block <= 6 && s.across >= 0 && s.across <= 4);
        std::vector<int> hit((size_t)w * h, 0);
        int64_t waves = 0;                                   // blocks with any pixel
        for (int py = 0; py < s.ny; ++py)
            for (int px = 0; px < s.nx; ++px)
                for (int q = 0; q < 16; ++q) {
                    bool any = false;
                    for (int lane = 0; lane < 64; ++lane) {
                        const PatchPixel p = patch_pixel(s, px, py, q, lane);
                        CHECK(p.i >= 0 && p.j >= 0);
                        if (p.i >= w || p.j >= h) continue;
                        any = true;
                        ++hit[(size_t)p.j * w + p.i];
                    }
                    waves += any;
                }
        for (int n : hit) CHECK(n == 1);
        // full blocks but for the last ones of each direction; never more patches than 4 x 4 blocks give
        CHECK(waves <= ((w + 7) / 8) * ((h + 7) / 8));
        CHECK((int64_t)s.nx * s.ny <= (int64_t)((w + 31) / 32) * ((h + 31) / 32));
        if (w == 1 || h == 1) CHECK(waves == (w * h + 63) / 64);
    }
    const int sizes[][2] = {{1, 1 << 30}, {1 << 30, 1}, {9, 119304647}, {119304647, 9}, {1 << 15, 1 << 15}, {2048, 2048},
                            {256, 256}, {33, 33}, {3, 5}};
    for (auto& z : sizes) {
        const int w = z[0], h = z[1];
        const PatchShape s = patch_shape(w, h);
        for (int n : {1, 3, 4096, 1 << 20}) {
            const int64_t fc = frames_per_launch(n, s);
            CHECK(fc >= 1 && fc <= n && (int64_t)s.nx * s.ny * fc * 256 <= 0xFFFFFFFFll);
        }
        const PatchPixel last = patch_pixel(s, s.nx - 1, s.ny - 1, 15, 63);
        CHECK(last.i >= w - 1 && last.j >= h - 1);
    }
    std::printf("patches host test ok\n");
    return 0;
}
