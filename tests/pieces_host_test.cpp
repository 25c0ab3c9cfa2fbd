// Host test of the split of coarse reslices over workgroups: row_tiles holds every tile with a pixel
// in reach of the grid, and the tiles of a batch that hold work in pieces get several workgroups each,
// however large the batch, while all others get one; a piece's lattice points never exceed their bound,
// however far from the world's origin it lies.
#include <cstdio>
#include <random>

#include "dare_pieces.h"

using namespace dare;

struct Unit {
    int r, tile;
};

#define CHECK(x)                                              \
    do {                                                      \
        if (!(x)) {                                           \
            std::printf("line %d: %s\n", __LINE__, #x);       \
            return 1;                                         \
        }                                                     \
    } while (0)

static PlaneView random_view(std::mt19937& g, int W, int H, int n, double pitch) {
    std::normal_distribution<double> d;
    std::uniform_real_distribution<double> u(0.2, 0.8);
    PlaneView v;
    double a[3], b[3], la = 0.0, ab = 0.0, lb = 0.0;
    for (int k = 0; k < 3; ++k) a[k] = d(g), b[k] = d(g), la += a[k] * a[k];
    if (g() % 4 == 0) a[0] = 1, a[1] = a[2] = 0, la = 1, b[0] = b[2] = 0, b[1] = 1;   // along the axes
    for (int k = 0; k < 3; ++k) a[k] /= std::sqrt(la), ab += a[k] * b[k];
    for (int k = 0; k < 3; ++k) b[k] -= ab * a[k], lb += b[k] * b[k];
    for (int k = 0; k < 3; ++k) {
        v.n[k] = 1 + (int)(g() % n);
        v.ex[k] = a[k] * pitch;
        v.ey[k] = b[k] / std::sqrt(lb) * pitch * 1.3;
        v.c00[k] = u(g) * v.n[k] - v.ex[k] * W / 2 - v.ey[k] * H / 2;
    }
    v.W = W;
    v.H = H;
    v.reach = 1 + (int)(g() % 8);
    return v;
}

int main() {
    std::mt19937 g(5);
    for (int trial = 0; trial < 3000; ++trial) {
        const double pitch = std::exp(std::uniform_real_distribution<double>(-1.0, 4.0)(g));
        const PlaneView v = random_view(g, 1 + g() % 120, 1 + g() % 120, 90, pitch);
        for (int ty = 0; ty < (v.H + 15) / 16; ++ty) {
            int t0, t1;
            row_tiles(v, ty, t0, t1);
            CHECK(t0 > t1 || (t0 >= 0 && t1 < (v.W + 15) / 16));
            for (int j = 16 * ty; j < std::min(16 * ty + 16, v.H); ++j)
                for (int i = 0; i < v.W; ++i) {
                    bool in = true;
                    for (int a = 0; a < 3; ++a) {
                        const double c = v.c00[a] + i * v.ex[a] + j * v.ey[a];
                        in = in && c > -v.reach + 1e-6 && c < v.n[a] - 1 + v.reach - 1e-6;
                    }
                    CHECK(!in || (i / 16 >= t0 && i / 16 <= t1));
                }
        }
    }
    for (int trial = 0; trial < 4000000; ++trial) {   // positions as the kernel computes them, along one axis
        std::uniform_real_distribution<double> u(0.0, 1.0);
        const double far = std::pow(10.0, 16.0 * u(g)), h = 0.125, inv_h = 1.0 / h;
        const double o = far * (u(g) < 0.5 ? -1.0 : 1.0) * (0.5 + 0.5 * u(g)), e0 = 1.0 - 2.0 * u(g), e1 = 1.0 - 2.0 * u(g);
        const int edge = 1 << (g() % 4), whole = 1 + (int)(g() % 8), i0 = edge * (int)(g() % 30), j0 = edge * (int)(g() % 30);
        // extents about whole numbers of voxels, where the roundings decide
        const double sx = whole * h / (std::max(edge - 1, 1) * (std::fabs(e0) + std::fabs(e1)) + 1e-300);
        const double t = o + h * (20.0 * u(g) - 10.0);
        double lo = 0.0, hi = 0.0;
        for (int k = 0; k < 4; ++k) {
            const double is = (double)(i0 + (k & 1 ? edge - 1 : 0)) * sx, js = (double)(j0 + (k & 2 ? edge - 1 : 0)) * sx;
            const double p = (t + is * e0) + js * e1, c = std::floor((p - o) * inv_h);
            lo = k ? std::min(lo, c) : c;
            hi = k ? std::max(hi, c) : c;
        }
        const double place = std::fabs(t) + std::fabs(o) + 512.0 * sx * (std::fabs(e0) + std::fabs(e1));
        const int points = piece_points(edge, sx * (std::fabs(e0) + std::fabs(e1)) * inv_h, place * inv_h);
        CHECK(hi - lo + 2.0 <= points || points >= 1024);
        CHECK(far > 1e4 || points <= whole + (edge > 1 ? 4 : 3));
    }
    CHECK(tile_pieces(0.5) == 1 && tile_pieces(1.1) == 4 && tile_pieces(16.0) == 256 && tile_pieces(1e30) == 256);
    for (int n : {1, 4, 16, 64, 400}) {       // coarse slices of a batch, and as many fine ones
        StagedUnits<Unit> u;
        std::vector<Unit> units;
        int32_t counts[4] = {0, 0, 0, 0};
        int64_t tiles = 0;
        for (int r = 0; r < 2 * n; ++r) {
            const PlaneView v = random_view(g, 512, 300, 256, r % 2 ? 0.5 : 16.0);
            if (r % 2) u.add_fine(r, v.W, v.H);
            else u.add_coarse(v, r, tile_pieces(16.0));
            tiles += 32 * 19;
        }
        const int grid = u.finish(counts, units);
        CHECK(counts[0] == (int)units.size() && counts[0] == tiles && counts[2] > 0 && counts[2] < 40 * n);
        CHECK(counts[3] >= std::min(256, 16384 / (40 * n)) && counts[3] <= 256 && grid >= 1 && grid <= 65535);
        for (int k = 0; k < counts[2]; ++k) CHECK(units[k].r % 2 == 0);
        std::vector<char> seen(tiles, 0);
        for (const Unit& q : units) CHECK(q.tile >= 0 && q.tile < 32 * 19 && !seen[q.r * 32 * 19 + q.tile]++);
    }
    std::printf("pieces host test ok\n");
    return 0;
}
