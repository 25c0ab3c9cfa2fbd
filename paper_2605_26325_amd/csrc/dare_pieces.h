// How reslices at radius 2..8 are split over workgroups where the output is too coarse for a 16 x
// 16 tile to be staged in one piece (dare_reslice_rs.hip).  Plain C++: the planners and the host
// tests use it.  The split only says which workgroup takes which piece; the pieces themselves and
// their results are the kernel's.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <vector>

namespace dare {

// Pieces of a tile at an output pitch of `pitch_vox` voxels: 1 up to an extent of about 10 voxels,
// then pieces of 8, 4, 2 or 1 pixels squared.
inline int tile_pieces(double pitch_vox) {
    int edge = 16;
    while (edge > 1 && (double)(edge - 1) * pitch_vox > 10.0) edge >>= 1;
    return (16 / edge) * (16 / edge);
}

// Lattice points per axis that a piece of `edge` pixels squared takes at most, wherever it falls: its cells
// span at most its extent's floor plus one, hence that plus three.  `step`: voxels per pixel along
// the axis, |i step| + |j step|; `place`: the largest magnitude, in voxels, that enters the
// positions, whose four roundings of 2^-53 each move the first and the last one.  (A margin of 1e-6
// voxels alone can be exceeded from about 1e9 voxels off the world's origin.)
constexpr int piece_points(int edge, double step, double place) {
    const double ext = (double)(edge - 1) * step * (1.0 + 1e-9) + 1e-6 + 1e-15 * place;
    return edge == 1 ? 2 : (int)(ext < 1024.0 ? ext : 1024.0) + 3;
}

// Workgroups per tile for `tiles` tiles of `pieces` pieces: up to 64 workgroups per CU in all.
inline int tile_parts(int64_t tiles, int pieces) {
    return (int)std::max<int64_t>(1, std::min<int64_t>(pieces, 16384 / std::max<int64_t>(tiles, 1)));
}

// A slice in voxel units, pixel (i, j) at c00 + i ex + j ey, over a grid of n voxels.
struct PlaneView {
    double c00[3], ex[3], ey[3];
    int32_t n[3];
    int32_t W, H;
    double reach;                          // voxels beyond the grid that its values still reach
};

// The tiles of tile row `ty` that may hold a pixel within reach of the grid: columns t0..t1, none
// if t0 > t1.  Each axis on its own, so an oblique plane's corners may be taken in needlessly.
inline void row_tiles(const PlaneView& v, int ty, int& t0, int& t1) {
    double lo = 0.0, hi = (double)(v.W - 1);
    const double j0 = 16.0 * ty, j1 = std::min(j0 + 15.0, (double)(v.H - 1));
    for (int a = 0; a < 3; ++a) {
        const double y0 = std::min(j0 * v.ey[a], j1 * v.ey[a]), y1 = std::max(j0 * v.ey[a], j1 * v.ey[a]);
        const double from = -v.reach - y1 - v.c00[a], to = (double)(v.n[a] - 1) + v.reach - y0 - v.c00[a];   // of i ex
        if (std::fabs(v.ex[a]) < 1e-12) {
            if (from > 1e-3 || to < -1e-3) hi = -1.0;
            continue;
        }
        const double p = from / v.ex[a], q = to / v.ex[a];
        lo = std::max(lo, std::min(p, q));
        hi = std::min(hi, std::max(p, q));
    }
    t0 = lo <= hi ? (int)(lo / 16.0) : 0;
    t1 = lo <= hi ? (int)(hi / 16.0) : -1;
}

// A batch's (request, tile) units: the tiles that hold work in pieces (of coarse requests, near the
// grid) first, with several workgroups each; every other tile, of fine requests and away from the
// grid, has one.  One number of workgroups for all tiles of a batch left the coarse requests of a
// large batch serial and gave the fine ones of a small batch idle workgroups.  32 slices of 512 x
// 512, 16 voxels apart, at R = 2 and 8: 1400 and 6540 us with one number, 303 and 1140 us so; one
// such slice with 16 fine ones of 256 x 256 at R = 2: 259 and 77 us.
template <class Unit>
struct StagedUnits {
    std::vector<Unit> coarse, fine;
    int most_pieces = 1;
    // The tiles of request `r`, staged in one piece each.
    void add_fine(int r, int W, int H) {
        const int n = ((W + 15) / 16) * ((H + 15) / 16);
        for (int t = 0; t < n; ++t) fine.push_back(Unit{r, t});
    }
    // The tiles of request `r`, in `pieces` pieces each where they hold work.
    void add_coarse(const PlaneView& v, int r, int pieces) {
        const int tx = (v.W + 15) / 16, ty = (v.H + 15) / 16;
        most_pieces = std::max(most_pieces, pieces);
        for (int y = 0; y < ty; ++y) {
            int t0, t1;
            row_tiles(v, y, t0, t1);
            for (int x = 0; x < tx; ++x) (x >= t0 && x <= t1 ? coarse : fine).push_back(Unit{r, y * tx + x});
        }
    }
    // The unit list in the kernel's order and its counts (dare_batch.h; counts[1] is the caller's);
    // returns the workgroups that it can use.
    int finish(int32_t counts[4], std::vector<Unit>& units) {
        counts[0] = (int32_t)(coarse.size() + fine.size());
        counts[2] = (int32_t)coarse.size();
        counts[3] = tile_parts((int64_t)coarse.size(), most_pieces);
        const int64_t groups = (int64_t)fine.size() + (int64_t)coarse.size() * counts[3];
        if (coarse.empty()) {
            units.swap(fine);
        } else {
            units.swap(coarse);
            units.insert(units.end(), fine.begin(), fine.end());
        }
        return (int)std::min<int64_t>(groups, 65535);
    }
};

}  // namespace dare
