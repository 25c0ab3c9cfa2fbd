// Reslice at interpolation radius 2..8 through the tent sums of the voxel lattice
// (dare_reslice_rs.hip).  Radius 1 runs the tile kernels of dare_tiles.hip.
#pragma once

#include "dare_batch.h"
#include "dare_pieces.h"

namespace dare {

// `pitch_vox`: the larger output pitch in voxels.
hipError_t launch_reslice_staged(const VolDev* vd, int dtype, int radius, const SliceArgs& s, double pitch_vox,
                                 hipStream_t stream);
// Batched form: counts[0] units, the first counts[2] of them with counts[3] workgroups each.
hipError_t launch_reslice_staged_batch(int dtype, int radius, const BatchReq* reqs, const int2* units,
                                       const int* counts, int grid, hipStream_t stream);
// Work units of a W x H request: its 16 x 16 tiles.
int64_t staged_tiles(int W, int H);
// Unit entries that a workspace holds for a W x H request at this radius (at least its tiles).
int64_t batch_units(int radius, int W, int H);

}  // namespace dare
