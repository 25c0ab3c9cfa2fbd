// Batched reslice: many requests (volumes, poses, sizes) in a fixed set of launches whose
// counts are read from device memory, so that a captured graph can replay any batch.
// Radius 1 runs the request setup pass and the persistent tile kernel (dare_tiles.hip); larger
// radii run the host-built (request, tile) table (dare_reslice_rs.hip).
#include "dare_staged.h"

namespace dare {

hipError_t launch_reslice_batch(int dtype, int radius, const BatchReq* reqs, SliceRec* recs, int2* units,
                                TileRec* tiles, int* counts, int nreq_max, int cap, int grid, hipStream_t stream) {
    if (radius <= 1) return launch_tiles_batch(dtype, reqs, recs, units, tiles, counts, nreq_max, cap, stream);
    return launch_reslice_staged_batch(dtype, radius, reqs, units, counts, grid, stream);
}

}  // namespace dare
