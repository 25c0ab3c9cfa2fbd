"""Dense sums and counts of grids about the widths at which the download's waves change their shape:
what was uploaded comes back, with nothing but zeros elsewhere.  Whole numbers: no tolerance."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_helpers import note
from helpers import random_grid

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx", [1, 7, 8, 9, 16, 17, 31, 32, 33, 64, 65, 130])
def test_widths(nx):
    import torch

    import paper_2605_26325_amd as dare
    note(f"dense download, {nx} voxels wide")
    rng = np.random.default_rng(nx)
    for ny, nz in ((9, 17), (40, 3), (1, 1)):
        K = 3
        S, C = random_grid(rng, K, (nx, ny, nz), p_empty=0.4)
        C[1, :, : ny // 2] = 0                              # whole bricks without a slot
        S[C == 0] = 0
        vol = dare.Volume(dare.make_geometry((0, 0, 0), 1.0, (nx, ny, nz), np.eye(4)), dare.default_params())
        St, Ct = (torch.from_numpy(x.astype(np.uint32).view(np.int32)).cuda() for x in (S, C))
        rn = np.array([[np.sin(k), 0.0, np.cos(k)] for k in range(K)])
        vol.upload_sums(rn, np.array([[0.0, 1.0, 0.0]] * K), St, Ct)
        torch.full((K, nz, ny, nx), 7, dtype=torch.int32, device="cuda")    # what the arrays' memory may hold before
        got_S, got_C = vol.download_sums()
        torch.cuda.synchronize()
        assert torch.equal(got_S, St) and torch.equal(got_C, Ct), (nx, ny, nz)
