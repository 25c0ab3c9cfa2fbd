"""A grid whose brick table has more entries than 32 bits index (64 bins of 4096 x 4096 x 1040
voxels): frames in the entries below 2^31 are compounded, a batch with a pixel above is refused and
leaves the volume as it was."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_helpers import note
from helpers import rodrigues

pytestmark = pytest.mark.gpu


def test_entries_past_32_bits_are_refused():
    import torch

    import paper_2605_26325_amd as dare
    dims, w, h = (4096, 4096, 1040), 40, 24
    per_bin = (dims[0] // 8) * (dims[1] // 8) * (dims[2] // 8)
    assert 63 * per_bin < 2 ** 31 < 64 * per_bin
    note("brick table of 2.18e9 entries")
    vol = dare.Volume(dare.make_geometry((0, 0, 0), 1.0, dims, np.eye(4)), dare.default_params(bin_tol_deg=2.0), dtype="bf16",
                      bricks=2000)

    def pose(k, z):                      # frame of bin k: its normal turned by 5 k degrees
        T = np.eye(4)
        T[:3, :3] = rodrigues(np.array([0.0, 1.0, 0.0]), np.deg2rad(5.0 * k))
        T[:3, 3] = (2000.0, 2000.0, z)
        return T
    frames = torch.full((64, h, w), 100, dtype=torch.uint8, device="cuda")

    def add(poses):
        p = torch.from_numpy(np.stack(poses).astype(np.float32)).cuda()
        return vol.reconstruct(frames[:len(poses)], p, (1.0, 1.0))
    add([pose(k, 500.0) for k in range(63)])
    before = vol.info()
    codebook = vol.codebook()
    assert before.bins == 63 and before.bricks_used > 63
    sl = vol.reslice(pose(3, 500.0), w, h, (1.0, 1.0)).cpu()
    assert bool(torch.isfinite(sl).any())
    # bin 63 in the last layers of bricks: entries of 2^31 and above
    with pytest.raises(dare.DareError) as e:
        add([pose(3, 520.0), pose(63, 1030.0)])
    assert e.value.status == dare.ERR_BUDGET
    after = vol.info()
    assert (after.bins, after.bricks_used, after.saturated) == (before.bins, before.bricks_used, before.saturated)
    assert all(np.array_equal(a, b) for a, b in zip(vol.codebook(), codebook))
    assert torch.equal(vol.reslice(pose(3, 500.0), w, h, (1.0, 1.0)).cpu().view(torch.int32), sl.view(torch.int32))
    # the same bin in its first layers, and the same place in another bin
    add([pose(63, -20.0), pose(3, 1030.0)])
    assert vol.info().bins == 64 and vol.info().bricks_used > before.bricks_used
    for k, z in ((63, -20.0), (3, 1030.0)):
        assert bool(torch.isfinite(vol.reslice(pose(k, z), w, h, (1.0, 1.0))).any())
