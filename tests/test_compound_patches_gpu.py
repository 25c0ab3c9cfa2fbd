"""Compounding at the edges of its pixel patches, bit for bit against the oracle: image sizes off the
32 x 32 patches and 8 x 8 blocks, several pixels in one voxel (merged before memory) and pixels
many bricks apart (more entries in a patch than its set holds), more frames than one chunk of the
bin assignment with many opened bins, grids off the dense download's rows, a second call into
resident bricks.  Whole numbers: no tolerance.
"""
from __future__ import annotations

import numpy as np
import pytest

import synth
from gpu_helpers import make_volume, note
from helpers import random_unit, rodrigues
from oracle import compound
from oracle.reslice import Params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,pv,dims,frames,spread,tol", [
    (1, 1, 1.0, (8, 8, 8), 5, 3.0, 5.0),
    (33, 31, 0.24, (21, 9, 65), 7, 4.0, 5.0),          # 16 pixels a voxel, ragged patches
    (64, 40, 0.5, (70, 66, 33), 9, 8.0, 5.0),
    (40, 70, 1.0, (64, 31, 72), 12, 8.0, 5.0),
    (47, 45, 9.5, (320, 96, 300), 3, 5.0, 5.0),        # every pixel in a brick of its own
    (5, 3, 2.0, (24, 24, 24), 1300, 40.0, 12.0),       # three chunks, bins opened in each
    (5, 3, 2.0, (24, 24, 24), 700, 40.0, 0.0),         # saturated codebook
])
def test_compound_patch_edges(w, h, pv, dims, frames, spread, tol):
    import torch
    note(f"compounding {frames} frames {w}x{h} at {pv} voxels into {dims}, spread {spread} tol {tol}")
    rng = np.random.default_rng(w * 1000 + h)
    sp, prm = 0.5, Params(bin_tol_deg=tol)
    pitch = (pv * sp, pv * sp * 0.97)
    calib = synth.make_calibration(w, pitch[0])
    origin = np.array([-850.0, 310.0, -1620.0])
    P = np.empty((frames, 4, 4), np.float32)
    for f in range(frames):
        R = rodrigues(random_unit(rng), np.deg2rad(rng.uniform(0, spread)))
        T = np.eye(4)
        T[:3, 0], T[:3, 1] = R @ [1.0, 0.0, 0.0], R @ [0.0, 0.0, 1.0]
        T[:3, 2] = np.cross(T[:3, 0], T[:3, 1])
        mid = origin + sp * (np.array(dims) - 1) * rng.uniform(0.3, 0.7, 3)
        T[:3, 3] = mid - T[:3, 0] * (w // 2) * pitch[0] - T[:3, 1] * (h // 2) * pitch[1]
        P[f] = (T @ np.linalg.inv(calib)).astype(np.float32)
    img = rng.integers(0, 256, (frames, h, w), dtype=np.uint8)
    vol = make_volume(origin, sp, dims, calib, prm, bricks=40_000)
    g = compound.empty_grid(origin, sp, dims, prm.bin_tol_deg, prm.max_bins)
    d_img, d_P = torch.from_numpy(img).cuda(), torch.from_numpy(P).cuda()
    for first, last in ((0, (frames + 1) // 2), (frames // 3, frames)):   # the second call meets resident bricks
        if tol == 0.0:
            with pytest.warns(RuntimeWarning):
                vol.reconstruct(d_img[first:last].contiguous(), d_P[first:last].contiguous(), pitch)
        else:
            vol.reconstruct(d_img[first:last].contiguous(), d_P[first:last].contiguous(), pitch)
        compound.compound(g, img[first:last], P[first:last], calib, pitch)
    S, C = vol.download_sums()
    torch.cuda.synchronize()
    assert C.shape[0] == g.C.shape[0]
    assert int(g.C.sum()) > 0
    assert np.array_equal(C.cpu().numpy(), g.C) and np.array_equal(S.cpu().numpy(), g.S)
