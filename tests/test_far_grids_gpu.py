"""Radii above 1 far from the world's origin, where a position's rounding is no longer small against a
voxel, at pitches whose tiles go in pieces: against the FP64 oracle (the same positions to the bit; a
spacing of a power of two), alone and batched.

Tolerance: |d| <= 1e-5 max(|ref|, 1) as for every reslice."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_helpers import assert_parity, make_volume, note, upload_grid
from helpers import random_grid
from oracle import quant, reslice
from oracle.reslice import Params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R", [2, 4, 7])
@pytest.mark.parametrize("place", [2.0 ** 31, 2.0 ** 36])
def test_far_from_the_origin(R, place):
    import torch

    import paper_2605_26325_amd as dare
    rng = np.random.default_rng(R)
    dims, h, K = (33, 28, 31), 0.5, 3
    S, C = random_grid(rng, K, dims, p_empty=0.4)
    origin = np.array([place, -0.7 * place, 0.9 * place])
    rn = np.array([[0.0, np.sin(0.05 * k), np.cos(0.05 * k)] for k in range(K)])
    rx = np.array([[1.0, 0.0, 0.0]] * K)
    prm = Params(radius_vox=R)
    vol = make_volume(origin, h, dims, np.eye(4), prm)
    upload_grid(vol, S, C, rn, rx)
    a, c = quant.storage(S, C, "fp32")
    specs, refs = [], []
    for pv in (0.7, 10.0 / 15.0, 8.0 / 7.0, 3.0, 5.0, 4.0 / 3.0):
        W, H, p = 37, 34, (pv * h, pv * h)
        T = np.eye(4)
        turn = rng.uniform(-0.2, 0.2)          # within the in-plane gate
        T[:3, 0], T[:3, 1] = [np.cos(turn), np.sin(turn), 0.0], [-np.sin(turn), np.cos(turn), 0.0]
        T[:3, 3] = origin + h * (np.array(dims) - 1) / 2 - T[:3, 0] * (W // 2) * p[0] - T[:3, 1] * (H // 2) * p[1]
        specs.append(dare.make_spec(T, W, H, p))
        refs.append(reslice.reslice(a, c, origin, h, rn, rx, np.eye(4), T, W, H, p, prm))
    note(f"far grid at {place:g} mm, R={R}")
    alone = [torch.full((s.height, s.width), -3.0, device="cuda") for s in specs]
    for s, o in zip(specs, alone):
        dare.dare_reslice(vol, s, o)
    outs = [torch.full((s.height, s.width), -7.0, device="cuda") for s in specs]
    vols = [vol] * len(specs)
    ws = torch.empty(dare.dare_reslice_batch_workspace_bytes(vols, specs), dtype=torch.uint8, device="cuda")
    dare.dare_reslice_batch(vols, specs, outs, ws)
    torch.cuda.synchronize()
    for k, ref in enumerate(refs):
        assert assert_parity(alone[k].cpu().numpy(), ref, what=f"R={R} {place:g} {k}") > 0
        assert torch.equal(outs[k].view(torch.int32), alone[k].view(torch.int32)), k
