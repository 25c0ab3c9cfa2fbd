"""Radii 2..8 against the FP64 oracle at the edges of the staged pieces: output pitches at which a
16 x 16 tile stages in one piece, in 8 x 8, 4 x 4 and 2 x 2 pieces and pixel by pixel, ragged
sizes, oblique planes partly outside the grid, more than 8 surviving bins; batched equals alone.

Tolerance: |d| <= 1e-5 max(|ref|, 1) as for every reslice.  The sums are FP32 with at most
3 (2R - 1) + 3 roundings of 2^-24 each on positive terms, under 3e-6 relative at R = 8.
"""
from __future__ import annotations

import numpy as np
import pytest

import synth
from gpu_helpers import assert_parity, make_volume, note, upload_grid
from helpers import random_grid, random_unit, rodrigues
from oracle import quant, reslice
from oracle.reslice import Params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,dtype", [(2, "f32"), (3, "bf16"), (4, "fp8"), (5, "f32"), (6, "f16"), (7, "fp8"), (8, "f32")])
def test_wide_radius_pieces_vs_oracle(R, dtype):
    import torch

    import paper_2605_26325_amd as dare
    rng = np.random.default_rng(700 + R)
    dims, h, K = (23, 18, 21), 0.5, 9
    S, C = random_grid(rng, K, dims, p_empty=0.6)
    n0, x0 = np.array([0.0, -1.0, 0.0]), np.array([1.0, 0.0, 0.0])
    turns = [rodrigues(random_unit(rng), np.deg2rad(rng.uniform(0, 6))) for _ in range(K)]
    calib = synth.make_calibration(16, 0.5)
    origin = np.array([-850.0, 310.0, -1620.0])
    prm = Params(radius_vox=R)
    form = {"f32": "fp32", "bf16": "bf16", "f16": "fp16", "fp8": "fp8"}[dtype]
    a, c = quant.storage(S, C, form)
    specs, refs, vols = [], [], []
    # axis-aligned, tilted about one axis, and steep on all three (the widest boxes)
    for base in (np.eye(3), rodrigues(np.array([0.0, 0.0, 1.0]), 0.6), rodrigues(np.array([1.0, 1.0, 0.0]) / 2 ** 0.5, 0.95)):
        rn = np.array([base @ t @ n0 for t in turns])
        rx = np.array([base @ t @ x0 for t in turns])
        vol = make_volume(origin, h, dims, calib, prm, dtype=dtype)
        upload_grid(vol, S, C, rn, rx)
        for pv in (0.4, 1.1, 3.0, 7.0, 21.0):
            W, H, p = 19, 18, (pv * h, 1.07 * pv * h)
            T = np.eye(4)
            T[:3, 0], T[:3, 2] = base @ x0, base @ n0
            T[:3, 1] = np.cross(T[:3, 2], T[:3, 0])
            mid = origin + h * (np.array(dims) - 1) / 2 + rng.normal(0, 1.5, 3) * h
            T[:3, 3] = mid - T[:3, 0] * (W // 2) * p[0] - T[:3, 1] * (H // 2) * p[1]
            P = T @ np.linalg.inv(calib)
            specs.append(dare.make_spec(P, W, H, p))
            vols.append(vol)
            refs.append(reslice.reslice(a, c, origin, h, rn, rx, calib, P, W, H, p, prm))
    alone = []
    for k, (v, s, ref) in enumerate(zip(vols, specs, refs)):
        note(f"R={R} {dtype} case {k}")
        out = torch.full((s.height, s.width), -3.0, device="cuda")
        dare.dare_reslice(v, s, out)
        torch.cuda.synchronize()
        alone.append(out)
        assert assert_parity(out.cpu().numpy(), ref, what=f"R={R} {dtype} case {k}") > 0
    outs = [torch.full((s.height, s.width), -7.0, device="cuda") for s in specs]
    ws = torch.empty(dare.dare_reslice_batch_workspace_bytes(vols, specs), dtype=torch.uint8, device="cuda")
    dare.dare_reslice_batch(vols, specs, outs, ws)
    torch.cuda.synchronize()
    for k, (o, x) in enumerate(zip(outs, alone)):
        assert torch.equal(o.view(torch.int32), x.view(torch.int32)), f"R={R} {dtype} case {k}: batched differs"


@pytest.mark.parametrize("R", [2, 5])
def test_only_a_far_corner_assigned(R):
    """Pixels a rounding error off a lattice point on every axis, where the only valid voxels lie R
    away on the far side: FP64 weights of about 1e-39 to 1e-48, whose quotient is the voxel's value."""
    import torch

    import paper_2605_26325_amd as dare
    note(f"far corner, R={R}")
    dims, h, N = (24, 24, 24), 1.0, 24
    S, C = np.zeros((1, N, N, N), np.int64), np.zeros((1, N, N, N), np.int64)
    S[0, 12, 12, 12], C[0, 12, 12, 12] = 3 * 97, 3
    prm = Params(radius_vox=R)
    calib = np.eye(4)
    origin = np.zeros(3)
    vol = make_volume(origin, h, dims, calib, prm)
    upload_grid(vol, S, C, np.array([[0.0, 0.0, 1.0]]), np.array([[1.0, 0.0, 0.0]]))
    a, c = quant.storage(S, C, "fp32")
    for eps in (1e-9, 1e-13, 1.8e-15):
        T = np.eye(4)
        T[:3, 3] = 12.0 + R - eps          # pixel (0, 0): R - eps from the voxel on every axis
        W = H = 3
        p = (1.0, 1.0)
        out = vol.reslice(T, W, H, p).cpu().numpy()
        ref = reslice.reslice(a, c, origin, h, np.array([[0.0, 0.0, 1.0]]), np.array([[1.0, 0.0, 0.0]]), calib, T, W, H, p, prm)
        assert not np.isnan(ref[0, 0])
        assert_parity(out, ref, what=f"R={R} eps={eps}")
