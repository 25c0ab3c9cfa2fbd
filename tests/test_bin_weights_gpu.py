"""Reslices whose Eq. 2 weights lie at the end of FP32's range, against the FP64 oracle, alone and
batched.  The blend depends on the weights' ratios only, so with one surviving bin every weight gives
the stored values.

Tolerance: |d| <= 1e-5 max(|ref|, 1) as for every reslice."""
from __future__ import annotations

import numpy as np
import pytest

import synth
from gpu_helpers import assert_parity, make_volume, note, upload_grid
from helpers import random_grid, rodrigues
from oracle import quant, reslice
from oracle.reslice import Params

pytestmark = pytest.mark.gpu

FORM = {"f32": "fp32", "bf16": "bf16", "f16": "fp16", "fp8": "fp8"}


def _check(dtype, angles_deg, prm, what):
    """Bins turned by `angles_deg` about the slices' lateral axis; fine and coarse pitches."""
    import torch

    import paper_2605_26325_amd as dare
    rng = np.random.default_rng(41)
    dims, h = (21, 17, 19), 0.5
    S, C = random_grid(rng, len(angles_deg), dims, p_empty=0.8)
    calib = synth.make_calibration(16, 0.5)
    origin = np.array([-850.0, 310.0, -1620.0])
    x0, n0 = np.array([1.0, 0.0, 0.0]), np.array([0.0, -1.0, 0.0])
    rn = np.array([rodrigues(x0, np.deg2rad(t)) @ n0 for t in angles_deg])
    rx = np.array([x0] * len(angles_deg))
    vol = make_volume(origin, h, dims, calib, prm, dtype=dtype)
    upload_grid(vol, S, C, rn, rx)
    a, c = quant.storage(S, C, FORM[dtype])
    specs, refs = [], []
    for pv in (0.45, 1.6, 9.0):
        W, H, p = 21, 18, (pv * h, 1.07 * pv * h)
        T = np.eye(4)
        T[:3, 0], T[:3, 2] = x0, n0
        T[:3, 1] = np.cross(n0, x0)
        mid = origin + h * (np.array(dims) - 1) / 2 + rng.normal(0, 1.0, 3) * h
        T[:3, 3] = mid - T[:3, 0] * (W // 2) * p[0] - T[:3, 1] * (H // 2) * p[1]
        P = T @ np.linalg.inv(calib)
        specs.append(dare.make_spec(P, W, H, p))
        refs.append(reslice.reslice(a, c, origin, h, rn, rx, calib, P, W, H, p, prm))
    note(f"bin weights: {what} {dtype} R={prm.radius_vox}")
    alone = [torch.full((s.height, s.width), -3.0, device="cuda") for s in specs]
    for s, o in zip(specs, alone):
        dare.dare_reslice(vol, s, o)
    outs = [torch.full((s.height, s.width), -7.0, device="cuda") for s in specs]
    vols = [vol] * len(specs)
    ws = torch.empty(dare.dare_reslice_batch_workspace_bytes(vols, specs), dtype=torch.uint8, device="cuda")
    dare.dare_reslice_batch(vols, specs, outs, ws)
    torch.cuda.synchronize()
    for k, ref in enumerate(refs):
        assert assert_parity(alone[k].cpu().numpy(), ref, what=f"{what} {k}") > 0
        assert torch.equal(outs[k].view(torch.int32), alone[k].view(torch.int32)), f"{what} {k}: batched differs"


# weights exp(-120.6), which FP32 does not hold, and exp(-100), 26 quanta of its smallest value
@pytest.mark.parametrize("R,dtype", [(2, "f32"), (3, "fp8"), (4, "bf16"), (6, "f16"), (8, "fp8")])
@pytest.mark.parametrize("k,angle", [(2000.0, 20.0), (300.0, 48.19)])
def test_one_bin_at_the_end_of_range(R, dtype, k, angle):
    _check(dtype, [angle], Params(radius_vox=R, k_normal=k, thr_normal_deg=60.0), f"k={k}")
