"""Radius-1 batches of requests too coarse to stage (per-pixel tiles near the grid and away from it, more
than one setup workgroup's 256 of them), mixed with fine requests and requests with no surviving bin:
every pixel written, bit for bit the requests resliced alone; calls of different sizes in a row on one
workspace."""
from __future__ import annotations

import numpy as np
import pytest

import synth
from gpu_helpers import make_volume, note, upload_grid
from helpers import random_grid, random_unit, rodrigues
from oracle.reslice import Params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16", "fp8"])
def test_coarse_mixes(dtype):
    import torch

    import paper_2605_26325_amd as dare
    rng = np.random.default_rng(17)
    dims, h, K = (45, 38, 41), 0.5, 4
    S, C = random_grid(rng, K, dims, p_empty=0.5)
    calib = synth.make_calibration(16, 0.5)
    origin = np.array([-850.0, 310.0, -1620.0])
    n0, x0 = np.array([0.0, -1.0, 0.0]), np.array([1.0, 0.0, 0.0])
    turns = [rodrigues(random_unit(rng), np.deg2rad(rng.uniform(0, 6))) for _ in range(K)]
    vol = make_volume(origin, h, dims, calib, Params(), dtype=dtype)
    upload_grid(vol, S, C, np.array([t @ n0 for t in turns]), np.array([t @ x0 for t in turns]))

    def spec(W, H, pv, angle=0.1, shift=0.0):
        T, p = np.eye(4), (pv * h, 1.1 * pv * h)
        turn = rodrigues(np.array([0.0, 0.0, 1.0]), angle)
        T[:3, 0], T[:3, 2] = turn @ x0, turn @ n0
        T[:3, 1] = np.cross(T[:3, 2], T[:3, 0])
        mid = origin + h * (np.array(dims) - 1) / 2 + rng.normal(0, 2.0, 3) * h + shift
        T[:3, 3] = mid - T[:3, 0] * (W // 2) * p[0] - T[:3, 1] * (H // 2) * p[1]
        return dare.make_spec(T @ np.linalg.inv(calib), W, H, p)
    gated = 1.2                                       # beyond both gates of every bin
    calls = [[spec(333, 300, 2.6), spec(64, 50, 0.5), spec(90, 70, 1.0, angle=gated), spec(17, 400, 9.0), spec(301, 299, 30.0),
              spec(200, 200, 6.0), spec(40, 40, 6.0, shift=500.0), spec(1, 1, 4.0), spec(600, 500, 4.0)],
             [spec(33, 31, 3.0), spec(400, 90, 2.2, angle=gated)],
             [spec(260, 270, 3.3) for _ in range(7)] + [spec(70, 300, 0.6)],
             [spec(2000, 1500, 2.4)], [spec(4200, 4100, 3.0)]]   # 1469 and 8449 tiles for each workgroup
    ws = torch.empty(max(dare.dare_reslice_batch_workspace_bytes([vol] * len(c), c) for c in calls), dtype=torch.uint8,
                     device="cuda")
    seen = 0
    for rep in range(2):
        for n, specs in enumerate(calls):
            note(f"coarse batch {dtype} call {n}")
            alone = [torch.full((s.height, s.width), -3.0, device="cuda") for s in specs]
            for s, o in zip(specs, alone):
                dare.dare_reslice(vol, s, o)
            outs = [torch.full((s.height, s.width), -7.0, device="cuda") for s in specs]
            dare.dare_reslice_batch([vol] * len(specs), specs, outs, ws)
            torch.cuda.synchronize()
            for k, (a, b) in enumerate(zip(alone, outs)):
                assert not bool((a == -3.0).any()) and not bool((b == -7.0).any()), (n, k)
                assert torch.equal(a.view(torch.int32), b.view(torch.int32)), (n, k)
                seen += int(torch.isfinite(b).sum())
    assert seen > 5000
