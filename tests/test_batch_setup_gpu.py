"""A few large requests in one batched call, whose setup is shared by several workgroups each: staged
in 32 x 32 and 16 x 16 tiles, gathered per pixel, and with no surviving bin; bit for bit the requests
resliced alone, in FP32 and BF16, twice with the same workspace."""
from __future__ import annotations

import numpy as np
import pytest

import synth
from gpu_helpers import make_volume, note, upload_grid
from oracle.reslice import Params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_large_requests_batched_equal_alone(dtype):
    import torch

    import paper_2605_26325_amd as dare
    note(f"batched setup of large requests, {dtype}")
    wl = synth.config1()
    rng = np.random.default_rng(8)
    K, dims = 3, (40, 36, 44)
    C = (rng.random((K, dims[2], dims[1], dims[0])) < 0.5).astype(np.int64) * rng.integers(1, 9, (K, dims[2], dims[1], dims[0]))
    S = C * rng.integers(0, 256, C.shape)
    vol = make_volume(wl.origin, wl.spacing, dims, wl.calib, Params(), dtype=dtype)
    upload_grid(vol, S, C, np.tile([0.0, -1.0, 0.0], (K, 1)), np.tile([1.0, 0.0, 0.0], (K, 1)))
    mid = wl.origin + wl.spacing * (np.array(dims) - 1) / 2
    specs = []
    for n, (W, H, pv, turn) in enumerate(((600, 517, 0.1, 0), (530, 511, 0.9, 0), (700, 300, 3.0, 0), (513, 600, 0.3, 1))):
        T = np.eye(4)
        T[:3, 0], T[:3, 2] = [1.0, 0.0, 0.0], ([0.0, -1.0, 0.0] if not turn else [0.0, 1.0, 0.0])
        T[:3, 1] = np.cross(T[:3, 2], T[:3, 0])
        p = pv * wl.spacing
        T[:3, 3] = mid + 0.13 * (n + 1) - T[:3, 0] * (W // 2) * p - T[:3, 1] * (H // 2) * p
        specs.append(dare.make_spec(T @ np.linalg.inv(wl.calib), W, H, (p, p)))
    alone = []
    for s in specs:
        o = torch.full((s.height, s.width), -3.0, device="cuda")
        dare.dare_reslice(vol, s, o)
        alone.append(o)
    torch.cuda.synchronize()
    assert [bool((~torch.isnan(o)).any()) for o in alone] == [True, True, True, False]
    vols = [vol] * len(specs)
    ws = torch.empty(dare.dare_reslice_batch_workspace_bytes(vols, specs), dtype=torch.uint8, device="cuda")
    for _ in range(2):
        outs = [torch.full((s.height, s.width), -7.0, device="cuda") for s in specs]
        dare.dare_reslice_batch(vols, specs, outs, ws)
        torch.cuda.synchronize()
        for k, (o, x) in enumerate(zip(outs, alone)):
            assert torch.equal(o.view(torch.int32), x.view(torch.int32)), k
