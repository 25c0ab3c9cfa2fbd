"""Served reslices at radii above 1: fine and coarse outputs in one tick (tiles staged whole and in
pieces, which take several workgroups each), into device and host memory, then a second tick of
another size on the same stream, through captured graphs and without; bit for bit the requests
resliced alone."""
from __future__ import annotations

import numpy as np
import pytest

import synth
from gpu_helpers import make_volume, note, upload_grid
from helpers import random_grid, random_unit, rodrigues
from oracle.reslice import Params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,dtype,graphs", [(2, "f32", True), (3, "fp8", True), (6, "bf16", True), (8, "f16", False)])
def test_fine_and_coarse_in_one_tick(R, dtype, graphs):
    import torch

    import paper_2605_26325_amd as dare
    rng = np.random.default_rng(60 + R)
    dims, h, K = (40, 33, 37), 0.5, 5
    S, C = random_grid(rng, K, dims, p_empty=0.5)
    calib = synth.make_calibration(16, 0.5)
    origin = np.array([-850.0, 310.0, -1620.0])
    n0, x0 = np.array([0.0, -1.0, 0.0]), np.array([1.0, 0.0, 0.0])
    turns = [rodrigues(random_unit(rng), np.deg2rad(rng.uniform(0, 8))) for _ in range(K)]
    vol = make_volume(origin, h, dims, calib, Params(radius_vox=R), dtype=dtype)
    upload_grid(vol, S, C, np.array([t @ n0 for t in turns]), np.array([t @ x0 for t in turns]))

    def request(W, H, pv):
        T, p = np.eye(4), (pv * h, 1.1 * pv * h)
        turn = rodrigues(random_unit(rng), np.deg2rad(rng.uniform(0, 12)))
        T[:3, 0], T[:3, 2] = turn @ x0, turn @ n0
        T[:3, 1] = np.cross(T[:3, 2], T[:3, 0])
        mid = origin + h * (np.array(dims) - 1) / 2 + rng.normal(0, 3.0, 3) * h
        T[:3, 3] = mid - T[:3, 0] * (W // 2) * p[0] - T[:3, 1] * (H // 2) * p[1]
        return T @ np.linalg.inv(calib), W, H, p
    ticks = [[request(W, H, pv) for W, H, pv in t] for t in (
        [(90, 70, 0.5), (33, 130, 12.0), (64, 64, 0.9), (5, 3, 20.0), (200, 180, 2.5)],
        [(40, 40, 16.0), (31, 17, 0.6)],
        [(130, 90, 0.4), (17, 100, 0.7), (250, 240, 14.0)])]
    srv = dare.Server(64 << 20, n_streams=1, max_tick_requests=8, use_graphs=1 if graphs else 0)
    vid = srv.add_volume(vol)
    for k, reqs in enumerate(ticks):
        note(f"served R={R} {dtype} tick {k}")
        ref = [vol.reslice(*q).cpu() for q in reqs]
        outs = [torch.full((q[2], q[1]), -5.0, device="cuda") if i % 3 != 1 else
                torch.full((q[2], q[1]), -5.0, pin_memory=True) for i, q in enumerate(reqs)]
        torch.cuda.synchronize()
        arr = dare.spec_array(*[[q[i] for q in reqs] for i in range(4)])
        tickets, _ = srv.submit_many([vid] * len(reqs), arr, [o.data_ptr() for o in outs])
        assert len(tickets) == len(reqs)
        while len(tickets):
            states, _ = srv.poll_many(tickets, 5.0)
            assert set(states.tolist()) <= {dare.OK, dare.ERR_NOT_READY}
            tickets = tickets[states == dare.ERR_NOT_READY]
        for i, (o, r) in enumerate(zip(outs, ref)):
            assert torch.isfinite(r).any(), (k, i)
            assert torch.equal(o.cpu().view(torch.int32), r.view(torch.int32)), (k, i)
    srv.close()
