"""Outstanding requests whose device destinations overlap, each in a tick of its own on another stream:
the last request's values stand, bit for bit the requests resliced alone, as for buffers of a
request's own beside them."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_helpers import note
from test_serving_gpu import _alone, env  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("streams,per_tick", [(3, 1), (2, 2)])
def test_overlaps_across_ticks(env, streams, per_tick):  # noqa: F811
    dare, torch, wl, vols = env
    note(f"overlapping device destinations, {streams} streams, {per_tick} requests a tick")
    rng = np.random.default_rng(7)
    W = H = 400
    reqs = [(int(rng.integers(2)), wl.slices.probe_poses[int(rng.integers(len(wl.slices.probe_poses)))], W, H, (0.08, 0.08))
            for _ in range(8)]
    ref = [torch.from_numpy(r.reshape(-1)).cuda().view(torch.int32) for r in _alone(dare, torch, vols, reqs)]
    n = W * H
    srv = dare.Server(64 << 20, n_streams=streams, max_tick_requests=per_tick)
    ids = [srv.add_volume(v) for v in vols]
    buf = torch.full((3 * n,), -5.0, device="cuda")
    own = torch.full((2, n), -5.0, device="cuda")
    # starts of the eight results in `buf`, None: a row of `own`
    starts = [0, n // 2, None, 0, n // 2, 2 * n, None, n // 3]
    ptr, rows = [], iter(range(2))
    for at in starts:
        ptr.append(own[next(rows)].data_ptr() if at is None else buf.data_ptr() + 4 * at)
    arr = dare.spec_array(*[[q[i] for q in reqs] for i in range(1, 5)])
    for rep in range(20):
        order = rng.permutation(len(reqs)) if rep else np.arange(len(reqs))
        buf.fill_(-5.0), own.fill_(-5.0)
        torch.cuda.synchronize()
        tickets, _ = srv.submit_many([ids[reqs[k][0]] for k in order], arr[order], [ptr[k] for k in order])
        assert len(tickets) == len(reqs)
        while len(tickets):
            states, _ = srv.poll_many(tickets, 5.0)
            assert set(states.tolist()) <= {dare.OK, dare.ERR_NOT_READY}
            tickets = tickets[states == dare.ERR_NOT_READY]
        want = torch.full((3 * n,), -5.0, device="cuda").view(torch.int32)
        for k in order:
            if starts[k] is not None:
                want[starts[k]:starts[k] + n] = ref[k]
        assert torch.equal(buf.view(torch.int32), want), rep
        assert torch.equal(own[0].view(torch.int32), ref[2]) and torch.equal(own[1].view(torch.int32), ref[6]), rep
    srv.close()
