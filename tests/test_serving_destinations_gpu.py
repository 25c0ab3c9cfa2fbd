"""Where served results go: device buffers (written by the kernels), parts of one buffer, buffers
that overlap in a tick (the later request's values stand), a result that would leave its
allocation's alignment, pinned and pageable host memory, all in one tick; bit for bit the requests
resliced alone, and nothing else written."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_helpers import note
from test_serving_gpu import _alone, _requests, env  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [0, 1])
def test_mixed_destinations_in_one_tick(env, order):  # noqa: F811
    dare, torch, wl, vols = env
    note(f"server destinations, order {order}")
    reqs = _requests(wl, 12, seed=91)
    ref = _alone(dare, torch, vols, reqs)
    n = [W * H for (_, _, W, H, _) in reqs]
    flat = torch.full((sum(n[:4]) + 64,), -5.0, device="cuda")             # 0..3: parts of one buffer
    both = torch.full((max(n[4], n[5]),), -5.0, device="cuda")             # 4, 5: the same memory
    odd = torch.zeros(4 * n[6] + 8, dtype=torch.uint8, device="cuda")      # 6: off the floats' alignment
    pinned = [torch.full((n[k],), -5.0, pin_memory=True) for k in (7, 8)]  # 7, 8
    pageable = torch.full((n[9],), -5.0)                                   # 9
    own = [torch.full((n[k],), -5.0, device="cuda") for k in (10, 11)]     # 10, 11
    at = np.cumsum([0] + n[:4])
    ptr = [flat.data_ptr() + 4 * int(at[k]) for k in range(4)] + [both.data_ptr()] * 2 + [odd.data_ptr() + 2] + \
        [t.data_ptr() for t in pinned] + [pageable.data_ptr()] + [t.data_ptr() for t in own]
    torch.cuda.synchronize()
    srv = dare.Server(64 << 20, n_streams=1, max_tick_requests=16)
    ids = [srv.add_volume(v) for v in vols]
    seq = list(range(12)) if order == 0 else [0, 2, 1, 3, 5, 4, 6, 8, 7, 9, 11, 10]
    arr = dare.spec_array([reqs[k][1] for k in seq], [reqs[k][2] for k in seq], [reqs[k][3] for k in seq],
                          [reqs[k][4] for k in seq])
    tickets, _ = srv.submit_many([ids[reqs[k][0]] for k in seq], arr, [ptr[k] for k in seq])
    assert len(tickets) == 12
    while len(tickets):
        states, _ = srv.poll_many(tickets, 5.0)
        assert set(states.tolist()) <= {dare.OK, dare.ERR_NOT_READY}
        tickets = tickets[states == dare.ERR_NOT_READY]
    srv.close()
    torch.cuda.synchronize()

    def same(t, k):
        assert np.array_equal(np.asarray(t).reshape(-1), ref[k].reshape(-1), equal_nan=True), k
    for k in range(4):
        same(flat[int(at[k]):int(at[k + 1])].cpu(), k)
    assert bool((flat[int(at[4]):] == -5.0).all())
    last = 5 if order == 0 else 4
    same(both[:n[last]].cpu(), last)
    raw = odd.cpu().numpy()
    same(np.frombuffer(raw[2:2 + 4 * n[6]].tobytes(), np.float32), 6)
    assert not raw[:2].any() and not raw[2 + 4 * n[6]:].any()
    same(pinned[0], 7), same(pinned[1], 8), same(pageable, 9)
    same(own[0].cpu(), 10), same(own[1].cpu(), 11)
