"""Image similarity: results into pageable and pinned host memory are the same bits and nothing beside
them is written; a call allocates no memory of its own."""
from __future__ import annotations

import ctypes as ct
import os
import re

import numpy as np
import pytest

from gpu_helpers import note

pytestmark = pytest.mark.gpu


def _inputs(torch, W, H):
    g = torch.Generator(device="cuda")
    g.manual_seed(W * 10 + H)
    frame = torch.randint(0, 256, (H, W), generator=g, device="cuda", dtype=torch.uint8)
    img = 0.6 * frame.float() + 80.0 * torch.rand((H, W), generator=g, device="cuda")
    img[: H // 4, : W // 3] = float("nan")
    return img, frame


@pytest.mark.parametrize("W,H", [(64, 48), (512, 300), (9, 40), (1, 1)])
def test_pageable_and_pinned(W, H):
    import torch

    import paper_2605_26325_amd as dare
    note(f"image similarity results, {W}x{H}")
    img, frame = _inputs(torch, W, H)
    ws = torch.empty(int(dare.lib.dare_compare_workspace_bytes()), dtype=torch.uint8, device="cuda")
    s = ct.c_void_p(torch.cuda.current_stream().cuda_stream)
    pageable = np.full(6, -5.0)
    pinned = torch.full((6,), -5.0, dtype=torch.float64, pin_memory=True)
    for p in (pageable.ctypes.data, pinned.data_ptr()):
        st = dare.lib.dare_compare_to_frame(ct.c_void_p(img.data_ptr()), ct.c_void_p(frame.data_ptr()), W, H,
                                            ct.c_void_p(ws.data_ptr()), ws.numel(), ct.cast(p + 8, ct.POINTER(ct.c_double)), s)
        assert st == dare.OK
    assert pageable.tobytes() == pinned.numpy().tobytes()
    assert pageable[0] == pageable[5] == -5.0
    r = dare.compare_to_frame(img, frame)
    assert np.array_equal(np.array(r), pageable[1:5], equal_nan=True)


def test_source_allocates_nothing():
    """The entry point takes its workspace and its result's memory from the caller."""
    src = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_26325_amd", "csrc", "dare_metrics.hip")
    with open(src) as f:
        assert not re.search(r"\bhip(Host)?Malloc|\bnew \w|\bmalloc\(", f.read())


def test_threads_have_results_of_their_own():
    import threading

    import torch

    import paper_2605_26325_amd as dare
    note("image similarity on four threads")
    pairs = [_inputs(torch, 60 + 9 * k, 50) for k in range(4)]
    ref = [dare.compare_to_frame(*p) for p in pairs]
    torch.cuda.synchronize()
    got = [[] for _ in pairs]

    def work(k):
        s = torch.cuda.Stream()
        for _ in range(50):
            got[k].append(dare.compare_to_frame(*pairs[k], stream=s))
    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for k, r in enumerate(ref):
        assert len(got[k]) == 50 and all(np.array_equal(g, r, equal_nan=True) for g in got[k])
