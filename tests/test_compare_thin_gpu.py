"""Image similarity of images too narrow or too flat for a window, and of the smallest that hold one,
against the oracle; 1e-9 absolute on NCC (both sides FP64), exact counts."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_helpers import note
from oracle import metrics

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w", [(1, 5000), (5000, 1), (10, 700), (700, 10), (11, 700), (700, 11), (2, 1), (10, 10), (3, 300000)])
def test_thin_images(h, w):
    import torch

    import paper_2605_26325_amd as dare
    note(f"image similarity, thin {h}x{w}")
    rng = np.random.default_rng(h * 7 + w)
    frame = rng.integers(0, 256, (h, w), dtype=np.uint8)
    img = (0.7 * frame + rng.normal(0, 20, (h, w))).astype(np.float32)
    img[rng.random((h, w)) < 0.1] = np.nan
    img[0, 0] = np.inf if w > 1 else img[0, 0]
    got = dare.compare_to_frame(torch.from_numpy(img).cuda(), torch.from_numpy(frame).cuda())
    with np.errstate(invalid="ignore"):
        refs = metrics.ncc(img, frame), metrics.ssim(img, frame)
    assert (got[2], got[3]) == (refs[0][1], refs[1][1])
    for g, r in zip(got, (refs[0][0], refs[1][0])):
        assert np.isnan(g) == np.isnan(r)
        assert np.isnan(r) or abs(g - r) <= 1e-9
