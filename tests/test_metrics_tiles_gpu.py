"""Image similarity at the edges of its 32 x 16 tiles and with more tiles than workgroups, against
the oracle; 1e-9 absolute on NCC and SSIM (both sides FP64) and exact counts."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_helpers import note
from oracle import metrics

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w,density", [
    (16, 32, 1.0), (17, 33, 1.0), (15, 31, 1.0), (11, 11, 1.0), (10, 40, 1.0), (48, 95, 0.999), (1, 1, 1.0),
    (1030, 545, 0.0),      # 65 x 18 tiles, assigned in a few blocks only
])
def test_tile_edges(h, w, density):
    import torch

    import paper_2605_26325_amd as dare
    note(f"image similarity {h}x{w} density {density}")
    rng = np.random.default_rng(h * 1000 + w)
    frame = rng.integers(0, 256, (h, w), dtype=np.uint8)
    img = (0.7 * frame + rng.normal(0, 20, (h, w))).astype(np.float32)
    if density == 0.0:
        keep = np.zeros((h, w), bool)
        for y, x in ((0, 0), (500, 250), (h - 14, w - 20), (1010, 3)):
            keep[y:y + 14, x:x + 20] = True
        img[~keep] = np.nan
    else:
        img[rng.random((h, w)) > density] = np.inf      # not finite, not NaN either
    got = dare.compare_to_frame(torch.from_numpy(img).cuda(), torch.from_numpy(frame).cuda())
    with np.errstate(invalid="ignore"):
        refs = metrics.ncc(img, frame), metrics.ssim(img, frame)
    assert (got[2], got[3]) == (refs[0][1], refs[1][1])
    for g, r in zip(got, (refs[0][0], refs[1][0])):
        assert np.isnan(g) == np.isnan(r)
        assert np.isnan(r) or abs(g - r) <= 1e-9
