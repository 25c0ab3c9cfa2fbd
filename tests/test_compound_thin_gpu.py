"""Compounding of thin and small frames, whose patches are not 4 x 4 blocks of 8 x 8 pixels, bit for
bit against the oracle.  Whole numbers: no tolerance."""
from __future__ import annotations

import pytest

from test_compound_patches_gpu import test_compound_patch_edges as _against_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,pv,dims,frames", [
    (1, 1100, 0.06, (24, 20, 70), 9), (1100, 1, 0.06, (70, 20, 24), 9), (2, 300, 0.3, (24, 24, 90), 7), (130, 3, 0.5, (66, 24, 20), 9),
    (4, 65, 1.0, (20, 20, 66), 11), (17, 9, 0.7, (30, 24, 24), 8), (33, 33, 1.0, (40, 40, 40), 9), (200, 33, 0.4, (90, 30, 30), 5),
    (7, 6, 6.0, (64, 48, 64), 5),
    (20, 20, 5.0, (112, 64, 112), 20),                 # the set of a patch's entries two thirds full
])
def test_thin_frames(w, h, pv, dims, frames):
    _against_oracle(w, h, pv, dims, frames, 5.0, 5.0)
