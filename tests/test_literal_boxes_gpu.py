"""Per-sample reslices at the edges of a tile's voxel box (taken from its corner pixels) against
`oracle.literal`, 1e-5 relative: ragged tiles, planes partly and wholly outside the grid, pitches
at which tiles stage and at which they sum per pixel, both readings."""
from __future__ import annotations

import pytest

from gpu_helpers import assert_parity, lib_params, note
from oracle import literal
from oracle.reslice import Params
from test_literal_gpu import _scene, _slice, _store

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H,pv,R,shift", [(21, 18, 0.2, 1, 0.0), (33, 17, 0.5, 2, 2.0), (18, 16, 1.5, 3, 0.0), (19, 17, 1.2, 2, 0.0),
                                            (17, 19, 6.0, 1, 1.0), (16, 16, 0.4, 1, 40.0)])
def test_boxes_vs_oracle(W, H, pv, R, shift):
    import torch

    import paper_2605_26325_amd as dare
    rng, origin, h, dims, calib, poses, frames, pitch, n0, x0, centre = _scene(77)
    note(f"per-sample store, {W}x{H} at {pv} voxels, R {R}, shifted {shift}")
    st = _store(dare, torch, origin, h, dims, calib, poses, frames, pitch)
    ref_store = literal.SampleStore(origin, h, dims, normal_axis=2)
    ref_store.add_frames(frames, poses.astype("float64"), calib, pitch)
    sp = (pv * h, 0.93 * pv * h)
    P = _slice(rng, calib, n0, x0, centre + shift, W, H, sp)
    prm = Params(radius_vox=R)
    for mode, spatial, norm in (("box", "box", "sample"), ("tent", "tent", "two_stage")):
        got = st.reslice(P, W, H, sp, lib_params(prm), mode).cpu().numpy()
        ref = literal.reslice(ref_store, calib, P, W, H, sp, prm, spatial=spatial, norm=norm)
        n = assert_parity(got, ref, what=mode)
        assert (n > 0) == (shift < 10.0)
