"""Lanes per ray of views whose rays lie more than a voxel apart or cross little: four
from 2^15 pixels on where rays are short, one from 2^18, sixteen below and where rays
are long -- the lanes the plan reports, the bits those of one lane per ray."""
import os
import re

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _context(vr, **env):
    env["VR_DEBUG_PLAN"] = "1"
    os.environ.update(env)
    try:
        return vr.vr_create(0)
    finally:
        for k in env:
            del os.environ[k]


@pytest.mark.parametrize("dims,image,extent,lanes", [
    ((9, 60, 70), (181, 181), 300.0, 16),    # 32761 pixels
    ((9, 60, 70), (182, 181), 300.0, 4),     # 32942
    ((9, 60, 70), (255, 258), 500.0, 4),
    ((3, 3, 3), (512, 511), 20.0, 4),        # 261632
    ((3, 3, 3), (512, 512), 20.0, 1),        # 262144
    ((9, 12, 13), (1003, 1001), 40.0, 1),    # 8 x 8 tiles past the border
    ((100, 90, 95), (200, 180), 230.0, 16),  # rays of 200 samples
    ((40, 35, 400), (130, 500), 500.0, 16),  # a tall frame, mostly empty, long rays
])
@pytest.mark.parametrize("bricks", [None, (40, 31, 33)])
def test_lanes_and_bits(dims, image, extent, lanes, bricks, capfd):
    import torch
    import paper_1008_0135_amd as vr
    a = torch.from_numpy(synth.cube(*dims, seed=8, n_sources=4, sigma_range=(1.5, 4.0))).cuda()
    mask = np.linspace(0.2, 1.0, dims[2], dtype=np.float32)
    auto, plain = _context(vr), _context(vr, VR_MARCH="gather")
    for eye, m, mode, scope in ((0.0, None, 0, 0), (700.0, None, 0, 0), (700.0, mask, 0, 1), (0.0, mask, 1, 0)):
        got = {}
        for c in (auto, plain):
            h = vr.vr_volume_create(c, a, dims)
            if bricks:
                vr.vr_volume_brick(h, vr.grid_spec(bricks))
            vr.vr_tf_set(c, synth.tf_colour(64), float(a.min()), float(a.max()))
            vr.vr_mask_set(c, m)
            out = torch.full((1, image[1], image[0], 4), 7.0, device="cuda")
            views = [vr.make_view(R, *image, eye_dist=eye, extent=extent) for R in synth.random_views(1, 6)]
            capfd.readouterr()
            vr.vr_render(c, h, views, vr.make_params(tau=0.95, mode=mode, ert_scope=scope), out)
            torch.cuda.synchronize()
            said = capfd.readouterr().err
            found = [int(x) for x in re.findall(r"gathers lanes (\d+)", said)]
            # (bricks are chosen for by their rectangles and their own rays: any; rays
            # through all bricks: four at least)
            want = (max(lanes, 4) if scope else found[0]) if bricks and found else lanes
            assert (found == [want] if c is auto else found == []), (eye, mode, scope, said)
            got[c] = out
            vr.vr_volume_destroy(h)
        assert torch.equal(got[auto], got[plain]), (eye, mode, scope)
    for c in (auto, plain):
        vr.vr_destroy(c)
