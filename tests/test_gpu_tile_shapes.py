"""Explicit tile shapes: one lane per ray, tiles of 4, 8 or 16 pixels dealt in
contiguous eighths -- views of fewer blocks than XCDs, of a ragged last eighth and
of many, whole and bricked, both ways of compositing, masked and unmasked, give the
bits of four and sixteen lanes per ray (the default choice)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H", [(1, 1), (5, 3), (33, 17), (70, 29), (161, 97)])
@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("masked", [False, True])
def test_same_bits_as_the_default(W, H, mode, masked):
    import torch
    import paper_1008_0135_amd as vr

    dims = (37, 24, 31)
    a = torch.from_numpy(synth.cube(*dims, seed=5, n_sources=4, sigma_range=(1.5, 4.0))).cuda()
    ctx = vr.vr_create(0)
    vr.vr_tf_set(ctx, synth.tf_colour(64), float(a.min()), float(a.max()))
    mask = np.linspace(0.2, 1.0, dims[2], dtype=np.float32) if masked else None
    vr.vr_mask_set(ctx, mask)
    for bricks in (None, (13, 9, 31)):
        h = vr.vr_volume_create(ctx, a, dims)
        if bricks:
            vr.vr_volume_brick(h, vr.grid_spec(bricks))
        for eye in (0.0, 60.0):
            views = [vr.make_view(R, W, H, eye_dist=eye) for R in synth.random_views(2, 3)]
            out = {}
            for tile in (0, 4, 8, 16):
                img = torch.full((2, H, W, 4), 7.0, device="cuda")
                p = vr.make_params(step=0.5, tau=0.95, mode=mode, tile=tile)
                vr.vr_render(ctx, h, views, p, img)
                torch.cuda.synchronize()
                out[tile] = img
            for tile in (4, 8, 16):
                assert torch.equal(out[0], out[tile]), (bricks, eye, tile)
        vr.vr_volume_destroy(h)
    vr.vr_destroy(ctx)
