"""Gather marches with several lanes per ray, macrocells passed over ray by ray
and rays taken through all bricks in one launch: the same bits as one lane per
ray stepping through its samples (the march VR_MARCH=gather selects)."""
import os

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _contexts():
    import torch
    torch.cuda.init()
    import paper_1008_0135_amd as vr
    os.environ["VR_MARCH"] = "gather"
    try:
        plain = vr.vr_create(0)
    finally:
        del os.environ["VR_MARCH"]
    return vr, vr.vr_create(0), plain


def _both(dims, image, spec, views, tf, mask=None, seed=5, shows=True, **par):
    """Images of the default context and of the one-lane-per-ray context."""
    import torch
    vr, auto, plain = _contexts()
    a = torch.from_numpy(synth.cube(*dims, seed=seed, n_sources=4)).cuda()
    out = []
    for ctx in (auto, plain):
        h = vr.vr_volume_create(ctx, a, dims)
        if spec is not None:
            vr.vr_volume_brick(h, spec(vr))
        vmin, vmax = vr.vr_volume_minmax(h)
        vr.vr_tf_set(ctx, tf(vmin, vmax))
        if mask is not None:
            vr.vr_mask_set(ctx, mask)
        o = torch.full((len(views), image[1], image[0], 4), 7.0, device="cuda")
        vr.vr_render(ctx, h, [vr.make_view(R, *image, eye_dist=e) for R, e in views], vr.make_params(**par), o)
        torch.cuda.synchronize()
        out.append(o)
        vr.vr_volume_destroy(h)
        vr.vr_destroy(ctx)
    assert not bool((out[0] == 7.0).any())  # every pixel written
    assert not shows or float(out[0].abs().max()) > 0.0
    return out


def _views(n, eye=0.0, seed=3):
    return [(R, eye) for R in synth.random_views(n, seed)]


def _opaque(vmin, vmax):
    # high opacity: rays stop after a few samples, anywhere in a group of lanes
    t = np.linspace(0, 1, 64)
    return np.stack([t, 1 - t, 0 * t + 0.3, 0.3 * t], axis=1).astype(np.float32)


def _ramp(vmin, vmax):
    return synth.tf_ramp(256)


# images below and past a tile, one pixel wide; rays of 0 to a few groups of 16 samples
@pytest.mark.parametrize("dims,image", [((2, 2, 2), (5, 3)), ((9, 31, 17), (33, 1)), ((40, 23, 65), (64, 66))])
@pytest.mark.parametrize("brick", [None, 8, 100])
@pytest.mark.parametrize("eye", [0.0, 200.0])
def test_lanes_per_ray(dims, image, brick, eye):
    import torch
    spec = None if brick is None else (lambda vr: vr.grid_spec((brick,) * 3))
    views = _views(2, eye) + [(np.eye(3), eye)]
    for tf, mode, tau in ((_ramp, 0, 0.99), (_opaque, 0, 0.9), (_ramp, 1, 0.99)):
        x, y = _both(dims, image, spec, views, tf, mode=mode, tau=tau)
        assert torch.equal(x, y)
    mask = np.linspace(0, 1, dims[2]).astype(np.float32)
    for mode in (0, 1):
        x, y = _both(dims, image, spec, views, _ramp, mask=mask, mode=mode)
        assert torch.equal(x, y)


# below kThruBelow: one launch through all bricks; above: launches per front of
# bricks, 4 lanes per ray (masked; rays 0.8 voxels apart) or 16 (2.5 voxels)
@pytest.mark.parametrize("dims,image,edge,masked", [((50, 41, 62), (70, 45), 16, False),
                                                    ((50, 41, 62), (70, 45), 16, True),
                                                    ((300, 300, 300), (640, 640), 64, True),
                                                    ((500, 500, 500), (340, 340), 50, False)])
@pytest.mark.parametrize("eye", [0.0, 1000.0])
def test_whole_ray_termination(dims, image, edge, masked, eye):
    import torch
    mask = np.linspace(1, 0.2, dims[2]).astype(np.float32) if masked else None
    for views in (_views(1, eye), _views(3, eye)):
        x, y = _both(dims, image, lambda vr: vr.grid_spec((edge,) * 3), views, _opaque, mask=mask, ert_scope=1, tau=0.95)
        assert torch.equal(x, y)


# macrocells below, at and above the 16 samples of a block; rays of more than
# 1024 samples (the walk's chunk); the table opaque nearly nowhere, half and everywhere
@pytest.mark.parametrize("dims,image,spec", [
    ((60, 45, 83), (50, 61), lambda vr, e: vr.grid_spec((100, 100, 100), macrocell=e)),
    ((60, 45, 83), (50, 61), lambda vr, e: vr.kd_spec(7, macrocell=e)),
    ((30, 20, 900), (40, 300), lambda vr, e: vr.grid_spec((64, 64, 900), macrocell=e))])
@pytest.mark.parametrize("edge", [2, 8, 16, 50])
@pytest.mark.parametrize("scope", [0, 1])
def test_macrocells_passed_over(dims, image, spec, edge, scope):
    import torch
    for thresh in (2.0, 5.0, 12.0):
        def tf(vmin, vmax):
            return synth.tf_noise_suppress(vmin, vmax, thresh=thresh, amax=0.6)
        for eye in (0.0, 1500.0):
            for mask in (None, np.linspace(0.3, 1, dims[2]).astype(np.float32)):
                # above 12 there may be nothing, or nothing that a ray meets
                x, y = _both(dims, image, lambda vr: spec(vr, edge), _views(2, eye), tf, mask=mask, ert_scope=scope,
                             tau=0.9, shows=thresh == 2.0)
                assert torch.equal(x, y)
