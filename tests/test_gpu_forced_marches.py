"""VR_MARCH=ring: every view by windows in LDS, whatever the estimates of the
default choice say, in each of its forms (footprint cells staged through
registers, with two or three LDS slots, in blocks, with pixels past a cell's
64th, and 8 x 8 pixel tiles) -- the march that ran as the plan reports it, the
bits those of one lane per ray stepping through its samples."""
import os
import re

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

DIMS = (160, 144, 176)
CELLS = {"ring": ({}, r"cells axis .* reg 1 .*blocks 0x0"),
         "ring2mem": ({"VR_RING_SLOTS": "2", "VR_RING_REG": "0"}, r"cells axis .* nslots 2 reg 0"),
         "ring3": ({"VR_RING_SLOTS": "3"}, r"cells axis .* nslots 3 reg 0"),
         "blk2x2": ({"VR_FOOT_BLOCK": "2x2"}, r"cells axis .*blocks 2x2"),
         "blk1x4": ({"VR_FOOT_BLOCK": "1x4"}, r"cells axis .*blocks 1x4"),
         "ovf": ({"VR_FOOT_RAYS": "64", "VR_FOOT_MAXPX": "4096"}, r"cells axis .* reg 1"),
         "tiles2": ({"VR_FOOT": "0", "VR_RING_SLOTS": "2"}, r"tiles axis .* nslots 2"),
         "tiles3": ({"VR_FOOT": "0", "VR_RING_SLOTS": "3"}, r"tiles axis .* nslots 3")}


def _context(vr, **env):
    env["VR_DEBUG_PLAN"] = "1"
    os.environ.update(env)
    try:
        return vr.vr_create(0)
    finally:
        for k in env:
            del os.environ[k]


def _layouts(vr):
    # bricks of 80 or 81 voxels along axis 1 (room for a block's rows), ragged along the others
    size = (80, 50, 61)
    return {"whole": None, "ragged": vr.grid_spec(size), "mat": vr.grid_spec(size, materialize=True),
            "cells": vr.grid_spec(size, macrocell=8), "narrow": vr.grid_spec((73, 50, 61))}


def _images(vr, ctx, a, layout, image, views, mask, mode, scope, capfd):
    import torch
    h = vr.vr_volume_create(ctx, a, DIMS)
    if layout is not None:
        vr.vr_volume_brick(h, layout)
    tf = synth.tf_noise_suppress(float(a.min()), float(a.max()), thresh=2.0, amax=0.5)
    vr.vr_tf_set(ctx, tf)
    vr.vr_mask_set(ctx, mask)
    out = torch.full((len(views), image[1], image[0], 4), 7.0, device="cuda")
    capfd.readouterr()
    vr.vr_render(ctx, h, [vr.make_view(R, *image, eye_dist=e) for R, e in views],
                 vr.make_params(tau=0.95, mode=mode, ert_scope=scope), out)
    torch.cuda.synchronize()
    said = [line for line in capfd.readouterr().err.splitlines() if line.startswith("[vr]")]
    vr.vr_volume_destroy(h)
    assert float(out.abs().max()) > 0 and not bool((out == 7.0).any())
    return out, said


@pytest.fixture(scope="module")
def cube():
    import torch
    torch.cuda.init()
    return torch.from_numpy(synth.cube(*DIMS, seed=27, n_sources=15, sigma_range=(2.0, 5.0))).cuda()


@pytest.mark.parametrize("march", list(CELLS))
@pytest.mark.parametrize("layout", ["whole", "ragged", "mat", "cells", "narrow"])
@pytest.mark.parametrize("image", [(97, 90), (331, 310)])
def test_parallel_views(march, layout, image, cube, capfd):
    import torch
    import paper_1008_0135_amd as vr
    env, says = CELLS[march]
    if "blk" in march and (layout == "narrow" or (march == "blk2x2" and layout != "whole" and image[0] == 97)):
        says = CELLS["ring"][1]  # bricks narrower than a block's rows: a wavefront per cell
    forced, plain = _context(vr, VR_MARCH="ring", **env), _context(vr, VR_MARCH="gather")
    views = [(R, 0.0) for R in synth.random_views(3, 28)]
    mask = np.random.default_rng(1).uniform(0, 1, DIMS[2]).astype(np.float32)
    spec = _layouts(vr)[layout]
    for m in (None, mask) if march in ("ring", "ring3", "ovf", "tiles3") else (None,):
        for mode, scope in ((0, 0), (1, 0), (0, 1)):
            x, said = _images(vr, forced, cube, spec, image, views, m, mode, scope, capfd)
            y, _ = _images(vr, plain, cube, spec, image, views, m, mode, scope, capfd)
            assert not any("gathers" in line for line in said), said
            assert sum(bool(re.search(says, line)) for line in said) >= (1 if "blk" in march else 2), said
            assert torch.equal(x, y), (mode, scope, m is not None)
    for c in (forced, plain):
        vr.vr_destroy(c)


@pytest.mark.parametrize("layout", ["ragged", "mat", "cells", "narrow"])
@pytest.mark.parametrize("image,eye", [((97, 90), 400.0), ((331, 310), 400.0), ((160, 170), 150.0)])
@pytest.mark.parametrize("past", [False, True])
def test_perspective_views(layout, image, eye, past, cube, capfd):
    import torch
    import paper_1008_0135_amd as vr
    env = CELLS["ovf"][0] if past else {}
    forced, plain = _context(vr, VR_MARCH="ring", **env), _context(vr, VR_MARCH="gather")
    views = [(R, eye) for R in synth.random_views(3, 29)]
    mask = np.random.default_rng(1).uniform(0, 1, DIMS[2]).astype(np.float32)
    spec = _layouts(vr)[layout]
    for m in (None, mask):
        for mode in (0, 1):
            x, said = _images(vr, forced, cube, spec, image, views, m, mode, 0, capfd)
            y, _ = _images(vr, plain, cube, spec, image, views, m, mode, 0, capfd)
            assert sum("cells class" in line for line in said) >= 3, said
            assert torch.equal(x, y), (mode, m is not None)
    for c in (forced, plain):
        vr.vr_destroy(c)
