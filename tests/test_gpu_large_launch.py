"""Calls whose launches pass 2^32 lanes along one dimension of the grid (several
lanes share a ray, one workgroup takes an item, one workgroup two planes of a
brick): they are rendered, batched and bricked like any other."""
import os

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _march(vr, mode):
    os.environ["VR_MARCH"] = mode
    try:
        return vr.vr_create(0)
    finally:
        del os.environ["VR_MARCH"]


@pytest.mark.parametrize("save", [False, True])
def test_march(save):
    # 16 lanes per ray of the largest image, rays 1.2 voxels apart
    import torch
    torch.cuda.init()
    import paper_1008_0135_amd as vr
    W = H = 16384
    dims = (40, 30, 50)
    a = torch.from_numpy(synth.cube(*dims, seed=5, n_sources=4)).cuda()
    outs = []
    for ctx in (vr.vr_create(0), _march(vr, "gather")):
        h = vr.vr_volume_create(ctx, a, dims)
        vr.vr_tf_set(ctx, synth.tf_ramp(64))
        out = torch.full((1, H, W, 4), 7.0, device="cuda")
        st = vr.vr_render(ctx, h, [vr.make_view(synth.rot_axis(2, 30.0), W, H, extent=20000.0)],
                          vr.make_params(ckpt_K=64), out, save=save and not outs)
        torch.cuda.synchronize()
        if st:
            vr.vr_state_destroy(st)
        outs.append(out)
        vr.vr_volume_destroy(h)
        vr.vr_destroy(ctx)
    assert float(outs[0].abs().max()) > 0
    assert torch.equal(*outs)


def test_batch():
    # a request of the largest image, 16 lanes per ray: four items a tile
    import torch
    torch.cuda.init()
    import paper_1008_0135_amd as vr
    W = H = 16384
    dims = (26000, 3, 4)
    ctx = vr.vr_create(0)
    a = torch.rand(dims[::-1], generator=torch.Generator("cuda").manual_seed(2), device="cuda")
    h = vr.vr_volume_create(ctx, a, dims)
    tf = synth.tf_ramp(64)
    vr.vr_tf_set(ctx, tf)
    t = torch.from_numpy(tf).cuda()
    R = synth.rot_axis(1, 20.0)
    batch = torch.full((H, W, 4), 7.0, device="cuda")
    plain = torch.full((1, H, W, 4), 7.0, device="cuda")
    cache = vr.vr_render_batch(ctx, [vr.make_request(h, R, W, H, t, 0.0, 0.0, batch)], vr.make_params())
    torch.cuda.synchronize()
    vr.vr_batch_destroy(cache)
    g = _march(vr, "gather")
    h2 = vr.vr_volume_create(g, a, dims)
    vr.vr_tf_set(g, tf)
    vr.vr_render(g, h2, [vr.make_view(R, W, H)], vr.make_params(), plain)
    torch.cuda.synchronize()
    assert float(batch.abs().max()) > 0
    assert torch.equal(batch, plain[0])
    for c, v in ((ctx, h), (g, h2)):
        vr.vr_volume_destroy(v)
        vr.vr_destroy(c)


def test_brick_ranges():
    # 65536 bricks of 600 planes
    import torch
    torch.cuda.init()
    import paper_1008_0135_amd as vr
    ctx = vr.vr_create(0)
    dims = (1025, 1025, 601)
    a = torch.rand(dims[::-1], generator=torch.Generator("cuda").manual_seed(2), device="cuda")
    h = vr.vr_volume_create(ctx, a, dims)
    vr.vr_volume_brick(h, vr.grid_spec((4, 4, 600)))
    d = vr.vr_volume_brick_info(h)
    assert len(d) == 65536
    for i in (0, 255, 256, 40000, 65535):
        lo, hi = list(d[i].slo), list(d[i].shi)
        box = a[lo[2]:hi[2] + 1, lo[1]:hi[1] + 1, lo[0]:hi[0] + 1]
        assert (d[i].vmin, d[i].vmax) == (float(box.min()), float(box.max()))
    vr.vr_volume_destroy(h)
    vr.vr_destroy(ctx)
