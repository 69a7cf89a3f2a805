"""Batched requests with 4 and with 16 lanes per ray: the bits of vr_render."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


# fewer than 512 tiles: 16 lanes for all; more: 4 where rays are less than 1.5
# voxels apart, 16 where they are more; images ragged against tiles and quarters
@pytest.mark.parametrize("shapes", [
    [((20, 31, 17), (9, 7)), ((2, 2, 2), (1, 1)), ((40, 33, 50), (67, 30))],
    [((60, 50, 70), (203, 201)), ((90, 80, 100), (33, 41)), ((2, 3, 4), (1, 3)), ((30, 31, 32), (17, 64))]])
def test_lanes(shapes):
    import torch
    torch.cuda.init()
    import paper_1008_0135_amd as vr
    ctx = vr.vr_create(0)
    tf = synth.tf_colour(64)
    dtf = torch.from_numpy(tf).cuda()
    p = vr.make_params(tau=0.9)
    reqs, want, got, keep = [], [], [], []
    for i, (dims, (W, H)) in enumerate(shapes):
        vol = torch.from_numpy(synth.cube(*dims, seed=i, n_sources=2)).cuda()
        h = vr.vr_volume_wrap(ctx, vol, dims)
        vmin, vmax = float(vol.min()), float(vol.max()) + 1e-3
        vr.vr_tf_set(ctx, tf, vmin, vmax)
        R = synth.random_views(1, i)[0]
        a, b = torch.full((1, H, W, 4), 7.0, device="cuda"), torch.full((H, W, 4), 7.0, device="cuda")
        vr.vr_render(ctx, h, [vr.make_view(R, W, H)], p, a)
        reqs.append(vr.make_request(h, R, W, H, dtf, vmin, vmax, b))
        want.append(a[0])
        got.append(b)
        keep.append((vol, h))
    cache = vr.vr_render_batch(ctx, reqs, p)
    torch.cuda.synchronize()
    for a, b in zip(want, got):
        assert torch.equal(a, b)
    for b in got:
        b.fill_(7.0)
    cache = vr.vr_render_batch(ctx, reqs, p, cache)  # the captured launch again
    torch.cuda.synchronize()
    for a, b in zip(want, got):
        assert torch.equal(a, b)
    vr.vr_batch_destroy(cache)
    for _, h in keep:
        vr.vr_volume_destroy(h)
    vr.vr_destroy(ctx)
