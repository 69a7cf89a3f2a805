"""The march that skips macrocells ray by ray, with small and with large tables
(one and four wavefronts per workgroup): the images of the same bricks without
the skip, bit for bit."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


# tables at both sides of the line; images of a few rays, of one tile and with
# ragged last tiles; early termination off, within a ray's brick, over the ray
@pytest.mark.parametrize("entries", [16, 1024, 1025])
@pytest.mark.parametrize("image", [(3, 2), (8, 8), (75, 53)])
@pytest.mark.parametrize("scope,tau", [(0, 2.0), (0, 0.9), (1, 0.9)])
@pytest.mark.parametrize("masked", [False, True])
def test_bits_of_the_plain_march(entries, image, scope, tau, masked):
    import torch
    import paper_1008_0135_amd as vr
    dims = (70, 90, 55)
    rng = np.random.default_rng(5)
    a = rng.uniform(0.0, 0.4, dims[::-1]).astype(np.float32)
    for x, y, z, r in ((20, 30, 20, 9), (41, 60, 40, 12), (60, 20, 11, 3)):
        a[z - r // 2:z + r // 2 + 1, y - r:y + r, x - r:x + r] += rng.uniform(0.0, 0.6, (2 * (r // 2) + 1, 2 * r, 2 * r))
    a[0, 0, 0], a[-1, -1, -1] = 0.0, 1.0
    tf = rng.uniform(0.0, 1.0, (entries, 4)).astype(np.float32)
    tf[:, 3] = np.where(np.arange(entries) < 0.5 * entries, 0.0, 0.3 * tf[:, 3])
    torch.cuda.init()
    ctx = vr.vr_create(0)
    views = [vr.make_view(synth.rot_axis(2, 40.0) @ synth.rot_axis(3, 25.0), *image),
             vr.make_view(synth.rot_axis(1, 70.0), *image)]
    h = vr.vr_volume_create(ctx, torch.from_numpy(a).cuda(), dims)
    vr.vr_volume_brick(h, vr.grid_spec((40, 40, 40), macrocell=4))
    vr.vr_tf_set(ctx, tf, 0.0, 1.0)
    if masked:
        vr.vr_mask_set(ctx, rng.permutation(np.linspace(0.0, 1.0, dims[2], dtype=np.float32)))
    for n in (1, 2):
        on, off = (torch.full((n, image[1], image[0], 4), -7.0, device="cuda") for _ in range(2))
        vr.vr_render(ctx, h, views[:n], vr.make_params(tau=tau, ert_scope=scope, ess=1), on)
        vr.vr_render(ctx, h, views[:n], vr.make_params(tau=tau, ert_scope=scope, ess=0), off)
        torch.cuda.synchronize()
        assert torch.equal(on, off)
        assert image == (3, 2) or on.abs().sum() > 0
    vr.vr_volume_destroy(h)
    vr.vr_destroy(ctx)
