"""Brick ranges taken from the macrocells' and the planes around them: every
brick's (min, max) is that of its stored box, exactly."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# boxes that start on macrocells, between them, and a last macrocell cut short;
# an extreme on a single voxel at the boxes' corners, edges and inside
@pytest.mark.parametrize("dims,size,edge", [((600, 40, 33), (300, 40, 33), 4), ((517, 70, 33), (256, 70, 33), 5),
                                            ((300, 130, 70), (150, 130, 35), 2), ((261, 33, 300), None, 6),
                                            ((2200, 9, 8), (1100, 9, 8), 3)])
@pytest.mark.parametrize("opt", [{}, {"materialize": True}, {"twin": True}])
def test_ranges_of_stored_boxes(dims, size, edge, opt):
    import torch
    import paper_1008_0135_amd as vr
    a = np.random.default_rng(dims[0]).standard_normal(dims[::-1], dtype=np.float32)
    torch.cuda.init()
    ctx = vr.vr_create(0)
    spec = (vr.grid_spec(size, macrocell=edge, **opt) if size else vr.kd_spec(3, macrocell=edge, **opt))
    h = vr.vr_volume_create(ctx, torch.from_numpy(a).cuda(), dims)
    vr.vr_volume_brick(h, spec)
    boxes = [(b.slo[:], b.shi[:]) for b in vr.vr_volume_brick_info(h)]
    vr.vr_volume_destroy(h)
    # minima and maxima of growing size at the first and last voxels of each box
    for k, (slo, shi) in enumerate(boxes):
        a[slo[2], shi[1], slo[0]] = -10.0 - k
        a[shi[2], slo[1], shi[0]] = 10.0 + k
    h = vr.vr_volume_create(ctx, torch.from_numpy(a).cuda(), dims)
    for _ in range(2):  # the second time over the first one's storage
        vr.vr_volume_brick(h, spec)
        for b in vr.vr_volume_brick_info(h):
            part = a[b.slo[2]:b.shi[2] + 1, b.slo[1]:b.shi[1] + 1, b.slo[0]:b.shi[0] + 1]
            assert (b.vmin, b.vmax) == (part.min(), part.max())
    vr.vr_volume_destroy(h)
    vr.vr_destroy(ctx)


# even edges of 24 and more are joined from cells of 12 to 23 voxels: no, one and
# more halvings, a volume smaller than a cell, last cells cut short in the middle of
# a small one; a voxel that is not a number marks every cell that touches it
@pytest.mark.parametrize("dims,edge", [((70, 41, 37), 18), ((200, 66, 65), 32), ((140, 70, 36), 34),
                                       ((97, 100, 33), 40), ((20, 31, 130), 128), ((51, 17, 20), 17)])
@pytest.mark.parametrize("wrapped", [False, True])
def test_large_macrocells(dims, edge, wrapped):
    import torch
    import paper_1008_0135_amd as vr
    a = np.random.default_rng(edge).standard_normal(dims[::-1], dtype=np.float32)
    if wrapped:
        a[tuple(n // 2 for n in a.shape)] = np.nan
    src = torch.from_numpy(a).cuda()
    ctx = vr.vr_create(0)
    h = vr.vr_volume_wrap(ctx, src, dims) if wrapped else vr.vr_volume_create(ctx, src, dims)
    vr.vr_volume_brick(h, vr.grid_spec(dims, macrocell=edge))
    e, cnt, mm = vr.vr_volume_macrocell_info(h)
    assert e == edge and tuple(cnt) == tuple(-(-(n - 1) // edge) for n in dims)
    for m in np.ndindex(cnt[2], cnt[1], cnt[0]):
        part = a[tuple(slice(k * e, min((k + 1) * e, n - 1) + 1) for k, n in zip(m, a.shape))]
        if np.isnan(part).any():
            assert np.isnan(mm[m][0])
        else:
            assert tuple(mm[m]) == (part.min(), part.max())
    vr.vr_volume_destroy(h)
    vr.vr_destroy(ctx)
