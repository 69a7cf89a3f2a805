"""Gradients of views whose workgroups take several tiles each (large tables, many
tiles): two and four tiles, a last run cut short, and the sizes on either side of
each line, against the FP64 oracle with the bound of the other gradient tests."""
import pytest

import synth
from test_gpu_adjoint_tiles import _check, _table, ctx  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("image", [(608, 640), (632, 624), (1001, 803)])  # 6080, 6162, 12726 tiles
@pytest.mark.parametrize("M,amax", [(2047, 0.2), (2048, 0.2), (2048, 0.95)])
def test_several_tiles(ctx, image, M, amax):  # noqa: F811
    # (a thin volume: tiles past its border, bands of unequal counts)
    _check(ctx, (6, 3, 7), image, synth.random_views(1, 9), _table(M, amax))
