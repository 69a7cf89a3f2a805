"""Table gradients of small tables, whose sums a tile keeps in several copies: at each
number of copies (64 down to one, the line between two and one at 128 and 129
entries) against the FP64 oracle, the bound of the other gradient tests; views whose
windows fill the LDS leave no room for copies."""
import numpy as np
import pytest

import synth
from test_gpu_adjoint_tiles import _check, _table, ctx  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [2, 3, 4, 7, 8, 16, 17, 33, 64, 65, 128, 129])
@pytest.mark.parametrize("amax", [0.2, 0.6])
def test_small_tables(ctx, M, amax):  # noqa: F811
    _check(ctx, (24, 20, 28), (33, 30), synth.random_views(2, 9), _table(M, amax))


@pytest.mark.parametrize("M", [2, 40])
def test_wide_windows(ctx, M):  # noqa: F811
    # rays several voxels apart: windows of thousands of floats
    _check(ctx, (150, 130, 140), (34, 30), synth.random_views(2, 9) + [np.eye(3)], _table(M, 0.2), K=4)
