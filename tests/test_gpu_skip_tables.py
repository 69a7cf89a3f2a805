"""The macrocell-skipping march with tables whose LDS copy, beside the march's own
LDS, passes 64 KB: the images of the same bricks without the skip."""
import pytest

import test_gpu_skip as skip

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("entries", [3100, 3300, 4096])
@pytest.mark.parametrize("scope,tau,masked", [(0, 2.0, False), (1, 0.9, False), (0, 0.9, True)])
def test_large_tables(entries, scope, tau, masked):
    skip.test_bits_of_the_plain_march(entries, (75, 53), scope, tau, masked)
