"""Random-order one-bit chains whose automatic tiles change during a call, against
the same chain with one shape throughout (every shape gives the same chain)."""
import numpy as np
import pytest

from gpu_helpers import need_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1537, 1600, 1792])
def test_change_of_shape(n):
    tl = need_gpu()
    say("domino change of tiles n=%d" % n)
    a = tl.Sampler(tl.domain(tl.TL_DOMINO, n=n), tl.weights(tl.TL_W_UNIFORM), 9, tl.options(colour_order=1))
    b = tl.Sampler(tl.domain(tl.TL_DOMINO, n=n), tl.weights(tl.TL_W_UNIFORM), 9,
                   tl.options(colour_order=1, kernel=3, tile_rows=32, tile_groups=2, sweeps_per_launch=8))
    for k in (n - 5, 1, 23, 100):   # the second but one call spans sweep n
        a.sweep(k)
        b.sweep(k)
        assert np.array_equal(a.export(), b.export()), k
