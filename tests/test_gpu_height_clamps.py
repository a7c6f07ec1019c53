"""Six-vertex tiles of one group asked for more rows than LDS holds (848, halo
included): the sweeps per launch are cut to what fits, bit for bit against the
oracle."""
import pytest

import oracle
from gpu_helpers import need_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("N,rows,spl", [(254, 100, 200), (255, 64, 1000), (30, 1, 255)])
def test_long_launches_are_clamped(N, rows, spl, order):
    tl = need_gpu()
    say("six-vertex clamped launch N=%d rows=%d S=%d order=%d" % (N, rows, spl, order))
    s = tl.Sampler(tl.domain(tl.TL_SIXVERTEX, n=N), tl.weights(tl.TL_W_SIXVERTEX, 4, 1, 2), 90 + N,
                   tl.options(tile_rows=rows, tile_groups=1, sweeps_per_launch=spl, colour_order=order))
    o = oracle.SixVertexOracle(N, oracle.table_from_ratios(oracle.sixv_ratios(2, 1, 2), False), seed=90 + N,
                               random_colours=bool(order))
    for k in (1, 260):
        s.sweep(k)
        o.sweep(k)
        assert (s.export() == o.export()).all(), "after %d sweeps" % o.t
