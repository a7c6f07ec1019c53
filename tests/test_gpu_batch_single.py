"""Batched chains alone in a batch, around the sizes where a chain begins to
list its movable tasks (more tasks than threads, or than 512), for each
work-group size, bit for bit against the oracle."""
from fractions import Fraction

import pytest

import oracle
from gpu_helpers import need_gpu, say

pytestmark = pytest.mark.gpu

MODES = {"one-bit": (False, False), "heat-bath": (True, False), "metropolis": (True, True)}


# order -> tasks: 64 -> 64, 65 -> 65, 128 -> 128, 129 -> 258, 256 -> 512,
# 257 -> 771, 341 -> 1023, 342 -> 1026
@pytest.mark.parametrize("threads", [64, 256, 512, 1024])
@pytest.mark.parametrize("mode", sorted(MODES))
def test_single_chains(mode, threads):
    tl = need_gpu()
    from paper_1804_07250_amd.serving import Batch
    two, metro = MODES[mode]
    w = tl.weights(tl.TL_W_TWO_PERIODIC, 1.0, 0.5) if two else tl.weights(tl.TL_W_UNIFORM)
    w.rule = tl.TL_METROPOLIS if metro else tl.TL_HEATBATH
    thr = oracle.table_from_ratios(oracle.domino_ratios("two", 1, Fraction(1, 2)) if two else oracle.domino_ratios(),
                                   metro)
    for i, n in enumerate((64, 65, 128, 129, 256, 257, 341, 342)):
        order = i % 2
        say("batch of one chain, order %d, %d threads, %s, colour order %d" % (n, threads, mode, order))
        b = Batch([tl.domain(tl.TL_DOMINO, n=n)], w, [50 + i], tl.options(colour_order=order, tile_rows=threads))
        o = oracle.DominoOracle(n, thr, metropolis=metro, seed=50 + i, random_colours=bool(order))
        for k in (1, 30):
            b.sweep(k)
            o.sweep(k)
        assert (b.export(0) == o.export()).all(), n
        b.destroy()
