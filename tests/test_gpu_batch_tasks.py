"""Batched chains that fill a work-group by themselves, bit for bit against the
oracle: as many tasks as threads, one row more, two passes over the tasks, words
and groups that end mid-way, every kind of decision and both colour orders."""
from fractions import Fraction

import pytest

import oracle
from gpu_helpers import need_gpu, say

pytestmark = pytest.mark.gpu

MODES = {"one-bit": (False, False), "heat-bath": (True, False), "metropolis": (True, True)}


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("mode", sorted(MODES))
def test_chains_alone(mode, order):
    tl = need_gpu()
    from paper_1804_07250_amd.serving import Batch
    two, metro = MODES[mode]
    sizes = [512, 511, 385, 384, 342, 257, 256, 129, 1]
    say("batch of chains alone in a work-group, %s order=%d" % (mode, order))
    w = tl.weights(tl.TL_W_TWO_PERIODIC, 1.0, 0.5) if two else tl.weights(tl.TL_W_UNIFORM)
    w.rule = tl.TL_METROPOLIS if metro else tl.TL_HEATBATH
    thr = oracle.table_from_ratios(oracle.domino_ratios("two", 1, Fraction(1, 2)) if two else oracle.domino_ratios(),
                                   metro)
    b = Batch([tl.domain(tl.TL_DOMINO, n=n) for n in sizes], w, list(range(len(sizes))), tl.options(colour_order=order))
    oras = [oracle.DominoOracle(n, thr, metropolis=metro, seed=i, random_colours=bool(order))
            for i, n in enumerate(sizes)]
    for k in (1, 30):
        b.sweep(k)
        b.sync()
        for i, o in enumerate(oras):
            o.sweep(k)
            assert (b.export(i) == o.export()).all(), "order %d after %d sweeps" % (sizes[i], o.t)
    b.destroy()
