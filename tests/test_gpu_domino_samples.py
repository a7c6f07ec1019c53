"""Samples taken inside the launches of a diamond that is one tile, against the
oracle's counts: the smallest and largest of them, words and groups that end
mid-way, bins of one face and of several, samples rarer than sweeps, calls that
begin and end between two samples, more samples than one launch counts, every
kind of decision and both colour orders."""
from fractions import Fraction

import pytest

import oracle
from gpu_helpers import need_gpu, say

pytestmark = pytest.mark.gpu

MODES = {"one-bit": (False, False), "heat-bath": (True, False), "metropolis": (True, True)}


def check(n, every, bin_, calls, mode="one-bit", order=0, spl=0):
    tl = need_gpu()
    say("domino samples n=%d every=%d bin=%d %s order=%d" % (n, every, bin_, mode, order))
    two, metro = MODES[mode]
    w = tl.weights(tl.TL_W_TWO_PERIODIC, 1.0, 0.5) if two else tl.weights(tl.TL_W_UNIFORM)
    w.rule = tl.TL_METROPOLIS if metro else tl.TL_HEATBATH
    s = tl.Sampler(tl.domain(tl.TL_DOMINO, n=n), w, 40 + n,
                   tl.options(obs_every=every, obs_bin=bin_, colour_order=order, sweeps_per_launch=spl))
    ratios = oracle.domino_ratios("two", 1, Fraction(1, 2)) if two else oracle.domino_ratios()
    o = oracle.DominoOracle(n, oracle.table_from_ratios(ratios, metro), metropolis=metro, seed=40 + n, obs_every=every,
                            bin_=bin_, random_colours=bool(order))
    for k in calls:
        s.sweep(k)
        o.sweep(k)
        obs = s.observables()
        assert obs["samples"] == int(o.samples[0])
        assert (obs["bin_sum"].reshape(-1) == o.bin_sum).all(), "after %d sweeps" % o.t
        assert obs["scalar_sum"] == int(o.scalar_sum[0])
    assert (s.export() == o.export()).all()


@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 64, 65, 127, 128, 129])
@pytest.mark.parametrize("every,bin_", [(1, 1), (3, 7), (2, 300)])
def test_sizes(n, every, bin_):
    check(n, every, bin_, (1, 7, 4, 12))


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("mode", sorted(MODES))
def test_rules_and_orders(mode, order):
    check(50, 2, 1, (5, 20), mode, order)


@pytest.mark.parametrize("every,calls,spl", [(1, (2050,), 0), (2, (2047, 2047), 0), (1, (50,), 7)])
def test_more_than_one_launch(every, calls, spl):
    check(20, every, 1, calls, spl=spl)
