"""The domino register-tile kernel at its edges, bit for bit against the oracle:
orders around the ends of words, groups and tiles, tiles of few and of many
groups (with and without the wavefronts that draw ahead), launches of more tiles
than compute units, where frozen tiles end early, both parities of the order
(which colour steps first), every kind of decision and both colour orders."""
from fractions import Fraction

import numpy as np
import pytest

import oracle
from gpu_helpers import need_gpu, say

pytestmark = pytest.mark.gpu

MODES = {"one-bit": (False, False), "heat-bath": (True, False), "metropolis": (True, True)}


def pair(tl, n, mode, order, rows, groups, spl):
    two, metro = MODES[mode]
    w = tl.weights(tl.TL_W_TWO_PERIODIC, 1.0, 0.5) if two else tl.weights(tl.TL_W_UNIFORM)
    w.rule = tl.TL_METROPOLIS if metro else tl.TL_HEATBATH
    s = tl.Sampler(tl.domain(tl.TL_DOMINO, n=n), w, 60 + n,
                   tl.options(kernel=3, tile_rows=rows, tile_groups=groups, sweeps_per_launch=spl, colour_order=order))
    ratios = oracle.domino_ratios("two", 1, Fraction(1, 2)) if two else oracle.domino_ratios()
    o = oracle.DominoOracle(n, oracle.table_from_ratios(ratios, metro), metropolis=metro, seed=60 + n,
                            random_colours=bool(order))
    return s, o


# (n, tile rows, groups, sweeps per launch): 64 and 65 rows; 127 .. 129 sites a
# row; tiles of 1, 6 and 12 groups; 130 and 400 tiles of which most are frozen
SHAPES = [(64, 64, 1, 4), (65, 32, 1, 16), (127, 62, 1, 1), (128, 40, 2, 6), (129, 24, 1, 20), (257, 33, 4, 3),
          (770, 50, 7, 2), (1300, 60, 10, 1), (1301, 10, 1, 9)]


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("mode", sorted(MODES))
@pytest.mark.parametrize("n,rows,groups,spl", SHAPES)
def test_register_tiles(n, rows, groups, spl, mode, order):
    tl = need_gpu()
    say("domino register tiles n=%d rows=%d groups=%d S=%d %s order=%d" % (n, rows, groups, spl, mode, order))
    s, o = pair(tl, n, mode, order, rows, groups, spl)
    for k in (1, 7, 25):
        s.sweep(k)
        o.sweep(k)
        assert (s.export() == o.export()).all(), "after %d sweeps" % o.t


@pytest.mark.parametrize("mode", sorted(MODES))
def test_frozen_tiles_follow_an_import(mode):
    """A frozen tile leaves words of the other buffer alone only where they
    agree: after an import of another state, both buffers hold the new one."""
    tl = need_gpu()
    n = 1301
    say("domino frozen tiles, import %s" % mode)
    s, o = pair(tl, n, mode, 0, 10, 1, 9)
    first = s.export()
    s.sweep(40)
    s.import_(first, 0)
    for k in (9, 13):
        s.sweep(k)
        o.sweep(k)
        assert np.array_equal(s.export(), o.export()), "after %d sweeps" % o.t
