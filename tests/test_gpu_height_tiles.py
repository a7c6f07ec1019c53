"""The height models' tile kernel at its edges, bit for bit against the oracle:
domains of one granule row less, exactly and one more than 16 task rows, whole
domains and tiles of more granules than wavefronts, words and groups that end
mid-way, starts with a frozen part, every kind of decision and both colour
orders."""
from fractions import Fraction

import pytest

import oracle
from gpu_helpers import need_gpu, say

pytestmark = pytest.mark.gpu

MODES = {"one-bit": (None, False), "heat-bath": (2, False), "metropolis": (2, True)}


def agree(s, o, sweeps):
    for k in sweeps:
        s.sweep(k)
        o.sweep(k)
        assert (s.export() == o.export()).all(), "after %d sweeps" % o.t


# (N, tile rows, sweeps per launch): 16 and 17 row pairs; 128 and 129 columns per
# plane; tiles of 22 granules (row pairs 86 .. 91 x 3 groups and more) and cut ones
SIXV = [(30, 0, 0), (31, 0, 0), (32, 0, 0), (33, 0, 0), (254, 0, 0), (255, 0, 0), (300, 150, 8), (300, 5, 3)]


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("mode", sorted(MODES))
@pytest.mark.parametrize("N,rows,spl", SIXV)
def test_six_vertex_tiles(N, rows, spl, mode, order):
    tl = need_gpu()
    c2, metro = MODES[mode]
    say("six-vertex tiles N=%d rows=%d S=%d %s order=%d" % (N, rows, spl, mode, order))
    w = tl.weights(tl.TL_W_UNIFORM) if c2 is None else tl.weights(tl.TL_W_SIXVERTEX, 4, 1, c2)
    w.rule = tl.TL_METROPOLIS if metro else tl.TL_HEATBATH
    s = tl.Sampler(tl.domain(tl.TL_SIXVERTEX, n=N), w, 90 + N,
                   tl.options(tile_rows=rows, sweeps_per_launch=spl, colour_order=order))
    ratios = oracle.sixv_ratios(1, 1, 1) if c2 is None else oracle.sixv_ratios(2, 1, c2)
    o = oracle.SixVertexOracle(N, oracle.table_from_ratios(ratios, metro), metropolis=metro, seed=90 + N,
                               random_colours=bool(order))
    agree(s, o, (1, 6, 33))


# (a, b, c, tile rows, sweeps per launch): 15, 16, 17 and 33 rows; 24 granules in one tile
LOZ = [(7, 6, 8, 0, 0), (7, 7, 8, 0, 0), (7, 8, 8, 0, 0), (300, 15, 17, 0, 0), (500, 120, 30, 100, 4), (129, 90, 60, 4, 5)]


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("mode", sorted(MODES))
@pytest.mark.parametrize("a,b,c,rows,spl", LOZ)
def test_lozenge_tiles(a, b, c, rows, spl, mode, order):
    tl = need_gpu()
    q, metro = (None, False) if mode == "one-bit" else (Fraction(9, 10), mode == "metropolis")
    say("lozenge tiles %s rows=%d S=%d %s order=%d" % ((a, b, c), rows, spl, mode, order))
    w = tl.weights(tl.TL_W_UNIFORM) if q is None else tl.weights(tl.TL_W_VOLUME, 9, 10)
    w.rule = tl.TL_METROPOLIS if metro else tl.TL_HEATBATH
    s = tl.Sampler(tl.domain(tl.TL_LOZENGE, a=a, b=b, c=c), w, 7,
                   tl.options(tile_rows=rows, sweeps_per_launch=spl, colour_order=order))
    thr = oracle.table_from_ratios(oracle.lozenge_ratios(q if q is not None else 1), metro)
    o = oracle.LozengeOracle(a, b, c, thr, metropolis=metro, seed=7, random_colours=bool(order))
    agree(s, o, (1, 6, 33))
