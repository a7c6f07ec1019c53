"""Served height-model jobs with ticks as long as their tiles allow, under both
colour orders: tiles with tall halos, which ask for nearly all of a compute
unit's LDS, beside small domains, bit for bit against the oracle."""
from fractions import Fraction

import pytest

import oracle
from gpu_helpers import need_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("quantum,sweeps", [(64, 70), (30, 61)])
def test_long_ticks(quantum, sweeps, order):
    tl = need_gpu()
    from paper_1804_07250_amd.serving import Server
    say("served ticks of %d sweeps, colour order %d" % (quantum, order))
    sv = Server(256 << 20, 8, tl.options(sweeps_per_launch=quantum, colour_order=order))
    jobs = []
    for i, (N, c, metro) in enumerate([(300, None, False), (400, 2, True), (502, None, False), (40, 2, False)]):
        w = tl.weights(tl.TL_W_UNIFORM) if c is None else tl.weights(tl.TL_W_SIXVERTEX, 1, 1, c)
        w.rule = tl.TL_METROPOLIS if metro else tl.TL_HEATBATH
        o = oracle.SixVertexOracle(N, oracle.table_from_ratios(oracle.sixv_ratios(1, 1, c or 1), metro),
                                   metropolis=metro, seed=70 + i, random_colours=bool(order))
        jobs.append((sv.submit(tl.domain(tl.TL_SIXVERTEX, n=N), w, 70 + i, sweeps), o, N))
    w = tl.weights(tl.TL_W_VOLUME, 9, 10)
    o = oracle.LozengeOracle(60, 300, 90, oracle.table_from_ratios(oracle.lozenge_ratios(Fraction(9, 10)), False),
                             seed=80, random_colours=bool(order))
    jobs.append((sv.submit(tl.domain(tl.TL_LOZENGE, a=60, b=300, c=90), w, 80, sweeps), o, "hexagon"))
    for ticket, o, name in jobs:
        r = sv.wait(ticket, 120.0)
        assert r["status"] == tl.TL_OK and r["sweeps"] == sweeps, name
        o.sweep(sweeps)
        assert r["hash"] == oracle.canonical_hash(o.export()), name
    sv.destroy()
