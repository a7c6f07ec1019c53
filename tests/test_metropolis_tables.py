"""Lazy Metropolis thresholds: of a weight ratio's two, current state down and up,
one is always 2^31 (the six-vertex tile kernels compare the other one alone)."""
import itertools

import pytest

import paper_1804_07250_amd as tl

HALF = 1 << 31


@pytest.mark.parametrize("free_side", [None, "north", "south", "east", "west"])
def test_one_of_each_pair_is_a_half(free_side):
    import numpy as np
    values = [1e-3, 0.25, 0.5, 1.0, 1.7320508, 3.0, 1000.0]
    for a, b, c in itertools.product(values, values, values):
        if free_side is None:
            dom = tl.domain(tl.TL_SIXVERTEX, n=8)
            w = tl.weights(tl.TL_W_SIXVERTEX, a, b, c, rule=tl.TL_METROPOLIS)
        else:
            dom = tl.domain(tl.TL_SIXVERTEX, mask=np.ones((6, 6), np.uint8), free_side=free_side)
            w = tl.weights(tl.TL_W_SIXVERTEX6, a, 1.0, b, 2.0, c, 0.75, rule=tl.TL_METROPOLIS)
        try:
            t = tl.thresholds(dom, w)
        except tl.TlError:
            continue   # weights too uneven for 32-bit thresholds
        assert len(t) % 2 == 0
        for down, up in zip(t[::2], t[1::2]):
            assert down == HALF or up == HALF, (a, b, c)
            assert down <= HALF <= up
