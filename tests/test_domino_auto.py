"""Automatic domino tile shapes on the host: in random order, where one-bit tiles
share compute units in the band that moves, fewer and wider ones take over after
as many sweeps as the order."""
from plan_helpers import plans  # noqa: F401  (fixture)


def ask(plans, n, order, weighted, t0, sweeps):
    return tuple(map(int, plans(["domino_auto %d %d %d %d %d" % (n, order, weighted, t0, sweeps)])[0].split()))


def test_random_order_shapes(plans):
    for n in (1537, 1600, 1700, 1792):   # 13 or 14 groups: 7 tiles a row
        narrow, wide = (32, 2, 8), (24, 3, 10)
        assert ask(plans, n, 1, 0, 0, 1000) == narrow + (1000,)
        assert ask(plans, n, 1, 0, 0, n) == narrow + (n,)
        assert ask(plans, n, 1, 0, 0, n + 500) == narrow + (n,) + wide
        assert ask(plans, n, 1, 0, n - 3, 10) == narrow + (3,) + wide
        assert ask(plans, n, 1, 0, n, 10) == narrow + (0,) + wide
        assert ask(plans, n, 1, 0, 0xFFFFFF00, 200) == narrow + (0,) + wide


def test_other_shapes_are_kept(plans):
    for n in (130, 1001, 1450, 1536, 1793, 2000, 2048, 2049, 4000):
        assert ask(plans, n, 1, 0, 5000, 1000) == (32, min(2, -(-n // 128)), 8, 1000)
    for n in (1400, 1600, 1700, 2048):
        assert ask(plans, n, 0, 0, 5000, 1000) == (32, 2, 16, 1000)
        assert ask(plans, n, 1, 1, 5000, 1000) == (32, 2, 8, 1000)
        assert ask(plans, n, 0, 1, 5000, 1000) == (32, 4, 16, 1000)
