"""Height tile plans on the host: tile rows, groups and sweeps per launch are
upper bounds, so every shape is given a plan that fits, and the plan keeps the
rules a launch rests on."""
import itertools

import pytest

from plan_helpers import plans  # noqa: F401  (fixture)
import paper_1804_07250_amd as tl

ROWS = [1, 5, 8, 32, 64, 100, 170, 254, 300, 600, 5000]
GROUPS = [1, 2, 3, 4, 8, 100]
SWEEPS = [1, 2, 8, 59, 64, 100, 127, 200, 1000, 1 << 30]


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("dom", [(tl.TL_SIXVERTEX, 0, 0, 0, N) for N in (3, 30, 100, 200, 254, 255, 256, 400, 511, 1024, 3000)]
                         + [(tl.TL_LOZENGE,) + abc + (0,) for abc in ((8, 8, 8), (60, 100, 100), (100, 1500, 100),
                                                                      (1024, 1024, 1024), (2000, 1000, 1000))])
def test_every_shape_has_a_plan(plans, dom, order):
    model, a, b, c, N = dom
    sixv = model == tl.TL_SIXVERTEX
    rows, sites = (N + 1, (N + 2) // 2) if sixv else (b + c + 1, (a + c + 3) // 3)
    ng = -(-sites // 128)
    per = (4 if order else 2) if sixv else 3   # halo rows a sweep
    shapes = list(itertools.product(ROWS, GROUPS, SWEEPS))
    ans = plans(["height %d %d %d %d %d %d %d %d %d %d" % (dom + (order,) + s + (s[2],)) for s in shapes])
    for (r, g, s), got in zip(shapes, ans):
        # halo of one sweep, a row and the tasks of 512 lanes: wider tiles than
        # these have none
        tg = min(g, ng)
        lg = tg + (2 if tg < ng else 0)
        if (2 if sixv else 1) * (512 // lg) < 2 * per + 3:
            assert got == "refused"
            continue
        assert got != "refused", (r, g, s)
        S, TR, TG, HR, HG, tiles, lds = map(int, got.split())
        assert 1 <= S <= s and 1 <= TR <= r and TG == tg and lds <= 160 * 1024, (r, g, s)
        cut = TR < rows
        assert HR == (per * S if cut else 0) and HG == (1 if tg < ng else 0), (r, g, s)
        assert tiles == -(-rows // TR) * -(-ng // TG), (r, g, s)
        height = TR + 2 * HR
        assert (-(-height // 2) if sixv else height) * (TG + 2 * HG) <= 512, (r, g, s)
