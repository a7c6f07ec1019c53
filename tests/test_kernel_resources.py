"""Kernels of the built library against the limits of a compute unit."""
import re

import kernel_resources as kr
from plan_helpers import plans  # noqa: F401  (fixture)


def test_height_plans_fit_with_the_kernels_static_lds(plans):
    """The largest LDS a height plan asks for, with what the tile kernels hold
    besides, is within a compute unit's 160 KB: rows to the limit of the tasks,
    long launches, both orders (two groups: N = 255 .. 510 have the most)."""
    import paper_1804_07250_amd as tl
    req = ["height %d 0 0 0 %d %d %d %d %d %d" % (tl.TL_SIXVERTEX, N, order, rows, groups, S, S)
           for N in (254, 256, 300, 400, 502, 503, 510, 1024) for order in (0, 1) for rows in (8, 16, 32, 100, 600)
           for groups in (1, 2, 4) for S in list(range(20, 66)) + [100, 1000]]
    req += ["height %d %d %d %d 0 %d %d %d %d %d" % ((tl.TL_LOZENGE,) + abc + (order, rows, groups, S, S))
            for abc in ((100, 1500, 100), (500, 500, 500)) for order in (0, 1) for rows in (8, 32, 300)
            for groups in (1, 2, 4) for S in list(range(20, 66)) + [100, 1000]]
    largest = max(int(a.split()[-1]) for a in plans(req) if a != "refused")
    assert largest > 140 * 1024   # (the requests do reach the limit)
    tiles = {n: k for n, k in kr.kernels().items()
             if re.search(r"(loz_tiled|height_tiled|height_items(_mixed)?)_kernel", n)}
    assert len(tiles) > 30
    for name, k in tiles.items():
        assert k[".group_segment_fixed_size"] + largest <= kr.LDS_BYTES, name


def test_kernels_keep_their_state_in_registers():
    """No kernel of a sweep spills or indexes its registers by a variable: private
    memory is device memory."""
    sweeps = {n: k for n, k in kr.kernels().items()
              if re.search(r"(tiled|reg|batch|items|items_mixed|sample|step)_kernel", n)}
    assert len(sweeps) > 60
    for name, k in sweeps.items():
        assert k[".private_segment_fixed_size"] == 0 and k[".vgpr_spill_count"] == 0, name
