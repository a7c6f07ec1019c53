"""Automatic height tile shapes on the host."""
import pytest

from plan_helpers import plans  # noqa: F401  (fixture)
import paper_1804_07250_amd as tl


def shape(plans, model, a, b, c, N, order, one_bit):
    return tuple(map(int, plans(["height_auto %d %d %d %d %d %d %d" % (model, a, b, c, N, order, one_bit)])[0].split()))


@pytest.mark.parametrize("order", [0, 1])
def test_whole_six_vertex_domains(plans, order):
    """Bit-serial six-vertex domains of more than 5 granules are cut into tiles
    (as one tile they took up to a third more time); one-bit ones of 16 are not."""
    for N in (20, 64, 100, 128, 140, 158):
        rows, groups, sweeps, granules = shape(plans, tl.TL_SIXVERTEX, 0, 0, 0, N, order, 0)
        assert rows == N + 1 and sweeps > 1 << 20 and granules <= 5, N
    for N in (160, 200, 254, 255, 300, 1000):
        rows, groups, sweeps, granules = shape(plans, tl.TL_SIXVERTEX, 0, 0, 0, N, order, 0)
        assert (rows, sweeps) == (16, 6 if order else 12) and granules <= 16, N
    for N in (20, 160, 200, 255):
        assert shape(plans, tl.TL_SIXVERTEX, 0, 0, 0, N, order, 1)[0] == N + 1, N


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("abc", [(100, 100, 100), (300, 200, 157), (400, 400, 400), (600, 600, 600), (100, 100, 1500),
                                 (1500, 500, 500), (1024, 1024, 1024), (2000, 1000, 1000), (3000, 400, 300)])
def test_one_bit_lozenge_granules(plans, abc, order):
    """Every granule of a one-bit lozenge tile has a wavefront (with more granules
    than the 16, taken in turns, wide hexagons took up to 1.3 times as long), and
    wide ones leave a SIMD no more than their share."""
    rows, groups, sweeps, granules = shape(plans, tl.TL_LOZENGE, *abc, 0, order, 1)
    assert granules <= 16
    ng = -(-((abc[0] + abc[2] + 3) // 3) // 128)
    if ng > 3 and rows < abc[1] + abc[2] + 1:
        assert groups == 2
