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
