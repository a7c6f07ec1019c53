"""Tile shapes measured with other tile kernels: a cache line without the
generation of the kernels, as it was written before they had one, or with another
one is not taken."""
import pytest

from gpu_helpers import need_gpu, say

pytestmark = pytest.mark.gpu


def test_lines_of_other_kernels_are_ignored(tmp_path):
    tl = need_gpu()
    say("tune cache of other kernels")
    path = str(tmp_path / "tiles.txt")
    dom = tl.domain(tl.TL_SIXVERTEX, n=300)
    w = tl.weights(tl.TL_W_UNIFORM)
    first = tl.Sampler(dom, w, 1, tl.options(tune_cache=path)).autotune(8)
    assert first["from_cache"] == 0
    key = open(path).read().split()[0]
    fields = key.split(":")
    assert ":gfx950" in key and "/" in fields[-2] and "/" not in fields[-1]   # the device, then the generation
    with open(path, "w") as f:
        f.write(":".join(fields[:-1]) + " 4 1 4 2\n")
        f.write(":".join(fields[:-1]) + ":other 4 1 4 2\n")
    again = tl.Sampler(dom, w, 1, tl.options(tune_cache=path)).autotune(8)
    assert again["from_cache"] == 0 and len(open(path).read().splitlines()) == 3
    third = tl.Sampler(dom, w, 1, tl.options(tune_cache=path)).autotune(8)
    assert third["from_cache"] == 1
    assert [third[k] for k in ("tile_rows", "tile_groups")] == [again[k] for k in ("tile_rows", "tile_groups")]
