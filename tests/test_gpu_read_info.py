"""clod_read_info's radix passes on both paths of the binning: three over the depth keys, then the row
and the column partition, or one per eight bits of the tile id in batches of more than 2,048 tile
rows or with frames beyond 256 x 256 tiles."""
import pytest

from paper_2510_09997_amd import _clod as C, synth
from paper_2510_09997_amd.render import Batch, Scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,sizes,passes", [
    (500, [(16, 16)], 5), (500, [(4096, 40)], 5), (500, [(32, 512)] * 64, 5),    # (row path)
    (500, [(4097, 40)], 5), (500, [(40, 4112)], 5),                              # (771 tiles: two passes of eight bits)
    (500, [(4112, 4112)], 6), (500, [(32, 512)] * 64 + [(16, 16)], 5),           # (66,049 and 4,097 tiles)
    (0, [(64, 64)], 0)])
def test_radix_passes(n, sizes, passes):
    print("case: radix passes", n, len(sizes), sizes[0], flush=True)
    scene = Scene(synth.make_scene(n, 0, "uniform", seed=1, log_scale_mean=-3.5))
    b = Batch(n, [synth.look_at((0.3, 0.2, -3.0), width=w, height=h) for w, h in sizes])
    b.project(scene)
    D = b.bin_sort()
    info = C.clod_read_info(b.c_struct())
    assert (info["n_dup"], info["overflow"], info["capacity"]) == (D, False, b.capacity)
    assert info["passes"] == passes
