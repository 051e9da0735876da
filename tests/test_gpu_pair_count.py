"""The pair count that an overflowed binning reports, in 64 bits, on both paths: frames that every
Gaussian covers whole (16,384 x 16,384 pixels, 2^20 tiles), where 4,096 records already hold 2^32
pairs."""
import numpy as np
import pytest

from paper_2510_09997_amd import _clod as C, synth
from paper_2510_09997_amd.render import Batch, Scene

pytestmark = pytest.mark.gpu


def covering(n):
    sc = synth.make_scene(n, 0, "uniform", seed=1, log_scale_mean=2.0)
    sc["mean"] *= np.float32(0.1)
    sc["decay"][:] = 100.0
    sc["opacity"][:] = 3.0
    return sc


@pytest.mark.parametrize("n,size,capacity", [(9000, 16384, 1 << 16), (9000, 16384, 64), (4097, 16384, 5000), (5000, 4096, 1 << 16),
                                             (5000, 4096, 64)])
def test_overflow_reports_every_pair(n, size, capacity):
    print("case: pair count", n, size, capacity, flush=True)
    b = Batch(n, [synth.look_at((0.0, 0.0, -3.0), width=size, height=size)], dup_capacity=capacity)
    b.project(Scene(covering(n)))
    rendered = int(b.counts[0, 2])
    assert rendered == n
    C.clod_bin_sort(b.c_struct(), sync_count=False)
    info = C.clod_read_info(b.c_struct())
    assert info["overflow"] and info["n_dup"] == n * (size // 16) ** 2
