"""The adjoint loop's work counters on an image of one 8x8 quadrant whose every pixel blends every
entry: the lanes walked, the exponentials and the contributing pairs are 64 per entry, whether the
number of entries of a batch is odd or even."""
import numpy as np
import pytest
import torch

from paper_2510_09997_amd import synth
from paper_2510_09997_amd.render import Batch, Scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 3, 8, 9, 63, 64, 65, 129])
def test_walked_lanes(n):
    print("case: adjoint counters", n, flush=True)
    sc = synth.make_scene(n, 0, "uniform", seed=n, log_scale_mean=2.0)
    sc["mean"][:2] *= np.float32(0.01)
    sc["log_scale"][:] = 2.0   # (the image is 0.3 of a standard deviation to each side)
    sc["mean"][2] = np.linspace(-0.1, 0.1, n)
    sc["decay"][:] = 100.0
    sc["opacity"][:] = -4.0   # (alpha 0.018: 129 of them leave a tenth of the light)
    scene = Scene(sc)
    b = Batch(n, [synth.look_at((0.0, 0.0, -3.0), width=8, height=8)])
    b.project(scene)
    assert b.bin_sort() == n
    rgb, T, last = b.render_fwd()
    assert bool((last == n).all())
    pairs = torch.zeros(3, dtype=torch.int64, device="cuda")
    b.render_bwd(scene, T, last, torch.ones_like(rgb), pairs=pairs)
    assert pairs.tolist() == [64 * n] * 3
