"""The blend adjoint at the edges of its batches (64 entries) and of its reductions over groups of
eight, with quadrants that end at different entries and with clamped opacities, element-wise against
FP64 autograd (relative to the magnitude of each element's chain-rule terms)."""
import numpy as np
import pytest

from helpers import _grad_case, check_grads
from paper_2510_09997_amd import synth

pytestmark = pytest.mark.gpu


def stack(n, opacity, scale, spread, seed):
    """n Gaussians before one another, all in sight of a small image."""
    sc = synth.make_scene(n, 1, "uniform", seed=seed, log_scale_mean=scale)
    r = np.random.default_rng(seed)
    sc["mean"][0] = r.uniform(-spread, spread, n)
    sc["mean"][1] = r.uniform(-spread, spread, n)
    sc["mean"][2] = np.linspace(-0.5, 0.5, n)
    sc["opacity"][:] = opacity + 0.2 * r.standard_normal(n)
    sc["decay"][:] = 30.0
    return sc


@pytest.mark.parametrize("n,opacity,scale,spread", [
    (1, -2.0, -1.5, 0.1), (6, -2.0, -1.5, 0.1), (7, -2.0, -1.5, 0.1), (8, -2.0, -1.5, 0.1), (9, -2.0, -1.5, 0.1),
    (63, -4.0, -1.5, 0.2), (64, -4.0, -1.5, 0.2), (65, -4.0, -1.5, 0.2), (200, -4.5, -1.5, 0.3),
    (40, 6.0, -2.0, 0.4),            # opaque: alpha clamped at 0.99, pixels end early
    (150, -1.0, -3.2, 0.5),          # small splats: a quadrant sees a few of a batch
])
def test_adjoint_edges(n, opacity, scale, spread):
    print("case: adjoint", n, opacity, scale, flush=True)
    sc = stack(n, opacity, scale, spread, seed=n)
    views = [synth.look_at((0.05, 0.03, -3.0), width=29, height=21, s_v=1.0),
             synth.look_at((-0.3, 0.1, -2.5), width=16, height=16, s_v=1.5)]
    got, want, S, _ = _grad_case(sc, views, seed=n, dL_deta=[0.3, -0.2])
    check_grads(got, want, S)
