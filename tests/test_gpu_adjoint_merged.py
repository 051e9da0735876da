"""The adjoint of records that cover many tiles, whose sums the four waves of a tile merge: gradients
element-wise against FP64 autograd in windows of 256 entries and their edges, with pixels that end
early and clamped opacities; both sides of the line (112 tiles to the record of a pair); the counters;
and the time against the forward's."""
import numpy as np
import pytest
import torch

from helpers import _grad_case, check_grads
from paper_2510_09997_amd import synth
from paper_2510_09997_amd.render import Batch, Scene

pytestmark = pytest.mark.gpu


def wide(n, opacity, scale, seed):
    sc = synth.make_scene(n, 1, "uniform", seed=seed, log_scale_mean=scale, log_scale_std=0.2)
    sc["mean"] *= np.float32(0.4)
    sc["opacity"][:] = opacity + 0.2 * np.random.default_rng(seed).standard_normal(n)
    sc["decay"][:] = 30.0
    return sc


@pytest.mark.parametrize("n,opacity,scale", [
    (1, -2.0, 0.2), (255, -4.5, 0.2), (256, -4.5, 0.2), (257, -4.5, 0.2), (600, -5.0, 0.2),
    (40, 6.0, 0.2),                   # opaque: alpha clamped at 0.99, pixels end early
    (150, -1.0, -0.2), (150, -1.0, -2.0)])
def test_merged_adjoint(n, opacity, scale):
    print("case: merged adjoint", n, opacity, scale, flush=True)
    sc = wide(n, opacity, scale, seed=n)
    views = [synth.look_at((0.05, 0.03, -3.0), width=203, height=160, s_v=1.0),
             synth.look_at((-0.3, 0.1, -2.5), width=197, height=165, s_v=1.5)]
    got, want, S, _ = _grad_case(sc, views, seed=n, dL_deta=[0.3, -0.2])
    check_grads(got, want, S)


@pytest.mark.parametrize("side", ["below", "above"])
def test_the_line_and_the_counters(side):
    """Records of exactly one row of 112 tiles, and of 111: the counters of a frame whose every pixel
    blends every entry are 256 per pair either way."""
    print("case: merged adjoint, line", side, flush=True)
    n, tiles = 9, 112 if side == "above" else 111
    sc = wide(n, -4.0, 2.0, seed=3)
    sc["log_scale"][:] = 2.0
    sc["mean"][:2] *= np.float32(0.001)
    sc["mean"][2] = np.linspace(-0.1, 0.1, n)
    scene = Scene(sc)
    b = Batch(n, [synth.look_at((0.0, 0.0, -3.0), width=16 * tiles, height=16)])
    b.project(scene)
    assert b.bin_sort() == n * tiles and int(b.counts[0, 2]) == n
    rgb, T, last = b.render_fwd()
    assert bool((last == n).all())
    pairs = torch.zeros(3, dtype=torch.int64, device="cuda")
    b.render_bwd(scene, T, last, torch.ones_like(rgb), pairs=pairs)
    assert pairs.tolist() == [256 * n * tiles] * 3


def test_few_large_records_take_no_longer():
    """3,000 Gaussians over the whole of a 1080p frame: the backward takes at most five times the
    forward blend (it took 7 to 11 times while every quadrant added to memory on its own)."""
    print("case: merged adjoint, time", flush=True)
    sc = synth.make_scene(3000, 3, "mixture", seed=1)
    sc["log_scale"][:] = 0.5
    sc["decay"][:] = 100.0
    scene = Scene(sc)
    b = Batch(3000, [synth.look_at((0.0, 0.0, -8.0), width=1920, height=1080)], dup_capacity=30_000_000)
    b.project(scene)
    b.bin_sort()
    rgb, T, last = b.render_fwd()
    grads = scene.zeros_like()

    def time(f):
        us = []
        for _ in range(9):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            f()
            e[1].record()
            torch.cuda.synchronize()
            us.append(1e3 * e[0].elapsed_time(e[1]))
        return float(np.median(us))

    fwd, bwd = time(lambda: b.render_fwd()), time(lambda: b.render_bwd(scene, T, last, rgb, grads=grads))
    print("  ", fwd, bwd, flush=True)
    assert bwd < 5.0 * fwd
