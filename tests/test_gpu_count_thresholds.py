"""Counting with thresholds that the estimate of the mask takes apart: 0 (alpha'' > 0, whose end is where
the exponential becomes 0), budgets of the whole scene or past the positive alpha'', thresholds near
the smallest and above the largest it takes, tiny epsilons and far scales, alone and mixed in a batch;
against the oracle.  And the time with a threshold of 0: masks left open are evaluated in full."""
import numpy as np
import pytest
import torch

from helpers import params_struct
from oracle import oracle as O
from paper_2510_09997_amd import synth
from paper_2510_09997_amd.render import Batch, Scene

pytestmark = pytest.mark.gpu


def edge_scene(n):
    """q within a tenth of the end of the exponential (86), alphas from far below 2^-20 to nearly 1."""
    sc = synth.make_scene(n, 0, "uniform", seed=4, log_scale_mean=-3.5)
    r = np.random.default_rng(4)
    pos = np.array((0.9, -0.6, -2.7))
    d = np.linalg.norm(sc["mean"].T - pos, axis=1)
    q = np.where(np.arange(n) % 4 == 0, 86.0 + r.uniform(-2e-4, 2e-4, n), r.uniform(85.9, 86.1, n))
    q[::7] = r.uniform(60.0, 130.0, len(q[::7]))
    sc["decay"][:] = np.sqrt(0.5 * (d / d.max()) ** 2 / q).astype(np.float32)
    sc["opacity"][:] = np.where(np.arange(n) % 3 == 0, r.uniform(-14.2, -13.5, n), r.uniform(-90.0, 8.0, n))
    return sc, pos


CASES = {   # tau, eps, s_v and budget per view, factor of the length unit
    "zero": (0.0, 1e-6, [(1.0, 0), (1.01, 0), (4.0, 0)], 1.0),
    "zero_and_budgets": (0.0, 1e-6, [(1.0, 0), (1.0, 9000), (1.0, 20000), (1.5, 700), (1.0, 19000)], 1.0),
    "budgets_at_zero": (0.0, 1e-6, [(1.0, 9000), (1.0, 20000), (1.0, 20003), (1.0, 19000)], 1.0),
    "whole_scene": (1.0 / 255.0, 1e-6, [(1.0, 20000), (2.0, 50000), (1.0, 0)], 1.0),
    "tiny": (2.0 ** -101, 1e-6, [(1.0, 0), (1.9, 0), (2.0, 0), (2.1, 0), (1e4, 0)], 1.0),
    "denormal": (1e-40, 1e-6, [(1.0, 0), (3.0, 0)], 1.0),
    "huge": (1e30, 1e-6, [(1.0, 0), (1e9, 0)], 1.0),
    "tiny_eps": (0.0, 1e-33, [(1.0, 0), (1.0, 20000)], 1.0),
    "least_eps": (1.0 / 255.0, 2e-38, [(1.0, 0), (3.0, 0)], 1.0),
    "large_unit": (0.0, 1e-6, [(1.0, 0), (2.0, 0)], 2.0 ** 45),
    "larger_unit": (1.0 / 255.0, 1e-6, [(1.0, 0), (2.0, 0)], 2.0 ** 55),
}


@pytest.mark.parametrize("name", list(CASES))
def test_counts_at_thresholds(name):
    print("case: count thresholds", name, flush=True)
    tau, eps, per_view, unit = CASES[name]
    n = 20_000
    sc, pos = edge_scene(n)
    f = np.float32(unit)
    sc["mean"] *= f
    sc["log_scale"] += np.float32(np.log(unit))
    views = []
    for s_v, budget in per_view:
        v = synth.look_at(pos, width=200, height=150, s_v=s_v)
        v.t, v.c = (v.t * f).astype(np.float32), (v.c * f).astype(np.float32)
        v.budget = budget
        views.append(v)
    p = dict(tau=tau, eps=float(np.float32(eps)))
    scene = Scene(sc)
    b = Batch(n, views, params_struct(p))
    counted = b.lod_count(scene).cpu().numpy()
    b.project(scene)
    assert np.array_equal(counted, b.counts.cpu().numpy())
    for j, v in enumerate(views):
        assert np.array_equal(counted[j], O.view_pass(sc, v, p)["counts"]), j


def test_a_threshold_of_zero_is_estimated():
    """The count of a scene without a mask takes less than twice that with the default threshold (it
    took 2.4 times as long when every mask was left open)."""
    print("case: count time", flush=True)
    scene = Scene(synth.make_scene(2_000_000, 0, "mixture", seed=0))
    views = synth.random_views(0, 16, radius=(4.0, 60.0), resolutions=((640, 480),), sv_range=(1.0, 8.0))

    def time(params):
        b = Batch(scene.n, views, params_struct(params), dup_capacity=1)
        ms = []
        for _ in range(9):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            b.lod_count(scene)
            e[1].record()
            torch.cuda.synchronize()
            ms.append(e[0].elapsed_time(e[1]))
        return float(np.median(ms))

    base, zero = time(None), time(dict(tau=0.0))
    print("  ", base, zero, flush=True)
    assert zero < 2.0 * base
