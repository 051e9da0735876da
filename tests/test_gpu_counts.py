"""Counts, flags and attenuated opacities over the forms that take the short ways of the per-Gaussian
stages (short root and quotients, estimated masks and projections in the counting entry points) and
the forms that must not: scales far from 1, a threshold of 0, budgets, viewports, degenerate
rotations, infinities and NaN, scenes of less and more than a block's share, against the oracle."""
import numpy as np
import pytest
import torch

from helpers import params_struct
from oracle import oracle as O
from paper_2510_09997_amd import _clod as C, synth
from paper_2510_09997_amd.render import Batch, Scene

pytestmark = pytest.mark.gpu


def views_at(dists, svs, w=320, h=200):
    return [synth.look_at((0.31 * d, -0.2 * d, -0.9 * d), width=w, height=h, s_v=s) for d in dists for s in svs]


def make(n, seed=0, scale=-3.5, **kw):
    return synth.make_scene(n, 0, "mixture" if n > 500 else "uniform", seed=seed, log_scale_mean=scale, **kw)


def scaled(sc, views, factor):
    """The scene and its cameras at another length unit."""
    f = np.float32(factor)
    sc["mean"] *= f
    sc["log_scale"] += np.float32(np.log(factor))
    for v in views:
        v.t, v.c = (v.t * f).astype(np.float32), (v.c * f).astype(np.float32)
    return sc, views


def case(name):
    p = None
    if name[1:].isdigit():
        sc, views = make(int(name[1:])), views_at([3.0, 9.0], [1.0, 4.0])
    elif name == "views70":
        sc, views = make(3000), views_at(np.geomspace(1.0, 90.0, 35), [1.0, 7.0])
    elif name == "tiny_unit":       # squared distances below 2^-80
        sc, views = scaled(make(2000), views_at([3.0, 8.0], [1.0, 2.0]), 2.0 ** -45)
        p = dict(near=1e-16)
    elif name == "large_unit":      # squared distances above 2^80
        sc, views = scaled(make(2000), views_at([3.0, 8.0], [1.0, 2.0]), 2.0 ** 45)
    elif name == "near_views":      # splats wider than the bound of the estimated projection
        sc, views = make(4000, scale=-1.5), views_at([0.5, 1.0, 2.0], [1.0, 3.0])
    elif name == "tau0":
        sc, views, p = make(3000), views_at([3.0, 9.0], [1.0, 16.0]), dict(tau=0.0)
    elif name == "dilation0":
        sc, views, p = make(3000), views_at([3.0, 9.0], [1.0, 2.0]), dict(dilation=0.0)
    elif name == "budget":
        sc, views = make(5000), views_at([3.0, 9.0], [1.0, 2.0])
        for v, k in zip(views, (0, 1, 777, 5000)):
            v.budget = k
    elif name == "viewports":
        sc = make(4000)
        views = synth.strips(views_at([4.0], [1.0])[0], [1.0, 2.0, 4.0])
    elif name == "thresholds":      # alpha'' at the threshold to within rounding
        sc, views = make(4000), views_at([3.0, 6.0], [1.0, 2.5])
        sc["decay"][:] = 1e18
        t = np.float64(np.float32(1.0 / 255.0)) * np.repeat([1.0, 2.5], 2000)
        sc["opacity"][:] = (np.log(t / (1.0 - t)) + np.linspace(-3e-6, 3e-6, 4000)).astype(np.float32)
    else:
        sc, views = make(3000), views_at([3.0, 7.0], [1.0, 2.0])
        r = np.random.default_rng(5)
        for k in ("mean", "log_scale", "quat", "opacity", "decay"):
            a = sc[k].reshape(-1, sc["n"])
            for val in (np.nan, np.inf, -np.inf, 0.0, 1e-30, 1e30, -1e30):
                if k == "mean" and not (abs(val) < 1e20):
                    continue
                a[r.integers(0, len(a), 20), r.integers(0, sc["n"], 20)] = val
        sc["quat"][:, 17] = 0.0
    return sc, views, p


@pytest.mark.parametrize("name", ["n1", "n255", "n1025", "n6001", "views70", "tiny_unit", "large_unit", "near_views", "tau0",
                                  "dilation0", "budget", "viewports", "thresholds", "odd_values"])
def test_counts_flags_and_opacities(name):
    print("case: counts", name, flush=True)
    sc, views, p = case(name)
    scene = Scene(sc)
    b = Batch(scene.n, views, params_struct(p))
    b.project(scene)
    counted = b.lod_count(scene)
    b.project(scene)                      # (the counting entry point shares the workspace)
    alpha = b.section(C.SEC_ALPHA).cpu().numpy().reshape(len(views), -1)
    flags = b.section(C.SEC_FLAGS).cpu().numpy().reshape(len(views), -1)
    assert torch.equal(counted, b.counts)
    for j, v in enumerate(views):
        want = O.view_pass(sc, v, p)
        assert np.array_equal(b.counts[j].cpu().numpy(), want["counts"]), j
        ok = ~np.isnan(want["rec"][:, 6])
        assert np.array_equal(np.isnan(alpha[j]), ~ok)
        assert np.array_equal(alpha[j][ok].view(np.uint32), want["rec"][:, 6][ok].view(np.uint32)), j
        assert np.array_equal(flags[j] & 7, want["flags"] & 7), j
