"""The first level of the budgeted selection, which takes its Gaussians through groups of views: batches
of one view to more than two groups, with and without budgets in a group, views that share a camera
and views that do not, scales at which the short root and quotients do not hold, odd parameters, and
fewer Gaussians than a block, against the oracle."""
import numpy as np
import pytest
import torch

from helpers import params_struct
from oracle import oracle as O
from paper_2510_09997_amd import _clod as C, synth
from paper_2510_09997_amd.render import Batch, Scene

pytestmark = pytest.mark.gpu


def batch_of(V, n, kind):
    sc = synth.make_scene(n, 0, "mixture" if n > 500 else "uniform", seed=V, log_scale_mean=-3.5)
    views = []
    for j in range(V):
        d = 3.0 + 1.5 * (j // 2 if kind == "runs" else j)   # two views of a camera in turn
        v = synth.look_at((0.31 * d, -0.2 * d, -0.9 * d), width=160, height=120, s_v=1.0 + 0.7 * j)
        v.budget = 0 if kind == "some" and j % 3 == 1 else 1 + (j * 7919 + n // 3) % n
        views.append(v)
    if kind in ("tiny_unit", "large_unit"):
        f = np.float32(2.0 ** (-45 if kind == "tiny_unit" else 45))
        sc["mean"] *= f
        sc["log_scale"] += np.float32(np.log(f))
        for v in views:
            v.t, v.c = (v.t * f).astype(np.float32), (v.c * f).astype(np.float32)
    if kind == "odd":
        r = np.random.default_rng(3)
        for k in ("opacity", "decay"):
            for val in (np.inf, -np.inf, 0.0, 1e-30, 1e30, -1e30):
                sc[k].reshape(-1)[r.integers(0, n, 20)] = val
    return sc, views, dict(near=1e-16) if kind == "tiny_unit" else None


@pytest.mark.parametrize("V,n,kind", [(1, 2, "runs"), (2, 255, "runs"), (4, 1025, "runs"), (5, 300_001, "some"), (9, 3000, "some"),
                                      (7, 263_000, "runs"), (4, 3000, "tiny_unit"), (4, 3000, "large_unit"), (6, 5000, "odd")])
def test_budget_first_level(V, n, kind):
    print("case: budget first level", V, n, kind, flush=True)
    sc, views, p = batch_of(V, n, kind)
    b = Batch(n, views, params_struct(p))
    b.project(Scene(sc))
    alpha = b.section(C.SEC_ALPHA).cpu().numpy().reshape(V, n)
    flags = b.section(C.SEC_FLAGS).cpu().numpy().reshape(V, n)
    counts = b.counts.clone()
    assert torch.equal(b.lod_count(Scene(sc)), counts)   # (without the plane of alpha'')
    for j, v in enumerate(views):
        want = O.view_pass(sc, v, p)
        assert np.array_equal(counts[j].cpu().numpy(), want["counts"]), j
        assert np.array_equal(alpha[j].view(np.uint32), want["rec"][:, 6].view(np.uint32)), j
        assert np.array_equal(flags[j] & 7, want["flags"] & 7), j
