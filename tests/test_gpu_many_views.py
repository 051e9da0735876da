"""Batches of many views, up to the most a call takes: the per-Gaussian stages keep a table of the
views in LDS, 80 bytes and more a view.  Every output against the same views in batches of 64."""
import numpy as np
import pytest
import torch

from paper_2510_09997_amd import _clod as C, synth
from paper_2510_09997_amd.render import Batch, Scene

pytestmark = pytest.mark.gpu


def views_of(V):
    rng = np.random.default_rng(V)
    eyes = rng.normal(size=(V, 3))
    eyes *= rng.uniform(2.5, 9.0, V)[:, None] / np.linalg.norm(eyes, axis=1)[:, None]
    return [synth.look_at(tuple(e), width=32, height=24, s_v=float(s))
            for e, s in zip(eyes, rng.uniform(1.0, 8.0, V))]


def run(scene, views, dL, grads, accumulate):
    b = Batch(scene.n, views, dup_capacity=1 << 20)
    b.project(scene)
    D = b.bin_sort()
    rgb, T, last = b.render_fwd()
    b.render_bwd(scene, T, last, dL, grads=grads, accumulate=accumulate)
    return dict(counts=b.counts.clone(), lod=b.lod_count(scene), flags=b.section(C.SEC_FLAGS), alpha=b.section(C.SEC_ALPHA),
                rgb=rgb, T=T, last=last), D


@pytest.mark.parametrize("V", [300, 777, 1024])
def test_many_views(V):
    sc = synth.make_scene(1100, 1, "mixture", seed=V, log_scale_mean=-3.5)
    scene, views = Scene(sc), views_of(V)
    px = 3 * 32 * 24
    dL = torch.from_numpy(np.random.default_rng(1).normal(size=V * px).astype(np.float32)).cuda()
    whole = scene.zeros_like()
    got, D = run(scene, views, dL, whole, False)
    parts, total, size, Dsum = [], scene.zeros_like(), scene.zeros_like(), 0
    for v0 in range(0, V, 64):
        g = scene.zeros_like()
        w, d = run(scene, views[v0:v0 + 64], dL[v0 * px:(v0 + 64) * px].clone(), g, False)
        parts.append(w)
        Dsum += d
        for k in total:
            total[k] += g[k]
            size[k] += g[k].abs()
    assert D == Dsum > 0
    for k in got:
        want = torch.cat([p[k].reshape(-1) for p in parts])
        assert torch.equal(got[k].reshape(-1), want), k
    assert torch.equal(got["counts"], got["lod"])
    # Sums of up to V terms in binary32: V 2^-24 of the terms' magnitudes, here 16 times that of the
    # batches' (their own terms and the chain behind the sums round too).
    for k in total:
        err = (whole[k] - total[k]).norm() / size[k].norm()
        assert float(err) <= 16 * V * 2.0 ** -24, (k, float(err))
