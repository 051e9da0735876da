"""The resident server's blend of sparse frames whose lists lie between the two lines of long tiles
(2,048 with block masks, 8,192 without, as in the server): bit-identical to the per-stage launches, and
as quick as lists of that length are as four quadrants."""
import time

import numpy as np
import pytest
import torch

from paper_2510_09997_amd import _clod as C, synth
from paper_2510_09997_amd.render import Batch, Scene
from test_gpu_persistent import Job, same_bits, start

pytestmark = pytest.mark.gpu


def slab(n):
    """Small faint Gaussians spread evenly over the image, one layer behind another."""
    sc = synth.make_scene(n, 0, "uniform", seed=2, log_scale_mean=-5.0)
    sc["mean"][:2] *= np.float32(1.8)
    sc["mean"][2] *= np.float32(0.2)
    sc["opacity"][:] = -3.0
    sc["decay"][:] = 100.0
    return sc


def run(n, view):
    """The server's result, the lists' lengths and the median time of its blend stage in us."""
    sc = slab(n)
    scene = Scene(sc, packed_sh=True)
    b = Batch(n, [view])
    b.project(scene)
    b.bin_sort()
    want = b.render_fwd()
    lists = np.diff(b.section(C.SEC_RANGES).cpu().numpy().astype(np.int64), axis=1).ravel()
    srv = start()
    blend = []
    try:
        job = Job(srv, scene, n, [view], dup_pairs=int(lists.sum()) + 65536)
        t0 = time.perf_counter()
        while C.clod_server_clock(srv) < 0:
            assert time.perf_counter() - t0 < 30.0
            time.sleep(1e-4)
        for _ in range(7):
            job.submit()
            job.wait()
            tl = C.clod_server_stage_times(srv, job.seq)
            blend.append((tl[-1][1] - tl[-2][1]) / 1e3)
    finally:
        C.clod_server_stop(srv)
    torch.cuda.synchronize()
    for got, ref in zip((job.rgb, job.T, job.last), want):
        assert same_bits(got, ref)
    return lists, float(np.median(blend))


def test_lists_between_the_lines():
    print("case: server long tiles", flush=True)
    view = synth.look_at((0.0, 0.0, -3.0), width=640, height=480)
    below, us_below = run(900_000, view)
    above, us_above = run(1_440_000, view)
    print("  lists", np.median(below), np.median(above), "blend", us_below, us_above, flush=True)
    assert 1000 < np.median(below) and below.max() < 2048
    assert 2048 < np.median(above) and above.max() < 8192
    # 1.6 times the entries: at most twice the time (a quarter above their ratio).
    assert us_above < 2.0 * us_below
