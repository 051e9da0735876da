"""Binning of records that cover many tiles: column parts that shrink to what fits and grow again (rows
of mixed widths up to 256 columns), the row kernels' shorter shares on both sides of their line (64
tiles a record on average), and the time, against as many pairs of ordinary records."""
import numpy as np
import pytest
import torch

from paper_2510_09997_amd import synth
from paper_2510_09997_amd.render import Batch, Scene
from test_gpu_binning import check_lists

pytestmark = pytest.mark.gpu


def scene(n, log_scale, seed=3):
    sc = synth.make_scene(n, 0, "uniform", seed=seed, log_scale_mean=-4.0)
    sc["log_scale"][:] = log_scale
    sc["decay"][:] = 100.0
    sc["opacity"][:] = 3.0
    return sc


@pytest.mark.parametrize("kind,n,size,tiles", [
    ("all", 700, (4096, 512), (2000, 9000)),        # every row pair covers up to 256 columns
    ("all", 1200, (1920, 1080), (2000, 9000)),
    ("mixed", 6000, (4096, 256), (64, 1500)),       # a wide record among narrow ones
    ("runs", 3000, (2048, 512), (64, 3000)),       # stretches of wide and of narrow ones
    ("below", 4000, (1024, 768), (40, 64)), ("above", 4000, (1024, 768), (64, 100))])
def test_lists_of_wide_records(kind, n, size, tiles):
    print("case: wide records", kind, n, flush=True)
    scale = np.full(n, {"below": -2.6, "above": -2.41}.get(kind, 0.6), np.float32)
    if kind == "mixed":
        scale[np.arange(n) % 9 != 0] = -4.0
    sc = scene(n, scale)
    if kind == "runs":                               # by depth, so that the lists alternate
        sc["log_scale"][:] = np.where(np.floor(sc["mean"][2] * 10) % 2 == 0, 0.2, -4.5).astype(np.float32)
    b, D = check_lists(Scene(sc), [synth.look_at((0.0, 0.0, -4.0), width=size[0], height=size[1])], capacity=12_000_000)
    rendered = int(b.counts[0, 2])
    print("  tiles a record", D / rendered, flush=True)
    assert tiles[0] * rendered <= D < tiles[1] * rendered


def test_wide_records_take_no_longer_than_others():
    """Ten million pairs of 1,400 records take at most half as long again as of a million (they took 1.6
    times as long while each pair was stored on its own and twelve waves shared the records)."""
    print("case: wide records, time", flush=True)
    view = synth.look_at((0.0, 0.0, -4.0), width=1920, height=1080)

    def run(n, log_scale):
        sc = Scene(scene(n, log_scale))
        b = Batch(n, [view], dup_capacity=30_000_000)
        b.project(sc)
        D = b.bin_sort()
        us = []
        for _ in range(9):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            b.bin_sort(sync=False)
            e[1].record()
            torch.cuda.synchronize()
            us.append(1e3 * e[0].elapsed_time(e[1]))
        return D, float(np.median(us))

    D0, ordinary = run(1_100_000, -4.35)
    D1, wide = run(1400, 0.6)
    print("  ", D0, ordinary, D1, wide, flush=True)
    assert abs(D1 / D0 - 1.0) < 0.4
    assert wide / D1 < 1.5 * ordinary / D0
