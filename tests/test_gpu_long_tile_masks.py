"""Long tiles of full batches, which get block masks only from 32,768 entries on (up to 4,096 filled tiles
from 8,192): bit-identical to the oracle where masked and unmasked long tiles meet in a batch, and no
slower where the lists grow behind pixels that end early."""
import numpy as np
import pytest
import torch

from helpers import compare_forward, gpu_forward
from oracle import oracle as O
from paper_2510_09997_amd import synth
from paper_2510_09997_amd.render import Batch, Scene

pytestmark = pytest.mark.gpu


def pile(n, seed, opacity):
    """Small Gaussians before one another, over a few tiles of the image's middle."""
    sc = synth.make_scene(n, 0, "uniform", seed=seed, log_scale_mean=-5.0)
    sc["mean"] *= np.float32(0.04)
    sc["opacity"][:] = opacity
    sc["decay"][:] = 30.0
    return sc


def join(*scenes):
    return dict(n=sum(s["n"] for s in scenes), sh_degree=0,
                **{k: np.ascontiguousarray(np.concatenate([s[k] for s in scenes], axis=-1))
                   for k in ("mean", "log_scale", "quat", "opacity", "decay", "sh")})


@pytest.mark.parametrize("frame,filled", [(960, (2049, 4096)), (1360, (4097, 8192))])
def test_masked_and_unmasked_tiles_of_a_batch(frame, filled):
    print("case: long tile masks", frame, flush=True)
    spread = synth.make_scene(60_000, 0, "uniform", seed=5, log_scale_mean=-4.5)
    side = pile(9000, 3, -4.5)
    side["mean"][0] += np.float32(0.6)
    sc = join(pile(33_500, 2, -5.2), side, spread)
    views = [synth.look_at((0.0, 0.0, -3.0), width=32, height=32, s_v=1.0), synth.look_at((0.0, 0.0, -3.2), width=frame, height=frame)]
    rs = [O.render32(sc, v) for v in views]
    lists = np.concatenate([np.diff(r["tile_off"]) for r in rs])
    assert filled[0] <= (lists > 0).sum() <= filled[1]
    assert lists.max() >= 32_768 and ((lists >= 8192) & (lists < 32_768)).any()
    g = gpu_forward(sc, views)
    compare_forward(g, sc, views)
    assert g["pairs"][0] == sum(r["pair_classes"][0] for r in rs)
    assert g["pairs"][2] == sum(r["pair_classes"][2] for r in rs)


def test_entries_behind_ended_pixels_cost_little():
    """Twice the Gaussians, all behind pixels that have ended: the blend takes at most half as long
    again (with masks over the whole of the longer lists it took 1.9 times as long)."""
    print("case: long tile masks, time", flush=True)
    view = synth.look_at((0.0, 0.0, -10.0), width=1920, height=1080)

    def run(n):
        sc = synth.make_scene(n, 0, "mixture", seed=1)
        sc["log_scale"][:] = -1.5
        sc["decay"][:] = 100.0
        scene = Scene(sc)
        b = Batch(n, [view], dup_capacity=60_000_000)
        b.project(scene)
        D = b.bin_sort()
        us = []
        for _ in range(9):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            b.render_fwd()
            e[1].record()
            torch.cuda.synchronize()
            us.append(1e3 * e[0].elapsed_time(e[1]))
        return D, float(np.median(us))

    few, many = run(100_000), run(200_000)
    print("  ", few, many, flush=True)
    assert many[1] < 1.5 * few[1]
