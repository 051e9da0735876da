"""Long tiles (sixteen 4x4 blocks per tile, entries in groups of four with one termination test per
group) at the lines where a tile becomes long, in sparse and in full batches, with pixels that end
inside a group, colours that are not finite and lists of every length modulo four: bit-identical to
the oracle, with the contract's pair counts."""
import numpy as np
import pytest

from helpers import compare_forward, gpu_forward
from oracle import oracle as O
from paper_2510_09997_amd import synth

pytestmark = pytest.mark.gpu


def cluster(n, opacity, scale, seed):
    sc = synth.make_scene(n, 0, "uniform", seed=seed, log_scale_mean=scale)
    sc["mean"] *= np.float32(0.05)
    sc["opacity"][:] = opacity + 0.3 * np.random.default_rng(seed).standard_normal(n)
    sc["decay"][:] = 30.0
    return sc


def join(a, b):
    return dict(n=a["n"] + b["n"], sh_degree=0, **{k: np.ascontiguousarray(np.concatenate([a[k], b[k]], axis=-1))
                                                  for k in ("mean", "log_scale", "quat", "opacity", "decay", "sh")})


@pytest.mark.parametrize("n,opacity,scale,colours", [
    (2047, -4.0, -4.0, ""), (2048, -4.0, -4.0, ""), (2049, -5.0, -4.0, ""), (2050, 3.0, -4.5, ""), (2051, -1.0, -5.0, ""),
    (5003, -4.5, -5.5, "inf"), (9001, 1.0, -5.5, ""), (9002, -4.8, -5.5, "full"), (4099, -3.0, -5.0, "noplanes")])
def test_long_tiles_bitexact(n, opacity, scale, colours):
    print("case: long tiles", n, opacity, scale, colours, flush=True)
    sc = cluster(n, opacity, scale, seed=n)
    views = [synth.look_at((0.0, 0.0, -3.0), width=32, height=32, s_v=1.0)]
    cap = None
    if colours == "inf":
        sc["sh"][0, 1, ::977] = np.inf
    if colours == "full":      # a batch of more than 2,048 filled tiles: the line is 8,192 entries
        spread = synth.make_scene(30_000, 0, "uniform", seed=5, log_scale_mean=-4.5)
        sc = join(sc, spread)
        views.append(synth.look_at((0.0, 0.0, -3.5), width=1040, height=1040, s_v=1.0))
    if colours == "noplanes":  # many empty tiles: the bit planes find no room
        views.append(synth.look_at((0.0, 0.0, -3.0), width=2560, height=1440, s_v=1e6))
    rs = [O.render32(sc, v) for v in views]
    lists = np.concatenate([np.diff(r["tile_off"]) for r in rs])
    if colours == "full":
        assert (lists > 0).sum() > 2048
    else:
        assert 0.9 * n < lists.max() <= n   # (the faintest may fall below the mask's threshold)
    if colours == "noplanes":
        cap = int(sum(r["entries"].size for r in rs)) + 64
        assert 16 * 8 * ((cap + 63) // 64 + lists.size + 1) > 8 * cap
    g = gpu_forward(sc, views, dup_capacity=cap)
    compare_forward(g, sc, views)
    assert g["pairs"][0] == sum(r["pair_classes"][0] for r in rs)
    assert g["pairs"][2] == sum(r["pair_classes"][2] for r in rs)
