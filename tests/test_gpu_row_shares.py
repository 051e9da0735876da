"""The row stage's unequal shares of the depth-sorted records, which it takes once they are more than
256 to a wave of its largest grid (262,144 records where a batch has over 1,024 tile rows) and cover
eight tiles or more on average: lists below either line and past both, with near records that cover
many rows."""
import pytest

from paper_2510_09997_amd import _clod as C, synth
from paper_2510_09997_amd.render import Scene
from test_gpu_binning import check_lists

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,scale,tiles", [(10_900, -3.3, (8, 40)), (13_200, -3.3, (8, 40)), (16_001, -3.3, (8, 40)),
                                           (23_001, -5.0, (1, 8))])
def test_lists_with_unequal_shares(n, scale, tiles):
    print("case: row shares", n, flush=True)
    sc = synth.make_scene(n, 0, "uniform", seed=5, log_scale_mean=scale)
    sc["decay"][:] = 100.0            # every Gaussian is kept at any distance
    sc["opacity"][:] = 3.0
    sc["log_scale"][:, : n // 100] = -1.0
    views = [synth.look_at((0.3, 0.2 + 0.01 * j, -4.0), width=400, height=720, s_v=1.0) for j in range(24)]
    b, D = check_lists(Scene(sc), views)
    records = int(((b.section(C.SEC_FLAGS).cpu().numpy() & 4) != 0).sum())
    print("  records", records, "pairs", D, flush=True)
    assert 0.9 * 24 * n < records <= 24 * n and tiles[0] * records <= D < tiles[1] * records
