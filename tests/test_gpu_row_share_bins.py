"""The row stage's unequal shares in each size of its tables: up to 256, 512 and 1,024 tile rows, past the
line that depends on them (256 records to a wave of the largest grid: 1,048,576 records with 256 or
512 rows, 524,288 with 1,024), in records of eight tiles or more; lists against the host's sort."""
import pytest

from paper_2510_09997_amd import _clod as C, synth
from paper_2510_09997_amd.render import Scene
from test_gpu_binning import check_lists

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,scale,sizes,rows,line", [
    (1_060_000, -4.3, [(1024, 1024)], (1, 256), 1 << 20),
    (180_000, -4.9, [(1280, 720), (1920, 1080), (2560, 2160)] * 2, (257, 512), 1 << 20),
    (37_000, -3.3, [(400, 720)] * 15, (513, 1024), 1 << 19)])
def test_unequal_shares_per_table(n, scale, sizes, rows, line):
    print("case: row share bins", n, rows, flush=True)
    sc = synth.make_scene(n, 0, "uniform", seed=6, log_scale_mean=scale)
    sc["decay"][:] = 100.0            # every Gaussian is kept at any distance
    sc["opacity"][:] = 3.0
    sc["log_scale"][:, : n // 500] = -1.5
    views = [synth.look_at((0.3, 0.2 + 0.01 * j, -4.0), width=w, height=h, s_v=1.0) for j, (w, h) in enumerate(sizes)]
    assert rows[0] <= sum((v.height + 15) // 16 for v in views) <= rows[1]
    b, D = check_lists(Scene(sc), views, capacity=40 * n * len(views))
    records = int(((b.section(C.SEC_FLAGS).cpu().numpy() & 4) != 0).sum())
    print("  records", records, "pairs", D, flush=True)
    assert records > line and D >= 8 * records
