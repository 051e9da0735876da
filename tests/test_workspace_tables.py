"""The binning's tables in the workspace, which are sized by the batch: every block count and column unit
that a pass over up to that many records can take fits them, and the workspace of a small batch is
small."""
import pytest

from hostprog import run
from paper_2510_09997_amd import _clod as C, synth

BODY = r"""
  unsigned bad = 0;
  for (int64_t VN : {1ll, 2ll, 63ll, 1000ll, 1024ll, 1025ll, 2048ll, 9999ll, 32768ll, 32769ll, 100000ll, 262143ll, 262144ll,
                     262145ll, 1000000ll, 1048576ll, 1048577ll, 4000000ll, 32000000ll, 4294967294ll})
    for (uint32_t tallest : {0u, 1u, 2u, 17u, 255u, 256u})
      for (uint32_t rows : {1u, 255u, 256u, 300u, 1025u, 2048u})
        for (uint32_t cols = 64; cols <= kColsMax; cols += 64) {
          if (tallest == 0 ? rows != 1 : rows < tallest) continue;   // 0: the general path, no rows
          const uint32_t words = tallest == 0 ? hist_words(VN, 0, 0, 0) : hist_words(VN, rows, cols, tallest);
          if (words > kHistWords) bad |= 1;
          for (uint32_t bins = 256; bins <= kRowBinsMax; bins *= 2)
            for (int64_t N : {(int64_t)0, (int64_t)1, VN / 3, VN - 1, VN}) {
              const RadixGeom G = radix_geom((uint64_t)N, bins);
              const uint32_t nb = G.nb > 0 ? G.nb : 1;               // (row 0 is read for no elements too)
              if ((uint64_t)nb * 4 * bins > words) bad |= 2;
              if (G.nb > pass_blocks(VN) || G.nb > pass_blocks(N < 1 ? 1 : N) || G.nb > radix_blocks(bins)) bad |= 4;
              if ((G.nb + kGroup - 1) / kGroup > sum_groups(VN)) bad |= 8;
              if ((uint64_t)G.kw * 4 * G.nb < (uint64_t)N || G.kw % 64 != 0) bad |= 16;
            }
          if (tallest == 0) continue;
          // The row kernels' shares where records cover many tiles.
          for (int64_t N : {(int64_t)1, VN / 3, VN}) {
            const RadixGeom G = radix_geom((uint64_t)N, row_bins_of(rows), kWaveMinWide);
            if ((uint64_t)G.nb * 4 * row_bins_of(rows) > words || G.nb > pass_blocks(N < 1 ? 1 : N, kWaveMinWide)) bad |= 512;
            if ((G.nb + kGroup - 1) / kGroup > sum_groups(VN)) bad |= 1024;
          }
          const uint32_t units_max = words / cols;
          if (units_max <= rows) { bad |= 32; continue; }
          // Row pairs: at most one per record and row of the tallest view.
          const uint64_t most = (uint64_t)VN * tallest < 0xFFFFFFFEull ? (uint64_t)VN * tallest : 0xFFFFFFFEull;
          for (uint64_t total : {(uint64_t)0, (uint64_t)1, most / 2, most}) {
            const uint32_t unit = unit_pairs((uint32_t)total, units_max - rows);
            // As if the tables had their full size.
            if (unit != unit_pairs((uint32_t)total, kHistWords / cols - rows)) bad |= 64;
            if (total >= rows && ceil_div((uint32_t)(total - rows + 1), unit) + rows - 1 > units_max) bad |= 128;
          }
        }
  if (sum_words(1, 256) != kDepthBins0 + 2 * kRowBinsMax + 256) bad |= 256;
  printf("%u\n", bad);
"""


def test_tables_hold_what_a_batch_can_need(tmp_path):
    assert run(tmp_path, BODY).strip() == "0"


# (What the sections before the tables, and 36 + 69 bytes per record, already took.)
@pytest.mark.parametrize("n,sizes,most", [
    (0, [(16, 16)], 0.10e6), (1, [(16, 16)], 0.15e6), (100, [(16, 16)], 0.15e6), (10_000, [(256, 256)], 1.6e6),
    (20_011, [(333, 217)] * 2, 6.0e6), (10_000, [(1920, 1080)], 2.4e6), (3_000_000, [(1920, 1080)], 337e6)])
def test_workspace_of_a_batch(n, sizes, most):
    views = C.make_views([synth.look_at((0, 0, -3), width=w, height=h) for w, h in sizes])
    assert 105 * n * len(sizes) < C.clod_ws_bytes(n, views) <= most
