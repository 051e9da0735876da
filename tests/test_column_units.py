"""Column units of the row path for pair counts up to the largest a pair buffer takes (2^32 - 2), where
32-bit sums of the sizing would wrap: units of at least kUnit pairs, whole multiples of it, as short
as the room allows, and never more of them than the tables hold, however the pairs lie in the rows."""
from hostprog import run

BODY = r"""
  unsigned long long x = 88172645463325252ull;
  auto next = [&]() { x ^= x << 13; x ^= x >> 7; x ^= x << 17; return x; };
  unsigned bad = 0;
  for (uint32_t cols = 64; cols <= kColsMax; cols += 64) {
    const uint32_t units_max = kHistWords / cols;
    for (uint32_t rows : {1u, 2u, 7u, 256u, 2047u, kRowBinsMax}) {
      const uint32_t room = units_max - rows;
      for (unsigned t = 0; t < 400; ++t) {
        const uint64_t span = (uint64_t)kUnit * room;
        uint64_t total = t == 0 ? 0 : t == 1 ? 1 : t < 40 ? span * (t / 4) + (t % 4) - 2 : t < 80 ? 0xFFFFFFFEull - (t - 40)
                       : t < 120 ? 0xFFFFFFFFull - span + (t - 100) : next() % 0xFFFFFFFFull;
        if (total > 0xFFFFFFFEull) total = 0xFFFFFFFEull;
        const uint64_t unit = unit_pairs((uint32_t)total, room);
        if (unit < kUnit || unit % kUnit != 0) bad |= 1;
        if (unit > kUnit && (unit - kUnit) * room >= total) bad |= 2;     // a shorter unit would do
        // The rows' pairs: even shares with odd remainders, one row with all of them, random cuts.
        for (int how = 0; how < 3; ++how) {
          uint64_t left = total, units = 0;
          for (uint32_t r = 0; r < rows; ++r) {
            uint64_t n = r + 1 == rows ? left : how == 0 ? total / rows : how == 1 ? (r == rows / 2 ? left : 0)
                       : left == 0 ? 0 : next() % (2 * (left / (rows - r)) + 1);
            if (n > left) n = left;
            left -= n;
            units += ceil_div((uint32_t)n, (uint32_t)unit);
            if (ceil_div((uint32_t)n, (uint32_t)unit) != (n + unit - 1) / unit) bad |= 4;
          }
          if (units > units_max) bad |= 8;
        }
      }
    }
  }
  printf("%u\n", bad);
"""


def test_units_fit_their_tables_for_every_pair_count(tmp_path):
    assert run(tmp_path, BODY).strip() == "0"
