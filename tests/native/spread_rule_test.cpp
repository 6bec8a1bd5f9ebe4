// Host-only test of the rules of the spread passes
// (paper_2511_16298_amd/csrc/spread_rule.hpp), built with sanitizers by
// tests/test_spread_rule_cpu.py.  Prints OK and exits 0 when every check holds.
#include <stdio.h>

#include <initializer_list>

#include "spread_rule.hpp"

using ss::SpreadShape;

static int g_fail = 0;
#define CHECK(c)                                                            \
  do {                                                                      \
    if (!(c)) {                                                             \
      fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #c); \
      ++g_fail;                                                             \
    }                                                                       \
  } while (0)

// `frames` frames of tx x ty tiles, `n` Gaussians each, a capacity of
// `per` pairs per Gaussian.
struct Call {
  uint32_t frames, n, tx, ty;
  SpreadShape sh;
  Call(uint32_t f, uint32_t n_, uint32_t x, uint32_t y) : frames(f), n(n_), tx(x), ty(y) {
    for (uint32_t i = 0; i < f; ++i) sh.add(n, x, y);
  }
  uint32_t cap(double per) const {
    const double c = per * frames * n;
    return c > 1073741823.0 ? 1073741823u : static_cast<uint32_t>(c);
  }
  bool pays(double per) const { return ss::spread_pays(frames * n, frames, cap(per), sh); }
  uint32_t items(double per) const { return ss::row_pass_items(frames * n, cap(per), sh); }
};

int main() {
  // the shape's sums
  const Call two(2, 3000, 40, 23);
  CHECK(two.sh.sum_tx == 80 && two.sh.max_tx == 40 && two.sh.max_ty == 23 && two.sh.max_tiles == 920);
  CHECK(two.sh.col_blocks == 4);   // two workgroups of 2,048 Gaussians per frame

  // room to spare is not work: the decision for thinly filled batches is the
  // one that a close capacity gets, whatever the capacity
  for (double per : {1.5, 4.7, 5.3, 14.0, 47.0, 500.0}) {
    CHECK(!Call(64, 5000, 120, 68).pays(per));
    CHECK(!Call(64, 15000, 120, 68).pays(per));
    CHECK(!Call(128, 5000, 40, 23).pays(per));
    CHECK(!Call(24, 8000, 120, 68).pays(per));
  }
  for (double per : {4.7, 5.3, 14.0, 47.0, 500.0}) {
    CHECK(Call(64, 50000, 120, 68).pays(per));
    CHECK(Call(16, 20000, 120, 68).pays(per));
    CHECK(Call(1, 1000000, 120, 68).pays(per));
    CHECK(Call(1, 50000, 40, 23).pays(per));
    CHECK(Call(16, 20000, 120, 68).items(per) == 1024);
    CHECK(Call(8, 100000, 80, 45).items(per) == 2048);
    CHECK(Call(1, 6000000, 120, 68).items(per) == 4096);
    CHECK(Call(1, 300000, 120, 100).items(per) == 2048);
  }

  // axes
  CHECK(!Call(1, 1000000, 161, 90).pays(4.7) && Call(1, 1000000, 160, 90).pays(4.7));
  CHECK(!Call(1, 1000000, 90, 161).pays(4.7) && Call(1, 1000000, 90, 160).pays(4.7));
  CHECK(!Call(1, 1000000, 120, 7).pays(4.7) && Call(1, 1000000, 120, 8).pays(4.7));
  CHECK(!Call(1, 1000000, 7, 120).pays(4.7) && Call(1, 1000000, 8, 120).pays(4.7));
  CHECK(!Call(1, 1000000, 256, 1).pays(4.7) && !Call(1, 1000000, 1, 1).pays(4.7));
  // one digit pass over the pairs: up to 256 tiles
  CHECK(Call(1, 200000, 16, 16).pays(4.7) && !Call(1, 1000000, 32, 8).pays(4.7));
  CHECK(Call(1, 131071, 16, 16).pays(7.9) && !Call(1, 131071, 16, 16).pays(8.1) && Call(1, 131072, 16, 16).pays(8.1));
  CHECK(!Call(2, 100000, 16, 16).pays(4.7) && Call(8, 100000, 16, 16).pays(4.7) && !Call(128, 10000, 16, 16).pays(4.7));
  // small splats on long axes
  CHECK(!Call(1, 1048576, 128, 128).pays(1.99) && Call(1, 1048576, 128, 128).pays(2.0));
  CHECK(Call(1, 1048575, 128, 128).pays(1.6) && Call(1, 2000000, 120, 68).pays(1.6));
  // nothing to do; the largest sizes do not overflow
  CHECK(!Call(1, 0, 120, 68).pays(0.0) && !ss::spread_pays(0, 1, 0, SpreadShape{}));
  CHECK(ss::mean_column_items(100, 100, SpreadShape{}) == 0);
  SpreadShape big;
  big.add(0x7FFFFFFFu, 120, 68);
  CHECK(ss::spread_pays(0x7FFFFFFFu, 1, 0x3FFFFFFFu, big) && ss::row_pass_items(0x7FFFFFFFu, 0x3FFFFFFFu, big) == 4096);
  if (g_fail == 0) printf("OK\n");
  return g_fail == 0 ? 0 : 1;
}
