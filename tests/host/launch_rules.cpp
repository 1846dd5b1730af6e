// Host-only checks of the launch rules (fstat_launch.hpp).  Built and run by
// tests/test_host_checks.py; no GPU is touched.
#include <cstdio>

#include "fstat_launch.hpp"

using namespace fstat;

static int fails = 0;
static void check(bool ok, const char* what) {
  if (!ok) {
    printf("FAIL %s\n", what);
    ++fails;
  }
}

// One block per tile wherever the launch is small enough to leave the chip
// idle otherwise; never more blocks than tiles, and a bounded launch.
static void point_launch() {
  for (int64_t tiles : {1, 24, 256, 257, 1954, 5076, 32767})
    for (int64_t n : {1, 2, 4, 16, 32}) {
      const int64_t b = point_blocks(tiles, n, true);
      check(b >= 1 && b <= tiles, "blocks within the tiles");
      if (n * tiles <= 32768) check(b == tiles, "a small launch has a block per tile");
      check(n * b <= 32768 || b == 256 || b == tiles, "a large launch is bounded");
      check(n * b >= 1024 || b == tiles, "four workgroups per compute unit");
      check(point_blocks(tiles, n, false) == tiles, "a block per tile where no other kernel runs");
    }
}

int main() {
  point_launch();
  printf(fails ? "FAIL\n" : "OK\n");
  return fails != 0;
}
