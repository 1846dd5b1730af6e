// Host-only checks of the launch rules (fstat_launch.hpp).  Built and run by
// tests/test_host_checks.py; no GPU is touched.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstring>

#include "fstat_launch.hpp"
#include "fstat_prologue.hpp"

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

// The parameter launch has a block for every template of any bank, and each of
// its dimensions stays below 2^32 threads (65535 blocks in the second one).
static void param_launch() {
  for (int64_t n : {int64_t(0), int64_t(1), int64_t(11), int64_t(65536), int64_t(65537),
                    (int64_t(1) << 25) - 1, int64_t(1) << 25, int64_t(3000000001)}) {
    const ParamGrid g = param_grid(n);
    check(g.x >= 1 && int64_t(g.x) * g.y >= n, "a block per template");
    check(g.y == 1 || g.x == 1u << kParamRowLog, "rows of the kernel's length");
    check(int64_t(g.x) * kParamThreads < int64_t(1) << 32 && g.y <= 65535, "launch limits");
    if (n > 0) check(int64_t(g.x) * (g.y - 1) < n, "no empty row of blocks");
  }
}

// Every set of outputs goes to an epilogue that writes all of them.
static void row_modes() {
  float f;
  float2 f2;
  fstat_candidate c;
  unsigned long long u;
  for (int m = 0; m < 32; ++m) {
    RowOutput o;
    std::memset(&o, 0, sizeof o);
    if (m & 1) o.twoF = &f;
    if (m & 2) o.fafb = &f2;
    if (m & 4) o.cand = &c;
    if (m & 8) o.best = &u;
    if (m & 16) o.acc = 1;
    const int mode = forward_row_mode(o);
    const bool stores = m & 19, keeps = m & 12;
    if (stores && keeps) check(mode == -1, "arrays and candidates in one transform");
    else if (keeps) check(mode == kRowCand, "candidates");
    else check(mode == (m == 1 ? kRow2F : kRow2FExt), "arrays");
  }
}

// The autotuners time every shape once, and the automatic line counts wherever
// those have small-launch items of their own.
static void autotuned_shapes() {
  for (int log_n = 12; log_n <= 24; ++log_n) {
    const auto shapes = tune_shapes(log_n);
    check(!shapes.empty(), "shapes to time");
    for (int lr = log_n / 2; lr <= (log_n + 1) / 2; ++lr) {
      const int lc = log_n - lr, cmax = cols_lines_max(lr), rmax = rows_lines_max(lc);
      bool automatic = false, full = false;
      for (size_t i = 0; i < shapes.size(); ++i) {
        const TuneShape& a = shapes[i];
        if (a.col_log_len != lr) continue;
        check(a.col_lines == 0 || a.col_lines == cmax || a.col_lines == cmax / 2, "column lines");
        check(a.row_lines == 0 || a.row_lines == rmax || a.row_lines == rmax / 2, "row lines");
        check(a.radix == 32 || (a.radix == 16 && (lr == 9 || lr == 10)), "stage plan");
        automatic |= a.col_lines == (lr <= 9 ? 0 : cmax / 2) && a.row_lines == (lc <= 9 ? 0 : rmax);
        full |= a.col_lines == cmax && a.row_lines == rmax / 2;
        for (size_t j = 0; j < i; ++j) {
          const TuneShape& b = shapes[j];
          check(a.col_log_len != b.col_log_len || a.col_lines != b.col_lines ||
                    a.row_lines != b.row_lines || a.radix != b.radix,
                "a shape timed twice");
        }
      }
      check(automatic && full, "the default shape and the opposite one");
    }
  }
}

int main() {
  point_launch();
  param_launch();
  row_modes();
  autotuned_shapes();
  printf(fails ? "FAIL\n" : "OK\n");
  return fails != 0;
}
