// Rules of the launches that need no device: how many blocks, which kernel.
// Host-only, so that they are checked without a GPU.
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

#include "fstat_common.hpp"
#include "fstat_prologue.hpp"

namespace fstat {

// Blocks per template of the kernels that solve every point (k_resample_bin,
// k_grad), for n templates of `tiles` tiles: one block per tile where every
// template takes them, and else (spans) while the launch stays below
// kPointBlocks; a larger launch walks the tiles.  A template that takes the other
// kernel of its pair leaves all its blocks empty: 160 000 of both kernels cost 100
// us (32 templates of 2.6 M points, 4350 us a call), 32 768 cost 40, 8192 cost
// 19.  Walking costs 3 % (32 templates of 1 M points with a sample every 5 s 4510
// us, 4395 with a block per tile), and 256 blocks per template are one workgroup
// per compute unit where four fit (one template 326 us against 186, two 373 /
// 319).
constexpr int64_t kPointBlocks = 32768;
inline unsigned point_blocks(int64_t tiles, int64_t n, bool spans) {
  if (!spans) return unsigned(tiles);
  return unsigned(std::min(tiles, std::max<int64_t>(256, kPointBlocks / std::max<int64_t>(n, 1))));
}

// Grid of k_params for n templates (and status words), one block each: a
// dimension of a launch holds fewer than 2^32 threads, which blocks of 128 pass
// at 2^25 templates, so the second one carries on from 2^kParamRowLog on (a
// constant: the kernel need not read the grid's size).  A walk of the templates
// in a loop took 206 registers instead of 110.
struct ParamGrid {
  unsigned x, y;
};
inline ParamGrid param_grid(int64_t n) {
  const int64_t x = std::max<int64_t>(1, std::min<int64_t>(n, int64_t(1) << kParamRowLog));
  return {unsigned(x), unsigned(std::max<int64_t>(1, (n + x - 1) / x))};
}

// The forward epilogue a RowOutput needs: plain 2F stores; candidates and
// loudest bin; Fa and Fb or sums (and nothing at all).  No row pass writes
// arrays and keeps candidates in one transform: -1, which the launch refuses.
inline int forward_row_mode(const RowOutput& out) {
  const bool keeps = out.cand || out.best, stores = out.twoF || out.fafb || out.acc;
  if (keeps) return stores ? -1 : int(kRowCand);
  return out.twoF && !out.fafb && !out.acc ? kRow2F : kRow2FExt;
}

// Lines per workgroup of the column pass (NL) and rows per workgroup of the
// row pass (RQ): at most as many as fit 128 KiB of LDS, capped for
// coalescing, with 512 threads; or half of that with 256 threads, so that two
// workgroups share a compute unit.
inline int cols_lines_max(int log_rr) { return std::min(64, 16384 >> log_rr); }
inline int rows_lines_max(int log_c) { return std::min(32, 8192 >> log_c); }

// Lines of up to 2^9 points have a variant for launches that leave the chip
// idle (cols_for, rows_for), which only the automatic line count takes.
constexpr int kFewMaxLog = 9;

// The launch shapes the autotuners time for transforms of 2^log_n points: both
// splits around the square root, for each pass two line counts, and both
// column stage plans where they differ (2^9 and 2^10 points).  The line counts
// are the automatic one and the one it does not take where lines are short (a
// fixed count never takes the small items of a small launch), else the full
// and the half count.
struct TuneShape {
  int col_log_len, col_lines, row_lines, radix;
};
inline std::vector<TuneShape> tune_shapes(int log_n) {
  std::vector<TuneShape> out;
  for (int lr = log_n / 2; lr <= (log_n + 1) / 2; ++lr) {
    const int lc = log_n - lr;
    if (lr < 6 || lr > 12 || lc < 6 || lc > 12) continue;
    const int cmax = cols_lines_max(lr), rmax = rows_lines_max(lc);
    const int cols[2] = {lr <= kFewMaxLog ? 0 : cmax / 2, cmax};
    const int rows[2] = {lc <= kFewMaxLog ? 0 : rmax, rmax / 2};
    for (int c : cols)
      for (int r : rows)
        for (int radix : {32, 16}) {
          if (radix == 16 && lr != 9 && lr != 10) continue;
          out.push_back({lr, c, r, radix});
        }
  }
  return out;
}

}  // namespace fstat
