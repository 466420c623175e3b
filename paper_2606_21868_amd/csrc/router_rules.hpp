// How a token batch's router logits are cut into workgroups (host code without HIP, so that the lines can be checked on the CPU).
#pragma once

#include <algorithm>

namespace wisp {

constexpr int kRouterMaxSplit = 8;   // column slices (partial sums) of a token batch's logits, at most
constexpr int kRouterChip = 256;     // compute units: workgroups that run side by side at full rate

struct RouterTiles {
  int slices, steps;   // column slices and 16-column steps of each
  int tb;              // 16-token blocks of a workgroup
  int groups, rb;      // groups of 64 rb router rows
};

// Column slices: at most kRouterMaxSplit, of at least four steps, while 64-token blocks of them fit the chip at
// once; they alone order a logit's sum.  Workgroups: either 64 tokens against all rows (the router matrix is then
// read once per 64 tokens), or 16 or 32 tokens against groups of 64 rows, which fill an empty chip: a wave's chain of
// fp32 matrix-core instructions is the time (64 x 128 x 256 columns take 6.8 us on one SIMD).  The time of either is
// its rounds over the chip times the 16 x 64 blocks of a workgroup (tb rb), but a small workgroup's block costs
// (3 + groups) / 3 of a large one's, as both operands are read more often: us a block and round, small against
// large, 10 / 8.4 (64 rows, d 7168), 3.5 / 2 (128, 2048), 5.7 / 2.6 (192, 4096), 9.3 / 3.9 (256, 7168).
// us a launch, small against large: 256 rows, d 7168 at 37 / 512 / 700 / 1000 / 1900 tokens 14 / 39 / 57 / 75 / 148 against
// 60 / 61 / 62 / 62 / 64; 128 rows, d 2048 at 37 / 1000 / 1900 tokens 5.8 / 14.9 / 25.2 against 12.2 / 15.5 / 17.7.
inline RouterTiles router_tiles(int T, int N, int d) {
  const int total = d / 16;
  auto blocks = [&](int tb) { return (T + 16 * tb - 1) / (16 * tb); };
  auto rounds = [&](int wgs) { return (wgs + kRouterChip - 1) / kRouterChip; };
  RouterTiles r{};
  int S = 1;
  while (2 * S <= kRouterMaxSplit && total / (2 * S) >= 4 && 2 * S * blocks(4) <= kRouterChip) S *= 2;
  r.steps = (total + S - 1) / S;
  r.slices = S = (total + r.steps - 1) / r.steps;
  const int nb = (N + 15) / 16, rows64 = (nb + 3) / 4;
  const int tb = blocks(2) * S * rows64 >= kRouterChip ? 2 : 1;
  const int small = rounds(blocks(tb) * S * rows64) * tb, large = rounds(blocks(4) * S) * 4 * rows64;
  const bool fine = small * (3 + rows64) < 3 * large;
  r.tb = fine ? tb : 4;
  r.groups = fine ? rows64 : 1;
  r.rb = fine ? 1 : rows64;
  return r;
}

}  // namespace wisp
