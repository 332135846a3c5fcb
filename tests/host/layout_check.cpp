// Host checks of the packed operators' index arithmetic, built with
// UndefinedBehaviorSanitizer by test_host_layout.py.
#include <cstdio>

#include "../../paper_2501_03377_amd/csrc/kp_layout.h"

int main() {
  // (groups, points): the last block of an operator of just below, at and above
  // 2^31 16-byte units of FP64 (128 a block), against 128-bit arithmetic
  const int cases[][2] = {{1, 16}, {2, 513}, {4, 512}, {1, 65536}, {1, 65552}, {2, 92688},
                          {2, 131072}, {4, 180224}};
  for (const auto& c : cases) {
    const int G = c[0], m = (c[1] + G - 1) / G, nf = (m + 15) / 16;
    const __int128 blocks = (__int128)G * nf * nf;
    volatile unsigned q = G - 1, j = nf - 1, n = nf;
    if ((__int128)kp::fold_units(kp::fold_block(q, j, j, n, n), 128) != (blocks - 1) * 128) {
      std::printf("FAILED: %d points in %d groups\n", c[1], G);
      return 1;
    }
  }
  // neighbours: k-blocks next to each other, then columns, then groups
  if (kp::fold_block(0, 0, 1, 5, 5) != 1 || kp::fold_block(0, 1, 0, 5, 5) != 5 ||
      kp::fold_block(1, 0, 0, 5, 5) != 25)
    return 1;
  std::printf("layout checks ok\n");
  return 0;
}
