// csrc/xcd_grid.h: every place has one workgroup per row of the grid, all of them on one XCD.
#include <cstdio>
#include <vector>

#include "xcd_grid.h"

int main() {
  for (int rows = 1; rows <= 3; ++rows)
    for (int wgs = 1; wgs <= 600; ++wgs) {
      const int all = jk::xcd_grid(wgs, rows);
      if (all < wgs || all >= wgs + jk::kXcds || (rows == 1 && all != wgs)) return std::printf("%d of %d\n", all, wgs), 1;
      std::vector<int> xcd(all, -1);
      for (int row = 0; row < rows; ++row) {
        std::vector<int> seen(all, 0);
        for (int blk = 0; blk < all; ++blk) {
          const int at = jk::xcd_place(blk, all), on = (row * all + blk) % jk::kXcds;
          if (at < 0 || at >= all || seen[at]++) return std::printf("%d workgroups: place %d of %d\n", wgs, at, blk), 1;
          if (row > 0 && xcd[at] != on) return std::printf("%d workgroups: place %d on XCDs %d and %d\n", wgs, at, xcd[at], on), 1;
          xcd[at] = on;
        }
      }
    }
  return 0;
}
