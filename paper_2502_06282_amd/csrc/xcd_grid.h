// Which workgroups of a grid of two dimensions run on one XCD, of which there are eight: workgroups go round them in the order
// of the grid.  Not installed.
#pragma once

namespace jk {
constexpr int kXcds = 8;

// The grid's first dimension for `wgs` places, each with a workgroup in every one of `rows` rows: those of a place run on one XCD
// if there are a multiple of the XCDs in a row.  (Workgroups of places beyond `wgs` have nothing to do.)
constexpr int xcd_grid(int wgs, int rows) { return rows > 1 ? (wgs + kXcds - 1) / kXcds * kXcds : wgs; }

// The place of workgroup `blk` of a row of `all`: neighbours run on one XCD
constexpr int xcd_place(int blk, int all) { return all % kXcds == 0 ? blk % kXcds * (all / kXcds) + blk / kXcds : blk; }
}  // namespace jk
