// Workgroups of the wide CG launches (cg_fused.hip).
#pragma once

namespace stag {

constexpr int kWideWG = 1024;   // lanes of a workgroup, one site each
constexpr int kWideGrid = 256;  // one workgroup per CU

// Tiles of kWideWG sites that each workgroup walks, for n problems of tiles[p] tiles and slots[p] right-hand sides:
// the smallest count that leaves kWideGrid workgroups in all, or 0 if there are more right-hand sides than that.
// A few workgroups more run a second round on an otherwise idle chip: 16^3x40 x 19, FP64, 266 workgroups, 444 us
// an iteration, where the launches with separate reductions take 412; 20^3x40 x 13, 260 workgroups, 617 and 572.
inline int wide_tiles(const int* tiles, const int* slots, int n) {
  long total = 0, nslots = 0;
  for (int p = 0; p < n; ++p) {
    total += (long)tiles[p] * slots[p];
    nslots += slots[p];
  }
  if (nslots > kWideGrid) return 0;
  for (int per = (int)((total + kWideGrid - 1) / kWideGrid);; ++per) {
    long grid = 0;
    for (int p = 0; p < n; ++p) grid += (long)((tiles[p] + per - 1) / per) * slots[p];
    if (grid <= kWideGrid) return per;
  }
}

}  // namespace stag
