// Workgroups of the two sweeps over K (score_sweep.h): plain arithmetic, the same on the host and on the device.
#ifndef AMS_SWEEP_GRID_H
#define AMS_SWEEP_GRID_H

namespace ams {

constexpr int kMaxGridRows = 65535;  // extent of a launch in y

struct SweepGrid {
  int x, y;
};

// A row holds one workgroup per chunk of a unit; under the causal window, rows after those of the units hold one more per unit
// for its newest keys, next to each other.  A launch of more rows than the grid takes (the window's, from 32768 units of one
// chunk on) has two of them abreast: the order of the workgroups stays.
constexpr int sweep_rows(int units, int n_chunks, bool causal) {
  return units + (causal ? (units + n_chunks - 1) / n_chunks : 0);
}
constexpr SweepGrid sweep_grid(int units, int n_chunks, bool causal) {
  const int rows = sweep_rows(units, n_chunks, causal), abreast = rows > kMaxGridRows ? 2 : 1;
  return SweepGrid{n_chunks * abreast, (rows + abreast - 1) / abreast};
}
// Row by and place bx in it of workgroup (x, y) of a grid grid_x wide.
constexpr void sweep_place(int x, int y, int grid_x, int n_chunks, int& bx, int& by) {
  bx = x;
  by = y;
  if (grid_x != n_chunks) {
    by = y * (grid_x / n_chunks) + x / n_chunks;
    bx = x % n_chunks;
  }
}
// The unit whose newest keys that workgroup takes, -1: none.
constexpr int sweep_tail(int bx, int by, int n_chunks, int units) {
  const int unit = (by - units) * n_chunks + bx;
  return unit < units ? unit : -1;
}

}  // namespace ams
#endif
